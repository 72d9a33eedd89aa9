"""GPU parity of the kernels at the sizes where their tiles, chunks and dispatch rules change: edges and
remainders of tiles, the smallest and largest sizes of a range."""
import numpy as np
import pytest
import torch

import vbm_inputs as vi
from oracle import binning
from oracle import dwt as odwt
from oracle import tf as otf
from tests.gpu_common import ITEM_MASK, dev, say, to_dev

pytestmark = pytest.mark.gpu


def _api():
    from paper_2601_09417_amd import api
    return api


# Sides 4 (the smallest), one output pair short of and beyond the 64 x 16 tile, odd coarse sides, several tiles
# and z chunks; offset 1: a field that starts on a 4-byte boundary only.
@pytest.mark.parametrize("G,J,wav,with_tf,offset", [
    (4, 1, "bior4.4", True, 0), (4, 1, "haar", False, 1), (6, 1, "bior4.4", False, 1), (62, 1, "bior4.4", True, 1),
    (66, 1, "bior4.4", False, 0), (66, 1, "haar", True, 1), (72, 3, "bior4.4", True, 0), (100, 2, "bior4.4", False, 0),
    (130, 1, "bior4.4", True, 0), (100, 2, "haar", True, 0)])
def test_dwt_tile_edges(G, J, wav, with_tf, offset):
    api = _api()
    say(f"dwt edges G={G} J={J} {wav} tf={with_tf} offset={offset}")
    rng = np.random.default_rng(G + J)
    xs = np.array([0.1, 0.3, 0.3, 0.55, 0.8], np.float32)          # values beyond both ends, a jump at 0.3
    rgba_pts = rng.uniform(size=(5, 4)).astype(np.float32)
    if with_tf:
        vol = rng.uniform(size=(G, G, G)).astype(np.float32)
        vol.reshape(-1)[: 5] = xs                                     # on the control points
        rgba = otf.apply(vol, xs, rgba_pts)
    else:
        vol = rng.uniform(size=(4, G ** 3)).astype(np.float32)
        rgba = vol.reshape(4, G, G, G)
    flat = torch.empty(vol.size + offset, device=dev())
    flat[offset:] = torch.from_numpy(vol.reshape(-1)).to(dev())
    x = flat[offset:].view(vol.shape)
    got = api.dwt3d(x, J, wav, (xs, rgba_pts) if with_tf else None).cpu().numpy()
    ref = odwt.dwt3d_rgba(rgba, J, wav)
    tol = 1e-6 if wav == "haar" else 1e-5
    for (j, o), (off, n) in odwt.block_offsets(G, J).items():
        blk = slice(off, off + n ** 3)
        scale = max(np.abs(ref[:, blk]).max(), 1e-6)
        err = np.abs(got[:, blk] - ref[:, blk]).max() / scale
        assert err <= tol, ((j, o), err)


# Item counts around the emission's 256-item blocks, the sorts' 4096- and 8192-key tiles and the 16384 elements up
# to which one block sorts; opacities with holes in the depth keys, none visible at all (0), footprints on either
# side of the 32-tile rule; a batch of one tile (no digits to sort), short and long.
@pytest.mark.parametrize("n,views,W,H,tile,bits,opacity,log_scale", [
    (1, 2, 131, 77, 16, 8, (0.5, 0.9), -3.0), (255, 2, 131, 77, 16, 8, (0.5, 0.9), -3.0),
    (256, 2, 131, 77, 8, 8, (0.5, 0.9), -2.0), (257, 2, 131, 77, 16, 4, (0.5, 0.9), -1.6),
    (300, 2, 131, 77, 16, 8, (0.001, 0.003), -3.0), (4097, 2, 131, 77, 16, 8, (0.001, 0.007), -3.5),
    (8192, 2, 131, 77, 32, 8, (0.5, 0.9), -4.0), (8193, 2, 131, 77, 16, 8, (0.001, 0.007), -3.5),
    (16500, 2, 131, 77, 8, 5, (0.001, 0.02), -3.8), (300, 1, 16, 16, 16, 8, (0.5, 0.9), -3.0),
    (20000, 1, 16, 15, 16, 8, (0.5, 0.9), -3.0), (700, 1, 640, 1100, 8, 8, (0.2, 0.9), -3.4)])
def test_pair_lists_at_block_edges(n, views, W, H, tile, bits, opacity, log_scale):
    api = _api()
    say(f"pair lists n={n} {views} views {W}x{H} tile={tile} digits={bits} opacity {opacity} log scale {log_scale}")
    gs = vi.random_gaussians(n, 31 + n, log_scale_mean=log_scale, opacity_range=opacity)
    cams = vi.orbit_cameras(views, W, H, azimuth0=0.2)
    ref = binning.pair_lists(gs, cams, tile)
    total = ref["tile"].size
    full = ref["ranges"][:, 1] > ref["ranges"][:, 0]
    # the exact capacity, and one beyond the one-block sort
    for capacity, mode in ((max(total, 1), "batched"), (total + 16385, "batched"), (total + 16385, "exact")):
        rp = api.plan_batch(cams, [0, n], tile=tile, sort_bits=bits, pair_capacity=capacity, mode=mode)
        for _ in range(2):      # the second pass finds the first one's counters, totals and look-back words
            out = api.render_fwd(rp, to_dev(gs))
        torch.cuda.synchronize()
        assert out.status[:2].tolist() == [0, total]
        assert int(out.status[2]) == sum(int((p["n_tiles"] > 0).sum()) for p in ref["proj"])
        assert np.array_equal(rp.region("pair_tile", torch.int32).cpu().numpy()[:total], ref["tile"])
        assert np.array_equal(rp.region("pair_item", torch.int32).cpu().numpy()[:total] & ITEM_MASK, ref["item"])
        ranges = rp.region("ranges", torch.int32).cpu().numpy().reshape(-1, 2)
        assert np.array_equal(ranges[full], ref["ranges"][full])
        assert not ranges[~full].any()
    if total > 1:           # one slot short: flagged
        rp = api.plan_batch(cams, [0, n], tile=tile, sort_bits=bits, pair_capacity=total - 1)
        out = api.render_fwd(rp, to_dev(gs))
        assert out.status.tolist()[:2] == [1, total]
