"""GPU parity of the kernels at the sizes where their tiles, chunks and dispatch rules change: edges and
remainders of tiles, the smallest and largest sizes of a range."""
import numpy as np
import pytest
import torch

import vbm_inputs as vi
from oracle import dwt as odwt
from oracle import tf as otf
from tests.gpu_common import dev, say

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
