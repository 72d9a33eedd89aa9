"""GPU parity of the kernels at the sizes where their tiles, chunks and dispatch rules change: edges and
remainders of tiles, the smallest and largest sizes of a range."""
import dataclasses

import numpy as np
import pytest
import torch

import vbm_inputs as vi
from oracle import binning, render
from oracle import dvr as odvr
from oracle import dwt as odwt
from oracle import select as oselect
from oracle import tf as otf
from tests.gpu_common import (GRAD_TOL, IMG_TOL, ITEM_MASK, ROWS, dev, flat, group_error, image_error, masked_dL, say,
                              to_dev)

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


# Item counts around the emission's 256-item blocks, the sorts' 4096- and 8192-key tiles and the 8192 elements up
# to which one block sorts; opacities with holes in the depth keys, none visible at all (0), footprints on either
# side of the 32-tile rule; a batch of one tile (no digits to sort), short and long.
@pytest.mark.parametrize("n,views,W,H,tile,bits,opacity,log_scale", [
    (1, 2, 131, 77, 16, 8, (0.5, 0.9), -3.0), (255, 2, 131, 77, 16, 8, (0.5, 0.9), -3.0),
    (256, 2, 131, 77, 8, 8, (0.5, 0.9), -2.0), (257, 2, 131, 77, 16, 4, (0.5, 0.9), -1.6),
    (4096, 2, 131, 77, 16, 8, (0.001, 0.007), -3.5),
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


# List lengths around what the compositing walks count in: 16 entries (shorter lists are not shared by four waves),
# batches of 64 and of 32, closed-up batches that are no multiple of four; faint lists that are walked to the end and
# dense ones whose pixels stop inside a batch; an image that ends inside a band.
@pytest.mark.parametrize("n,H,tile,opacity,log_scale", [
    (15, 16, 16, (0.2, 0.6), -2.0), (16, 16, 16, (0.2, 0.6), -2.0), (17, 13, 16, (0.9, 1.0), -1.5),
    (33, 16, 8, (0.2, 0.6), -2.0), (64, 16, 16, (0.2, 0.6), -2.0), (65, 10, 16, (0.02, 0.1), -2.0),
    (130, 16, 16, (0.5, 1.0), -1.6), (200, 16, 32, (0.5, 1.0), -1.6), (400, 16, 16, (0.01, 0.05), -2.6),
    (400, 16, 8, (0.5, 1.0), -2.0)])
def test_compositing_walks_at_batch_edges(n, H, tile, opacity, log_scale):
    api = _api()
    say(f"walks n={n} 24x{H} tile={tile} opacity {opacity} log scale {log_scale}")
    gs = vi.random_gaussians(n, 71 + n, log_scale_mean=log_scale, opacity_range=opacity)
    cams = vi.orbit_cameras(1, 24, H, azimuth0=0.9)
    P = to_dev(gs)
    rp = api.plan_batch(cams, [0, n], tile=tile, pair_capacity=1 << 16)
    batch = render.Batch(gs, cams, tile)
    ref = render.render_forward(batch)
    dL = masked_dL(cams, [r["flagged"] for r in ref], seed=n)
    g_ref, _ = render.render_backward(batch, dL)
    for _ in range(2):
        out = api.render_fwd(rp, P)
        assert image_error(api.split_views(out.image, cams)[0].cpu().numpy(), ref[0]["image"],
                           ref[0]["flagged"]) <= IMG_TOL
        ok = ~ref[0]["flagged"]
        nc = out.n_contrib.cpu().numpy().reshape(H, 24)
        assert np.array_equal(nc[ok], ref[0]["n_visited"][ok])
        G = api.render_bwd(rp, P, flat(dL), out).cpu().numpy()
        for name, rows in ROWS.items():
            assert group_error(G[rows], g_ref[name].reshape(rows.stop - rows.start, -1)) <= GRAD_TOL, name


def test_counters_agree_between_walks():
    """The evaluation counters count list entries up to a pixel's stop and contributions; they do not depend on how
    a list is walked: 16x16 tiles shared by four waves (few tiles), 8x8 and 32x32 tiles see the same contributions
    (opacities up to 0.3: the reach of alpha >= 1/255 stays within three sigma, so the tilings list the same)."""
    import ctypes

    from paper_2601_09417_amd import _lib as L
    api = _api()
    gs = vi.random_gaussians(3000, 5, log_scale_mean=-2.6, opacity_range=(0.05, 0.3))
    cams = vi.orbit_cameras(2, 131, 77)
    used = []
    for tile in (8, 16, 32):
        rp = api.plan_batch(cams, [0, gs.n], tile=tile, pair_capacity=1 << 18)
        c = torch.zeros(4, dtype=torch.int64, device=dev())
        L.check(L.load().vbm_profile_counters(ctypes.c_void_p(c.data_ptr())), "vbm_profile_counters")
        try:
            out = api.render_fwd(rp, to_dev(gs))
            api.render_bwd(rp, to_dev(gs), torch.ones_like(out.image), out)
            torch.cuda.synchronize()
        finally:
            L.load().vbm_profile_counters(None)
        ev_f, us_f, ev_b, us_b = c.tolist()
        assert us_f == us_b and ev_b == int(out.n_contrib.sum()) and ev_f >= ev_b
        used.append(us_f)
    assert used[0] == used[1] == used[2] > 0


# The selection's candidate pass: grids below, at and above its 4096-location regions and the size from which a sample
# bounds the candidates; K of 1, of everything and between; planes that start on a 4-byte boundary only; a sample that
# misleads (only the sampled locations are large, so the bound leaves too few); ties at the K-th key; NaN and
# infinities.
@pytest.mark.parametrize("G,K,kind", [
    (4, 1, "plain"), (16, 4096, "plain"), (18, 1000, "odd"), (64, 5000, "plain"), (66, 1, "plain"), (66, 20000, "odd"),
    (72, 72 ** 3, "plain"), (96, 50000, "mislead"), (96, 300000, "ties"), (96, 2000, "special")])
def test_selection_candidates(G, K, kind):
    api = _api()
    say(f"selection G={G} K={K} {kind}")
    M = G ** 3
    rng = np.random.default_rng(G + K)
    c = (rng.normal(size=(4, M)) * np.exp(rng.normal(size=M))).astype(np.float32)
    if kind == "mislead":
        c *= np.where(np.arange(M) % 2048 < 16, 100.0, 1.0).astype(np.float32)
    if kind == "ties":
        c = np.round(c).astype(np.float32)
    if kind == "special":
        c[0, 7::5000] = np.inf
        c[2, 11::9000] = np.nan
    flat_c = torch.empty(4 * M + 1, device=dev())
    off = 1 if kind == "odd" else 0
    x = flat_c[off:off + 4 * M].view(4, M)
    x.copy_(torch.from_numpy(c))
    bank = np.zeros((8, 12), np.float32)
    bank[:, 0] = 1.0
    bank[:, 4:8] = 1.0
    P, kept = api.build_gaussians(x, G, 1, bank, K, s_mode="none")
    kept = kept.cpu().numpy()
    if kind == "special":
        # key order of the bit patterns: NaN above infinity above the finite keys
        with np.errstate(invalid="ignore"):
            square = ((c[0] * c[0] + c[1] * c[1]) + c[2] * c[2]) + c[3] * c[3]
            v = np.sqrt(square.astype(np.float64)).astype(np.float32)
        order = np.lexsort((np.arange(M), -np.nan_to_num(v, nan=np.inf).astype(np.float64), ~np.isnan(v)))
        ref = np.sort(order[:K])
    else:
        ref = oselect.topk(c, K)
    assert np.array_equal(kept, ref)
    ok = np.isfinite(c[3][ref])
    assert np.array_equal(P[10].cpu().numpy()[ok], np.clip(np.abs(c[3][ref][ok]), np.float32(1e-3), np.float32(0.99)))


# Views of several sizes in one call, more than one launch holds and none a multiple of the 16x16 blocks; the smallest
# volume; steps other than half a voxel; a transfer function with a jump and values beyond both its ends.
@pytest.mark.parametrize("G,step,n_views", [(2, 0.5, 1), (21, 0.5, 10), (21, 0.75, 2), (33, 1.0, 3)])
def test_dvr_views_and_steps(G, step, n_views):
    api = _api()
    say(f"dvr G={G} step={step} views={n_views}")
    rng = np.random.default_rng(G)
    vol = rng.uniform(size=(G, G, G)).astype(np.float32)
    xs = np.array([0.1, 0.4, 0.4, 0.7, 0.9], np.float32)
    rgba = rng.uniform(size=(5, 4)).astype(np.float32)
    rgba[:, 3] *= np.float32(0.2)
    # intrinsics rounded to float32, the values the library receives
    cams = [dataclasses.replace(c, fx=float(np.float32(c.fx)), fy=float(np.float32(c.fy)))
            for v in range(n_views) for c in [vi.orbit_cameras(n_views, 17 + 3 * v, 33 - 2 * v, azimuth0=0.1)[v]]]
    img = api.dvr_render(torch.from_numpy(vol).to(dev()), (xs, rgba), cams, step_vox=step)
    for got, cam in zip(api.split_views(img, cams), cams):
        ref, _, near = odvr.render(vol, xs, rgba, cam, step_vox=step, flag_rel=1e-6)
        assert near.sum() <= 2
        err = np.abs(got.cpu().numpy() - ref)[:, ~near].max()
        assert err <= 1e-5 * max(float(np.abs(ref).max()), 1e-6)


# The loss value comes from one block that takes 2048 partial sums at a time: one partial, a single pass of the
# block, a remainder after it, and view groups whose last one is a single tile.  The bounds are those of the
# repository's loss comparison.
@pytest.mark.parametrize("kind", ["l1", "l1_dssim"])
@pytest.mark.parametrize("dims", [[(1, 1)], [(33, 31)], [(900, 905)], [(640, 512), (640, 512), (129, 500), (5, 3)]])
def test_loss_partials(dims, kind):
    from oracle import loss as oloss
    api = _api()
    say(f"loss partials {dims} {kind}")
    rng = np.random.default_rng(len(dims))
    imgs = [rng.uniform(size=(3, h, w)).astype(np.float32) for w, h in dims]
    tgts = [np.clip(i + 0.1 * rng.normal(size=i.shape), 0, 1).astype(np.float32) for i in imgs]
    x = torch.from_numpy(np.concatenate([i.reshape(-1) for i in imgs])).to(dev())
    y = torch.from_numpy(np.concatenate([t.reshape(-1) for t in tgts])).to(dev())
    g = torch.empty_like(x)
    value = float(api.ImageLoss(dims, kind, 0.2)(x, y, g).item())
    ref_loss, ref_g = oloss.loss_and_grad(imgs, tgts, kind)
    assert abs(value - ref_loss) <= 1e-5 * abs(ref_loss)
    rg = np.concatenate([a.reshape(-1) for a in ref_g])
    assert np.abs(g.cpu().numpy() - rg).max() <= 1e-4 * np.abs(rg).max()


# Subbands of one part of a chunk, of one chunk and of a chunk and a short part; blocks without coefficients; many equal
# norms (zeros, halves); infinities; budgets of 0 and of more than a subband holds.  The results match the oracle's.
@pytest.mark.parametrize("G,J,values,K_tot,params", [
    (8, 1, "normal", 100, dict(alpha=0.0, beta=0.0)), (16, 1, "normal", 7, dict(alpha=0.0, beta=0.0, min_band=0)),
    (32, 1, "infinite", 2048, dict(alpha=0.0, beta=0.0)), (32, 1, "zeros", 512, dict(alpha=0.0, beta=0.0, lam=0.0)),
    (52, 1, "sparse", 9001, dict(lam=0.5)), (52, 1, "halves", 20001, dict(lam=1.0)),
    (64, 1, "normal", 4, dict(min_band=40000)), (66, 1, "normal", 30011, dict(lam=0.0))])
def test_adaptive_parts(G, J, values, K_tot, params):
    from tests.gpu_common import adaptive_check
    api = _api()
    say(f"adaptive parts G={G} J={J} {values} K_tot={K_tot} {params}")
    rng = np.random.default_rng(G + K_tot)
    c = rng.normal(size=(4, G ** 3)).astype(np.float32)
    if values == "zeros":
        c[:] = 0.0
    elif values == "sparse":
        c *= rng.uniform(size=(1, G ** 3)) < 0.03
    elif values == "halves":
        c = (np.round(2 * c) / 2).astype(np.float32)
    elif values == "infinite":
        c[rng.uniform(size=c.shape) < 0.01] = -np.inf
    kept, stats = api.adaptive_select(torch.from_numpy(c).to(dev()), G, J, K_tot, **params)
    adaptive_check(c, G, J, kept.cpu().numpy(), stats.cpu().numpy(), K_tot, **params)


# Batches of 3,000 longest lists or more take the backward's sums through LDS, two list entries at a time; each view
# alone is below that and is reduced in registers, which the comparisons with the oracle cover.  The batch's gradient
# is the sum of the views', to the same bound: lists of one entry and of odd and even length, alphas beyond the clamp
# (opacity 1), images that end inside a tile.
@pytest.mark.parametrize("n,views,W,H,tile,opacity,log_scale", [
    (400, 400, 120, 116, 16, (0.5, 1.0), -3.4), (400, 160, 120, 116, 8, (0.5, 1.0), -3.4),
    (600, 400, 128, 120, 16, (0.02, 0.3), -3.2), (200, 240, 100, 90, 8, (0.9, 1.0), -4.0)])
def test_backward_sums_through_lds(n, views, W, H, tile, opacity, log_scale):
    api = _api()
    say(f"sums through LDS n={n} {views} views {W}x{H} tile={tile} opacity {opacity} log scale {log_scale}")
    gs = vi.random_gaussians(n, 171 + n, log_scale_mean=log_scale, opacity_range=opacity)
    cams = vi.orbit_cameras(views, W, H)
    P = to_dev(gs)
    rng = np.random.default_rng(n)
    dL = torch.from_numpy(rng.normal(size=len(cams) * 3 * W * H).astype(np.float32)).to(dev())

    def grad(batch, dl, at_least):
        rp = api.plan_batch(batch, [0, n], tile=tile, pair_capacity=1 << 20)
        out = api.render_fwd(rp, P)
        lists = rp.region("ranges", torch.int32).cpu().numpy().reshape(-1, 2)
        lists = lists[:, 1] - lists[:, 0]
        assert (lists.sum() >= 3100 * lists.max()) == at_least
        return api.render_bwd(rp, P, dl.contiguous(), out).cpu().numpy().astype(np.float64)

    G = grad(cams, dL, True)
    ref = sum(grad(cams[v:v + 1], dL[3 * W * H * v:3 * W * H * (v + 1)], False) for v in range(len(cams)))
    for name, rows in ROWS.items():
        assert group_error(G[rows], ref[rows]) <= GRAD_TOL, name


# Footprints from a pixel to the whole image and from round to thin (axes 10^4 apart), where the tile test's short form
# meets its margin: the same pairs as the oracle's four-edge test.
@pytest.mark.parametrize("tile", [8, 16, 32])
def test_pair_lists_of_thin_footprints(tile):
    api = _api()
    say(f"thin footprints tile={tile}")
    gs = vi.random_gaussians(1500, 77, log_scale_mean=-3.5, log_scale_std=2.5, opacity_range=(0.004, 0.99))
    cams = vi.orbit_cameras(2, 301, 203)
    ref = binning.pair_lists(gs, cams, tile)
    total = ref["tile"].size
    rp = api.plan_batch(cams, [0, gs.n], tile=tile, pair_capacity=total)
    out = api.render_fwd(rp, to_dev(gs))
    assert out.status[:2].tolist() == [0, total]
    assert np.array_equal(rp.region("pair_tile", torch.int32).cpu().numpy()[:total], ref["tile"])
    assert np.array_equal(rp.region("pair_item", torch.int32).cpu().numpy()[:total] & ITEM_MASK, ref["item"])


def _stop_at_the_threshold(alpha):
    """Entries i, j, k, s and a pixel p whose transmittance is exactly float32(1e-4) after i, j and k, and for which
    T - s T + s T, each step rounded, falls below it: alpha float32 [entries][pixels], all at least one half, so that
    every product below is exact in float64 before its one rounding."""
    f = np.float32
    c = float(f(1e-4))
    i, j = np.triu_indices(alpha.shape[0])
    for p in range(alpha.shape[1]):
        a = alpha[:, p].astype(np.float64)
        order = np.argsort(a)
        T1 = 1.0 - a[i]
        T2 = (T1 - T1 * a[j]).astype(f).astype(np.float64)
        at = np.searchsorted(a[order], 1.0 - c / T2)
        low = np.nonzero(f(c) * a.astype(f) + (c - c * a).astype(f) < f(c))[0]
        for step in (-1, 0):
            k = order[np.clip(at + step, 0, a.size - 1)]
            hit = np.nonzero((T2 - T2 * a[k]).astype(f) == f(c))[0]
            if hit.size and low.size:
                return p, [int(i[hit[0]]), int(j[hit[0]]), int(k[hit[0]]), int(low[0])]
    raise AssertionError("no such entries")


# A pixel that an entry has stopped stays as that entry left it, whatever rounding made of its transmittance: the
# entries behind it, and the padding of a group of four, neither move its count nor get a gradient from it.  (Gaussians
# at one place, which the lists keep in the order they are given in.)
@pytest.mark.parametrize("tile,behind", [(8, 2), (8, 9), (8, 70), (16, 2), (16, 13), (16, 70)])
def test_stopped_pixel_stays_stopped(tile, behind):
    api = _api()
    n = 400
    rng = np.random.default_rng(tile)
    cam = vi.orbit_cameras(1, tile, tile, azimuth0=0.9)[0]
    f = np.float32
    gs = vi.GaussianSet(np.zeros((3, n), f), np.full((3, n), 3.0, f), np.tile(np.array([[1], [0], [0], [0]], f), (1, n)),
                        rng.uniform(0.93, 0.985, n).astype(f), rng.uniform(0.2, 1.0, (3, n)).astype(f))
    # every entry's alpha, alone in a view of its own (1 - T is exact from one half on)
    rp = api.plan_batch([cam] * n, np.arange(n + 1), list(range(n)), tile=tile, pair_capacity=1 << 16)
    alpha = f(1.0) - api.render_fwd(rp, to_dev(gs)).final_T.cpu().numpy().reshape(n, tile * tile)
    assert alpha.min() >= 0.5
    p, entries = _stop_at_the_threshold(alpha)
    say(f"stopped pixel tile={tile}: pixel {p}, entries {entries}, {behind} behind")
    idx = np.array(entries + list(range(behind)))
    P = to_dev(gs.subset(idx))
    rp = api.plan_batch([cam], [0, idx.size], tile=tile, pair_capacity=1 << 16)
    out = api.render_fwd(rp, P)
    assert out.status.tolist()[:2] == [0, idx.size]
    assert int(out.n_contrib[p]) == 3
    assert abs(float(out.final_T[p]) - float(f(1e-4))) <= 2 ** -37   # one unit in the last place
    dL = torch.zeros_like(out.image)
    dL[p::tile * tile] = 1.0
    G = api.render_bwd(rp, P, dL, out).cpu().numpy()
    assert not G[:, 3:].any()
    a = alpha[idx[:3], p].astype(np.float64)
    w = a * np.concatenate([[1.0], np.cumprod(1.0 - a)[:2]])
    assert np.abs(G[11] - np.concatenate([w, np.zeros(idx.size - 3)])).max() <= GRAD_TOL * w.max()


# Voxels that are not numbers or infinite: a sample that is not a number takes the first control point's colour, an
# infinite one that of its end, as any value beyond the end points does.
@pytest.mark.parametrize("step", [0.5, 0.75])
def test_dvr_samples_that_are_not_finite(step, monkeypatch):
    api = _api()
    say(f"dvr of voxels that are not finite, step {step}")
    rng = np.random.default_rng(3)
    G = 21
    vol = rng.uniform(size=(G, G, G)).astype(np.float32)
    special = rng.choice(G ** 3, 90, replace=False)
    vol.reshape(-1)[special] = np.repeat(np.array([np.nan, np.inf, -np.inf], np.float32), 30)
    xs = np.array([0.1, 0.4, 0.4, 0.7, 0.9], np.float32)
    rgba = rng.uniform(size=(5, 4)).astype(np.float32)
    rgba[:, 3] *= np.float32(0.2)

    def trilinear(v, p):
        u = np.clip((p + 1.0) / (2.0 / G) - 0.5, 0.0, G - 1.0)
        i = np.minimum(np.floor(u).astype(np.int64), G - 2)
        f = u - i
        x, y, z = i[..., 0], i[..., 1], i[..., 2]
        lerp = lambda t, a, b: a + t * (b - a)  # noqa: E731
        with np.errstate(invalid="ignore"):
            row = [[lerp(f[..., 0], v[z + dz, y + dy, x], v[z + dz, y + dy, x + 1]) for dy in (0, 1)] for dz in (0, 1)]
            s = lerp(f[..., 2], lerp(f[..., 1], *row[0]), lerp(f[..., 1], *row[1]))
        return np.where(np.isnan(s), -np.inf, s)

    monkeypatch.setattr(odvr, "trilinear", trilinear)
    cams = [dataclasses.replace(c, fx=float(np.float32(c.fx)), fy=float(np.float32(c.fy)))
            for c in vi.orbit_cameras(2, 61, 45, azimuth0=0.1)]
    img = api.dvr_render(torch.from_numpy(vol).to(dev()), (xs, rgba), cams, step_vox=step)
    for got, cam in zip(api.split_views(img, cams), cams):
        ref, _, near = odvr.render(vol, xs, rgba, cam, step_vox=step, flag_rel=1e-6)
        assert np.isfinite(ref).all() and near.sum() <= 2
        err = np.abs(got.cpu().numpy() - ref)[:, ~near].max()
        assert err <= 1e-5 * float(np.abs(ref).max())


def _dwt_call(vol_ptr, G, J, wav, tf, coeffs):
    import ctypes as C

    from paper_2601_09417_amd import _lib as L
    lib = L.load()
    ws = torch.empty(lib.vbm_dwt3d_workspace_size(G, J), dtype=torch.uint8, device=dev())
    t = _api().make_tf(*tf) if tf is not None else None
    L.check(lib.vbm_dwt3d(vol_ptr, G, J, L.WAVELETS[wav], C.byref(t) if t else None, coeffs.data_ptr(), ws.data_ptr(),
                          ws.numel(), torch.cuda.current_stream().cuda_stream), "vbm_dwt3d")


# The coefficients may take the field's own memory: the whole of it (RGBA), or any part.
@pytest.mark.parametrize("G,J,wav,with_tf,offset", [
    (130, 1, "bior4.4", False, 0), (100, 2, "haar", False, 0), (4, 1, "haar", False, 0), (72, 3, "bior4.4", False, 0),
    (130, 1, "bior4.4", True, 130 ** 3), (100, 1, "haar", True, 1001), (64, 5, "bior4.4", True, 0),
    (64, 2, "bior4.4", True, 4 * 64 ** 3 - 7)])
def test_dwt_over_its_own_input(G, J, wav, with_tf, offset):
    api = _api()
    say(f"dwt over its input G={G} J={J} {wav} tf={with_tf} offset={offset}")
    g = torch.Generator(device="cuda").manual_seed(G)
    vol = torch.rand((G, G, G) if with_tf else (4, G ** 3), generator=g, device=dev())
    tf = (np.array([0.1, 0.3, 0.8], np.float32), np.linspace(0.0, 1.0, 12, dtype=np.float32).reshape(3, 4))
    ref = api.dwt3d(vol, J, wav, tf if with_tf else None)
    shared = torch.full((4 * G ** 3 + vol.numel(),), float("nan"), device=dev())
    shared[offset:offset + vol.numel()] = vol.reshape(-1)
    _dwt_call(shared[offset:].data_ptr(), G, J, wav, tf if with_tf else None, shared)
    assert torch.equal(shared[:4 * G ** 3].view(4, -1), ref)


# Segments whose width has no float32 reciprocal (infinite, or below the normal range), and colours that are infinite
# beyond an end point.
@pytest.mark.parametrize("kind,wav", [("infinite", "haar"), ("infinite", "bior4.4"), ("subnormal", "haar"),
                                      ("subnormal", "bior4.4"), ("wide", "haar"), ("wide", "bior4.4"),
                                      ("colour", "haar")])
def test_dwt_transfer_function_segments(kind, wav):
    api = _api()
    G = 8
    say(f"dwt transfer function {kind} {wav}")
    rng = np.random.default_rng(9)
    rgba = rng.uniform(size=(3, 4)).astype(np.float32)
    vol = rng.uniform(size=(G, G, G)).astype(np.float32)
    xs = np.array([0.1, 0.5, 0.8], np.float32)
    if kind == "infinite":
        xs[2] = np.inf
    elif kind == "wide":
        xs[:] = [-3e38, 1e37, 3.3e38]
        vol = (vol.astype(np.float64) * 6e38 - 3e38).astype(np.float32)
    elif kind == "subnormal":
        xs[:] = [0.0, 2.0 ** -138, 1.0]
        vol.reshape(-1)[::2] = (rng.integers(0, 2 ** 11, vol.size // 2) * 2.0 ** -149).astype(np.float32)
    elif kind == "colour":
        rgba[2, 3] = np.inf
        vol[:] = 0.9
    # t = (f - x0) / (x1 - x0) in the segment, the end point's colour outside
    e = np.clip(np.searchsorted(xs, vol, side="right") - 1, 0, 1)
    with np.errstate(invalid="ignore", over="ignore"):
        x0, x1 = xs[e].astype(np.float64), xs[e + 1].astype(np.float64)
        t = np.clip((vol - x0) / (x1 - x0), 0.0, 1.0)[None]
        c0, c1 = np.moveaxis(rgba[e], -1, 0).astype(np.float64), np.moveaxis(rgba[e + 1], -1, 0).astype(np.float64)
        c = np.where(t >= 1.0, c1, c0 + t * (c1 - c0))
    got = api.dwt3d(torch.from_numpy(vol).to(dev()), 1, wav, (xs, rgba)).cpu().numpy()
    if kind == "colour":
        assert np.isposinf(got[3, :(G // 2) ** 3]).all() and np.isfinite(got[:3]).all()
        return
    ref = odwt.dwt3d_rgba(c, 1, wav)
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()


# Lists beyond the 2,040 entries at which the launch order's length steps end: two scenes of one tile each, the longer
# list second; sorted by one block (room for 8,192 pairs) and by the radix passes.
@pytest.mark.parametrize("capacity", [8192, 40000])
@pytest.mark.parametrize("tile", [8, 16])
def test_lists_beyond_the_length_steps(tile, capacity):
    api = _api()
    counts = [2100, 5000]
    say(f"long lists tile={tile} capacity={capacity}")
    gs = vi.random_gaussians(sum(counts), 5, log_scale_mean=-1.0, log_scale_std=0.1, opacity_range=(0.004, 0.01))
    so = np.concatenate([[0], np.cumsum(counts)])
    cams = vi.orbit_cameras(2, tile, tile, azimuth0=0.4)
    P = to_dev(gs)
    rp = api.plan_batch(cams, so, [0, 1], tile=tile, pair_capacity=capacity)
    out = api.render_fwd(rp, P)
    lists = rp.region("ranges", torch.int32).cpu().numpy().reshape(-1, 2)
    lists = lists[:, 1] - lists[:, 0]
    assert int(out.status[0]) == 0 and lists[0] >= 2040 and lists[1] >= lists[0] + 1000
    assert int(rp.region("counters", torch.int32)[8]) == lists.max()
    batch = render.Batch(gs, cams, tile, [0, 1], so)
    ref = render.render_forward(batch)
    for v, got in enumerate(api.split_views(out.image, cams)):
        assert image_error(got.cpu().numpy(), ref[v]["image"], ref[v]["flagged"]) <= IMG_TOL
    dL = masked_dL(cams, [r["flagged"] for r in ref], seed=tile)
    g_ref, _ = render.render_backward(batch, dL)
    G = api.render_bwd(rp, P, flat(dL), out).cpu().numpy()
    for name, rows in ROWS.items():
        assert group_error(G[rows], g_ref[name].reshape(rows.stop - rows.start, -1)) <= GRAD_TOL, name


# The levels that the small tile takes: sides of one and of several of its four rows, with a remainder or none, and of
# one and two outputs per block along z (30 to 36: one, 46 and 64: two).
@pytest.mark.parametrize("G,J,with_tf,offset", [(10, 1, True, 0), (30, 1, False, 1), (36, 2, True, 1), (46, 1, True, 0),
                                                (64, 1, False, 0)])
def test_dwt_small_levels(G, J, with_tf, offset):
    test_dwt_tile_edges(G, J, "bior4.4", with_tf, offset)


# The lists that four waves share in the backward: some of an uneven batch's (a view with a dense middle), none of a batch
# whose longest list is a small share of its pairs and that has many of that length.  Either way the gradient is that of
# the views alone.
@pytest.mark.parametrize("n,views,W,H,log_scale,shared",
                         [(1500, 2, 480, 360, -2.2, True), (300, 6, 480, 320, -1.0, False)])
def test_backward_shares_lists_of_uneven_batches(n, views, W, H, log_scale, shared):
    api = _api()
    say(f"shared lists n={n} {views} views {W}x{H} log scale {log_scale}")
    gs = vi.random_gaussians(n, 41 + n, log_scale_mean=log_scale, opacity_range=(0.02, 0.3))
    cams = vi.orbit_cameras(views, W, H)
    P = to_dev(gs)
    dL = torch.from_numpy(np.random.default_rng(n).normal(size=views * 3 * W * H).astype(np.float32)).to(dev())

    def grad(batch, dl, tile):
        rp = api.plan_batch(batch, [0, n], tile=tile, pair_capacity=1 << 22)
        out = api.render_fwd(rp, P)
        lists = rp.region("ranges", torch.int32).cpu().numpy().reshape(-1, 2)
        lists = lists[:, 1] - lists[:, 0]
        split, longest = rp.region("counters", torch.int32)[7:9].tolist()
        assert longest == lists.max()
        many = np.count_nonzero(lists >> 3 >= max(16, lists.sum() // 2048) >> 3)
        if tile == 16:
            assert split == (many if many <= 256 or longest >= lists.sum() // 700 else 0)
        return split, api.render_bwd(rp, P, dl.contiguous(), out).cpu().numpy().astype(np.float64)

    split, G = grad(cams, dL, 16)
    assert (split > 256) == shared and (split == 0) == (not shared)
    ref = sum(grad(cams[v:v + 1], dL[3 * W * H * v:3 * W * H * (v + 1)], 32)[1] for v in range(views))
    for name, rows in ROWS.items():
        assert group_error(G[rows], ref[rows]) <= GRAD_TOL, name


def test_walks_leave_the_same_transmittance():
    """Pixels that stop go back to the transmittance before the entry that stopped them; the walks of 8x8, shared 16x16
    and 32x32 tiles leave the same value and image bit for bit (opacities up to 0.34: the tilings list the same)."""
    api = _api()
    say("walks leave the same transmittance")
    gs = vi.random_gaussians(20000, 5, log_scale_mean=-2.6, opacity_range=(0.05, 0.34))
    cams = vi.orbit_cameras(2, 131, 77)
    P = to_dev(gs)
    outs = [api.render_fwd(api.plan_batch(cams, [0, gs.n], tile=t, pair_capacity=1 << 19), P) for t in (8, 16, 32)]
    assert int((outs[0].final_T < 1.2e-4).sum()) > 1000      # many have stopped
    for o in outs[1:]:
        assert torch.equal(o.final_T, outs[0].final_T) and torch.equal(o.image, outs[0].image)
