"""GPU parity where the tile kernels' selection can go wrong: equal depths inside and across the
16 kept fragments, lists at the sizes between which the kernels change, parts of a tile that
start inside a word of the kept bits; against the oracle with the tolerances of gpu_util."""
import numpy as np
import pytest

import scenes
from gpu_util import GRAD_KEY, PARAMS, assert_lists, assert_pyramid, grad_close, to_device
from oracle import oracle

pytestmark = pytest.mark.gpu


def _check(sc, dev, tuning=None, include_coarser=False, seed=0):
    """Lists, colours and gradients of one view; returns the renderer."""
    import torch
    import paper_2401_06003_amd as tp
    cam, nl, D = sc["cams"][0], sc["nlayers"], sc["D"]
    r = tp.Renderer([cam], nl, D, len(sc["points"]["x"]), tuning=tuning, device=dev,
                    include_coarser=include_coarser)
    t = to_device(sc["points"], dev)
    args = [t[k] for k in PARAMS]
    out = r.forward(*args)
    counts, ids = r.export_fragments()
    P = r.texels
    G = scenes.upstream_gradient(seed, P * D).reshape(P, D)
    outs = r.backward(*args, torch.from_numpy(G.reshape(-1)).to(dev))
    torch.cuda.synchronize()
    f = oracle.forward_ex(sc["points"], cam, nl, coarser=include_coarser)
    assert_lists(counts.cpu().numpy(), ids.cpu().numpy().astype(np.int64), f["counts"], f["ids"])
    assert_pyramid(out.cpu().numpy().astype(np.float64).reshape(P, D), f["pyr"])
    b = oracle.backward_ex(sc["points"], cam, nl, G.astype(np.float64), coarser=include_coarser)
    for k, o in zip(PARAMS, outs):
        g = o.cpu().numpy().astype(np.float64)
        grad_close(g, b[GRAD_KEY[k]].reshape(g.shape), k)
    return r


@pytest.mark.parametrize("D,coarser,item,n", [(4, False, 0, 4000), (8, False, 300, 4000),
                                              (4, True, 0, 1500), (4, False, 0, 700)])
def test_equal_depths_in_the_lists(gpu, D, coarser, item, n):
    """Four depths for all points: a texel's kept list holds equal depths, and the 16th kept
    fragment has the depth of fragments that are not kept."""
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(21, n=n, W=45, H=37, nlayers=4, D=D, s_lo=0.5, s_hi=14.0,
                             depth_ties=True)
    r = _check(sc, gpu, tp.make_tuning(16, 0, item), coarser)
    assert r.tile_stats()[0].max() > 256


@pytest.mark.parametrize("n,tile_w,item", [(1, 16, 0), (1023, 8, 256), (4095, 64, 0),
                                           (4096, 16, 300), (4097, 16, 300)])
def test_point_counts_around_the_single_workgroup_binning(gpu, n, tile_w, item):
    """Up to 4096 points in one view are binned by one workgroup, more by four passes: one point,
    a count no thread count divides, both sides of the limit, tiles cut into several items."""
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(30 + n % 7, n=n, W=150, H=99, nlayers=5, s_lo=0.3, s_hi=30.0)
    r = _check(sc, gpu, tp.make_tuning(tile_w, 256, item))
    st = r.stats()
    assert st["entries"] >= st["visible"]
    if n >= 4096:
        assert st["items"] > st["bins"]  # some tile has several items


@pytest.mark.parametrize("n,W,H,nl,item,ties", [
    (1500, 16, 16, 1, 0, False),     # one tile, more fragments than fit, hundreds per texel
    (1500, 16, 16, 1, 0, True),      # ... of four depths: bins divided down to single keys
    (20000, 24, 20, 2, 0, True),     # items of 8192 entries, thousands of equal depths per texel
    (20000, 70, 50, 3, 777, False),  # tiles of many items, partial lists merged
    (1300, 33, 17, 3, 0, False)])    # around the item size whose fragments all fit
def test_lists_selected_by_counting(gpu, n, W, H, nl, item, ties):
    """Items of a few hundred to thousands of entries, whose kept lists are selected by depth bins
    where their fragments do not fit in LDS."""
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(40, n=n, W=W, H=H, nlayers=nl, s_lo=0.4, s_hi=10.0, depth_ties=ties)
    r = _check(sc, gpu, tp.make_tuning(16, 0, item))
    assert r.tile_stats()[0].max() > 300


@pytest.mark.parametrize("n,D", [(3000, 4), (5000, 4), (5000, 8)])
def test_points_with_more_than_four_entries(gpu, n, D):
    """Tiles of 8 texels: one point in some forty crosses a tile corner in one of its layers and
    has five to eight entries; binned by one workgroup and by four passes."""
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(50, n=n, W=96, H=80, nlayers=4, D=D, s_lo=0.5, s_hi=8.0)
    _check(sc, gpu, tp.make_tuning(8, 0, 0))


@pytest.mark.parametrize("tile_w,nl,D,n", [(16, 3, 4, 8000), (64, 6, 4, 8000), (8, 7, 8, 8000),
                                           (16, 8, 4, 3000)])
def test_inclusion_with_long_own_lists(gpu, tile_w, nl, D, n):
    """Own lists of up to 16 fragments in the finer layers, merged with full covering lists; layer
    counts whose coarsest group has one layer, several, or as many as one launch takes."""
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(60, n=n, W=61, H=52, nlayers=nl, D=D, s_lo=0.5, s_hi=20.0)
    _check(sc, gpu, tp.make_tuning(tile_w, 0, 0), include_coarser=True)


@pytest.mark.parametrize("n,pb", [(30000, 16384), (40000, 32768), (66000, 65535)])
def test_large_point_blocks(gpu, n, pb):
    """Binning workgroups of more than 4096 points, a partly filled last one; tiles with tens of
    thousands of entries from one block."""
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(70, n=n, W=40, H=24, nlayers=3, s_lo=0.3, s_hi=6.0)
    _check(sc, gpu, tp.make_tuning(16, pb, 0))


def test_default_point_blocks_of_large_tables(gpu):
    """Eight 2560x1440 views of 1.2M points, whose default block is larger than 4096 points: the
    pyramid and the gradients are those of blocks of 4096."""
    import torch
    import paper_2401_06003_amd as tp
    n, V = 1200000, 8
    gen = torch.Generator(device=gpu).manual_seed(3)
    u = lambda lo, hi: lo + (hi - lo) * torch.rand(n, generator=gen, device=gpu)
    eye = [1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 1.0]
    cams = [{"R": eye, "t": [0.01 * v, 0.0, 3.0], "fx": 1500.0, "fy": 1500.0, "cx": 1280.0,
             "cy": 720.0, "W": 2560, "H": 1440, "znear": 0.01} for v in range(V)]
    args = [u(-1.5, 1.5), u(-1.0, 1.0), u(-0.5, 0.5), u(0.001, 0.01), u(0.1, 1.0),
            torch.rand(n, 4, generator=gen, device=gpu)]
    got = []
    for tuning in (None, tp.make_tuning(0, 4096, 0)):
        r = tp.Renderer(cams, 6, 4, n, tuning=tuning, device=gpu)
        out = r.forward(*args).clone()
        G = torch.linspace(-1.0, 1.0, out.numel(), device=gpu)
        got.append([out] + [g.clone() for g in r.backward(*args, G)])
        del r
    for a, b in zip(*got):
        assert torch.equal(a, b)


def _tile_entries(sc, tile_w):
    """Entries of every point that writes a fragment: the tiles of its fragments."""
    f = oracle.fragments(sc["points"], sc["cams"][0], sc["nlayers"])
    touched = np.unique(np.stack([f["idx"], f["L"], f["i"] // tile_w, f["j"] // (256 // tile_w)], 1),
                        axis=0)
    return np.bincount(touched[:, 0])


@pytest.mark.parametrize("n,D,tile_w", [(3000, 4, 8), (4096, 8, 16), (6000, 4, 16), (6000, 8, 8)])
def test_points_on_tile_corners(gpu, n, D, tile_w):
    """A third of the points within half a texel of a corner where four tiles of layer 0 and four
    of layer 1 meet, so that hundreds have five to eight entries and use the second table of entry
    positions; binned by one workgroup and by four passes.  (Random points do so only about once
    in 200: in test_points_with_more_than_four_entries four to seven of all.)"""
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(51, n=n, W=96, H=160, nlayers=4, D=D, s_lo=0.5, s_hi=8.0)
    cam, p = sc["cams"][0], sc["points"]
    rng = np.random.default_rng(52)
    m = n // 3
    step = (2 * tile_w, 512 // tile_w)  # corners common to layers 0 and 1
    for k, c, f, size, s in (("x", "cx", "fx", 96, step[0]), ("y", "cy", "fy", 160, step[1])):
        at = s * rng.integers(1, -(-size // s), m) + rng.uniform(-0.4, 0.4, m)
        p[k][:m] = (at - float(cam[c])) * p["z"][:m] / float(cam[f])
    per = _tile_entries(sc, tile_w)
    assert (per > 4).sum() > 100 and (per == 8).sum() > 50, ((per > 4).sum(), (per == 8).sum())
    _check(sc, gpu, tp.make_tuning(tile_w, 0, 0))


@pytest.mark.parametrize("item", [0, 256])
@pytest.mark.parametrize("n", [257, 1025])
def test_as_many_items_as_entries_allow(gpu, n, item):
    """Every point on a corner of four tiles in both of its layers: eight entries each, in eight
    tiles of n entries, so that (n = 257, items of 256) one item fewer than a launch provides for
    is in use."""
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(53, n=n, W=64, H=64, nlayers=3, s_lo=1.1, s_hi=1.9)
    cam, p = sc["cams"][0], sc["points"]
    rng = np.random.default_rng(54)
    for k, c, f in (("x", "cx", "fx"), ("y", "cy", "fy")):
        p[k][:] = (32.0 + rng.uniform(-0.4, 0.4, n) - float(cam[c])) * p["z"] / float(cam[f])
    assert (_tile_entries(sc, 16) == 8).all()
    r = _check(sc, gpu, tp.make_tuning(16, 0, item))
    assert (r.tile_stats()[0] == n).sum() == 8


@pytest.mark.parametrize("n,D,tile_w,item", [(150000, 4, 16, 256), (300000, 8, 8, 500),
                                             (200000, 4, 64, 300)])
def test_backward_of_joined_items(gpu, n, D, tile_w, item):
    """More small items than fit the chip at once: the backward takes those of a tile in runs, the
    last of them short; with a background gradient, which one run of a tile writes."""
    import torch
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(55, n=n, W=150, H=99, nlayers=4, D=D, s_lo=0.4, s_hi=14.0)
    cam, nl = sc["cams"][0], sc["nlayers"]
    t = to_device(sc["points"], gpu)
    args = [t[k] for k in PARAMS]
    got = []
    for it in (item, 65536):
        r = tp.Renderer([cam], nl, D, n, tuning=tp.make_tuning(tile_w, 0, it), device=gpu)
        P = r.texels
        rng = np.random.default_rng(56)
        bg = rng.uniform(0.0, 1.0, (P, D)).astype(np.float32)
        G = scenes.upstream_gradient(57, P * D).reshape(P, D).astype(np.float32)
        d_bg, d_G = (torch.from_numpy(a.reshape(-1)).to(gpu) for a in (bg, G))
        gbg = torch.zeros(P * D, device=gpu)
        r.forward(*args, background=d_bg)
        if it == item:
            assert r.stats()["items"] > r.stats()["bins"] + 512
        got.append(r.backward(*args, d_G, background=d_bg, grad_background=gbg) + [gbg])
    for a, b in zip(*got):  # whole tiles and cut ones
        assert torch.equal(a, b)
    want = oracle.backward_ex(sc["points"], cam, nl, G.astype(np.float64),
                              background=bg.astype(np.float64))
    for k, o in zip(PARAMS + ("bg",), got[0]):
        g = o.cpu().numpy().astype(np.float64)
        w = want["gbg"] if k == "bg" else want[GRAD_KEY[k]]
        grad_close(g, w.reshape(g.shape), k)
