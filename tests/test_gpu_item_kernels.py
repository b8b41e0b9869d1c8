"""The item kernels of the forward give the same texels.  Calls of few (point, view) pairs select
a tile's lists by counting (k_fwd_select), larger ones sort in rounds (k_fwd_items): every
small scene here is rendered twice, alone and followed by points behind the camera that raise the
count, so the same lists come from both.  Against each other bit for bit, and the larger call
against the oracle with the tolerances of gpu_util."""
import numpy as np
import pytest

import scenes
from gpu_util import GRAD_KEY, PARAMS, assert_lists, assert_pyramid, grad_close, to_device
from oracle import oracle

pytestmark = pytest.mark.gpu

BEHIND = 1500000
ALPHA_ATOL = 1e-5  # as in the coarser-layer tests


def _with_points_behind(pts, D):
    """`pts` followed by points that no camera at the origin looking along +z sees: they write
    nothing, and the indices of the others (ties in depth go by index) stay."""
    out = {}
    for k in PARAMS:
        v = np.asarray(pts[k], dtype=np.float32)
        tail = (BEHIND, D) if k == "desc" else (BEHIND,)
        fill = {"z": -1.0, "sw": 0.01, "alpha": 0.5}.get(k, 0.0)
        out[k] = np.concatenate([v, np.full(tail, fill, dtype=np.float32)])
    return out


def _render(points, sc, dev, tuning, coarser, bg, G, Ga):
    import torch
    import paper_2401_06003_amd as tp
    cam, nl, D = sc["cams"][0], sc["nlayers"], sc["D"]
    n = len(points["x"])
    r = tp.Renderer([cam], nl, D, n, tuning=tuning, device=dev, include_coarser=coarser)
    t = to_device(points, dev)
    args = [t[k] for k in PARAMS]
    alpha = torch.empty(r.texels, device=dev)
    gbg = torch.empty(r.texels * D, device=dev)
    pyr = r.forward(*args, background=bg, alpha_out=alpha)
    counts, ids = r.export_fragments()
    outs = r.backward(*args, G, background=bg, grad_alpha=Ga, grad_background=gbg)
    torch.cuda.synchronize()
    most = int(r.tile_stats()[0].max())
    res = {"pyr": pyr, "coverage": alpha, "counts": counts, "ids": ids, "gbg": gbg}
    res.update(zip(PARAMS, outs))
    return {k: v.cpu().numpy() for k, v in res.items()}, most


@pytest.mark.parametrize("seed,n,W,H,nl,D,tile_w,item,ties,coarser", [
    (90, 6000, 61, 45, 4, 4, 16, 0, False, False),      # whole tiles of thousands of entries
    (91, 6000, 61, 45, 4, 8, 16, 300, False, False),    # tiles cut into many items
    (92, 5000, 45, 37, 4, 4, 16, 0, True, False),       # four depths for all points
    (93, 5000, 45, 37, 4, 8, 8, 300, True, False),      # ... across items, 8x32 tiles
    (94, 6000, 150, 33, 5, 4, 64, 700, False, False),   # 64x4 tiles
    (95, 12000, 16, 16, 1, 4, 16, 8192, True, False),   # one tile, a second item of few entries
    (96, 1100, 33, 17, 3, 8, 32, 256, False, False),    # items of the smallest size
    (97, 6000, 61, 52, 5, 4, 16, 300, False, True),     # coarser layers taking part
    (98, 5000, 45, 37, 4, 8, 8, 0, True, True)])
def test_both_item_kernels(gpu, seed, n, W, H, nl, D, tile_w, item, ties, coarser):
    import torch
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(seed, n=n, W=W, H=H, nlayers=nl, D=D, s_lo=0.4, s_hi=12.0,
                             depth_ties=ties)
    cam = sc["cams"][0]
    P = oracle.num_pixels(W, H, nl)
    rng = np.random.default_rng(seed)
    bg = rng.uniform(0.0, 1.0, (P, D)).astype(np.float32)
    G = scenes.upstream_gradient(seed, P * D).reshape(P, D).astype(np.float32)
    Ga = rng.standard_normal(P).astype(np.float32)
    dev = [torch.from_numpy(a.reshape(-1)).to(gpu) for a in (bg, G, Ga)]
    tuning = tp.make_tuning(tile_w, 0, item)
    few, most = _render(sc["points"], sc, gpu, tuning, coarser, *dev)
    many, most_many = _render(_with_points_behind(sc["points"], D), sc, gpu, tuning, coarser, *dev)
    assert most == most_many and most > 256  # (up to 256 entries another kernel renders the tile)
    if item:
        assert most > item
    for k in few:
        a, b = few[k], many[k]
        if k in PARAMS:
            assert not b[n:].any(), k
            b = b[:n]
        assert np.array_equal(a, b), k
    f = oracle.forward_ex(sc["points"], cam, nl, background=bg.astype(np.float64), coarser=coarser)
    assert_lists(many["counts"], many["ids"].astype(np.int64), f["counts"], f["ids"])
    assert_pyramid(many["pyr"].astype(np.float64).reshape(P, D), f["pyr"])
    assert np.abs(many["coverage"] - f["alpha"]).max() <= ALPHA_ATOL
    b = oracle.backward_ex(sc["points"], cam, nl, G.astype(np.float64),
                           background=bg.astype(np.float64), grad_alpha=Ga.astype(np.float64),
                           coarser=coarser)
    for k in PARAMS:
        g = many[k][:n].astype(np.float64)
        grad_close(g, b[GRAD_KEY[k]].reshape(g.shape), k)
