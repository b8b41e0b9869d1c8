"""What the renderer reads and writes of the buffers a caller hands it, on the GPU."""
import numpy as np
import pytest

import scenes
from gpu_util import PARAMS, renderer, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,nl,D,tile_w", [(61, 52, 5, 4, 16), (33, 17, 2, 8, 64),
                                             (130, 19, 8, 4, 8)])
def test_inclusion_ignores_what_the_buffers_held(gpu, W, H, nl, D, tile_w):
    """Tiles that reach beyond the layer (the last of every row and column here, the table's last
    tile among them): the words of texels outside it are never written, so a backward must not
    take them for list lengths.  0x1f bytes would be lengths of 31, beyond the 16 slots of a list;
    0xff bytes are NaNs in the workspace.  The gradients are those of cleared buffers, bit for
    bit."""
    import torch
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(80, n=3000, W=W, H=H, nlayers=nl, D=D, s_lo=0.5, s_hi=12.0)
    r = renderer(sc, gpu, tp.make_tuning(tile_w, 0, 0), include_coarser=True)
    t = to_device(sc["points"], gpu)
    args = [t[k] for k in PARAMS]
    G = torch.from_numpy(scenes.upstream_gradient(81, r.texels * D)).to(gpu)
    got = []
    for saved, work in ((0, 0), (0x1f, 0xff), (0xff, 0x1f)):
        r.saved.fill_(saved)
        r.workspace.fill_(work)
        pyr = r.forward(*args).clone()
        got.append([pyr] + [g.cpu() for g in r.backward(*args, G)])
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)
    assert all(float(np.abs(g.numpy()).max()) > 0 for g in got[0][1:])


@pytest.mark.parametrize("n,D,coarser", [(300, 4, False), (9000, 8, False), (5000, 4, True)])
def test_backward_leaves_saved_as_it_was(gpu, n, D, coarser):
    """`saved` is const to the backward: not a byte of it changes, and a second backward from it,
    into a workspace that held something else, gives the same gradients."""
    import torch
    sc = scenes.random_small(85, n=n, W=90, H=61, nlayers=5, D=D, s_lo=0.4, s_hi=12.0)
    r = renderer(sc, gpu, include_coarser=coarser)
    t = to_device(sc["points"], gpu)
    args = [t[k] for k in PARAMS]
    r.saved.zero_()
    r.forward(*args)
    before = r.saved.clone()
    G = torch.from_numpy(scenes.upstream_gradient(86, r.texels * D)).to(gpu)
    first = r.backward(*args, G)
    assert torch.equal(r.saved, before)
    r.workspace.fill_(0xff)
    for a, b in zip(first, r.backward(*args, G)):
        assert torch.equal(a, b)
    assert torch.equal(r.saved, before)
