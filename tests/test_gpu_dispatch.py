"""Which kernels a call takes, seen by the library's own stage times, and that calls on both sides
of a rule agree."""
import pytest

import scenes
from gpu_util import PARAMS, renderer, to_device

pytestmark = pytest.mark.gpu


def _launches(fn):
    """{stage: kernel launches} of fn()."""
    import torch
    import paper_2401_06003_amd as tp
    tp.timing_enable(True)
    try:
        fn()
        torch.cuda.synchronize()
        return {k: v[1] for k, v in tp.timing_read().items()}
    finally:
        tp.timing_enable(False)


def test_every_stage_is_some_kernel(gpu):
    """Binning of a few points by one workgroup is a stage of its own, not a scatter without its
    count and scans, and every stage of the table is recorded by some call."""
    import torch
    import paper_2401_06003_amd as tp
    sc = scenes.random_small(100, n=9000, W=61, H=45, nlayers=4)
    few = scenes.random_small(101, n=300, W=61, H=45, nlayers=4)

    def call(scene, **kw):
        r = renderer(scene, gpu, **kw)
        t = to_device(scene["points"], gpu)
        args = [t[k] for k in PARAMS]
        out = r.forward(*args)
        r.backward(*args, torch.ones_like(out))
        r.export_fragments()

    small = _launches(lambda: call(few))
    assert small["front"] == 1
    assert not any(small[k] for k in ("count", "colscan", "binscan", "scatter"))
    large = _launches(lambda: call(sc, tuning=tp.make_tuning(16, 0, 256)))
    assert large["front"] == 0
    assert all(large[k] == 1 for k in ("count", "colscan", "binscan", "scatter"))
    inclusion = _launches(lambda: call(sc, include_coarser=True))
    assert [k for k in small if not (small[k] or large[k] or inclusion[k])] == []
