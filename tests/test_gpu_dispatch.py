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


@pytest.mark.parametrize("n", [1, 700, 4096])
def test_one_workgroup_binning_up_to_11264_tiles(gpu, n):
    """A view of 11,200 tiles is binned by one workgroup, one of 11,300 by the four passes; the
    second is the first with one more column of tiles to the right of every point, so the common
    texels and the gradients are the same, bit for bit."""
    import torch
    sc = scenes.random_small(110 + n, n=n, W=1792, H=1600, nlayers=1, s_lo=0.3, s_hi=3.0)
    t = to_device(sc["points"], gpu)
    args = [t[k] for k in PARAMS]
    cam = dict(sc["cams"][0])
    px = args[0] / args[2] * float(cam["fx"]) + float(cam["cx"])
    args[0] = torch.where(px < 1780.0, args[0], -args[0]).contiguous()
    G = torch.from_numpy(scenes.upstream_gradient(111, 1808 * 1600 * 4)).to(gpu).view(1600, 1808, 4)
    got = []
    for W in (1792, 1808):
        r = renderer(sc, gpu, cams=[dict(cam, W=W)])
        res = []
        lt = _launches(lambda: res.append(r.forward(*args)))
        assert r.stats()["bins"] == W // 16 * 100
        assert (lt["front"], lt["count"]) == ((1, 0) if W == 1792 else (0, 1))
        assert r.stats()["visible"] > 0
        g = r.backward(*args, G[:, :W].contiguous().view(-1))
        got.append([res[0].view(1600, W, 4)[:, :1792]] + g)
    for a, b in zip(*got):
        assert torch.equal(a, b)
    assert float(got[0][0].abs().max()) > 0


def test_small_calls_while_another_thread_captures(gpu):
    """A call of a few points on the null stream, which asks whether its stream is being captured,
    is accepted while another thread captures a stream of its own, as a larger call is."""
    import ctypes
    import threading

    import torch
    sc = scenes.random_small(120, n=300, W=61, H=45, nlayers=4)
    big = scenes.random_small(121, n=30000, W=61, H=45, nlayers=4)
    calls = []
    for s in (sc, big):
        r = renderer(s, gpu)
        t = to_device(s["points"], gpu)
        args = [t[k] for k in PARAMS]
        out = r.forward(*args)
        G = torch.ones_like(out)
        want = [out.clone()] + [g.clone() for g in r.backward(*args, G)]
        outs = [torch.empty_like(g) for g in want[1:]]
        calls.append((r, args, out, G, outs, want))
    torch.cuda.synchronize()
    assert torch.cuda.current_stream().cuda_stream == 0
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    stream, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(stream)) == 0
    begun, finish, codes = threading.Event(), threading.Event(), []

    def capture():
        codes.append(hip.hipStreamBeginCapture(stream, 1))  # hipStreamCaptureModeThreadLocal
        begun.set()
        finish.wait(30)
        codes.append(hip.hipStreamEndCapture(stream, ctypes.byref(graph)))

    th = threading.Thread(target=capture)
    th.start()
    assert begun.wait(30)
    try:
        for r, args, out, G, outs, want in calls:
            r.forward(*args, out=out)
            r.backward(*args, G, outs=outs)
    finally:
        finish.set()
        th.join()
    torch.cuda.synchronize()
    assert codes == [0, 0]
    assert hip.hipGraphDestroy(graph) == 0 and hip.hipStreamDestroy(stream) == 0
    for r, args, out, G, outs, want in calls:
        for a, b in zip([out] + outs, want):
            assert torch.equal(a, b)
