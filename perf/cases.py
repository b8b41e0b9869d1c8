"""Workloads of the point renderer and the reconstruction network, through the public entry
points of `paper_2401_06003_amd`, with seeded synthetic inputs.

`listed()` names the workloads, `draw()` gives further ones of the same ranges, `prepare()`
makes what a program holds before the call, `run()` is one pass, `work()` counts the bytes and
operations a pass cannot do without, and `exact()` evaluates the same outputs in 64 bits with
plain torch.

A render case is a dict with
  op       "forward" (a view is rendered), "train" (forward and backward calls), "autograd"
           (render() and a mean squared error through torch.autograd) or "plan" (a captured
           forward + backward, replayed)
  scene    "cube" (points uniform in a cube in front of one camera), "clusters" (anisotropic
           clusters and planar patches, one camera), "orbit" (the clusters with fixed world
           sizes, cameras of mixed resolutions and distances) or "ring" (cameras on a circle)
  points, width, height, layers, channels, views
  order    "shuffled" (no order in the point index) or "morton" (a spatially coherent cloud)
  extras   background, coverage and their gradients and the camera gradient as well
  coarser  coarser-layer inclusion
A decoder case has op "decode" and width, height, layers, channels, outputs.
"""
import math

import torch

import paper_2401_06003_amd as tp

KEEP = 16
EPS = 0.25
ZNEAR = 0.01
FEATURES = 32
RESOLUTIONS = [(640, 480), (800, 600), (1024, 768), (1280, 720), (1600, 900), (1920, 1080)]


def _render(name, op, scene, points, width, height, layers, channels=4, views=1,
            order="shuffled", extras=False, coarser=False):
    return {"name": name, "op": op, "scene": scene, "points": points, "width": width,
            "height": height, "layers": layers, "channels": channels, "views": views,
            "order": order, "extras": extras, "coarser": coarser}


def _decode(name, width, height, layers, channels, outputs):
    return {"name": name, "op": "decode", "width": width, "height": height, "layers": layers,
            "channels": channels, "outputs": outputs}


def listed():
    return [
        # a thumbnail of a few points: the smallest call, nothing but latency
        _render("thumb_forward", "forward", "cube", 300, 97, 61, 4),
        # a first optimisation on a toy scene (the size that is checked against a CPU)
        _render("cube_train", "train", "cube", 4096, 256, 256, 5),
        # the same size as a captured graph: the inner loop of a program that cannot afford
        # host calls
        _render("cube_plan", "plan", "cube", 4096, 256, 256, 5),
        # one training step of a scene with every optional term, at a size no tile divides
        _render("ragged_extras_train", "train", "clusters", 350001, 1237, 823, 7, channels=8,
                extras=True),
        # the step of the headline scene
        _render("clusters2m_train", "train", "clusters", 2000000, 1920, 1080, 8),
        # showing a reconstruction in scan order over an environment: forward alone
        _render("scan2m_forward", "forward", "clusters", 2000000, 1920, 1080, 8, order="morton",
                extras=True),
        # a dense cloud at the same resolution
        _render("clusters8m_train", "train", "clusters", 8000000, 1920, 1080, 8),
        # the step with coarser layers taking part in the blending
        _render("coarser2m_train", "train", "clusters", 2000000, 1920, 1080, 8, coarser=True),
        # a batch of camera views of different sizes in one call
        _render("orbit16_train", "train", "orbit", 4000000, 1920, 1080, 8, views=16),
        # an iteration of a whole optimisation: eight large views, wide descriptors, a loss
        # and its gradients through autograd
        _render("ring8_autograd", "autograd", "ring", 8000000, 2560, 1440, 8, channels=8,
                views=8),
        # the image of a frame from its pyramid, and of a small odd one with wide descriptors
        _decode("decode_1080p", 1920, 1080, 8, 4, 3),
        _decode("decode_ragged", 643, 477, 5, 8, 3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.2:
        width = _log_int(rng, 32, 2560)
        return {"op": "decode", "width": width,
                "height": max(16, min(1440, int(width * rng.uniform(0.5, 1.0)))),
                "layers": rng.randint(1, 9), "channels": rng.choice([4, 8]),
                "outputs": rng.choice([3, 3, 3, 1, 4, 8])}
    width = _log_int(rng, 48, 2560)
    height = max(32, min(1440, int(width * rng.uniform(0.5, 1.0))))
    scene = rng.choice(["cube", "clusters", "clusters", "orbit", "ring"])
    views = rng.randint(2, 6) if scene in ("orbit", "ring") else 1
    coarser = views == 1 and rng.random() < 0.2
    # between one point in 256 pixels of a view and 8 points per pixel, and no more work than
    # the largest listed cases
    least = max(64, width * height // 256)
    most = min(8 * width * height, 2000000 if coarser or views > 1 else 8000000)
    points = _log_int(rng, least, most)
    case = _render("", rng.choice(["forward", "train", "train", "autograd", "plan"]), scene,
                   points, width, height, rng.randint(1, 9), rng.choice([4, 4, 8]), views,
                   rng.choice(["shuffled", "morton"]), rng.random() < 0.3, coarser)
    del case["name"]
    if case["op"] == "autograd":
        case["extras"] = False  # render() takes the points alone
    return case


# -------------------------------------------------------------------------------------
# Inputs (made from the seed alone)

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _camera(R, t, width, height):
    f = (width / 2.0) / math.tan(math.radians(60.0) / 2.0)
    f32 = torch.float32
    return {"R": torch.tensor(R, dtype=f32).reshape(9).tolist(),
            "t": torch.tensor(t, dtype=f32).tolist(),
            "fx": torch.tensor(f, dtype=f32).item(), "fy": torch.tensor(f, dtype=f32).item(),
            "cx": width / 2.0, "cy": height / 2.0, "W": width, "H": height,
            "znear": torch.tensor(ZNEAR, dtype=f32).item()}


def _look_at(eye, target, width, height):
    eye = torch.tensor(eye, dtype=torch.float64)
    fwd = torch.tensor(target, dtype=torch.float64) - eye
    fwd = fwd / fwd.norm()
    up = torch.tensor([0.0, -1.0, 0.0], dtype=torch.float64)
    if abs(float(up @ fwd)) > 0.99:
        up = torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64)
    right = torch.linalg.cross(up, fwd)
    right = right / right.norm()
    R = torch.stack([right, torch.linalg.cross(fwd, right), fwd])
    return _camera(R.reshape(9).tolist(), (-R @ eye).tolist(), width, height)


def _clusters(gen, cpu_gen, n, dev, plane_frac, clusters=64, planes=8):
    """Points of anisotropic Gaussian clusters and of random planar patches, shuffled, and the
    cluster centres."""
    f64 = torch.float64
    n_plane = int(round(n * plane_frac))
    n_clu = n - n_plane
    centres = torch.rand(clusters, 3, generator=cpu_gen, dtype=f64) * 2 - 1
    rots = torch.linalg.qr(torch.randn(clusters, 3, 3, generator=cpu_gen, dtype=f64))[0]
    sig = torch.exp(math.log(0.01) + torch.rand(clusters, 3, generator=cpu_gen, dtype=f64) *
                    math.log(0.2 / 0.01))
    axes = (rots * sig[:, None, :]).float().to(dev)  # columns scaled by the axis lengths
    cid = torch.randint(clusters, (n_clu,), generator=gen, device=dev)
    g = torch.randn(n_clu, 3, generator=gen, device=dev)
    xyz = centres.float().to(dev)[cid]
    for j in range(3):
        xyz = xyz + axes[:, :, j][cid] * g[:, j:j + 1]
    if n_plane:
        pc = torch.rand(planes, 3, generator=cpu_gen, dtype=f64) * 2 - 1
        nrm = torch.randn(planes, 3, generator=cpu_gen, dtype=f64)
        nrm = nrm / nrm.norm(dim=1, keepdim=True)
        e1 = torch.linalg.cross(nrm, torch.randn(planes, 3, generator=cpu_gen, dtype=f64))
        e1 = e1 / e1.norm(dim=1, keepdim=True)
        e2 = torch.linalg.cross(nrm, e1)
        side = 0.5 + 1.5 * torch.rand(planes, 1, generator=cpu_gen, dtype=f64)
        pid = torch.randint(planes, (n_plane,), generator=gen, device=dev)
        a = torch.rand(n_plane, 2, generator=gen, device=dev) - 0.5
        xyz_p = (pc.float().to(dev)[pid] + a[:, :1] * (side * e1).float().to(dev)[pid] +
                 a[:, 1:] * (side * e2).float().to(dev)[pid])
        xyz = torch.cat([xyz, xyz_p])
    return xyz[torch.randperm(n, generator=gen, device=dev)], centres


def _morton(xyz, bits=10):
    """The permutation that puts points along a Z-order curve."""
    lo, hi = xyz.min(dim=0)[0], xyz.max(dim=0)[0]
    q = ((xyz - lo) / (hi - lo).clamp_min(1e-30) * ((1 << bits) - 1)).long()
    code = torch.zeros(len(xyz), dtype=torch.int64, device=xyz.device)
    for b in range(bits):
        for a in range(3):
            code |= ((q[:, a] >> b) & 1) << (3 * b + a)
    return torch.sort(code, stable=True)[1]


def _pyramid_texels(width, height, layers):
    return sum((-(-width // (1 << L))) * (-(-height // (1 << L))) for L in range(layers))


def _scene(case, seed):
    """(points x, y, z, sw, alpha, desc; cameras; background; upstream gradients)."""
    dev = _device()
    gen = torch.Generator(device=dev).manual_seed(seed)
    cpu_gen = torch.Generator().manual_seed(seed)
    n, D, W, H = case["points"], case["channels"], case["width"], case["height"]
    centres = None
    if case["scene"] == "cube":
        xyz = torch.rand(n, 3, generator=gen, device=dev) - 0.5
        cams = [_camera([1, 0, 0, 0, 1, 0, 0, 0, 1], [0, 0, 2.5], W, H)]
        s_hi, alpha_lo = 32.0, 0.2
    else:
        xyz, centres = _clusters(gen, cpu_gen, n, dev,
                                 0.0 if case["scene"] == "orbit" else 0.3)
        cams = [_camera([1, 0, 0, 0, 1, 0, 0, 0, 1], [0, 0, 3.0], W, H)]
        s_hi, alpha_lo = 128.0, 0.1
    if case["scene"] == "orbit":
        cams = []
        for v in range(case["views"]):
            # resolutions in turn, none larger than the case's own; directions spread over the
            # sphere; distances from near (few large splats) to far (all points small)
            w, h = RESOLUTIONS[v % len(RESOLUTIONS)]
            w, h = (w, h) if w <= W and h <= H else (W, H)
            cz = 1.0 - 2.0 * (v + 0.5) / case["views"]
            az = v * math.pi * (3.0 - math.sqrt(5.0))
            r = math.sqrt(1.0 - cz * cz)
            dist = 1.2 * (8.0 / 1.2) ** (((v * 7) % case["views"]) / max(case["views"] - 1, 1))
            target = centres[int(torch.randint(len(centres), (1,), generator=cpu_gen))].tolist()
            eye = [target[0] + dist * r * math.cos(az), target[1] + dist * cz,
                   target[2] + dist * r * math.sin(az)]
            cams.append(_look_at(eye, target, w, h))
    elif case["scene"] == "ring":
        el = math.radians(15.0)
        cams = []
        for v in range(case["views"]):
            az = 2.0 * math.pi * v / case["views"]
            cams.append(_look_at([3.0 * math.cos(el) * math.sin(az), -3.0 * math.sin(el),
                                  -3.0 * math.cos(el) * math.cos(az)], [0.0, 0.0, 0.0], W, H))
    if case["order"] == "morton":
        xyz = xyz[_morton(xyz)]
    u = torch.rand(n, generator=gen, device=dev)
    if case["scene"] == "orbit":
        sw = 0.002 * torch.exp(u * math.log(0.05 / 0.002))
    else:
        s = 0.5 * torch.exp(u * math.log(s_hi / 0.5))
        depth = 3.0 if case["scene"] == "ring" else xyz[:, 2] + cams[0]["t"][2]
        sw = s * depth / cams[0]["fx"]
    alpha = alpha_lo + (1.0 - alpha_lo) * torch.rand(n, generator=gen, device=dev)
    desc = torch.rand(n, D, generator=gen, device=dev)
    x, y, z = (xyz[:, k].contiguous() for k in range(3))
    texels = sum(_pyramid_texels(c["W"], c["H"], case["layers"]) for c in cams)
    up = torch.randn(texels * D, generator=gen, device=dev)  # gradient, or the loss's target
    bg = ga = None
    if case["extras"]:
        bg = torch.rand(texels * D, generator=gen, device=dev)
        ga = torch.randn(texels, generator=gen, device=dev)
    if case["op"] == "autograd":
        up = torch.rand(texels * D, generator=gen, device=dev)
    return (x, y, z, sw.contiguous(), alpha, desc), cams, bg, up, ga


def _decoder_inputs(case, seed):
    """(weights as Decoder takes them, flat pyramid): normal kernels scaled by their fan-in,
    features in [0, 1] with a fifth of the texels empty."""
    dev = _device()
    gen = torch.Generator(device=dev).manual_seed(seed)
    D, nl = case["channels"], case["layers"]
    w, b = [], []
    for L in range(nl):
        cin = D if L == nl - 1 else D + FEATURES
        k = torch.randn(3, 3, cin, 2 * FEATURES, generator=gen, device=dev)
        w.append((k / math.sqrt(9.0 * cin)).half())
        b.append(0.1 * torch.randn(2 * FEATURES, generator=gen, device=dev))
    wo = torch.randn(FEATURES, case["outputs"], generator=gen, device=dev) / math.sqrt(FEATURES)
    bo = 0.1 * torch.randn(case["outputs"], generator=gen, device=dev)
    texels = _pyramid_texels(case["width"], case["height"], nl)
    pyr = torch.rand(texels, D, generator=gen, device=dev)
    pyr *= (torch.rand(texels, 1, generator=gen, device=dev) >= 0.2).float()
    return {"w": w, "b": b, "wo": wo, "bo": bo}, pyr.reshape(-1)


# -------------------------------------------------------------------------------------
# The calls

def prepare(case, seed):
    if case["op"] == "decode":
        weights, pyr = _decoder_inputs(case, seed)
        dec = tp.Decoder(case["width"], case["height"], case["layers"], case["channels"],
                         weights)
        return {"case": case, "decoder": dec, "pyramid": pyr}
    points, cams, bg, up, ga = _scene(case, seed)
    r = tp.Renderer(cams, case["layers"], case["channels"], case["points"], EPS,
                    device=points[0].device, include_coarser=case["coarser"])
    st = {"case": case, "renderer": r, "points": points, "up": up, "bg": bg, "ga": ga}
    new = points[0].new_empty
    if case["extras"]:
        st["alpha"] = new(r.texels)
        st["gbg"] = new(r.texels * r.D)
        st["gcam"] = new(r.V, 16)
    if case["op"] == "autograd":
        st["points"] = tuple(p.requires_grad_(True) for p in points)
    if case["op"] == "plan":
        st["pyramid"] = new(r.texels * r.D)
        st["grads"] = [new(r.n) for _ in range(5)] + [new(r.n, r.D)]
        extras = {}
        if case["extras"]:
            extras = {"background": bg, "alpha_out": st["alpha"], "grad_alpha": ga,
                      "grad_background": st["gbg"], "grad_camera": st["gcam"]}
        st["plan"] = tp.Plan(r, *points, st["pyramid"], up, st["grads"], **extras)
    return st


def run(state):
    case = state["case"]
    if case["op"] == "decode":
        return state["decoder"].forward(state["pyramid"])
    r, points = state["renderer"], state["points"]
    if case["op"] == "forward":
        out = r.forward(*points, background=state["bg"], alpha_out=state.get("alpha"))
        return [out, state["alpha"]] if case["extras"] else [out]
    if case["op"] == "autograd":
        out = tp.render(*points, r)
        loss = torch.nn.functional.mse_loss(out, state["up"])
        return [out.detach()] + list(torch.autograd.grad(loss, points))
    if case["op"] == "plan":
        state["plan"].launch(forward=True, backward=True)
        out, grads = state["pyramid"], state["grads"]
    else:
        out = r.forward(*points, background=state["bg"], alpha_out=state.get("alpha"))
        grads = r.backward(*points, state["up"], background=state["bg"],
                           grad_alpha=state["ga"], grad_background=state.get("gbg"),
                           grad_camera=state.get("gcam"))
    if case["extras"]:
        return [out] + list(grads) + [state["alpha"], state["gbg"], state["gcam"]]
    return [out] + list(grads)


def _views(case):
    """(width, height) of every view."""
    W, H = case["width"], case["height"]
    if case["scene"] != "orbit":
        return [(W, H)] * case["views"]
    sizes = [RESOLUTIONS[v % len(RESOLUTIONS)] for v in range(case["views"])]
    return [(w, h) if w <= W and h <= H else (W, H) for w, h in sizes]


def work(case):
    D, nl = case["channels"], case["layers"]
    if case["op"] == "decode":
        W, H, out = case["width"], case["height"], case["outputs"]
        flops, weights = 2.0 * W * H * FEATURES * out, 4.0 * (FEATURES + 1) * out
        for L in range(nl):
            cin = D if L == nl - 1 else D + FEATURES
            flops += 2.0 * _pyramid_texels(-(-W // (1 << L)), -(-H // (1 << L)), 1) * 9 * cin * 64
            weights += 2.0 * 9 * cin * 64 + 4.0 * 64
        return {"bytes": 4.0 * _pyramid_texels(W, H, nl) * D + weights + 4.0 * W * H * out,
                "flops": flops}
    n, V = case["points"], case["views"]
    texels = sum(_pyramid_texels(w, h, nl) for w, h in _views(case))
    # points read, pyramid written; backward: gradient (or target) read, point gradients written
    b = 4.0 * n * (5 + D) + 4.0 * texels * D
    if case["extras"]:
        b += 4.0 * texels * (D + 1)
    back = case["op"] != "forward"
    if back:
        b += 4.0 * texels * D + 4.0 * n * (5 + D)
        if case["extras"]:
            b += 4.0 * texels * (D + 1) + 64.0 * V
    # projection and footprint of every point in every view, and the blend of about two
    # fragments per texel (each as often again in the backward)
    flops = (60.0 * n * V + 2.0 * texels * (2 * D + 8)) * (3 if back else 1)
    return {"bytes": b, "flops": flops}


# -------------------------------------------------------------------------------------
# The same outputs in 64 bits.  Which layer, texel and place in a list a fragment gets is
# decided in single precision, as the method states it; every weight, colour and gradient
# follows from there in double precision.

def _fma32(a, b, c):
    return (a.double() * b.double() + c.double()).float()


def _fragments(points, cam, nl):
    """All fragments of one view, sorted by (texel, depth, point index)."""
    x, y, z, sw, alpha, _ = points
    dev = x.device
    f32, f64 = torch.float32, torch.float64
    R = [torch.tensor(v, dtype=f32, device=dev) for v in cam["R"]]
    t = [torch.tensor(v, dtype=f32, device=dev) for v in cam["t"]]
    fx, fy, cx, cy = (torch.tensor(cam[k], dtype=f32, device=dev)
                      for k in ("fx", "fy", "cx", "cy"))
    Xc, Yc, Zc = (_fma32(R[3 * k], x, _fma32(R[3 * k + 1], y, _fma32(R[3 * k + 2], z, t[k])))
                  for k in range(3))
    qx = (Xc.double() / Zc.double()).float()
    qy = (Yc.double() / Zc.double()).float()
    sx, sy = _fma32(fx, qx, cx), _fma32(fy, qy, cy)
    s = ((fx * sw).double() / Zc.double()).float()
    ok = (Zc > cam["znear"]) & sx.isfinite() & sy.isfinite() & s.isfinite() & (s > 0)
    bits = s.view(torch.int32)
    e = (bits >> 23) - 127
    tm = ((bits & 0x7fffff) | (127 << 23)).view(f32)
    below, above = s < 1.0, s >= float(1 << (nl - 1))
    one = below | above | (tm == 1.0)
    L0 = torch.where(below, torch.zeros_like(e), torch.where(above, torch.full_like(e, nl - 1), e))
    s64, tm64 = s.double(), tm.double()
    io0 = torch.where(below, EPS + (1.0 - EPS) * s64,
                      torch.where(one, torch.ones_like(s64), 2.0 - tm64))
    dio0 = torch.where(below, torch.full_like(s64, 1.0 - EPS),
                       torch.where(one, torch.zeros_like(s64), -torch.exp2(-e.double())))
    zkey = Zc.view(torch.int32).long()
    dims = [(-(-cam["W"] // (1 << L)), -(-cam["H"] // (1 << L))) for L in range(nl)]
    offs = [0]
    for w, h in dims:
        offs.append(offs[-1] + w * h)
    parts = []
    for L in range(nl):
        for sel in range(2):
            pick = ok & (L0 + sel == L) & (~one if sel else torch.ones_like(one))
            p = pick.nonzero()[:, 0]
            if not len(p):
                continue
            W, H = dims[L]
            u = sx[p] * (2.0 ** -L) - 0.5
            v = sy[p] * (2.0 ** -L) - 0.5
            ins = (u > -1) & (u < W) & (v > -1) & (v < H)
            p, u, v = p[ins], u[ins], v[ins]
            fu, fv = u - u.floor(), v - v.floor()
            i0, j0 = u.floor().long(), v.floor().long()
            io = (tm64[p] - 1.0) if sel else io0[p]
            dio = torch.exp2(-e[p].double()) if sel else dio0[p]
            for c in range(4):
                di, dj = c & 1, c >> 1
                wx32, wy32 = (fu if di else 1.0 - fu), (fv if dj else 1.0 - fv)
                i, j = i0 + di, j0 + dj
                m = ((i >= 0) & (i < W) & (j >= 0) & (j < H) & (wx32 != 0) & (wy32 != 0))
                m = m.nonzero()[:, 0]
                wx = fu.double()[m] if di else 1.0 - fu.double()[m]
                wy = fv.double()[m] if dj else 1.0 - fv.double()[m]
                q = p[m]
                key = ((offs[L] + j[m] * W + i[m]) << 32) | zkey[q]
                parts.append((key, q, wx, wy, io[m], dio[m],
                              torch.full_like(wx, (2.0 if di else 0.0) - 1.0),
                              torch.full_like(wx, (2.0 if dj else 0.0) - 1.0),
                              torch.full_like(wx, 2.0 ** -L)))
    if not parts:
        zi, zf = torch.zeros(0, dtype=torch.int64, device=dev), torch.zeros(0, dtype=f64, device=dev)
        parts = [(zi, zi, zf, zf, zf, zf, zf, zf, zf)]
    key, q, wx, wy, io, dio, dx, dy, sc = (torch.cat(c) for c in zip(*parts))
    del parts
    o = torch.sort(q, stable=True)[1]  # by point index, then by (texel, depth)
    o = o[torch.sort(key[o], stable=True)[1]]
    f = {"key": key[o], "p": q[o], "wx": wx[o], "wy": wy[o], "io": io[o], "dio": dio[o],
         "dx": dx[o], "dy": dy[o], "sc": sc[o]}
    f["al"] = alpha.double()[f["p"]]
    f["gamma"] = f["wx"] * f["wy"] * f["io"] * f["al"]
    geo = {"Xc": Xc, "Yc": Yc, "Zc": Zc, "s": s}
    return f, geo, dims, offs


def _lists(f, P, dims, offs, coarser):
    """[P, 16] fragment numbers of every texel's blended list, -1 where it is shorter."""
    texel = f["key"] >> 32
    dev = texel.device
    start = torch.searchsorted(texel, torch.arange(P + 1, device=dev))
    rank = torch.arange(len(texel), device=dev) - start[texel]
    lists = torch.full((P, KEEP), -1, dtype=torch.int64, device=dev)
    kept = (rank < KEEP).nonzero()[:, 0]
    lists[texel[kept], rank[kept]] = kept
    if not coarser:
        return lists
    order = ((f["key"] & 0xffffffff) << 32) | f["p"]  # depth, then point index
    order = torch.cat([order, order.new_full((1,), 2 ** 63 - 1)])
    for L in range(len(dims) - 2, -1, -1):
        (W, H), Wc = dims[L], dims[L + 1][0]
        j, i = torch.meshgrid(torch.arange(H, device=dev) >> 1, torch.arange(W, device=dev) >> 1,
                              indexing="ij")
        up = lists[offs[L + 1] + (j * Wc + i).reshape(-1)]
        both = torch.cat([lists[offs[L]:offs[L + 1]], up], dim=1)  # own first on equal keys
        first = torch.sort(order[both], dim=1, stable=True)[1][:, :KEEP]
        lists[offs[L]:offs[L + 1]] = torch.gather(both, 1, first)
    return lists


def _exact_view(points, cam, nl, coarser, bg, up, ga, grads, gcam):
    """Pyramid, coverage, background gradient of one view; adds to the gradients.  up is the
    upstream gradient [P, D] or a function of the pyramid that gives it, or None."""
    f, geo, dims, offs = _fragments(points, cam, nl)
    P, D = offs[-1], points[5].shape[1]
    lists = _lists(f, P, dims, offs, coarser)
    f64 = torch.float64
    dev = lists.device
    desc = points[5].double()
    gamma = torch.cat([f["gamma"], f["gamma"].new_zeros(1)])  # (-1 reads the last, zero)
    pt = torch.cat([f["p"], f["p"].new_zeros(1)])
    C = torch.zeros(P, D, dtype=f64, device=dev)
    T = torch.ones(P, dtype=f64, device=dev)
    for m in range(KEEP):
        g = gamma[lists[:, m]]
        if len(desc):
            C += (T * g)[:, None] * desc[pt[lists[:, m]]]
        T = T * (1.0 - g)
    if bg is not None:
        C += T[:, None] * bg
    if up is None:
        return C, 1.0 - T, None
    G = up(C) if callable(up) else up
    gbg = T[:, None] * G
    # back to front: T_m by division would lose digits, so the fronts are kept
    fronts = torch.empty(P, KEEP, dtype=f64, device=dev)
    Tm = torch.ones(P, dtype=f64, device=dev)
    for m in range(KEEP):
        fronts[:, m] = Tm
        Tm = Tm * (1.0 - gamma[lists[:, m]])
    B = (G * bg).sum(1) if bg is not None else torch.zeros(P, dtype=f64, device=dev)
    dgam = torch.zeros(len(gamma), dtype=f64, device=dev)
    for m in range(KEEP - 1, -1, -1):
        k = lists[:, m]
        on = (k >= 0).nonzero()[:, 0]
        ko = k[on]
        g, p, To, Go = gamma[ko], pt[ko], fronts[on, m], G[on]
        gm = (Go * desc[p]).sum(1)
        if ga is not None:
            gm = gm + ga[on]
        dgam.index_add_(0, ko, To * (gm - B[on]))
        grads[5].index_add_(0, p, (To * g)[:, None] * Go)
        B[on] = g * gm + (1.0 - g) * B[on]
    del fronts, lists
    d, p = dgam[:-1], f["p"]
    n = len(points[0])

    def per_point(val):
        return torch.zeros(n, dtype=f64, device=dev).index_add_(0, p, val)

    grads[4] += per_point(d * f["wx"] * f["wy"] * f["io"])
    gs = per_point(d * f["wx"] * f["wy"] * f["al"] * f["dio"])
    gxs = per_point(d * f["dx"] * f["wy"] * f["io"] * f["al"] * f["sc"])
    gys = per_point(d * f["wx"] * f["dy"] * f["io"] * f["al"] * f["sc"])
    hit = per_point(torch.ones_like(d)) > 0
    one = torch.ones((), dtype=f64, device=dev)
    iz = torch.where(hit, 1.0 / geo["Zc"].double(), one)
    qx = torch.where(hit, geo["Xc"].double(), one) * iz
    qy = torch.where(hit, geo["Yc"].double(), one) * iz
    s = torch.where(hit, geo["s"].double(), one)
    dX, dY = gxs * cam["fx"] * iz, gys * cam["fy"] * iz
    dZ = -(gxs * cam["fx"] * qx + gys * cam["fy"] * qy + gs * s) * iz
    R = cam["R"]
    for k in range(3):
        grads[k] += R[k] * dX + R[3 + k] * dY + R[6 + k] * dZ
    grads[3] += gs * cam["fx"] * iz
    if gcam is not None:
        xyz = [c.double() for c in points[:3]]
        for a, dv in enumerate((dX, dY, dZ)):
            for k in range(3):
                gcam[3 * a + k] = (dv * xyz[k]).sum()
            gcam[9 + a] = dv.sum()
        gcam[12] = (gxs * qx + gs * points[3].double() * iz).sum()
        gcam[13] = (gys * qy).sum()
        gcam[14], gcam[15] = gxs.sum(), gys.sum()
    return C, 1.0 - T, gbg


def _exact_decoder(case, seed):
    weights, pyr = _decoder_inputs(case, seed)
    D, nl = case["channels"], case["layers"]
    dims = [(-(-case["width"] // (1 << L)), -(-case["height"] // (1 << L))) for L in range(nl)]
    offs = [0]
    for w, h in dims:
        offs.append(offs[-1] + w * h * D)
    out = None
    for L in range(nl - 1, -1, -1):
        W, H = dims[L]
        feat = pyr[offs[L]:offs[L + 1]].double().reshape(H, W, D)
        up = None
        if out is not None:
            up = out
            for axis, size in ((0, H), (1, W)):
                i = torch.arange(size, device=pyr.device)
                last = up.shape[axis] - 1
                near = (i >> 1).clamp(0, last)
                far = ((i >> 1) + (i & 1) * 2 - 1).clamp(0, last)
                up = 0.75 * up.index_select(axis, near) + 0.25 * up.index_select(axis, far)
            feat = torch.cat([feat, up], dim=2)
        pad = torch.nn.functional.pad(feat, (0, 0, 1, 1, 1, 1))
        k = weights["w"][L].double()
        acc = weights["b"][L].double().expand(H * W, -1).clone()
        for dy in range(3):
            for dx in range(3):
                acc += pad[dy:dy + H, dx:dx + W].reshape(H * W, -1) @ k[dy, dx]
        a, g = acc[:, :FEATURES], acc[:, FEATURES:]
        out = (torch.where(a > 0, a, torch.expm1(a)) * torch.sigmoid(g)).reshape(H, W, FEATURES)
        if up is not None:
            out = out + up
    return out @ weights["wo"].double() + weights["bo"].double()


def exact(case, seed):
    if case["op"] == "decode":
        return _exact_decoder(case, seed)
    points, cams, bg, up, ga = _scene(case, seed)
    D, nl, back = case["channels"], case["layers"], case["op"] != "forward"
    f64, dev = torch.float64, points[0].device
    grads = [torch.zeros_like(p, dtype=f64) for p in points]
    gcam = torch.zeros(len(cams), 16, dtype=f64, device=dev)
    sizes = [_pyramid_texels(c["W"], c["H"], nl) for c in cams]
    total = sum(sizes) * D
    outs, o = [], 0

    def part(a, width):
        return None if a is None else a[o * width:(o + sizes[v]) * width].double().reshape(
            (-1, D) if width == D else (-1,))

    for v, cam in enumerate(cams):
        upv = part(up, D) if back else None
        if case["op"] == "autograd":
            target = upv
            upv = lambda C, target=target: 2.0 * (C - target) / total
        outs.append(_exact_view(points, cam, nl, case["coarser"], part(bg, D), upv, part(ga, 1),
                                grads, gcam[v] if case["extras"] else None))
        o += sizes[v]
    pyr = torch.cat([c[0].reshape(-1) for c in outs])
    alpha = torch.cat([c[1] for c in outs])
    if not back:
        return [pyr, alpha] if case["extras"] else [pyr]
    res = [pyr] + grads
    if case["extras"]:
        res += [alpha, torch.cat([c[2].reshape(-1) for c in outs]), gcam]
    return res
