"""The work that users of this package have it do, as measurable cases.

Every case is one call (or one round of calls) through the public entry points: ``Plan`` (one
frame pair per call on one stream), ``Batch`` (many pairs per call), and the serving loop over
host frames.  Frames are synthetic particle images (Gaussian spots on a dim background with
noise, moved by a shear layer and vortices), made on the GPU from the seed alone.
``exact`` evaluates the same method in 64-bit torch.
"""
from __future__ import annotations

import math

import torch

import paper_1306_2461_amd as ofmi
from paper_1306_2461_amd.serve import GpuExecutor, Server

# ------------------------------------------------------------------------------ the cases

# Sizes of the mixed batch and of the served streams (H, W), in the proportions of the
# benchmark's 64-pair batch and 8-stream run.
MIXED = [(512, 512), (768, 1024), (2048, 2048), (768, 1024)] * 6
STREAMS = [(480, 640), (1024, 1024), (2048, 2048), (480, 640), (1024, 1024), (480, 640), (1024, 1024), (2048, 2048)]


def _sizes(text):
    return [tuple(int(x) for x in s.split("x")) for s in text.split()]


def _text(sizes):
    return " ".join(f"{h}x{w}" for h, w in sizes)


def _case(kind, sizes, levels, radius, iters, **more):
    c = {"kind": kind, "sizes": _text(sizes), "levels": levels, "radius": radius, "iters": iters, "fp16": False,
         "f32": False, "gauss": False, "normalize": False, "mask": False}
    c.update(more)
    return c


def listed():
    cases = {
        # a single small pair: launches and latency decide
        "plan_256": _case("plan", [(256, 256)], 3, 4, 4),
        # the headline workload: one 1024x1024 camera pair after another on one stream
        "plan_1024": _case("plan", [(1024, 1024)], 4, 8, 4),
        # the same with the pyramid stored in FP16
        "plan_1024_fp16": _case("plan", [(1024, 1024)], 4, 8, 4, fp16=True),
        # the paper's 1792x384 region of interest, r = 10, frames equalised first
        "plan_roi_normalized": _case("plan", [(384, 1792)], 4, 10, 4, normalize=True),
        # an odd crop of float frames (already preprocessed by the caller), small window
        "plan_odd_f32": _case("plan", [(479, 637)], 3, 5, 3, f32=True),
        # a large camera
        "plan_2048": _case("plan", [(2048, 2048)], 4, 8, 4),
        # the Gaussian-weighted window option
        "plan_1024_gauss": _case("plan", [(1024, 1024)], 4, 8, 4, gauss=True),
        # an obstacle and side walls masked out
        "plan_1024_mask": _case("plan", [(1024, 1024)], 4, 8, 4, mask=True),
        # a batch of small, odd-sized regions (many regions of interest of one recording)
        "batch_small_odd": _case("batch", [(181, 243), (256, 256), (97, 310), (333, 200)] * 4, 3, 4, 4),
        # offline processing of a recording: many pairs of one camera per call
        "batch_16x1024": _case("batch", [(1024, 1024)] * 16, 4, 8, 4),
        # offline processing of recordings of several cameras, FP16 storage
        "batch_mixed_fp16": _case("batch", MIXED, 4, 8, 4, fp16=True),
        # eight live streams through the serving loop, frames in pinned host memory
        "serve_8": _case("serve", STREAMS, 4, 8, 4, fp16=True),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _levels_max(sizes):
    return int(math.log2(min(min(s) for s in sizes))) + 1


def draw(rng):
    def side(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["plan", "plan", "plan", "batch", "batch", "serve"])
    if kind == "plan":
        option = rng.choice(["", "", "fp16", "f32", "gauss", "normalize", "mask"])
        top = 1024 if option in ("gauss", "normalize") else 2048
        sizes = [(side(128, top), side(128, top))]
        radius, iters = rng.randint(2, 10), rng.randint(1, 6)
        more = {option: True} if option else {}
    elif kind == "batch":
        n = rng.randint(2, 24)
        top = 512 if n > 12 else 1024
        some = [(side(96, top), side(96, top)) for _ in range(rng.randint(1, 4))]
        sizes = [some[i % len(some)] for i in range(n)]
        radius, iters = rng.randint(2, 10), rng.randint(2, 5)
        more = {"fp16": rng.random() < 0.5, "mask": rng.random() < 0.2}
    else:
        sizes = [(side(240, 1100), side(240, 1100)) for _ in range(rng.randint(1, 8))]
        radius, iters = rng.choice([4, 8, 10]), rng.randint(2, 4)
        more = {"fp16": rng.random() < 0.7}
    levels = min(rng.randint(2, 4), _levels_max(sizes))
    return _case(kind, sizes, levels, radius, iters, **more)


# ------------------------------------------------------------------------------ inputs

def _device():
    return torch.device("cuda", torch.cuda.current_device())


def _gen(seed, item):
    g = torch.Generator(device=_device())
    g.manual_seed(int(seed) * 1009 + item)
    return g


def _field(H, W, g, dmax):
    """Displacement field of one pair: a shear layer and one vortex, at most `dmax` px."""
    r = torch.rand(5, generator=g, device=g.device, dtype=torch.float64)
    yc, cx, cy = (0.3 + 0.4 * r[0]) * H, (0.2 + 0.6 * r[1]) * W, (0.2 + 0.6 * r[2]) * H
    rc, shift = 0.05 * min(H, W) + 4.0, r[3:] - 0.5

    def f(x, y):
        su = 0.4 * dmax * (1.0 + torch.tanh((y - yc) / (0.04 * H + 2.0)))
        dx, dy = x - cx, y - cy
        q = (dx * dx + dy * dy) / (rc * rc)
        c = 0.15 * dmax * torch.exp(-q) / rc
        return 0.8 * su - c * dy + 0.1 * dmax * shift[0], c * dx + 0.1 * dmax * shift[1]

    return f


def _render(xp, yp, amp, H, W, sigma, g):
    """Particle frame (uint8): spots summed in integers, so the same seed gives the same bits."""
    R = int(math.ceil(4.0 * sigma))
    off = torch.arange(-R, R + 1, device=xp.device)
    img = torch.zeros(H * W, dtype=torch.int64, device=xp.device)
    for s in range(0, xp.numel(), 1 << 18):
        px, py, pa = xp[s:s + (1 << 18)], yp[s:s + (1 << 18)], amp[s:s + (1 << 18)]
        ix, iy = px.round().long()[:, None] + off, py.round().long()[:, None] + off
        gx = torch.exp(-(ix - px[:, None]) ** 2 / (2 * sigma * sigma)) * ((ix >= 0) & (ix < W))
        gy = torch.exp(-(iy - py[:, None]) ** 2 / (2 * sigma * sigma)) * ((iy >= 0) & (iy < H))
        val = (pa[:, None, None] * gy[:, :, None] * gx[:, None, :] * 65536.0).round().long()
        at = iy.clamp(0, H - 1)[:, :, None] * W + ix.clamp(0, W - 1)[:, None, :]
        img.index_add_(0, at.reshape(-1), val.reshape(-1))
    out = img.double() / 65536.0 + 10.0 + 3.0 * torch.randn(H * W, generator=g, device=xp.device, dtype=torch.float64)
    return out.clamp(0, 255).round().to(torch.uint8).reshape(H, W)


def _pair(H, W, levels, seed, item):
    g = _gen(seed, item)
    dmax = min(2.5 * 2 ** (levels - 1), 8.0)
    field = _field(H, W, g, dmax)
    sigma, rho, m = 1.2, 0.03, 14
    n = int(rho * (H + 2 * m) * (W + 2 * m))
    q = torch.rand(3, n, generator=g, device=g.device, dtype=torch.float64)
    xp, yp, amp = q[0] * (W + 2 * m) - m, q[1] * (H + 2 * m) - m, 150.0 + 105.0 * q[2]
    du, dv = field(xp, yp)
    return _render(xp, yp, amp, H, W, sigma, g), _render(xp + du, yp + dv, amp, H, W, sigma, g)


def _inputs(case, seed):
    """The pairs of a case as the caller holds them (device tensors)."""
    pairs = [_pair(h, w, case["levels"], seed, i) for i, (h, w) in enumerate(_sizes(case["sizes"]))]
    if case["f32"]:   # frames a caller has scaled already
        pairs = [((a.float() * 0.7310 - 11.3).contiguous(), (b.float() * 0.7310 - 11.3).contiguous()) for a, b in pairs]
    return pairs


def _mask(H, W):
    """Side walls and an obstacle (a disc) excluded: nonzero = compute."""
    y, x = torch.meshgrid(torch.arange(H, device=_device()), torch.arange(W, device=_device()), indexing="ij")
    m = (y >= H // 8) & (y < H - H // 8)
    m &= (x - W // 3) ** 2 + (y - H // 2) ** 2 > (min(H, W) // 6) ** 2
    return m.to(torch.uint8).contiguous()


def prepare(case, seed):
    sizes = _sizes(case["sizes"])
    pairs = _inputs(case, seed)
    p = (case["levels"], case["radius"], case["iters"])
    if case["kind"] == "plan":
        H, W = sizes[0]
        plan = ofmi.Plan(H, W, *p, fp16=case["fp16"], input_f32=case["f32"], normalize=case["normalize"],
                         gaussian_window=case["gauss"], device=_device())
        if case["mask"]:
            plan.set_mask(_mask(H, W))
        u = torch.empty((H, W), dtype=torch.float32, device=_device())
        return {"kind": "plan", "plan": plan, "pair": pairs[0], "out": (u, torch.empty_like(u))}
    if case["kind"] == "batch":
        b = ofmi.Batch(sizes, *p, fp16=case["fp16"], input_f32=case["f32"], gaussian_window=case["gauss"],
                       device=_device())
        if case["mask"]:
            b.set_masks([_mask(h, w) for h, w in sizes])
        us, vs = b.outputs()
        return {"kind": "batch", "batch": b, "I1": [a for a, _ in pairs], "I2": [c for _, c in pairs], "out": (us, vs)}
    srv = Server(GpuExecutor(*p, fp16=case["fp16"], device=_device()))
    host = [[f.cpu().pin_memory() for f in pair] for pair in pairs]
    for i, pair in enumerate(host):   # the streams are running: each has its previous frame
        srv.open_stream(i, tuple(pair[0].shape))
        srv.submit(i, pair[0])
    srv.drain()
    srv.done.clear()
    return {"kind": "serve", "server": srv, "host": host}


def run(state):
    if state["kind"] == "plan":
        return state["plan"].compute(*state["pair"], *state["out"])
    if state["kind"] == "batch":
        us, vs = state["batch"].compute(state["I1"], state["I2"], *state["out"])
        return {"u": us, "v": vs}
    # two frames per stream: forth to the second frame and back to the first
    srv, reqs = state["server"], []
    for k in (1, 0):
        for i, pair in enumerate(state["host"]):
            reqs.append(srv.submit(i, pair[k]))
        srv.step()
    srv.drain()
    srv.done.clear()
    return {"u": [r.u for r in reqs], "v": [r.v for r in reqs]}


# Arithmetic of one pixel and iteration: two coordinates split, three interpolations, two
# gradients, the temporal difference, five products, five two-way window sums as suffix plus
# prefix (3 additions per direction), the 2x2 solve.
_FLOPS = 4 + 9 + 4 + 5 + 5 + 30 + 30


def work(case):
    nbytes = flops = 0.0
    passes = 2 if case["kind"] == "serve" else 1
    for h, w in _sizes(case["sizes"]):
        px = h * w
        per = 4 if case["f32"] else 1
        frames = 1 if case["kind"] == "serve" else 2    # a served stream keeps its previous frame
        nbytes += passes * px * (frames * per + 8)
        level = sum(math.ceil(h / 2 ** k) * math.ceil(w / 2 ** k) for k in range(case["levels"]))
        taps = 2 * (2 * case["radius"] + 1) * 5 * 2 - 30 if case["gauss"] else 0
        flops += passes * (level * case["iters"] * (_FLOPS + taps) + frames * 18.0 * (level - px))
        if case["normalize"]:
            flops += 2 * 14.0 * px
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------------------ 64 bits

def _shift(a, d, dim):
    """a at index + d along dim, clamped to the edge."""
    n = a.shape[dim]
    i = (torch.arange(n, device=a.device) + d).clamp(0, n - 1)
    return a.index_select(dim, i)


def _reduce(a):
    for dim in (1, 0):
        a = (_shift(a, -2, dim) + _shift(a, 2, dim) + 4 * (_shift(a, -1, dim) + _shift(a, 1, dim)) + 6 * a) / 16
    return a[::2, ::2]


def _window(a, r, taps):
    """Window sum truncated at the border, separable, with the given taps."""
    for dim in (1, 0):
        n = a.shape[dim]
        z = torch.zeros_like(a.narrow(dim, 0, 1)).expand([r if k == dim else s for k, s in enumerate(a.shape)])
        p = torch.cat([z, a, z], dim)
        s = torch.zeros_like(a)
        for k, t in enumerate(taps):
            s = s + t * p.narrow(dim, k, n)
        a = s
    return a


def _bilinear(a, x, y):
    H, W = a.shape
    x, y = x.clamp(0, W - 1), y.clamp(0, H - 1)
    x0, y0 = x.floor(), y.floor()
    fx, fy = x - x0, y - y0
    x0, y0 = x0.long(), y0.long()
    x1, y1 = (x0 + 1).clamp(max=W - 1), (y0 + 1).clamp(max=H - 1)
    top = a[y0, x0] * (1 - fx) + a[y0, x1] * fx
    return top * (1 - fy) + (a[y1, x0] * (1 - fx) + a[y1, x1] * fx) * fy


def _equalised(a, r=5, eps=1.0):
    one = [1.0] * (2 * r + 1)
    n = _window(torch.ones_like(a), r, one)
    m = _window(a, r, one) / n
    var = _window(a * a, r, one) / n - m * m
    return (a - m) / (var.clamp(min=0).sqrt() + eps)


def _flow64(case, I1, I2, mask=None):
    L, r, K = case["levels"], case["radius"], case["iters"]
    P1, P2 = [I1.double()], [I2.double()]
    if case["normalize"]:
        P1, P2 = [_equalised(P1[0])], [_equalised(P2[0])]
    M = [None if mask is None else mask.bool()]
    for _ in range(1, L):
        for P in (P1, P2):
            c = _reduce(P[-1])
            P.append(c.half().double() if case["fp16"] else c)   # the storage the caller chose
        if M[-1] is None:
            M.append(None)
        else:
            m = M[-1] | _shift(M[-1], 1, 0)
            M.append((m | _shift(m, 1, 1))[::2, ::2])
    taps = [1.0] * (2 * r + 1)
    if case["gauss"] and r > 0:
        taps = [math.exp(-2.0 * d * d / (r * r)) for d in range(-r, r + 1)]
    u = v = None
    for l in range(L - 1, -1, -1):
        A1, A2 = P1[l], P2[l]
        H, W = A1.shape
        y, x = torch.meshgrid(torch.arange(H, device=A1.device, dtype=torch.float64),
                              torch.arange(W, device=A1.device, dtype=torch.float64), indexing="ij")
        if u is None:
            u, v = torch.zeros_like(A1), torch.zeros_like(A1)
        else:
            u, v = 2 * _bilinear(u, x / 2, y / 2), 2 * _bilinear(v, x / 2, y / 2)
        for _ in range(K):
            w = _bilinear(A2, x + u, y + v)
            ix = 0.5 * (_shift(w, 1, 1) - _shift(w, -1, 1))
            iy = 0.5 * (_shift(w, 1, 0) - _shift(w, -1, 0))
            it = w - A1 - ix * u - iy * v
            A, B, C, sx, sy = (_window(q, r, taps) for q in (ix * ix, ix * iy, iy * iy, ix * it, iy * it))
            bx, by = sx + A * u + B * v, sy + B * u + C * v
            T, D = A + C, A * C - B * B
            ok, some = D > 1e-5 * T * T, T > 0
            d, t = torch.where(ok, D, 1.0), torch.where(some, T * T, 1.0)
            du = torch.where(ok, -(C * bx - B * by) / d, torch.where(some, -(A * bx + B * by) / t, 0.0))
            dv = torch.where(ok, -(A * by - B * bx) / d, torch.where(some, -(B * bx + C * by) / t, 0.0))
            u, v = u + du, v + dv
            if M[l] is not None:
                u, v = u * M[l], v * M[l]
    return u, v


def exact(case, seed):
    pairs = _inputs(case, seed)
    flows = [_flow64(case, a, b, _mask(*a.shape) if case["mask"] else None) for a, b in pairs]
    if case["kind"] == "plan":
        return flows[0]
    if case["kind"] == "serve":
        flows += [_flow64(case, b, a) for a, b in pairs]
    return {"u": [f[0] for f in flows], "v": [f[1] for f in flows]}
