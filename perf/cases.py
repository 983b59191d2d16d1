"""The work that this library is measured on, as a user's program calls it.

A case is a dict with a ``kind``; every kind goes through the public binding the way the README's
examples do -- plan, tuner where a program would tune, caller-owned buffers and workspace in
``prepare``, and one call (or a few, where an entry point does one part) in ``run``.

  run      iterated 2D Jacobi steps: star and box footprints of radius 1 to 4, FP32 / BF16 / FP16
           storage, constant, periodic and framed halos, widths of any remainder, tuned plans and
           plans left as ``stencil_plan`` makes them
  run3d    the 3D form: star and box footprints of radius 1 and 2, every storage type
  batch    many grids of different shapes and stencils in one call
  varcoef  variable-coefficient heat steps
  solve    iteration to a tolerance with periodic convergence checks
  norms    the FP64 reductions of a field and its predecessor
  infer    the CNN surrogate's forward pass
  grad     its loss and gradient on a batch of crops
  train    optimiser steps of the whole training loop (fields, targets, crops, gradient, Adam)
"""
import math
import random

import numpy as np
import torch

import paper_2605_07954_amd as st

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
CHANNELS = (2, 32, 32, 32, 32, 32, 1)  # of the surrogate's six 3x3 convolutions
CNN_FLOPS = 18 * sum(a * b for a, b in zip(CHANNELS, CHANNELS[1:]))  # multiply-adds of one pixel, times 2
EXACT_LIMIT = 3e12  # tap products that exact() computes in a few seconds


def listed():
    return [
        # the smallest earnest run: a grid that fits the L2, where launches and latency count
        dict(name="heat5_512", kind="run", rows=512, cols=512, shape="star", r=1, storage="f32", steps=100, tune=True),
        # the headline stencil at its headline size: 49 taps, bound by the vector units
        dict(name="box49_16384", kind="run", rows=16384, cols=16384, shape="box", r=3, storage="f32", steps=60, tune=True),
        # a bandwidth-hungry star on a large grid, and the same with 16-bit storage
        dict(name="star9_8192", kind="run", rows=8192, cols=8192, shape="star", r=2, storage="f32", steps=120, tune=True),
        dict(name="star9_8192_bf16", kind="run", rows=8192, cols=8192, shape="star", r=2, storage="bf16", steps=120,
             tune=True),
        # a grid whose sides are no multiple of anything, with a halo that is not zero
        dict(name="star13_ragged", kind="run", rows=4099, cols=5003, shape="star", r=3, storage="f32", steps=48, b=1.5,
             tune=True),
        # a plan that the program does not tune
        dict(name="box9_untuned", kind="run", rows=2000, cols=3000, shape="box", r=1, storage="f32", steps=50, tune=False),
        # the 3D form at the size the benchmark runs
        dict(name="star7_3d_512", kind="run3d", planes=512, rows=512, cols=512, shape="star", r=1, storage="f32", steps=20),
        # 256 grids of mixed shapes and stencils, a parameter study in one graph launch
        dict(name="batch_256", kind="batch", grids=256, lo=64, hi=2048, steps=40, spec=3),
        # the variable-coefficient heat steps that the surrogate replaces
        dict(name="varcoef_1024", kind="varcoef", rows=1024, cols=1024, steps=16),
        # run to convergence, a check every 20 steps
        dict(name="solve_2048", kind="solve", rows=2048, cols=2048, every=20, tol=2e-4),
        # the surrogate: one field, and four optimiser steps of its training
        dict(name="infer_1024", kind="infer", batch=1, rows=1024, cols=1024),
        dict(name="train_1024", kind="train", batch=8, grid=1024, crop=256, K=16, steps=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    """A side between lo and hi: half of them a multiple of 16, the others as they fall."""
    n = _log(rng, lo, hi)
    return max(16, n // 16 * 16) if rng.random() < 0.5 else n


def draw(rng: random.Random):
    kind = rng.choice(["run", "run", "run", "run", "run3d", "run3d", "batch", "varcoef", "varcoef", "solve", "norms",
                       "infer", "grad", "train"])
    if kind == "run":
        c = dict(kind=kind, rows=_side(rng, 128, 8192), cols=_side(rng, 128, 8192), shape=rng.choice(["star", "box"]),
                 r=rng.choice([1, 1, 2, 2, 3, 4]), storage=rng.choice(["f32", "f32", "bf16", "f16"]),
                 steps=_log(rng, 8, 120), tune=rng.random() < 0.7)
        halo = rng.choice(["zero", "zero", "value", "periodic", "frame"])
        if halo == "value":
            c["b"] = round(rng.uniform(-2, 2), 3)
        elif halo != "zero":
            c["bc"] = halo
        return c
    if kind == "run3d":
        return dict(kind=kind, planes=_side(rng, 32, 512), rows=_side(rng, 32, 512), cols=_side(rng, 32, 512),
                    shape=rng.choice(["star", "star", "box"]), r=rng.choice([1, 1, 2]),
                    storage=rng.choice(["f32", "f32", "bf16", "f16"]), steps=_log(rng, 4, 24),
                    b=rng.choice([0.0, 0.0, 0.5]))
    if kind == "batch":
        return dict(kind=kind, grids=_log(rng, 8, 128), lo=64, hi=rng.choice([256, 1024, 2048]), steps=_log(rng, 10, 60),
                    spec=rng.randrange(1000))
    if kind == "varcoef":
        return dict(kind=kind, rows=_side(rng, 64, 4096), cols=_side(rng, 64, 4096), steps=_log(rng, 4, 64))
    if kind == "solve":
        return dict(kind=kind, rows=_side(rng, 256, 4096), cols=_side(rng, 256, 4096), every=_log(rng, 5, 50),
                    tol=rng.choice([5e-4, 3e-4, 2e-4]))
    if kind == "norms":
        return dict(kind=kind, rows=_side(rng, 512, 16384), cols=_side(rng, 512, 16384),
                    storage=rng.choice(["f32", "f32", "bf16", "f16"]))
    if kind == "infer":
        return dict(kind=kind, batch=rng.choice([1, 1, 2, 4]), rows=_side(rng, 100, 1500), cols=_side(rng, 100, 1500))
    if kind == "grad":
        return dict(kind=kind, batch=rng.choice([1, 2, 4, 8]), rows=_side(rng, 48, 320), cols=_side(rng, 48, 320))
    grid = _side(rng, 192, 1024)
    return dict(kind=kind, batch=rng.choice([2, 4, 8]), grid=grid, crop=rng.choice([64, 100, 128, 192]), K=rng.choice([4, 8, 16]),
                steps=rng.choice([1, 2, 4]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _mask(shape, r, dims):
    """Footprint of a star (the axes) or a box (all of it)."""
    n = 2 * r + 1
    if shape == "box":
        return np.ones((n,) * dims, bool)
    off = np.indices((n,) * dims) != r
    return off.sum(0) <= 1


def _weights(shape, r, seed, dims=2):
    """Positive weights on the footprint that sum to 1, so that a field neither grows nor dies."""
    m = _mask(shape, r, dims)
    w = np.zeros(m.shape)
    v = np.random.default_rng(seed).random(int(m.sum()))
    w[m] = v / v.sum()
    return w.astype(np.float32)


def _heat5():
    w = np.zeros((3, 3), np.float32)
    w[1, 1] = 0.6
    w[0, 1] = w[2, 1] = w[1, 0] = w[1, 2] = 0.1
    return w


def _uniform(dims, storage, g):
    return torch.rand(dims, device="cuda", generator=g).to(DTYPES[storage])


def _weights_of(c, seed):
    return _heat5() if c["shape"] == "star" and c["r"] == 1 and c["kind"] == "run" else _weights(
        c["shape"], c["r"], seed, 3 if c["kind"] == "run3d" else 2)


def _frame(c, g):
    return _uniform((2 * c["r"] * (c["cols"] + 2 * c["r"]) + 2 * c["r"] * c["rows"],), c["storage"], g)


def _grids(c):
    """(rows, cols, shape, r) of each grid: sides log-uniform, a 5-point star, 9-point box or 13-point star."""
    rng = np.random.default_rng(c["spec"])
    a, b = math.log(c["lo"]), math.log(c["hi"])
    return [(int(round(math.exp(rng.uniform(a, b)))), int(round(math.exp(rng.uniform(a, b)))),
             *(("star", 1), ("box", 1), ("star", 3))[int(rng.integers(3))]) for _ in range(c["grids"])]


def _coefficients(n, seed):
    """n rows of 16 sine modes (p, q, a, 0) of a start field and 8 cosine modes (kx, ky, b, phase) of a diffusivity."""
    rng = np.random.default_rng(seed)
    t = np.zeros((n, 24, 4), np.float32)
    t[:, :16, :2] = rng.integers(1, 7, (n, 16, 2))
    t[:, :16, 2] = rng.standard_normal((n, 16)) / np.hypot(t[:, :16, 0], t[:, :16, 1])
    t[:, 16:, :2] = rng.integers(0, 4, (n, 8, 2))
    t[:, 16:, 2] = rng.standard_normal((n, 8))
    t[:, 16:, 3] = rng.uniform(0, 2 * math.pi, (n, 8))
    return t.reshape(n, 96)


def _fields(n, rows, cols, seed):
    """n smooth fields and diffusivities in [0.05, 0.2], each (n, rows, cols) FP32."""
    t = torch.from_numpy(_coefficients(n, seed)).double().cuda().reshape(n, 24, 4)
    i = torch.arange(rows, device="cuda", dtype=torch.float64)
    j = torch.arange(cols, device="cuda", dtype=torch.float64)
    u, k = [], []
    for f in range(n):
        p, q, a = (t[f, :16, m, None] for m in range(3))
        u.append((a * torch.sin(p * math.pi * (i + 1) / (rows + 1))).T.contiguous()
                 @ torch.sin(q * math.pi * (j + 1) / (cols + 1)))
        kx, ky, b, ph = (t[f, 16:, m, None] for m in range(4))
        y, x = 2 * math.pi * ky * i / rows + ph, 2 * math.pi * kx * j / cols
        g = (b * torch.cos(y)).T.contiguous() @ torch.cos(x) - (b * torch.sin(y)).T.contiguous() @ torch.sin(x)
        k.append(0.125 + 0.075 * g / b.abs().sum())
    return torch.stack(u).float(), torch.stack(k).float()


def _params(seed):
    """Weights of a network in the middle of training: He-normal, small biases; [ky][kx][ci][co] then b, layer by layer."""
    rng = np.random.default_rng(seed)
    v = []
    for ci, co in zip(CHANNELS, CHANNELS[1:]):
        v += [rng.standard_normal(9 * ci * co) * math.sqrt(2 / (9 * ci)), rng.standard_normal(co) * 0.05]
    return torch.from_numpy(np.concatenate(v).astype(np.float32)).cuda()


def _crops(c, seed):
    """Fields, diffusivities, targets and loss windows (the 6 cells next to a cut edge left out) of a gradient case."""
    u, k = _fields(c["batch"], c["rows"], c["cols"], seed)
    target = u.double()
    for _ in range(4):
        target = _varcoef_step(target, k.double())
    return u, k, target.float(), np.array([[6, c["rows"] - 6, 6, c["cols"] - 6]] * c["batch"], np.int32)


# ---------------------------------------------------------------------------
# what a program holds before the call
# ---------------------------------------------------------------------------

class State:
    """Buffers and handles of one case; the handles go when it does."""

    def __init__(self, **kw):
        self.__dict__.update(kw)
        self.close = kw.get("close", [])

    def __del__(self):
        try:
            torch.cuda.synchronize()
            for destroy, handle in self.close:
                destroy(handle)
        except Exception:  # noqa: BLE001 - at interpreter exit the modules may be gone
            pass


def _bytes(n):
    return torch.empty(max(int(n), 1), dtype=torch.uint8, device="cuda")


def _raw(t):
    """The tensor as the binding takes it: 16-bit fields as bit patterns."""
    return t if t.dtype == torch.float32 else t.view(torch.int16)


def prepare(case, seed):
    c, kind, g = case, case["kind"], _gen(seed)
    if kind == "run":
        x = _uniform((c["rows"], c["cols"]), c["storage"], g)
        out = torch.empty_like(x)
        plan = st.stencil_plan(c["rows"], c["cols"], c["r"], _weights_of(c, seed), c.get("b", 0.0), c["storage"],
                               st.ST_FLAG_GRAPH if c["tune"] else 0)
        frame = None
        if c.get("bc") == "frame":
            frame = _frame(c, g)
            st.stencil_set_boundary(plan, st.ST_BC_FRAME, _raw(frame))
        elif c.get("bc") == "periodic":
            st.stencil_set_boundary(plan, st.ST_BC_PERIODIC)
        ws = torch.empty_like(x)
        if c["tune"]:
            ws = _bytes(x.numel() * x.element_size() + (1 << 17))  # the resident variant's counters, too
            st.stencil_autotune(plan, _raw(x), _raw(out), ws, min(24, c["steps"]))
        return State(c=c, plan=plan, x=x, out=out, ws=ws, frame=frame, close=[(st.stencil_destroy, plan)])
    if kind == "run3d":
        x = _uniform((c["planes"], c["rows"], c["cols"]), c["storage"], g)
        plan = st.stencil_plan3d(c["planes"], c["rows"], c["cols"], c["r"], _weights_of(c, seed), c.get("b", 0.0),
                                 c["storage"], 0)
        return State(c=c, plan=plan, x=x, out=torch.empty_like(x), ws=torch.empty_like(x),
                     close=[(st.stencil_destroy, plan)])
    if kind == "batch":
        specs = _grids(c)
        plans = [st.stencil_plan(h, w, r, _weights(s, r, seed * 1000 + i), 0.0, "f32", 0)
                 for i, (h, w, s, r) in enumerate(specs)]
        ins = [_uniform((h, w), "f32", g) for h, w, _, _ in specs]
        outs = [torch.empty_like(x) for x in ins]
        batch = st.stencil_batch_create(plans, [c["steps"]] * len(plans), st.ST_FLAG_GRAPH)
        ws = _bytes(st.stencil_batch_workspace_bytes(batch))
        st.stencil_batch_autotune(batch, ins, outs, ws)
        return State(c=c, batch=batch, ins=ins, outs=outs, ws=ws,
                     close=[(st.stencil_batch_destroy, batch)] + [(st.stencil_destroy, p) for p in plans])
    if kind == "varcoef":
        u, k = (t[0].contiguous() for t in _fields(1, c["rows"], c["cols"], seed))
        out, ws = torch.empty_like(u), torch.empty_like(u)
        plan = st.stencil_plan_varcoef(c["rows"], c["cols"], 0.0, st.ST_FLAG_GRAPH)
        st.stencil_autotune_varcoef(plan, u, k, out, ws, min(16, c["steps"]))
        return State(c=c, plan=plan, u=u, k=k, out=out, ws=ws, close=[(st.stencil_destroy, plan)])
    if kind == "solve":
        x = _uniform((c["rows"], c["cols"]), "f32", g)
        out = torch.empty_like(x)
        plan = st.stencil_plan(c["rows"], c["cols"], 1, _heat5(), 0.0, "f32", 0)
        tune_ws = _bytes(4 * x.numel() + (1 << 17))
        st.stencil_autotune(plan, x, out, tune_ws, min(24, c["every"]))
        ws = _bytes(st.stencil_solve_ws_bytes(plan, c["every"]))
        return State(c=c, plan=plan, x=x, out=out, ws=ws, close=[(st.stencil_destroy, plan)])
    if kind == "norms":
        u = _uniform((c["rows"], c["cols"]), c["storage"], g)
        prev = _uniform((c["rows"], c["cols"]), c["storage"], g)
        plan = st.stencil_plan(c["rows"], c["cols"], 1, _heat5(), 0.0, c["storage"], 0)
        return State(c=c, plan=plan, u=u, prev=prev, ws=_bytes(st.stencil_norms_ws_bytes(plan)),
                     out=torch.empty(4, dtype=torch.float64, device="cuda"), close=[(st.stencil_destroy, plan)])
    m, params = st.surrogate_create(), _params(seed)
    if kind == "infer":
        u, k = _fields(c["batch"], c["rows"], c["cols"], seed)
        return State(c=c, m=m, params=params, u=u, k=k, out=torch.empty_like(u),
                     ws=_bytes(st.surrogate_workspace_bytes(m, c["batch"], c["rows"], c["cols"])),
                     close=[(st.surrogate_destroy, m)])
    if kind == "grad":
        u, k, target, window = _crops(c, seed)
        return State(c=c, m=m, params=params, u=u, k=k, target=target, window=window, grad=torch.empty_like(params),
                     loss=torch.zeros(1, dtype=torch.float64, device="cuda"),
                     ws=_bytes(st.surrogate_workspace_bytes(m, c["batch"], c["rows"], c["cols"])),
                     close=[(st.surrogate_destroy, m)])
    n = c["steps"] * c["batch"]
    yx = np.random.default_rng(seed).integers(0, c["grid"] - c["crop"] + 1, (n, 2)).astype(np.int32)
    return State(c=c, m=m, params=params, yx=yx, at=0,
                 optim=torch.zeros(2 * st.SG_PARAM_COUNT, dtype=torch.float32, device="cuda"),
                 coef=torch.from_numpy(_coefficients(n, seed)).cuda(),
                 losses=torch.zeros(c["steps"], dtype=torch.float64, device="cuda"),
                 ws=_bytes(st.surrogate_train_ws_bytes(m, c["grid"], c["grid"], c["crop"], c["batch"], c["K"], c["steps"])),
                 close=[(st.surrogate_destroy, m)])


def run(state):
    s, c = state, state.c
    kind = c["kind"]
    if kind in ("run", "run3d"):
        st.stencil_run(s.plan, _raw(s.x), _raw(s.out), c["steps"], s.ws)
        return s.out
    if kind == "batch":
        st.stencil_run_batched(s.batch, s.ins, s.outs, s.ws)
        return s.outs[:60]  # (of more grids, the first 60 are compared)
    if kind == "varcoef":
        st.stencil_run_varcoef(s.plan, s.u, s.k, s.out, c["steps"], s.ws)
        return s.out
    if kind == "solve":
        steps, rel = st.stencil_solve(s.plan, s.x, s.out, 5000, c["every"], c["tol"], s.ws)
        return {"field": s.out, "steps": steps, "residual": rel}
    if kind == "norms":
        st.stencil_norms(s.plan, s.prev, s.u, s.out, s.ws)
        return s.out
    if kind == "infer":
        st.surrogate_infer(s.m, s.params, s.u, s.k, s.out, c["batch"], c["rows"], c["cols"], s.ws)
        return s.out
    if kind == "grad":
        st.surrogate_loss_grad(s.m, s.params, s.u, s.k, s.target, s.window, c["batch"], c["rows"], c["cols"], s.grad, s.loss,
                               s.ws)
        return {"grad": s.grad, "loss": s.loss}
    # the next optimiser steps of a long schedule: params and optim are updated in place
    st.surrogate_train(s.m, s.params, s.optim, s.coef, s.yx, s.losses, s.ws, c["grid"], c["grid"], c["crop"], c["batch"],
                       c["K"], c["steps"], s.at, 10_000_000, 1e-3)
    s.at += c["steps"]
    return {"params": s.params, "optim": s.optim, "losses": s.losses}


# ---------------------------------------------------------------------------
# work and exact values
# ---------------------------------------------------------------------------

def _taps(c):
    return int(_mask(c["shape"], c["r"], 3 if c["kind"] == "run3d" else 2).sum())


def work(case):
    c, kind = case, case["kind"]
    if kind in ("run", "run3d"):
        cells = c["rows"] * c["cols"] * c.get("planes", 1)
        return {"bytes": 2 * cells * (4 if c["storage"] == "f32" else 2),
                "flops": c["steps"] * cells * (2 * _taps(c) - 1)}
    if kind == "batch":
        taps = {("star", 1): 5, ("box", 1): 9, ("star", 3): 13}
        return {"bytes": sum(8 * h * w for h, w, _, _ in _grids(c)),
                "flops": sum(c["steps"] * h * w * (2 * taps[(s, r)] - 1) for h, w, s, r in _grids(c))}
    if kind == "norms":
        cells = c["rows"] * c["cols"]
        return {"bytes": 2 * cells * (4 if c["storage"] == "f32" else 2), "flops": 8 * cells}
    if kind == "train":  # fields, K plain steps, and three passes' worth of convolutions on the crops, per trajectory
        n = c["steps"] * c["batch"]
        return {"bytes": n * 4 * 3 * c["crop"] ** 2,
                "flops": n * (c["K"] * 14 * c["grid"] ** 2 + 3 * CNN_FLOPS * c["crop"] ** 2)}
    cells = c["rows"] * c["cols"] * c.get("batch", 1)
    if kind == "varcoef":
        return {"bytes": 12 * cells, "flops": 14 * c["steps"] * cells}
    if kind == "solve":  # about 0.05 / tol steps until the noise of the start field is that small
        return {"bytes": 8 * cells, "flops": 9 * cells * int(0.05 / c["tol"])}
    if kind == "infer":
        return {"bytes": 12 * cells, "flops": CNN_FLOPS * cells}
    return {"bytes": 12 * cells, "flops": 3 * CNN_FLOPS * cells}


def _jacobi_step(u, w, pad):
    """One step on an FP64 field; `pad` extends it by the halo."""
    r, dims, e = w.shape[0] // 2, u.dim(), pad(u)
    out = torch.zeros_like(u)
    for at in np.argwhere(w != 0):
        v = e
        for d in range(dims):
            v = v.narrow(d, int(at[d]), u.shape[d])
        out.add_(v, alpha=float(w[tuple(at)]))
    return out


def _constant(r, b):
    return lambda u: torch.nn.functional.pad(u, (r,) * (2 * u.dim()), value=b)


def _periodic(r):
    def pad(u):
        for d in range(u.dim()):
            i = torch.arange(-r, u.shape[d] + r, device=u.device) % u.shape[d]
            u = u.index_select(d, i)
        return u
    return pad


def _framed(c, frame):
    r, h, w = c["r"], c["rows"], c["cols"]
    f = frame.double()
    a, b = r * (w + 2 * r), r * h

    def pad(u):
        mid = torch.cat([f[2 * a:2 * a + b].view(h, r), u, f[2 * a + b:].view(h, r)], 1)
        return torch.cat([f[:a].view(r, -1), mid, f[a:2 * a].view(r, -1)], 0)
    return pad


def _varcoef_step(u, k):
    """u' = u + sum over the four faces of (k + k_nb) / 2 (u_nb - u): outside the grid u_nb = 0 and k_nb = k."""
    e = torch.nn.functional.pad(u, (1, 1, 1, 1))
    q = torch.cat([k[..., :1, :], k, k[..., -1:, :]], -2)
    q = torch.cat([q[..., :1], q, q[..., -1:]], -1)
    h, w, out = u.shape[-2], u.shape[-1], u.clone()
    for y, x in ((0, 1), (1, 0), (1, 2), (2, 1)):
        out += 0.5 * (k + q[..., y:y + h, x:x + w]) * (e[..., y:y + h, x:x + w] - u)
    return out


def _network(params, u, k):
    """The surrogate on FP64 fields (n, rows, cols); params: the flat buffer, FP64."""
    n, h, w = u.shape
    s = u.reshape(n, -1).square().mean(1).sqrt().view(n, 1, 1)
    x, at = torch.stack([u / s, (k - 0.125) / 0.075], -1), 0
    for l, (ci, co) in enumerate(zip(CHANNELS, CHANNELS[1:])):
        W, b = params[at:at + 9 * ci * co].view(9, ci, co), params[at + 9 * ci * co:at + 9 * ci * co + co]
        at += 9 * ci * co + co
        e = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
        y = b.expand(n * h * w, co)
        for t in range(9):
            y = y + e[:, t // 3:t // 3 + h, t % 3:t % 3 + w].reshape(-1, ci) @ W[t]
        x = y.view(n, h, w, co)
        if l < 5:
            x = x * 0.5 * (1 + torch.erf(x / math.sqrt(2)))
    return u + s * 2.0 ** -11 * x[..., 0]


def exact(case, seed):
    c, kind, g = case, case["kind"], _gen(seed)
    if kind in ("run", "run3d"):
        if work(c)["flops"] > 2 * EXACT_LIMIT:
            return None
        dims = (c["rows"], c["cols"]) if kind == "run" else (c["planes"], c["rows"], c["cols"])
        u = _uniform(dims, c["storage"], g).double()
        if c.get("bc") == "frame":
            pad = _framed(c, _frame(c, g))
        else:
            b = float(torch.tensor(c.get("b", 0.0)).to(DTYPES[c["storage"]]))
            pad = _periodic(c["r"]) if c.get("bc") else _constant(c["r"], b)
        w = _weights_of(c, seed).astype(np.float64)
        for _ in range(c["steps"]):
            u = _jacobi_step(u, w, pad)
        return u
    if kind == "batch":
        outs = []
        for i, (h, w, s, r) in enumerate(_grids(c)):
            u = _uniform((h, w), "f32", g).double()
            if i < 60:
                for _ in range(c["steps"] if h * w < 1 << 20 else 0):
                    u = _jacobi_step(u, _weights(s, r, seed * 1000 + i).astype(np.float64), _constant(r, 0.0))
                outs.append(u if h * w < 1 << 20 else None)
        return outs
    if kind == "varcoef":
        u, k = (t[0].double() for t in _fields(1, c["rows"], c["cols"], seed))
        for _ in range(c["steps"]):
            u = _varcoef_step(u, k)
        return u
    if kind == "solve":
        u, w, n = _uniform((c["rows"], c["cols"]), "f32", g).double(), _heat5().astype(np.float64), 0
        while n < 5000:
            for _ in range(min(c["every"], 5000 - n)):
                last, u, n = u, _jacobi_step(u, w, _constant(1, 0.0)), n + 1
            rel = float((u - last).norm() / u.norm())
            if rel <= c["tol"]:
                break
        return {"field": u, "steps": None, "residual": rel}
    if kind == "norms":
        u, prev = (_uniform((c["rows"], c["cols"]), c["storage"], g).double() for _ in range(2))
        nxt = _jacobi_step(u, _heat5().astype(np.float64), _constant(1, 0.0))
        return torch.stack([(u - prev).square().sum(), u.square().sum(), u.sum(), nxt.sum()])
    if kind == "infer":
        u, k = _fields(c["batch"], c["rows"], c["cols"], seed)
        p = _params(seed).double()
        return torch.cat([_network(p, u[i:i + 1].double(), k[i:i + 1].double()) for i in range(c["batch"])])
    if kind == "grad":
        u, k, target, win = _crops(c, seed)
        p = _params(seed).double().requires_grad_()
        loss = 0.0
        n = sum((b - a) * (d - e) for a, b, e, d in win.tolist())
        for i, (a, b, e, d) in enumerate(win.tolist()):
            part = (_network(p, u[i:i + 1].double(), k[i:i + 1].double()) - target[i].double())[0, a:b, e:d].square().sum() / n
            part.backward()
            loss += float(part)
        return {"grad": p.grad, "loss": torch.tensor([loss], dtype=torch.float64)}
    return None  # Adam's first steps divide each gradient by its own size: no digits of the update are left to compare
