"""GPU parity of runs long enough to be replayed from a plan's cached hipGraph (more than eight passes): the
first run, replays on new contents, and each change of what the graph was captured for -- input, output,
workspace, step count, diffusivity -- every one bit for bit against the FP32 oracle, with the program's own
work and synchronisations between them."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpuhelp
    return gpuhelp


def _replays(g, run, ref, fields, spare, steps):
    """run(x, out, ws, steps) on changing buffers; ref(u0, steps) is what it must give."""
    import torch
    x = [g.to_dev(f) for f in fields]
    a, b, ws, ws2 = (torch.empty_like(x[0]) for _ in range(4))
    calls = [(x[0], a, ws, steps), (x[0], a, ws, steps), (x[1], a, ws, steps), (x[1], b, ws, steps), (x[1], b, ws2, steps),
             (x[1], b, ws2, steps + 3), (x[0], a, ws, steps)]
    for k, (inp, out, w, n) in enumerate(calls):
        if k == 1:  # new contents in the captured input
            x[0].copy_(g.to_dev(spare))
        out.fill_(0)
        _ = (x[1].float() * 3).sum().item()  # eager work between replays
        run(inp, out, w, n)
        u0 = (spare if k else fields[0]) if inp is x[0] else fields[1]
        np.testing.assert_array_equal(g.to_host(out), ref(u0, n), err_msg=f"call {k}")


@pytest.mark.parametrize("shape,r,tb,storage,variant", [("star", 1, 2, "f32", "tiled"), ("box", 2, 1, "bf16", "tiled"),
                                                        ("star", 2, 3, "f16", "march"), ("box", 1, 2, "f32", "march8")])
def test_replays_2d(g, shape, r, tb, storage, variant):
    import paper_2605_07954_amd as lib
    rng = np.random.default_rng(r)
    W = wl.random_footprint_weights(rng, shape, r)
    fields = [rng.random((150, 264), dtype=np.float32) for _ in range(3)]
    if storage != "f32":
        fields = [oracle.to_bits(f, storage) for f in fields]
    plan = lib.stencil_plan(150, 264, r, W, 0.5, storage, lib.ST_FLAG_GRAPH)
    try:
        lib.stencil_set_blocking(plan, tb)
        if variant != "tiled":
            lib.stencil_set_variant(plan, {"march": lib.ST_VARIANT_MARCH, "march8": lib.ST_VARIANT_MARCH8}[variant])
        _replays(g, lambda x, o, w, n: lib.stencil_run(plan, x, o, n, w),
                 lambda u, n: oracle.stencil_f32(u, W, 0.5, n) if storage == "f32" else oracle.stencil_lowp(u, W, 0.5, n, storage),
                 fields[:2], fields[2], 10 * tb + 1)
    finally:
        lib.stencil_destroy(plan)


def test_replays_3d(g):
    import paper_2605_07954_amd as lib
    rng = np.random.default_rng(3)
    W = np.where((np.indices((5, 5, 5)) != 2).sum(0) <= 1, rng.random((5, 5, 5)), 0.0)
    W = (W / W.sum()).astype(np.float32)
    fields = [rng.random((11, 37, 70), dtype=np.float32) for _ in range(3)]
    plan = lib.stencil_plan3d(11, 37, 70, 2, W, 0.25, "f32", lib.ST_FLAG_GRAPH)
    try:
        _replays(g, lambda x, o, w, n: lib.stencil_run(plan, x, o, n, w), lambda u, n: oracle.stencil3d_f32(u, W, 0.25, n),
                 fields[:2], fields[2], 21)
    finally:
        lib.stencil_destroy(plan)


def test_replays_varcoef(g):
    import paper_2605_07954_amd as lib
    rng = np.random.default_rng(4)
    fields = [rng.random((130, 201), dtype=np.float32) for _ in range(3)]
    kappas = [(0.05 + 0.15 * rng.random((130, 201))).astype(np.float32) for _ in range(2)]
    dev = [g.to_dev(k) for k in kappas]
    plan = lib.stencil_plan_varcoef(130, 201, 0.0, lib.ST_FLAG_GRAPH)
    try:
        lib.stencil_set_blocking(plan, 1)
        for k in (0, 1, 0):  # the graph of one diffusivity must not replay for another
            _replays(g, lambda x, o, w, n: lib.stencil_run_varcoef(plan, x, dev[k], o, n, w),
                     lambda u, n: oracle.varcoef_f32(u, kappas[k], 0.0, n), fields[:2], fields[2], 10)
    finally:
        lib.stencil_destroy(plan)


@pytest.mark.parametrize("bc", ["periodic", "frame"])
def test_replays_with_other_boundaries(g, bc):
    import torch
    import paper_2605_07954_amd as lib
    rng = np.random.default_rng(5)
    W = wl.random_footprint_weights(rng, "star", 2)
    u0 = rng.random((90, 260), dtype=np.float32)
    plan = lib.stencil_plan(90, 260, 2, W, 0.0, "f32", lib.ST_FLAG_GRAPH)
    try:
        frame = dev = None
        if bc == "frame":
            frame = rng.random(lib.stencil_frame_elems(plan), dtype=np.float32)
            dev = g.to_dev(frame)
        lib.stencil_set_boundary(plan, lib.ST_BC_PERIODIC if bc == "periodic" else lib.ST_BC_FRAME, dev)
        lib.stencil_set_blocking(plan, 2)
        ref = oracle.stencil_bc_f32(u0, W, bc, 21, frame)
        for shift in (0, 1):  # the second time off a 16-byte boundary
            x = torch.empty(u0.size + shift, device=g.DEV)[shift:]
            x.copy_(g.to_dev(u0).reshape(-1))
            out, ws = torch.empty(u0.size + shift, device=g.DEV)[shift:], torch.empty_like(x)
            for _ in range(3):
                out.fill_(0)
                _ = x.sum().item()
                lib.stencil_run(plan, x, out, 21, ws)
                np.testing.assert_array_equal(g.to_host(out).reshape(u0.shape), ref)
    finally:
        lib.stencil_destroy(plan)
