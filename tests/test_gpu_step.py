"""GPU parity of single steps on LDS tiles: grids whose sides sit at the edges of the 128 x 64 tile, every
footprint and storage type, bit for bit against the FP32 oracle (the same operations in the same order, so the
tolerance is zero); runs of large boxes, which take nothing but single steps; a solve made of them."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [(1, 8), (3, 128), (63, 120), (64, 136), (65, 264), (130, 16), (200, 384)]


@pytest.fixture(scope="module")
def g():
    import gpuhelp
    return gpuhelp


def _run(g, u0, W, b, steps, storage, noalloc=False, tb=0):
    import torch
    import paper_2605_07954_amd as lib
    rows, cols = u0.shape
    plan = lib.stencil_plan(rows, cols, (W.shape[0] - 1) // 2, W, b, storage, 0)
    try:
        if tb:
            lib.stencil_set_blocking(plan, tb)
        x = g.to_dev(u0) if storage == "f32" else g.to_dev(oracle.to_bits(u0, storage))
        out, ws = torch.empty_like(x), torch.empty_like(x)
        if noalloc:
            lib.stencil_run_noalloc(plan, x, out, steps)
        else:
            lib.stencil_run(plan, x, out, steps, ws)
        return g.to_host(out)
    finally:
        lib.stencil_destroy(plan)


def _ref(u0, W, b, steps, storage):
    return (oracle.stencil_f32(u0, W, b, steps) if storage == "f32"
            else oracle.stencil_lowp(oracle.to_bits(u0, storage), W, b, steps, storage))


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", ["star", "box"])
@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_single_step_bitwise(g, shape, r, storage):
    W = wl.random_footprint_weights(np.random.default_rng(r), shape, r)
    for k, (rows, cols) in enumerate(SIZES):
        u0 = np.random.default_rng(k).random((rows, cols), dtype=np.float32)
        b = (0.0, -1.25, 0.75)[k % 3]
        np.testing.assert_array_equal(_run(g, u0, W, b, 1, storage), _ref(u0, W, b, 1, storage), err_msg=f"{rows}x{cols} b {b}")
        np.testing.assert_array_equal(_run(g, u0, W, b, 3, storage, tb=1), _ref(u0, W, b, 3, storage), err_msg=f"{rows}x{cols} b {b}")


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("r,storage", [(4, "f32"), (3, "bf16")])
@pytest.mark.parametrize("steps", [2, 3, 6])
def test_large_box_bitwise(g, steps, noalloc, r, storage):
    W = wl.random_footprint_weights(np.random.default_rng(r), "box", r)
    u0 = np.random.default_rng(8).random((1210, 1264), dtype=np.float32)
    np.testing.assert_array_equal(_run(g, u0, W, 0.5, steps, storage, noalloc), _ref(u0, W, 0.5, steps, storage))


def test_solve_of_single_steps(g):
    import torch
    import paper_2605_07954_amd as lib
    W = wl.random_footprint_weights(np.random.default_rng(1), "star", 1)
    u0 = np.random.default_rng(2).random((130, 264), dtype=np.float32)
    plan = lib.stencil_plan(130, 264, 1, W, 0.0, "f32", 0)
    try:
        lib.stencil_set_blocking(plan, 1)
        x = g.to_dev(u0)
        out = torch.empty_like(x)
        ws = torch.empty(lib.stencil_solve_ws_bytes(plan, 3), dtype=torch.uint8, device=g.DEV)
        steps, rel = lib.stencil_solve(plan, x, out, 90, 3, 5e-3, ws)[:2]
        got = g.to_host(out)
    finally:
        lib.stencil_destroy(plan)
    assert 3 < steps < 90 and rel <= 5e-3
    np.testing.assert_array_equal(got, oracle.stencil_f32(u0, W, 0.0, steps))
