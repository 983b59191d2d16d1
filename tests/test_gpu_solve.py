"""GPU parity of the solve's intervals: the last pass sums the residual beside its levels, on grids and
intervals at the edges of the tiles and of the split into passes.

The field is bitwise the FP32 oracle's.  The residual is two FP64 sums of at most 40,000 exact products in
another order than numpy's, so it differs by at most 40,000 * 2^-53 < 1e-11 of itself.
"""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

TILED, MARCH, MARCH1 = 0, 2, 4


@pytest.fixture(scope="module")
def g():
    import gpuhelp
    return gpuhelp


@pytest.mark.parametrize("variant,shape,r,tb,tile", [
    (TILED, "star", 1, 16, (256, 32)), (TILED, "star", 1, 3, (64, 64)), (TILED, "box", 1, 5, (128, 32)),
    (TILED, "star", 2, 8, (128, 64)), (TILED, "box", 2, 8, (128, 32)), (TILED, "box", 3, 2, (64, 64)),
    (TILED, "star", 4, 2, (128, 64)), (TILED, "box", 4, 1, (64, 64)), (MARCH, "star", 1, 6, None),
    (MARCH1, "box", 2, 2, None), (MARCH, "star", 3, 2, None), (MARCH, "box", 4, 1, None)])
def test_solve_intervals(g, variant, shape, r, tb, tile):
    import torch
    import paper_2605_07954_amd as lib
    W = wl.random_footprint_weights(np.random.default_rng(r), shape, r)
    for k, (rows, cols, every) in enumerate([(1, 1, 2), (3, 130, tb), (33, 65, 1), (96, 129, tb + 1), (150, 260, 2 * tb + 1),
                                             (64, 64, 3 * tb)]):
        storage, b = (("f32", 0.0), ("bf16", 0.5), ("f32", -1.25), ("f16", 0.0), ("f32", 0.0), ("bf16", 0.0))[k]
        u0 = np.random.default_rng(10 * r + k).random((rows, cols), dtype=np.float32)
        steps = 2 * every + 1  # (the third interval holds one step)
        plan = lib.stencil_plan(rows, cols, r, W, b, storage, 0)
        try:
            lib.stencil_set_blocking(plan, 1, 0, 0)
            lib.stencil_set_variant(plan, variant)
            lib.stencil_set_blocking(plan, tb, *(tile or (0, 0)))
            x = g.to_dev(u0) if storage == "f32" else g.to_dev(oracle.to_bits(u0, storage))
            out = torch.empty_like(x)
            ws = torch.empty(lib.stencil_solve_ws_bytes(plan, every), dtype=torch.uint8, device=g.DEV)
            results = []
            for budget, tol in ((steps, 0.0), (steps, 1e30)):
                done, res = lib.stencil_solve(plan, x, out, budget, every, tol, ws)
                results.append((done, res, g.to_host(out).copy()))
        finally:
            lib.stencil_destroy(plan)

        def at(t):
            if storage == "f32":
                return oracle.stencil_f32(u0, W, b, t)
            return oracle.stencil_lowp(oracle.to_bits(u0, storage), W, b, t, storage)

        def value(f):
            return (f if storage == "f32" else oracle.from_bits(f, storage)).astype(np.float64)

        def rel(t):
            now, before = value(at(t)), value(at(t - 1))
            return np.sqrt(np.sum((now - before) ** 2) / np.sum(now * now))

        # a 16-bit field can come to rest: then the check of a tolerance of zero passes
        ends = [t for t in (every, 2 * every) if rel(t) == 0.0] + [steps]
        for (done, res, got), want in zip(results, (ends[0], every)):
            msg = f"{rows}x{cols} {storage} b {b} every {every}"
            assert done == want, msg
            np.testing.assert_array_equal(got, at(want), err_msg=msg)
            assert abs(res - rel(want)) <= 1e-11 * rel(want), msg
