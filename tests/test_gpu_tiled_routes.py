"""GPU parity of large untuned plans on each kernel that their passes may take -- one, four and eight columns
per marching lane, register tiles for narrow grids -- bit for bit against the FP32 oracle on whole fields (the
same operations in the same order, so the tolerance is zero)."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,shape,r,b,steps", [
    (1231, 1223, "box", 3, 0.5, 5), (5801, 5808, "box", 3, 0.0, 4), (5801, 5804, "box", 3, 0.0, 2), (64600, 520, "box", 3, -1.0, 4),
    (590000, 57, "box", 3, 0.0, 2), (200003, 41, "star", 2, 0.5, 7), (200003, 41, "box", 1, 0.0, 7), (200003, 41, "star", 3, 0.0, 5)])
def test_large_untuned_plans_bitwise(rows, cols, shape, r, b, steps):
    import gpuhelp as g
    W = wl.random_footprint_weights(np.random.default_rng(r), shape, r)
    u0 = np.random.default_rng(rows).random((rows, cols), dtype=np.float32)
    import torch
    import paper_2605_07954_amd as lib
    plan = lib.stencil_plan(rows, cols, r, W, b, "f32", 0)
    try:
        x = g.to_dev(u0)
        out, ws = torch.empty_like(x), torch.empty_like(x)
        lib.stencil_run(plan, x, out, steps, ws)
        got = g.to_host(out)
    finally:
        lib.stencil_destroy(plan)
    np.testing.assert_array_equal(got, oracle.stencil_f32(u0, W, b, steps))
