"""GPU parity of single levels of large FP32 3D stars, on LDS tiles that march along z: grids just large
enough for them, with sides that are no multiple of a tile, against the FP32 oracle bit for bit (the same
operations in the same order, so the tolerance is zero)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,r,b,steps", [((257, 241, 272), 1, 0.5, 1), ((5, 3499, 976), 1, -1.0, 1), ((67, 1001, 1008), 2, 0.0, 1),
                                             ((257, 241, 272), 1, 0.0, 3)])
def test_single_levels_bitwise(shape, r, b, steps):
    import gpuhelp as g
    import paper_2605_07954_amd as lib
    import torch
    rng = np.random.default_rng(5)
    k = 2 * r + 1
    W = rng.random((k, k, k)).astype(np.float32)
    W[(np.indices(W.shape) != r).sum(0) > 1] = 0.0
    W /= W.sum()
    u = rng.random(shape, dtype=np.float32)
    plan = lib.stencil_plan3d(*shape, r, W, b, "f32", 0)
    try:
        x = g.to_dev(u)
        out, ws = torch.empty_like(x), torch.empty_like(x)
        lib.stencil_run(plan, x, out, steps, ws)
        got = g.to_host(out)
    finally:
        lib.stencil_destroy(plan)
    np.testing.assert_array_equal(got, oracle.stencil3d_f32(u, W, b, steps))
