"""GPU parity of the field synthesis at the edges of its tiles: each field against the reference formula in
FP64, and the same field made by either kernel (one field alone, or many at once) bit for bit -- the factors
and the order of the FMAs are the same."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(1, 1), (16, 64), (17, 65), (15, 63), (64, 256), (65, 257), (130, 3)])
def test_synthesis_kernels_agree(rows, cols):
    import gpuhelp as g
    import torch
    import paper_2605_07954_amd as lib
    n = min(3000000 // (rows * cols) + 1, 40000)  # enough fields for the kernel of large ones (but for 1 x 1)
    coef = np.tile(wl.field_coefficients(2, 9), (n // 2 + 1, 1))[:n].astype(np.float32)
    u, k = (torch.empty((n, rows, cols), device=g.DEV) for _ in range(2))
    lib.surrogate_synth_fields(g.to_dev(coef), n, rows, cols, u, k)
    one_u, one_k = (torch.empty((2, rows, cols), device=g.DEV) for _ in range(2))
    lib.surrogate_synth_fields(g.to_dev(coef[:2]), 2, rows, cols, one_u, one_k)
    for t in range(2):
        hu, hk = wl.synth_fields(coef[t], rows, cols)
        # sums of 16 and 8 terms of size 1 in FP32 with rounded factors
        np.testing.assert_allclose(g.to_host(one_u[t]), hu, atol=2e-6)
        np.testing.assert_allclose(g.to_host(one_k[t]), hk, atol=2e-6)
        np.testing.assert_array_equal(g.to_host(u[t]), g.to_host(one_u[t]))
        np.testing.assert_array_equal(g.to_host(k[t]), g.to_host(one_k[t]))
