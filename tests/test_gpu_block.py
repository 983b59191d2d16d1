"""GPU parity of the register-tile kernels: constant-weight passes and variable-coefficient steps on
grids whose sides sit at the edges of the tiles, bit for bit against the FP32 oracle.

Both sides run the same FP32 operations in the same order, so the tolerance is zero (up to the sign of
an exact zero, which numpy's comparison ignores).
"""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

# cells a workgroup keeps: (tile_x, tile_y) -> columns x rows; the last one takes the deepest passes
TILES = {(64, 64): (64, 64), (128, 32): (128, 32), (128, 64): (128, 64), (256, 32): (256, 32)}


@pytest.fixture(scope="module")
def g():
    import gpuhelp
    return gpuhelp


def _sides(tile, halo):
    """Grid sides at one and two tiles' worth of stored cells, one less and one more, and a sliver."""
    out = max(tile - 2 * halo, 8)
    return [out - 1, out, out + 1, 2 * out + 1, 3]


@pytest.mark.parametrize("tile", sorted(TILES))
@pytest.mark.parametrize("shape,r,tb", [("star", 1, 1), ("star", 1, 5), ("star", 1, 16), ("box", 1, 7), ("star", 2, 6),
                                        ("box", 2, 3), ("star", 3, 4), ("box", 3, 2), ("star", 4, 7), ("box", 4, 2)])
def test_register_tiles_bitwise(g, tile, shape, r, tb):
    import torch
    import paper_2605_07954_amd as lib
    W = wl.random_footprint_weights(np.random.default_rng(r), shape, r)
    cs, rs = _sides(TILES[tile][0], r * tb), _sides(TILES[tile][1], r * tb)
    for k, (rows, cols) in enumerate(zip(rs, cs[1:] + cs[:1])):
        storage, b = (("f32", 0.0), ("f32", -1.25), ("bf16", 0.0), ("f16", 0.75), ("f32", 0.0))[k]
        u0 = np.random.default_rng(100 * r + k).random((rows, cols), dtype=np.float32)
        steps = tb + 1 + k
        plan = lib.stencil_plan(rows, cols, r, W, b, storage, 0)
        try:
            try:
                lib.stencil_set_blocking(plan, tb, *tile)
            except lib.StencilError:
                pytest.skip("depth beyond this tile's budget")
            x = g.to_dev(u0) if storage == "f32" else g.to_dev(oracle.to_bits(u0, storage))
            out, ws = torch.empty_like(x), torch.empty_like(x)
            lib.stencil_run(plan, x, out, steps, ws)
            got = g.to_host(out)
        finally:
            lib.stencil_destroy(plan)
        ref = (oracle.stencil_f32(u0, W, b, steps) if storage == "f32"
               else oracle.stencil_lowp(oracle.to_bits(u0, storage), W, b, steps, storage))
        np.testing.assert_array_equal(got, ref, err_msg=f"{rows}x{cols} {storage} b {b} steps {steps}")


@pytest.mark.parametrize("tile", sorted(TILES))
@pytest.mark.parametrize("tb", [1, 4, 9, 16])
def test_register_tiles_varcoef_bitwise(g, tile, tb):
    import torch
    import paper_2605_07954_amd as lib
    for k, (rows, cols) in enumerate(zip(_sides(TILES[tile][1], tb), _sides(TILES[tile][0], tb)[::-1])):
        rng = np.random.default_rng(k)
        u0 = rng.random((rows, cols), dtype=np.float32)
        kap = (0.05 + 0.15 * rng.random((rows, cols), dtype=np.float32)).astype(np.float32)
        b, steps = (0.0, 0.5)[k % 2], tb + k
        plan = lib.stencil_plan_varcoef(rows, cols, b, 0)
        try:
            try:
                lib.stencil_set_blocking(plan, tb, *tile)
            except lib.StencilError:
                pytest.skip("depth beyond this tile's budget")
            x, kd = g.to_dev(u0), g.to_dev(kap)
            out, ws = torch.empty_like(x), torch.empty_like(x)
            lib.stencil_run_varcoef(plan, x, kd, out, steps, ws)
            got = g.to_host(out)
        finally:
            lib.stencil_destroy(plan)
        np.testing.assert_array_equal(got, oracle.varcoef_f32(u0, kap, b, steps), err_msg=f"{rows}x{cols} steps {steps}")


def test_tiled_plan_of_a_large_grid(g):
    """A grid large enough that the tiled variant's passes run on the marching kernels, whole passes and a
    shallower last one: the whole field equals the oracle's."""
    import torch
    import paper_2605_07954_amd as lib
    rows, cols, r, tb, steps = 2899, 2903, 1, 6, 8
    W = wl.random_footprint_weights(np.random.default_rng(3), wl.BOX, r)
    u0 = np.random.default_rng(4).random((rows, cols), dtype=np.float32)
    plan = lib.stencil_plan(rows, cols, r, W, 0.25, "f32", 0)
    try:
        lib.stencil_set_blocking(plan, tb, 128, 64)
        x = g.to_dev(u0)
        out, ws = torch.empty_like(x), torch.empty_like(x)
        lib.stencil_run(plan, x, out, steps, ws)
        got = g.to_host(out)
    finally:
        lib.stencil_destroy(plan)
    np.testing.assert_array_equal(got, oracle.stencil_f32(u0, W, 0.25, steps))


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape,r", [("star", 1), ("star", 2), ("box", 1)])
def test_3d_register_tiles_bitwise(g, shape, r, storage):
    """3D passes of one to several levels on grids at the tiles' edges (64 x 64 or 64 x 32 cells less the
    margins) and with few and many planes per segment."""
    import torch
    import paper_2605_07954_amd as lib
    rng = np.random.default_rng(r)
    k = 2 * r + 1
    W = rng.random((k, k, k))
    if shape == "star":
        W = np.where((np.indices((k, k, k)) != r).sum(0) <= 1, W, 0.0)
    W = (W / W.sum()).astype(np.float32)
    grids = [(1, 52, 53, 7), (2, 64, 65, 1), (71, 57, 63, 6), (9, 61, 129, 4), (150, 8, 5, 13), (33, 105, 31, 3), (5, 1, 200, 12)]
    for planes, rows, cols, steps in grids:
        b = (0.0, -0.75)[steps % 2]
        u0 = rng.random((planes, rows, cols), dtype=np.float32)
        x = u0 if storage == "f32" else oracle.to_bits(u0, storage)
        plan = lib.stencil_plan3d(planes, rows, cols, r, W, b, storage, 0)
        try:
            xd = g.to_dev(x)
            out, ws = torch.empty_like(xd), torch.empty_like(xd)
            lib.stencil_run(plan, xd, out, steps, ws)
            got = g.to_host(out)
        finally:
            lib.stencil_destroy(plan)
        if storage == "f32":
            ref = oracle.stencil3d_f32(u0, W, b, steps)
        else:
            ref = x
            for _ in range(steps):
                ref = oracle.to_bits(oracle.stencil3d_f32(oracle.from_bits(ref, storage), W, b, 1), storage)
        np.testing.assert_array_equal(got, ref, err_msg=f"{planes}x{rows}x{cols} steps {steps}")
