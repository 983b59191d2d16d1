"""GPU parity of batched grids on register tiles: whole grids at the edges of the one tile they run in,
passes at the edges of tiles, and classes whose wide grids march while the narrow ones run on tiles.  Every
grid equals the FP32 oracle bit for bit: the same operations in the same order, so the tolerance is zero."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpuhelp
    return gpuhelp


def _check(g, grids, steps, flags, setup=None):
    """grids: (rows, cols, shape, r, b)."""
    import torch
    import paper_2605_07954_amd as lib
    rng = np.random.default_rng(7)
    W = [wl.random_footprint_weights(np.random.default_rng(k), s, r) for k, (_, _, s, r, _) in enumerate(grids)]
    u0 = [rng.random((h, w), dtype=np.float32) for h, w, _, _, _ in grids]
    plans = [lib.stencil_plan(h, w, r, W[k], b, "f32", 0) for k, (h, w, _, r, b) in enumerate(grids)]
    batch = lib.stencil_batch_create(plans, steps, flags)
    try:
        if setup:
            setup(lib, batch)
        ins = [g.to_dev(u) for u in u0]
        outs = [torch.empty_like(x) for x in ins]
        ws = torch.empty(lib.stencil_batch_workspace_bytes(batch), dtype=torch.uint8, device=g.DEV)
        for _ in range(2):
            for o in outs:
                o.fill_(float("nan"))
            lib.stencil_run_batched(batch, ins, outs, ws)
            got = [g.to_host(o) for o in outs]
            for k, (h, w, s, r, b) in enumerate(grids):
                np.testing.assert_array_equal(got[k], oracle.stencil_f32(u0[k], W[k], b, steps[k]),
                                              err_msg=f"{h}x{w} {s} r {r} b {b} steps {steps[k]}")
    finally:
        lib.stencil_batch_destroy(batch)
        for p in plans:
            lib.stencil_destroy(p)


@pytest.mark.parametrize("shape", ["star", "box"])
@pytest.mark.parametrize("r", [1, 2, 3])
def test_whole_grids(g, shape, r):
    # the tile holds 128 - 2r rows and 128 - r - (r rounded up to even) columns; LDS takes the longer sides
    h, w = 128 - 2 * r, 128 - r - 2 * ((r + 1) // 2)
    sizes = [(1, 1), (h, 60), (h + 1, 60), (50, w), (50, w + 1), (8, 9), (h - 1, 7), (3, 200)]
    grids = [(a, c, shape, r, (0.0, 1.5, -2.0)[k % 3]) for k, (a, c) in enumerate(sizes)]
    _check(g, grids, [1 + 5 * (k % 4) for k in range(len(grids))], (0, 2)[r % 2])


@pytest.mark.parametrize("shape", ["star", "box"])
@pytest.mark.parametrize("r", [1, 2, 3])
@pytest.mark.parametrize("depth", [1, 4, 16])
def test_tile_passes(g, shape, r, depth):
    sizes = [(129, 131), (257, 300), (40, 611), (700, 33), (220, 256 - 2 * r * min(depth, 13)), (128, 128)]
    grids = [(a, c, shape, r, (0.0, 0.5)[k % 2]) for k, (a, c) in enumerate(sizes)]
    _check(g, grids, [2, 9, 17, 16, 33, 5], 2 * (depth == 4),
           lambda lib, b: lib.stencil_batch_set_class(b, shape, r, "tiles", depth))


@pytest.mark.parametrize("shape,r,depth", [("star", 1, 8), ("star", 2, 5), ("star", 3, 4), ("box", 1, 6), ("box", 3, 2)])
def test_march_beside_tiles(g, shape, r, depth):
    # narrow and wide, odd widths, halos of zero (bands that start at the sides) and not
    sizes = [(300, 255), (300, 256), (200, 259), (190, 511), (180, 512), (170, 515), (90, 1027), (640, 130)]
    grids = [(a, c, shape, r, (0.0, 0.0, -1.0)[k % 3]) for k, (a, c) in enumerate(sizes)]
    _check(g, grids, [3, 10, 17, 8, 9, 16, 7, 12], 2 * (r == 1),
           lambda lib, b: lib.stencil_batch_set_class(b, shape, r, "march", depth))
