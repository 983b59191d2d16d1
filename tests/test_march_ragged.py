"""Row marching at odd widths: the layout that keeps every lane's vector inside the grid or outside it
(CPU), and bitwise parity with the FP32 oracle at the widths where bands move and on buffers that start
on no vector boundary (GPU)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
import workloads as wl

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="hipcc not found")
def test_ragged_layout(tmp_path):
    exe = str(tmp_path / "march_ragged_check")
    hipcc = HIPCC if os.path.exists(HIPCC) else shutil.which("hipcc")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", os.path.join(HERE, "march_ragged_check.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout + out.stderr


@pytest.fixture(scope="module")
def g():
    import gpuhelp
    return gpuhelp


@pytest.mark.gpu
@pytest.mark.parametrize("cols", [255, 256, 257, 263, 485, 487, 511, 513, 515, 751])
@pytest.mark.parametrize("shape,r,tb,storage,bc", [
    ("star", 1, 8, "f32", 0.5), ("star", 3, 4, "f32", 0.0), ("box", 2, 3, "f32", -1.0), ("star", 2, 5, "bf16", 0.0),
    ("box", 1, 4, "f16", 0.25), ("star", 2, 3, "f32", "periodic"), ("box", 3, 2, "f32", "frame"),
    ("star", 1, 6, "f16", "periodic")])
def test_ragged_march_bitwise(g, cols, shape, r, tb, storage, bc):
    """Zero tolerance: both sides run the same FP32 operations in the same order."""
    import torch
    import paper_2605_07954_amd as lib
    rows, steps = 37, tb + 1
    W = wl.random_footprint_weights(np.random.default_rng(r), shape, r)
    rng = np.random.default_rng(cols)
    u0 = rng.random((rows, cols), dtype=np.float32)
    host = u0 if storage == "f32" else oracle.to_bits(u0, storage)
    fixed = not isinstance(bc, str)
    frame = rng.random(oracle.frame_elems(rows, cols, r), dtype=np.float32) if bc == "frame" else None
    x0 = g.to_dev(host)

    def shifted(t):  # the same field one element past a vector boundary
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        v = buf[1:].view(t.shape)
        v.copy_(t)
        return v

    x, out, ws = shifted(x0), shifted(x0), shifted(x0)
    plan = lib.stencil_plan(rows, cols, r, W, bc if fixed else 0.0, storage, 0)
    fdev = g.to_dev(frame) if frame is not None else None
    try:
        lib.stencil_set_blocking(plan, 1, 0, 0)
        lib.stencil_set_variant(plan, lib.ST_VARIANT_MARCH)
        if not fixed:
            lib.stencil_set_boundary(plan, {"periodic": lib.ST_BC_PERIODIC, "frame": lib.ST_BC_FRAME}[bc], fdev)
        lib.stencil_set_blocking(plan, tb, 0, 0)
        lib.stencil_run(plan, x, out, steps, ws)
        got = g.to_host(out.contiguous())
    finally:
        lib.stencil_destroy(plan)
    if fixed:
        ref = (oracle.stencil_f32(u0, W, bc, steps) if storage == "f32" else oracle.stencil_lowp(host, W, bc, steps, storage))
    else:
        ref = (oracle.stencil_bc_f32(u0, W, bc, steps, frame) if storage == "f32"
               else oracle.stencil_bc_lowp(host, W, bc, steps, storage))
    np.testing.assert_array_equal(got, ref)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,shape,r,tb,storage,bc", [
    (37, 485, "box", 4, 2, "f32", "periodic"), (37, 515, "box", 4, 2, "bf16", "periodic"), (37, 751, "box", 4, 2, "f32", "frame"),
    (5000, 501, "star", 1, 4, "f32", "const"), (12000, 501, "star", 1, 6, "f16", "const"),
    (8003, 751, "box", 1, 6, "f32", "const"), (30001, 501, "star", 4, 3, "bf16", "const")])
def test_ragged_march_with_element_accesses(g, rows, cols, shape, r, tb, storage, bc):
    """Zero tolerance: both sides run the same FP32 operations in the same order."""
    import paper_2605_07954_amd as lib
    W = wl.random_footprint_weights(np.random.default_rng(r), shape, r)
    rng = np.random.default_rng(cols)
    u0 = rng.random((rows, cols), dtype=np.float32)
    host = u0 if storage == "f32" else oracle.to_bits(u0, storage)
    frame = rng.random(oracle.frame_elems(rows, cols, r), dtype=np.float32) if bc == "frame" else None
    x = g.to_dev(host)
    out, ws = x.clone(), x.clone()
    fdev = g.to_dev(frame) if frame is not None else None
    plan = lib.stencil_plan(rows, cols, r, W, 0.0, storage, 0)
    try:
        lib.stencil_set_blocking(plan, 1, 0, 0)
        lib.stencil_set_variant(plan, lib.ST_VARIANT_MARCH)
        if bc != "const":
            lib.stencil_set_boundary(plan, {"periodic": lib.ST_BC_PERIODIC, "frame": lib.ST_BC_FRAME}[bc], fdev)
        lib.stencil_set_blocking(plan, tb, 0, 0)
        lib.stencil_run(plan, x, out, tb + 1, ws)
        got = g.to_host(out)
    finally:
        lib.stencil_destroy(plan)
    if bc == "const":
        ref = (oracle.stencil_f32(u0, W, 0.0, tb + 1) if storage == "f32" else oracle.stencil_lowp(host, W, 0.0, tb + 1, storage))
    else:
        ref = (oracle.stencil_bc_f32(u0, W, bc, tb + 1, frame) if storage == "f32"
               else oracle.stencil_bc_lowp(host, W, bc, tb + 1, storage))
    np.testing.assert_array_equal(got, ref)
