"""What the library asks of the HIP runtime, on a host without a GPU: each test runs the library's host side
in a process of its own on a runtime that only writes the calls down (hip_stub.cpp).  Run as a script, this
file is that process; the tests read its log."""
import ctypes
import json
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = "/opt/rocm/include"
CALLER = 1000001  # the caller's stream

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM), reason="needs g++ and HIP headers")


# ---- in the process of its own ----------------------------------------------------------------------------
class Host:
    """The library on the stub, with its log."""

    def __init__(self, stub):
        self.stub = ctypes.CDLL(stub, mode=ctypes.RTLD_GLOBAL)
        self.stub.stub_log.restype = ctypes.c_char_p
        sys.modules["torch"] = None  # its own runtime stays out of this process
        sys.path.insert(0, os.path.dirname(HERE))
        import paper_2605_07954_amd as st
        self.st, self.lib = st, st.lib()

    def log(self):
        text = self.stub.stub_log().decode()
        self.stub.stub_clear()
        return [line.split(" ") for line in text.splitlines()]

    def weights(self, shape, r):
        k = 2 * r + 1
        w = np.full((k, k), 1.0 / (k * k), np.float32)
        if shape == "star":
            m = np.zeros((k, k), bool)
            m[r, :] = m[:, r] = True
            w[~m] = 0.0
        return w

    def fail(self, what, after):
        self.stub.stub_fail(what.encode(), after)


def case_batch(h, flags, fail=None, capturing=False):
    """Two runs of a batch of every kind of branch, a class changed by hand, a third run; its end."""
    grids = [(300, 700, "star", 1), (300, 700, "box", 2), (200, 90, "star", 1), (40, 50, "star", 3), (30, 40, "box", 1),
             (5, 900, "star", 2)]
    plans = [h.st.stencil_plan(a, c, r, h.weights(s, r), 0.0, "f32", 0) for a, c, s, r in grids]
    batch = h.st.stencil_batch_create(plans, [9] * len(grids), flags)
    fields = [[np.zeros((a, c), np.float32) for a, c, _, _ in grids] for _ in range(2)]
    ins, outs = ((ctypes.c_void_p * len(grids))(*[f.ctypes.data for f in fs]) for fs in fields)
    ws = np.zeros(h.st.stencil_batch_workspace_bytes(batch), np.uint8)

    def run():
        rc = h.lib.stencil_run_batched(batch, ins, outs, ws.ctypes.data, ws.nbytes, CALLER)
        return rc, h.log()

    if capturing:
        h.stub.stub_capturing(ctypes.c_void_p(CALLER))
    out = {"runs": [run(), run()]}
    h.st.stencil_batch_set_class(batch, "star", 1, "march", 4)
    if fail:
        h.fail(*fail)
    out["runs"].append(run())
    h.st.stencil_batch_destroy(batch)
    out["end"] = h.log()
    return out


def case_solve(h, first, gap=0):
    """A solve whose workspace lies right above its fields or right below them (or over the end of `out`)."""
    rows, cols = 200, 256
    plan = h.st.stencil_plan(rows, cols, 1, h.weights("star", 1), 0.0, "f32", 0)
    field, need = rows * cols * 4, h.st.stencil_solve_ws_bytes(plan, 8)
    mem = np.zeros(2 * field + need + 256, np.uint8)
    base = mem.ctypes.data + -mem.ctypes.data % 256
    ws, x = (base, base + (need + 255) // 256 * 256) if first == "workspace" else (base + 2 * field - gap, base)
    steps, rel = ctypes.c_int64(), ctypes.c_double()
    rc = h.lib.stencil_solve(plan, x, x + field, 16, 8, 0.0, ctypes.byref(steps), ctypes.byref(rel), ws, need, CALLER)
    return {"rc": rc, "kernels": [c[1].split("<")[0] for c in made(h.log(), "launch")]}


def case_run3d(h, dims, shape, r, storage, steps):
    """The kernels of a 3D run (on made-up device addresses)."""
    k = 2 * r + 1
    w = np.full((k, k, k), 0.01, np.float32)
    if shape == "star":
        w[(np.indices((k, k, k)) != r).sum(0) > 1] = 0.0
    plan = h.st.stencil_plan3d(*dims, r, w, 0.0, storage, 0)
    rc = h.lib.stencil_run(plan, 1 << 40, 2 << 40, steps, 3 << 40, h.st.stencil_workspace_bytes(plan, steps), CALLER)
    return {"rc": rc, "launches": made(h.log(), "launch")}


def case_synth(h, n, rows, cols):
    rc = h.lib.surrogate_synth_fields(1 << 40, n, rows, cols, 2 << 40, 3 << 40, CALLER)
    return {"rc": rc, "launches": made(h.log(), "launch")}


def case_run(h, rows, cols, shape, r, steps, storage="f32", tb=0, tile=(0, 0), shift=0):
    """The kernels of an untuned 2D run (on made-up device addresses, `shift` bytes off a 256-byte boundary)."""
    plan = h.st.stencil_plan(rows, cols, r, h.weights(shape, r), 0.5, storage, 0)
    if tb:
        h.st.stencil_set_blocking(plan, tb, *tile)
    rc = h.lib.stencil_run(plan, (1 << 40) + shift, 2 << 40, steps, 3 << 40, h.st.stencil_workspace_bytes(plan, steps), CALLER)
    return {"rc": rc, "launches": made(h.log(), "launch")}


def case_march(h, rows, cols, shape, r, storage, tb, bc):
    """The kernel of one pass of the marching variant."""
    plan = h.st.stencil_plan(rows, cols, r, h.weights(shape, r), 0.0, storage, 0)
    h.st.stencil_set_blocking(plan, 1)
    h.st.stencil_set_variant(plan, h.st.ST_VARIANT_MARCH)
    if bc != "const":
        frame = ctypes.c_void_p(4 << 40) if bc == "frame" else None
        assert h.lib.stencil_set_boundary(plan, {"periodic": h.st.ST_BC_PERIODIC, "frame": h.st.ST_BC_FRAME}[bc], frame) == 0
    h.st.stencil_set_blocking(plan, tb)
    rc = h.lib.stencil_run(plan, 1 << 40, 2 << 40, tb, 3 << 40, h.st.stencil_workspace_bytes(plan, tb), CALLER)
    return {"rc": rc, "kernels": [c[1] for c in made(h.log(), "launch") if "march" in c[1]]}


def case_varcoef(h, rows, cols, steps, tb, tile):
    plan = h.st.stencil_plan_varcoef(rows, cols, 0.0, 0)
    h.st.stencil_set_blocking(plan, tb, *tile)
    rc = h.lib.stencil_run_varcoef(plan, 1 << 40, 2 << 40, 3 << 40, steps, 4 << 40, h.st.stencil_workspace_bytes(plan, steps), CALLER)
    return {"rc": rc, "launches": made(h.log(), "launch")}


def case_occupancy(h):
    """Workgroups at once of one kernel, asked for 256, 1024 and 256 threads a workgroup."""
    fn = h.lib._ZN2st18resident_blocks_ofEPKvmiPi
    out = []
    for threads in (256, 1024, 256):
        n = ctypes.c_int()
        fn(ctypes.c_void_p(64), ctypes.c_size_t(0), ctypes.c_int(threads), ctypes.byref(n))
        out.append(n.value)
    return out


def case_batch_tuner(h, cols):
    """What the tuner picks for a class of grids of these widths, and how many runs of the batch it times."""
    plans = [h.st.stencil_plan(700, c, 2, h.weights("star", 2), 0.0, "f32", 0) for c in cols]
    batch = h.st.stencil_batch_create(plans, [30] * len(cols), 0)
    ptrs = [(ctypes.c_void_p * len(cols))(*[(f + 1 << 40) + (k << 32) for k in range(len(cols))]) for f in range(2)]
    ws = np.zeros(h.st.stencil_batch_workspace_bytes(batch), np.uint8)
    depth, engine = (ctypes.c_int * 6)(), (ctypes.c_int * 6)()
    rc = h.lib.stencil_batch_autotune(batch, *ptrs, ws.ctypes.data, ws.nbytes, depth, engine, CALLER)
    log = h.log()
    last = max(i for i, c in enumerate(log) if c[0] == "record")
    return {"rc": rc, "depth": depth[1], "engine": engine[1], "marched": any("march" in c[1] for c in log[:last] if c[0] == "launch"),
            "runs": len(made(log, "record"))}


def case_graph(h, kind):
    """Graphs made and replayed by runs of a plan, each call a change of one thing (or of none)."""
    heat = kind == "varcoef"
    plan = h.st.stencil_plan_varcoef(64, 64, 0.0, 2) if heat else h.st.stencil_plan(64, 64, 1, h.weights("star", 1), 0.0, "f32", 2)
    h.st.stencil_set_blocking(plan, 2)
    base = dict(x=1 << 40, k=2 << 40, out=3 << 40, ws=4 << 40, steps=24, stream=CALLER)
    out = []
    for change in ({}, {}, {"x": 5 << 40}, {}, {"out": 6 << 40}, {"ws": 7 << 40}, {"steps": 26}, {"stream": CALLER + 1}, {},
                   {"k": 8 << 40}, {}, {"steps": 16}, {"steps": 24}):
        base.update(change)
        a = [base["x"]] + ([base["k"]] if heat else []) + [base["out"], base["steps"], base["ws"], 64 * 64 * 4, base["stream"]]
        rc = (h.lib.stencil_run_varcoef if heat else h.lib.stencil_run)(plan, *a)
        log = h.log()
        live = len(made(log, "exec")) - len(made(log, "exec-"))
        out.append([rc, len(made(log, "captured")), len(made(log, "replay")), live])
    h.st.stencil_destroy(plan)
    return {"calls": out, "end": len(made(h.log(), "exec-"))}


def case_tuner(h, rows, cols, steps):
    """The register-tile kernels that the tuner of a star of r = 1 times, and the tile and depth it keeps."""
    plan = h.st.stencil_plan(rows, cols, 1, h.weights("star", 1), 0.0, "f32", 0)
    tb, tx, ty = (ctypes.c_int() for _ in range(3))
    need = h.st.stencil_workspace_bytes(plan, 2) + (64 << 20)
    rc = h.lib.stencil_autotune(plan, 1 << 40, 2 << 40, 3 << 40, need, steps, *map(ctypes.byref, (tb, tx, ty)), CALLER)
    return {"rc": rc, "launches": made(h.log(), "launch"), "kept": [tb.value, tx.value, ty.value]}


CASES = {k[5:]: f for k, f in list(globals().items()) if k.startswith("case_")}


# ---- the tests --------------------------------------------------------------------------------------------
@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    r = subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM,
                        os.path.join(HERE, "hip_stub.cpp"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return so


def ask(stub, case, **kw):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, case, json.dumps(kw)], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    return json.loads(r.stdout)


def unjoined(log):
    """Streams that hold a launch which the caller's stream does not wait for by the end of the log."""
    dirty, at = set(), {}
    for c in log:
        if c[0] == "launch" and c[-1] != str(CALLER):
            dirty.add(c[-1])
        elif c[0] == "record":
            at[c[1]] = c[2]
        elif c[0] == "wait" and c[1] == str(CALLER):
            dirty.discard(at.get(c[2]))
        elif c[0] == "sync":
            dirty.discard(c[1])
    return dirty


def made(log, what):
    return [c for c in log if c[0] == what]


@pytest.mark.parametrize("flags", [0, 2])
def test_batch_captures_nothing(stub, flags):
    res = ask(stub, "batch", flags=flags)
    whole = [c for _, log in res["runs"] for c in log] + res["end"]
    assert all(rc == 0 for rc, _ in res["runs"])
    for what in ("capture", "captured", "exec", "replay"):
        assert not made(whole, what)
    streams = {c[-1] for c in made(whole, "launch")}
    assert (len(streams) > 3) if flags else streams == {str(CALLER)}
    for _, log in res["runs"]:
        assert made(log, "launch") and not unjoined(log)
        assert not made(log, "stream-") and not made(log, "event-")
    assert not made(res["runs"][1][1], "stream") and not made(res["runs"][1][1], "event")  # made once
    # the end waits for each stream before it goes
    gone = {c[1] for c in made(res["end"], "stream-")}
    assert gone == {c[1] for c in made(whole, "stream")}
    for s in gone:
        assert res["end"].index(["sync", s]) < res["end"].index(["stream-", s])


@pytest.mark.parametrize("what,after", [("launch", 0), ("launch", 2), ("launch", 6), ("wait", 3), ("wait", 4), ("stream", 0)])
def test_batch_joins_what_a_failed_run_enqueued(stub, what, after):
    res = ask(stub, "batch", flags=2, fail=[what, after])
    rc, log = res["runs"][2]
    assert rc == -4 and not unjoined(log)


def test_batch_under_capture_stays_on_the_stream(stub):
    res = ask(stub, "batch", flags=2, capturing=True)
    for rc, log in res["runs"]:
        assert rc == 0 and {c[-1] for c in made(log, "launch")} == {str(CALLER)}
        assert not made(log, "wait") and not made(log, "stream")


def test_solve_does_not_depend_on_where_its_buffers_lie(stub):
    above, below = ask(stub, "solve", first="fields"), ask(stub, "solve", first="workspace")
    assert above["kernels"].count("sweep_block_sums") == 2  # the residual comes from each interval's last pass
    assert above == below
    # a workspace that overlaps `out` is refused, as stencil_run refuses it
    assert ask(stub, "solve", first="fields", gap=256)["rc"] == -2


@pytest.mark.parametrize("dims,shape,r,storage,ring", [
    ((512, 512, 512), "star", 1, "f32", True), ((256, 256, 256), "star", 1, "f32", True), ((512, 512, 512), "star", 2, "f32", True),
    ((300, 300, 300), "star", 1, "f32", False), ((128, 128, 128), "star", 1, "f32", False), ((400, 400, 400), "star", 2, "f32", False),
    ((512, 512, 512), "star", 1, "bf16", False), ((512, 512, 512), "box", 1, "f32", False)])
def test_3d_single_levels(stub, dims, shape, r, storage, ring):
    """One level of a large FP32 star goes where it is fastest; runs of several levels stay on register tiles."""
    one = ask(stub, "run3d", dims=dims, shape=shape, r=r, storage=storage, steps=1)
    assert one["rc"] == 0 and len(one["launches"]) == 1
    assert one["launches"][0][1].startswith("sweep3d<") == ring
    for c in ask(stub, "run3d", dims=dims, shape=shape, r=r, storage=storage, steps=8)["launches"]:
        assert c[1].startswith("sweep3d_block")


@pytest.mark.parametrize("n,rows,cols,kernel,grid", [(1, 100, 100, "<16,4>", 14), (1, 1024, 1024, "<16,4>", 1024),
                                                     (4, 1024, 1024, "<64,1>", 256)])
def test_synthesis_tiles(stub, n, rows, cols, kernel, grid):
    """Small fields share a column's factors among threads; a thread alone takes as long as a large field."""
    res = ask(stub, "synth", n=n, rows=rows, cols=cols)
    assert res["rc"] == 0 and res["launches"] == [["launch", "synth_kernel" + kernel, str(grid), "256", str(CALLER)]]


@pytest.mark.parametrize("rows,shape,r,tb,tile,kernel", [
    (2000, "star", 3, 8, (64, 64), "2,8,16"), (2000, "star", 4, 4, (64, 64), "2,8,16"), (300, "star", 4, 4, (128, 32), "1,8,8"),
    (2000, "star", 1, 8, (64, 64), "1,8,8"), (2000, "star", 1, 6, (128, 64), "2,8,8"), (2000, "box", 2, 4, (256, 32), "4,4,8")])
def test_tiles_that_margins_use_up(stub, rows, shape, r, tb, tile, kernel):
    """A pass whose margins would leave little of the plan's tile takes another; the others keep it."""
    res = ask(stub, "run", rows=rows, cols=rows, shape=shape, r=r, steps=3 * tb, tb=tb, tile=tile)
    assert res["rc"] == 0
    assert {c[1] for c in res["launches"]} == {f"sweep_block<0,{r},{int(shape == 'box')},{kernel}>"}


@pytest.mark.parametrize("rows,cols,shape,r,tb,tile,kernel", [
    (1040, 432, "star", 1, 16, (64, 64), "1,8,8"), (1500, 900, "star", 3, 3, (256, 32), "4,4,8"),
    (2000, 2000, "box", 1, 12, (64, 64), "2,8,8")])
def test_tiles_by_the_most_one_unit_gets(stub, rows, cols, shape, r, tb, tile, kernel):
    """Tiles whose margins are wide are weighed by how many of them the busiest compute unit takes."""
    res = ask(stub, "run", rows=rows, cols=cols, shape=shape, r=r, steps=3 * tb, tb=tb, tile=tile)
    assert res["rc"] == 0
    assert {c[1] for c in res["launches"]} == {f"sweep_block<0,{r},{int(shape == 'box')},{kernel}>"}


@pytest.mark.parametrize("rows,cols,shape,r,storage,kw,kernel", [
    (1024, 1024, "star", 1, "f32", {}, "sweep_step"), (8192, 8192, "star", 1, "f32", {}, "sweep_step"),
    (2000, 3000, "star", 4, "bf16", {}, "sweep_step"), (4096, 4096, "box", 4, "bf16", {}, "sweep_step"),
    (4096, 4096, "star", 1, "bf16", {}, "sweep_march"), (4096, 4096, "star", 3, "f16", {}, "sweep_march"),
    (8192, 8192, "star", 1, "f16", {}, "sweep_step"), (4096, 4096, "box", 3, "f32", {}, "sweep_march"),
    (250000, 40, "box", 4, "f32", {}, "sweep_march"), (1024, 1023, "star", 1, "f32", {}, "sweep_block"),
    (1024, 1020, "star", 1, "bf16", {}, "sweep_block"), (1024, 1024, "star", 1, "f32", {"shift": 4}, "sweep_block"),
    (1024, 1024, "star", 1, "f32", {"shift": 16}, "sweep_step"), (300, 300, "box", 3, "f32", {"tb": 1, "tile": (64, 64)}, "sweep_block"),
    (2000, 3000, "box", 4, "f32", {"tb": 1, "tile": (64, 64)}, "sweep_step"),
    (300, 300, "box", 4, "f32", {"tb": 1, "tile": (256, 32)}, "sweep_step"), (60000, 200, "box", 3, "f32", {}, "sweep_march"),
    (40, 250000, "star", 3, "f32", {}, "sweep_march"), (100000, 256, "box", 1, "bf16", {}, "sweep_step")])
def test_single_steps(stub, rows, cols, shape, r, storage, kw, kernel):
    """One step of an untuned plan runs where it is fastest; what LDS tiles cannot load whole goes elsewhere."""
    res = ask(stub, "run", rows=rows, cols=cols, shape=shape, r=r, steps=1, storage=storage, **kw)
    assert res["rc"] == 0 and [c[1].split("<")[0] for c in res["launches"]] == [kernel]


@pytest.mark.parametrize("rows,cols,r,storage,single", [
    (1000, 2000, 4, "f32", True), (1000, 2000, 3, "bf16", True), (4096, 4096, 3, "f16", True), (15625, 128, 3, "f32", True), (5000, 400, 4, "f32", False), (666, 3000, 3, "bf16", False),
    (1000, 1000, 4, "f32", False), (4096, 4096, 3, "f32", False), (6000, 8192, 3, "f32", False)])
def test_large_boxes_take_single_steps(stub, rows, cols, r, storage, single):
    runs = {n: ask(stub, "run", rows=rows, cols=cols, shape="box", r=r, steps=n, storage=storage) for n in (2, 7)}
    assert all(run["rc"] == 0 for run in runs.values())
    assert len(runs[2]["launches"]) == 1  # no workspace was asked for
    assert len(runs[7]["launches"]) == (7 if single else 4)
    assert not single or {c[1].split("<")[0] for c in runs[7]["launches"]} == {"sweep_step"}


@pytest.mark.parametrize("rows,cols,shape,r,kernel", [
    (625000, 64, "box", 3, "sweep_march<0,3,1,"), (40000, 1000, "box", 3, "sweep_march<0,3,8,"), (76923, 520, "box", 3, "sweep_march<0,3,1,"),
    (57142, 700, "box", 3, "sweep_march_w3<0,3,4,"), (250000, 40, "star", 2, "sweep_block"), (250000, 40, "box", 1, "sweep_block"),
    (250000, 40, "star", 3, "sweep_march"), (3000, 4000, "star", 2, "sweep_march<0,2,4,")])
def test_marching_of_narrow_grids(stub, rows, cols, shape, r, kernel):
    """Bands that a narrow grid would leave empty are not taken, however many rows it has."""
    res = ask(stub, "run", rows=rows, cols=cols, shape=shape, r=r, steps=12)
    assert res["rc"] == 0 and all(c[1].startswith(kernel) for c in res["launches"])


@pytest.mark.parametrize("rows,cols,shape,r,storage,tb,bc,elements", [
    (1000, 701, "box", 4, "bf16", 2, "periodic", True), (1000, 701, "box", 4, "f32", 2, "frame", True),
    (1000, 701, "box", 4, "bf16", 2, "frame", False), (1000, 701, "box", 4, "f32", 1, "periodic", False),
    (1000, 704, "box", 4, "f32", 2, "periodic", False), (2000, 2003, "star", 1, "f32", 4, "const", True),
    (1000, 701, "star", 1, "f32", 4, "const", False), (2000, 2003, "star", 1, "bf16", 4, "const", False),
    (2000, 2003, "box", 1, "f16", 6, "const", True), (2000, 2003, "star", 1, "f32", 6, "const", False),
    (3000, 3002, "star", 1, "bf16", 6, "const", True), (3000, 3002, "star", 1, "f16", 5, "const", True),
    (4099, 5003, "star", 4, "f16", 3, "const", True), (4099, 5003, "star", 4, "f32", 3, "const", False)])
def test_marching_with_element_accesses(stub, rows, cols, shape, r, storage, tb, bc, elements):
    res = ask(stub, "march", rows=rows, cols=cols, shape=shape, r=r, storage=storage, tb=tb, bc=bc)
    assert res["rc"] == 0 and len(res["kernels"]) == 1
    args = res["kernels"][0].split("<")[1].split(">")[0].split(",")
    assert args[2] == "4" and (args[5] == "false") == elements, res["kernels"]


@pytest.mark.parametrize("case,kw,blocks", [
    ("varcoef", dict(rows=140000, cols=140000, steps=8, tb=8, tile=(64, 64)), 2917 ** 2),
    ("run", dict(rows=140000, cols=140000, shape="box", r=4, storage="bf16", steps=2, tb=2, tile=(64, 64)), 2917 ** 2),
    ("run3d", dict(dims=(1, 150000, 150001), shape="star", r=1, storage="f32", steps=1), 2420 ** 2),
    ("run3d", dict(dims=(2, 150000, 150001), shape="box", r=1, storage="bf16", steps=1), None)])
def test_more_threads_than_a_launch_holds(stub, case, kw, blocks):
    """Fields that fit the device's memory with more tiles than one launch has threads for."""
    res = ask(stub, case, **kw)
    assert res["rc"] == 0
    work = [int(c[2]) * int(c[3]) for c in res["launches"]]
    assert len(work) > 1 and sum(work) >= 2 ** 32 > max(work)
    assert blocks is None or blocks == sum(int(c[2]) for c in res["launches"])


def test_occupancy_is_kept_by_workgroup_size(stub):
    assert ask(stub, "occupancy") == [1024, 256, 1024]  # the stub's compute units hold 1024 threads


def test_batch_tuner_of_narrow_grids(stub):
    """A class that never marches (all its grids narrower than a band) is tuned over its tiles alone."""
    narrow, wide = ask(stub, "batch_tuner", cols=[100, 200, 255]), ask(stub, "batch_tuner", cols=[100, 200, 256])
    assert narrow["rc"] == wide["rc"] == 0
    assert wide["engine"] == 1 and wide["marched"]
    assert narrow["engine"] == 0 and not narrow["marched"] and narrow["depth"] in (1, 2, 3, 4, 6, 8, 12, 16)
    assert narrow["runs"] < wide["runs"]


@pytest.mark.parametrize("kind", ["const", "varcoef"])
def test_graph_is_made_again_for_whatever_changes(stub, kind):
    """Runs of more than eight passes replay one graph per (input, diffusivity, output, workspace, steps, stream)."""
    res = ask(stub, "graph", kind=kind)
    k = int(kind == "varcoef")  # a constant plan has no diffusivity to change
    # 16 steps are eight passes, enqueued directly; 24 after them find the graph as it was, but for their steps
    assert [c[0] for c in res["calls"]] == [0] * 13
    assert [c[1] for c in res["calls"]] == [1, 0, 1, 0, 1, 1, 1, 1, 0, k, 0, 0, 1]
    assert [c[2] for c in res["calls"]] == [1] * 11 + [0, 1]
    assert sum(c[3] for c in res["calls"]) == 1 == res["end"]  # one graph at a time


def test_tuner_times_a_replaced_tile_once(stub):
    """48 steps of 2048^2 at 16 levels: three passes each on the tallest tile, for the tiles that cannot hold the
    depth at all; the ones it replaces are not timed again under their own name."""
    res = ask(stub, "tuner", rows=2048, cols=2048, steps=48)
    assert res["rc"] == 0
    tall = [c for c in res["launches"] if c[1] == "sweep_block<0,1,0,2,8,16>" and int(c[2]) == 22 * 22]
    assert len(tall) == 2 * 3 * 3  # two tiles, three runs of three passes


if __name__ == "__main__":
    print(json.dumps(CASES[sys.argv[2]](Host(sys.argv[1]), **json.loads(sys.argv[3]))))
