"""The host runtime's launches, streams and captures, on the CPU: dock_runtime.cpp built
against a model of HIP streams (tests/host/hip_stub.cpp)."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libdock_stub.so")
    inc = [a for d in ("/opt/rocm/include", os.path.join(ROOT, "include"),
                       os.path.join(ROOT, "paper_2209_05069_amd", "csrc")) for a in ("-I", d)]
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-Wl,-Bsymbolic",
                    "-D__HIP_PLATFORM_AMD__", *inc,
                    os.path.join(ROOT, "tests", "host", "hip_stub.cpp"), "-o", so], check=True)
    return so


@pytest.fixture
def D(stub, monkeypatch):
    from paper_2209_05069_amd import dock
    monkeypatch.setattr(dock, "LIBPATH", stub)
    monkeypatch.setattr(dock, "_lib", None)
    L = dock.lib()
    L.stub_log.restype = ctypes.c_char_p
    for f in (L.stub_hold, L.stub_capture):
        f.argtypes = [ctypes.c_void_p, ctypes.c_int]
    L.stub_idle.argtypes = [ctypes.c_void_p]
    L.stub_fail.argtypes = [ctypes.c_char_p, ctypes.c_int]
    L.stub_allocs.restype = ctypes.c_longlong
    return dock


@pytest.fixture
def ctx(D):
    c = D.dock_create(0)
    yield c
    D.dock_destroy(c)


def _job(D, ctx, ligands, atoms=(12, 40), pid=None, restarts=None, **kw):
    # (large lists have restarts enough to run in thirds)
    restarts = restarts or (4 if ligands < 2000 else 256)
    pk = synth.pocket_gaussians(7, 2, 8, 0.5, 4, 1.0)
    if pid is None:
        pid = D.dock_pocket_load(ctx, pk.values, pk.spacing, pk.origin)
    lib = synth.library_uniform(ligands, ligands, atoms, (0, 2))
    params = D.SearchParams(synth.start_quats(3, restarts), torsion_steps=8, sweep_passes=1, **kw)
    dl = D.DeviceLibrary(lib, device="cpu")
    res = D.DeviceResults(ligands, dl.n_atoms_total, dl.n_rot_total, params, device="cpu")
    return pid, dl, params, res


def _log(D):
    return D.lib().stub_log().decode().splitlines()


# ---------------------------------------------------------------------------


@pytest.mark.parametrize("top_k", [1, 2, 30])
@pytest.mark.parametrize("waves", [2, 4, 8])
@pytest.mark.parametrize("ligands", [1, 2, 3, 7, 40, 2100])
def test_every_share_of_a_split_final_step_has_a_workgroup(D, ctx, ligands, waves, top_k):
    # with the per-XCD split, share x of a list's ligands is taken by the workgroups
    # b with b % xcds == x: fewer workgroups than shares leave ligands undone
    job = _job(D, ctx, ligands, top_k=top_k)
    pid, dl, params, res = job
    tile = dict(ligands=1, dock_waves=4, select_waves=4, falign_waves=waves, falign_xcd=1)
    D.dock_set_tuning(ctx, params, [tile] * D.NUM_BINS)
    _log(D)
    D.dock_ligands_batch(ctx, pid, dl, params, res, 0x77)
    seen = [m.groups() for m in (re.match(r"falign .* blocks=(\d+) .*xcds=(\d+)", line)
                                 for line in _log(D)) if m]
    assert seen
    for blocks, xcds in seen:
        assert int(xcds) <= 1 or int(blocks) >= int(xcds)
    if ligands >= 2000:  # still split where there are workgroups enough
        assert any(int(x) == 8 for _, x in seen)


@pytest.mark.parametrize("ligands,bin_mode", [(7, 0), (2100, 0), (60, 1)])
def test_calls_on_other_streams_do_not_wait_for_a_stuck_one(D, ctx, ligands, bin_mode):
    # stream 0x51 still runs something of the caller's: its call waits for that, and
    # calls on other streams and submitted work do not
    L = D.lib()
    pid, dl, params, res = _job(D, ctx, ligands, (12, 200), bin_mode=bin_mode)
    other = _job(D, ctx, 5, (12, 200), pid=pid)
    _, _, params2, _ = other
    host = synth.library_uniform(4, 4, (12, 100), (0, 2))
    hres = D.HostResults(4, int(host.atom_off[-1]), int(host.rot_off[-1]), params2)
    D.dock_ligands_batch(ctx, pid, dl, params, res, 0x51)
    L.stub_all_idle()
    L.stub_hold(0x51, 1)
    _log(D)
    D.dock_ligands_batch(ctx, pid, dl, params, res, 0x51)
    # nothing waits for it in another stream (whose hardware queue others may share)
    assert {line.split("stream=")[1].split()[0] for line in _log(D)} == {str(0x51)}
    D.dock_ligands_batch(ctx, pid, other[1], params2, other[3], 0x52)
    assert L.stub_idle(0x52)
    D.dock_ligands_batch_noalloc(ctx, pid, other[1], params2, other[3], 0x53)
    assert L.stub_idle(0x53)
    tickets = [D.dock_submit(ctx, pid, host, params2, hres) for _ in range(5)]
    assert all(D.dock_poll(ctx, t) for t in tickets)
    assert not L.stub_idle(0x51)
    L.stub_hold(0x51, 0)
    assert L.stub_idle(0x51) and L.stub_all_idle()
    # the side streams are free: the next calls run their lists side by side, one behind
    # the other on one stream too
    for _ in range(3):
        _log(D)
        D.dock_ligands_batch(ctx, pid, dl, params, res, 0x54)
        assert len({line.split("stream=")[1] for line in _log(D) if line.startswith("dock ")}) == 3
    L.stub_all_idle()


def test_captured_sequences_keep_to_one_stream(D, ctx):
    # two requests of different lists in flight: what is captured for a replay is one
    # stream's sequence (no branches)
    L = D.lib()
    pid, dl, params, res = _job(D, ctx, 40, (12, 200))
    for held in (False, True):
        D.dock_ligands_batch(ctx, pid, dl, params, res, 0x61)
        L.stub_hold(0x61, 1 if held else 0)
        for _ in range(3):
            D.dock_ligands_batch(ctx, pid, dl, params, res, 0x61)
            D.dock_ligands_batch(ctx, pid, dl, params, res, 0x62)
    L.stub_hold(0x61, 0)
    log = _log(D)
    assert any(line.startswith("graph ") for line in log)
    captured = [line for line in log if line.endswith("captured")]
    assert captured and {re.search(r"stream=(\d+)", line).group(1) for line in captured} == {str(0x62)}
    assert L.stub_all_idle()


def test_cached_sequences_are_not_destroyed_in_flight(D, ctx):
    # more distinct repeated requests than the cache holds, all still running
    L = D.lib()
    big = _job(D, ctx, 60, (20, 20))
    pid = big[0]
    # (of one list each: a list for one stream has no side streams to use)
    jobs = [_job(D, ctx, 1 + i % 3, (9, 9 + i // 12), pid=pid) for i in range(40)]
    D.dock_ligands_batch(ctx, pid, *big[1:], 0x63)  # the stream's workspace
    L.stub_hold(0x63, 1)
    for _ in range(2):
        for _, dl, params, res in jobs:
            D.dock_ligands_batch(ctx, pid, dl, params, res, 0x63)
    log = _log(D)
    assert sum(line.startswith("graph stream") for line in log) >= 8, log
    assert not any("in flight" in line for line in log)
    L.stub_hold(0x63, 0)
    assert L.stub_all_idle()
    for _, dl, params, res in jobs[20:] + jobs[20:]:  # done: they make room
        D.dock_ligands_batch(ctx, pid, dl, params, res, 0x63)
    log = _log(D)
    assert any(line.startswith("graph destroyed") for line in log)
    L.stub_all_idle()


@pytest.mark.parametrize("ligands", [40, 2100])
@pytest.mark.parametrize("name", ["launch", "hipEventRecord", "hipStreamWaitEvent"])
def test_a_failed_call_leaves_nothing_beside_its_stream(D, ctx, name, ligands):
    # whatever call of the runtime fails: what was launched on side streams is behind the
    # caller's stream, or waited for, when the entry point returns (the caller may free
    # its buffers then)
    L = D.lib()
    pid, dl, params, res = _job(D, ctx, ligands, (12, 200))
    D.dock_ligands_batch(ctx, pid, dl, params, res, 0x71)
    L.stub_all_idle()
    failed = 0
    for nth in range(1, 60):
        _log(D)
        L.stub_fail(name.encode(), nth)
        try:
            D.dock_ligands_batch(ctx, pid, dl, params, res, 0x71)
        except D.DockError:
            failed += 1
        L.stub_fail(name.encode(), 0)
        ops = [re.match(r"(.*) stream=(\d+)", line).groups() for line in _log(D)]
        for t in {s for _, s in ops} - {str(0x71)}:
            mine = [i for i, (op, s) in enumerate(ops) if s == t and op not in ("record", "wait")]
            if not mine or ops[mine[-1]][0] == "synchronize":
                continue
            rec = [i for i, (op, s) in enumerate(ops) if s == t and op == "record" and i > mine[-1]]
            assert rec and ("wait", str(0x71)) in ops[rec[0]:], (nth, t, ops)
        assert L.stub_all_idle()
    assert failed >= (30 if name == "launch" else 4)
    D.dock_ligands_batch(ctx, pid, dl, params, res, 0x71)  # the context is as before


@pytest.mark.parametrize("ligands,atoms", [(40, (12, 200)), (5, (9, 20)), (2100, (12, 60))])
def test_a_callers_capture_keeps_to_its_stream(D, ctx, ligands, atoms):
    # also of a call that the stream has had before, and of one with a cached replay: the
    # launches go to the caller's capture, and no later call frees what they use
    L = D.lib()
    pid, dl, params, res = _job(D, ctx, ligands, atoms)
    big = _job(D, ctx, 2 * ligands, atoms, pid=pid)
    for warm in range(4):
        L.stub_all_idle()
        L.stub_capture(0x81, 1)
        _log(D)
        D.dock_ligands_batch(ctx, pid, dl, params, res, 0x81)
        log = _log(D)
        L.stub_capture(0x81, 0)
        assert any(line.startswith("dock ") for line in log)
        assert all(line.split("stream=")[1] == str(0x81) for line in log)
        assert not any(line.startswith(("graph", "beginCapture", "synchronize")) for line in log)
        D.dock_ligands_batch(ctx, pid, dl, params, res, 0x81)
    L.stub_all_idle()
    _log(D)
    D.dock_ligands_batch(ctx, big[0], big[1], big[2], big[3], 0x81)
    assert not any(line.startswith("free") for line in _log(D))
    L.stub_all_idle()


def test_bounds_are_taken_where_few_orientations_stay(D, ctx):
    # per atom bin; a pocket where they pay for no bin gives the tables' memory back
    L = D.lib()

    def route(pid=None):
        pid, dl, params, res = _job(D, ctx, 40, (20, 250), pid=pid)
        _log(D)
        D.dock_ligands_batch(ctx, pid, dl, params, res, 0x91)
        L.stub_all_idle()
        pairs = [re.match(r"(align\w*) bin=(\d)", line) for line in _log(D)]
        return pid, {int(m.group(2)): m.group(1) for m in pairs if m}

    few, _ = route()
    assert set(route(few)[1].values()) == {"align_bound"}
    for b in (1, 4, 7):
        L.stub_stay(b, 900)
    before = L.stub_allocs()
    some, got = route()
    assert got == {b: "align" if b in (1, 4, 7) else "align_bound" for b in range(8)}
    with_tables = L.stub_allocs() - before
    for b in range(8):
        L.stub_stay(b, 900)
    before = L.stub_allocs()
    none, got = route()
    assert set(got.values()) == {"align"}
    assert L.stub_allocs() - before == with_tables - 1
    for b in range(8):
        L.stub_stay(b, 0)
    assert set(route(few)[1].values()) == {"align_bound"}  # each pocket keeps its own


@pytest.mark.parametrize("shape,bins", [((64, 64, 64), range(8)), ((24, 24, 24), (0, 1)),
                                        ((64, 64, 24), (0, 1)), ((8, 8, 8), ())])
def test_bounds_need_fewer_orientations_where_ligands_reach_out_of_the_grid(D, ctx, shape, bins):
    # 60 of 900 are few for every bin inside the grid (its limits are 95 to 200)
    L = D.lib()
    for b in range(8):
        L.stub_stay(b, 60)
    pid = D.dock_pocket_load(ctx, np.zeros((2,) + shape, np.float32), 0.5, (0.0, 0.0, 0.0))
    for b in range(8):
        L.stub_stay(b, 0)
    _, dl, params, res = _job(D, ctx, 40, (20, 250), pid=pid)
    _log(D)
    D.dock_ligands_batch(ctx, pid, dl, params, res, 0x92)
    L.stub_all_idle()
    pairs = [re.match(r"(align\w*) bin=(\d)", line) for line in _log(D)]
    got = {int(m.group(2)): m.group(1) for m in pairs if m}
    assert got == {b: "align_bound" if b in bins else "align" for b in range(8)}


@pytest.mark.parametrize("ligands,atoms,restarts,parts", [
    (2047, (200, 250), 256, 1), (2048, (200, 250), 256, 3), (2048, (200, 250), 4, 1),
    (2100, (1, 1), 256, 1), (9000, (1, 12), 20, 1), (9000, (1, 12), 400, 3)])
def test_libraries_with_little_work_are_not_split(D, ctx, ligands, atoms, restarts, parts):
    # in thirds from 2,048 ligands and 10 million restarts x atoms on
    pid, dl, params, res = _job(D, ctx, ligands, atoms, restarts=restarts)
    _log(D)
    D.dock_ligands_batch(ctx, pid, dl, params, res, 0xA2)
    D.lib().stub_all_idle()
    bins = [m.group(1) for m in (re.match(r"dock bin=(\d)", line) for line in _log(D)) if m]
    assert bins and {bins.count(b) for b in bins} == {parts}


@pytest.mark.parametrize("sample", [60, 2100])
def test_tuned_tiles_are_those_of_the_form_that_runs(D, ctx, sample):
    # the model's selection is faster alone with 16 waves, and slower beside a sweep: a
    # library in thirds keeps 4 waves, a short list takes the 16
    pid, dl, params, res = _job(D, ctx, sample, (12, 120), restarts=256)
    table = D.dock_autotune(ctx, pid, dl, params, 0xA1)
    assert {t["select_waves"] for t in table if t["ligands"]} == {16 if sample < 2048 else 4}
    for n, waves in ((60, 16), (2100, 4)):
        _, dl, _, res = _job(D, ctx, n, (12, 120), pid=pid, restarts=256)
        _log(D)
        D.dock_ligands_batch(ctx, pid, dl, params, res, 0xA1)
        D.lib().stub_all_idle()
        seen = [re.match(r"select .* waves=(\d+)", line) for line in _log(D)]
        assert {int(m.group(1)) for m in seen if m} == {waves}
