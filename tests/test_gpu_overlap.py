"""Work lists side by side on several streams: the same results as one list after the
other, for lists on streams of their own, for a library split into parts, with the
next call on the same stream right behind, and under a caller's capture."""
import numpy as np
import pytest

import synth
from tests.test_gpu_parity import D, ctx  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
KEYS = ("best_score", "n_poses", "status", "pose_score", "pose_restart", "pose_xyz")


def _setup(D, ctx, L, atoms, seed, **kw):  # noqa: F811
    pk = synth.pocket_gaussians(seed, 4, 32, 0.5, 40, 4.0)
    lib = synth.library_uniform(seed, L, atoms, (0, 3))
    params = D.SearchParams(synth.start_quats(seed, 4), torsion_steps=16, sweep_passes=1,
                            top_k=2, **kw)
    pid = D.dock_pocket_load(ctx, pk.values, pk.spacing, pk.origin)
    dl = D.DeviceLibrary(lib)
    return pid, params, dl, [D.DeviceResults(L, dl.n_atoms_total, dl.n_rot_total, params)
                             for _ in range(3)]


def _same(a, b):
    for k in KEYS:
        np.testing.assert_array_equal(getattr(a, k).cpu().numpy(), getattr(b, k).cpu().numpy(),
                                      err_msg=k)


@pytest.mark.parametrize("L,atoms,bin_mode", [
    (1, (9, 9), 0), (7, (3, 200), 0), (60, (3, 256), 1), (2047, (3, 40), 0),
    (2048, (3, 70), 0), (2050, (3, 33), 0), (2100, (3, 70), 1)])
def test_overlapped_lists_are_the_sequence(D, ctx, L, atoms, bin_mode):  # noqa: F811
    # (phase timing keeps a call to one stream: the sequence to compare with)
    pid, params, dl, (ref, got, rep) = _setup(D, ctx, L, atoms, 90 + L % 7, bin_mode=bin_mode)
    print(f"[case] overlap L={L} bin_mode={bin_mode}", flush=True)
    D.dock_set_timing(ctx, True)
    D.dock_ligands_batch(ctx, pid, dl, params, ref)
    D.dock_set_timing(ctx, False)
    D.dock_get_timing(ctx)
    D.dock_ligands_batch(ctx, pid, dl, params, got)
    # repeated on a stream of its own: eager, captured, replayed, with eager calls between
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    for _ in range(4):
        D.dock_ligands_batch(ctx, pid, dl, params, rep, st)
        D.dock_ligands_batch(ctx, pid, dl, params, got, st)
    torch.cuda.synchronize()
    _same(ref, got)
    _same(ref, rep)
    D.dock_pocket_unload(ctx, pid)


@pytest.mark.parametrize("L,atoms,restarts,kw", [
    (2048, (60, 70), 80, {}),                  # the least in thirds: 10 million atoms to place
    (2050, (3, 70), 256, {}), (2100, (200, 256), 40, {}),
    (2100, (3, 70), 256, dict(bin_mode=1))])
def test_thirds_of_a_library_are_the_sequence(D, ctx, L, atoms, restarts, kw):  # noqa: F811
    pid, _, dl, _ = _setup(D, ctx, L, atoms, 90 + L % 7)
    params = D.SearchParams(synth.start_quats(7, restarts), torsion_steps=16, sweep_passes=1,
                            top_k=5, **kw)
    ref, got, rep = [D.DeviceResults(L, dl.n_atoms_total, dl.n_rot_total, params) for _ in range(3)]
    print(f"[case] thirds L={L} R={restarts} {kw}", flush=True)
    D.dock_set_timing(ctx, True)
    D.dock_ligands_batch(ctx, pid, dl, params, ref)
    D.dock_set_timing(ctx, False)
    D.dock_get_timing(ctx)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    for _ in range(3):
        D.dock_ligands_batch(ctx, pid, dl, params, got)
        torch.cuda.synchronize()
        D.dock_ligands_batch(ctx, pid, dl, params, rep, st)
        D.dock_ligands_batch(ctx, pid, dl, params, got, st)
    torch.cuda.synchronize()
    _same(ref, got)
    _same(ref, rep)
    D.dock_pocket_unload(ctx, pid)


def test_overlapped_lists_under_a_callers_capture(D, ctx):  # noqa: F811
    pid, params, dl, (ref, got, _) = _setup(D, ctx, 40, (3, 100), 95)
    st = torch.cuda.Stream()
    D.dock_ligands_batch_noalloc(ctx, pid, dl, params, ref, st)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    print("[case] overlap under capture", flush=True)
    with torch.cuda.graph(g, stream=st):
        D.dock_ligands_batch_noalloc(ctx, pid, dl, params, got, st)
    for _ in range(3):
        for k in KEYS:
            getattr(got, k).zero_()
        g.replay()
        torch.cuda.synchronize()
        _same(ref, got)
    D.dock_pocket_unload(ctx, pid)


def test_plain_calls_in_flight_keep_their_poses_apart(D, ctx):  # noqa: F811
    # plain calls of different sizes on two streams, in flight together on the same
    # inner streams: each has the batched form's results
    print("[case] plain calls in flight", flush=True)
    a = _setup(D, ctx, 9, (60, 250), 97)
    b = _setup(D, ctx, 30, (3, 30), 98)
    runs = []
    for pid, params, dl, (ref, got, _) in (a, b):
        plain = D.SearchParams(params.quat, **dict(params.values, mode=D.DOCK_MODE_PLAIN))
        D.dock_ligands_batch(ctx, pid, dl, params, ref)
        runs.append((pid, plain, dl, got, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(3):
        for pid, plain, dl, got, st in runs:
            D.dock_ligands_batch(ctx, pid, dl, plain, got, st)
    torch.cuda.synchronize()
    for pid, params, dl, (ref, got, _) in (a, b):
        _same(ref, got)
        D.dock_pocket_unload(ctx, pid)


@pytest.mark.parametrize("top_k", [1, 30])
@pytest.mark.parametrize("L", [1, 2, 3, 7])
def test_split_final_step_of_few_ligands(D, ctx, L, top_k):  # noqa: F811
    # a table tuned on a large sample, with the final step split over the XCDs, used on
    # a list too short for a workgroup per share
    pk = synth.pocket_gaussians(99, 4, 32, 0.5, 40, 4.0)
    lib = synth.library_uniform(99, L, (9, 60), (0, 3))
    params = D.SearchParams(synth.start_quats(99, 40), torsion_steps=16, sweep_passes=1,
                            top_k=top_k, dedup_rmsd=0.5)
    pid = D.dock_pocket_load(ctx, pk.values, pk.spacing, pk.origin)
    dl = D.DeviceLibrary(lib)
    ref, got = [D.DeviceResults(L, dl.n_atoms_total, dl.n_rot_total, params) for _ in range(2)]
    D.dock_ligands_batch(ctx, pid, dl, params, ref)
    for waves in (2, 4, 8):
        print(f"[case] split final step L={L} K={top_k} waves={waves}", flush=True)
        tile = dict(ligands=1, dock_waves=4, select_waves=4, falign_waves=waves, falign_xcd=1)
        D.dock_set_tuning(ctx, params, [tile] * D.NUM_BINS)
        for k in KEYS:
            getattr(got, k).zero_()
        D.dock_ligands_batch(ctx, pid, dl, params, got)
        torch.cuda.synchronize()
        _same(ref, got)
    D.dock_set_tuning(ctx, params, None)
    D.dock_pocket_unload(ctx, pid)


def test_calls_in_flight_on_several_streams(D, ctx):  # noqa: F811
    # batched calls of different sizes on streams of their own, split, unsplit and by
    # buckets, with submitted work between them: each has the results it has alone
    jobs = [_setup(D, ctx, L, atoms, 100 + L % 9, **kw) for L, atoms, kw in
            ((2100, (3, 70), {}), (40, (3, 200), {}), (300, (3, 50), {}),
             (60, (3, 256), dict(bin_mode=1)), (3, (9, 9), {}))]
    for pid, params, dl, (ref, _, _) in jobs:
        D.dock_ligands_batch(ctx, pid, dl, params, ref)
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in jobs]
    lib = jobs[1][2].host
    sizes = (lib.n_ligands, int(lib.atom_off[-1]), int(lib.rot_off[-1]))
    for rep in range(3):
        print(f"[case] calls in flight, round {rep}", flush=True)
        out = []
        for (pid, params, dl, (_, got, _)), st in zip(jobs, streams):
            for k in KEYS:
                getattr(got, k).zero_()
        torch.cuda.synchronize()
        for (pid, params, dl, (_, got, again)), st in zip(jobs, streams):
            D.dock_ligands_batch(ctx, pid, dl, params, got, st)
            D.dock_ligands_batch(ctx, pid, dl, params, again, st)
            h = D.HostResults(*sizes, jobs[1][1])
            out.append((D.dock_submit(ctx, jobs[1][0], lib, jobs[1][1], h), h))
        for t, _ in out:
            D.dock_wait(ctx, t)
        torch.cuda.synchronize()
        for pid, params, dl, (ref, got, again) in jobs:
            _same(ref, got)
            _same(ref, again)
        for _, h in out:
            for k in KEYS:
                np.testing.assert_array_equal(getattr(h, k), getattr(jobs[1][3][0], k).cpu().numpy(),
                                              err_msg=k)
    for pid, params, dl, _ in jobs:
        D.dock_pocket_unload(ctx, pid)


def test_warmed_up_calls_under_a_callers_capture(D, ctx):  # noqa: F811
    # dock_ligands_batch captured by the caller after eager and replayed calls on the
    # stream, and replayed behind a larger call that grows the stream's workspace
    pid, params, dl, (ref, got, _) = _setup(D, ctx, 40, (3, 100), 96)
    one = _setup(D, ctx, 6, (20, 20), 96)
    big = _setup(D, ctx, 300, (3, 100), 97)
    for pid_, params_, dl_, (ref_, got_, _) in ((pid, params, dl, (ref, got, None)), one):
        st = torch.cuda.Stream()
        for _ in range(4):
            D.dock_ligands_batch(ctx, pid_, dl_, params_, ref_, st)
            D.dock_ligands_batch(ctx, pid_, dl_, params_, got_, st)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        print("[case] warmed up, then captured", flush=True)
        with torch.cuda.graph(g, stream=st):
            D.dock_ligands_batch(ctx, pid_, dl_, params_, got_, st)
        for rep in range(3):
            for k in KEYS:
                getattr(got_, k).zero_()
            torch.cuda.synchronize()
            if rep == 1:
                D.dock_ligands_batch(ctx, big[0], big[2], big[1], big[3][0], st)
            with torch.cuda.stream(st):
                g.replay()
            torch.cuda.synchronize()
            _same(ref_, got_)
    for j in (pid, one[0], big[0]):
        D.dock_pocket_unload(ctx, j)
