"""Selection at a rounding of the duplicate test: two poses exactly as far apart as
dedup_rmsd by one order of summation, and not by another, are kept or dropped alike
whatever the selection's tile and whatever the number of ligands in the call."""
import numpy as np
import pytest

import synth
from tests.test_gpu_parity import D, ctx  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
f32 = np.float32


def _fma(a, b, c):  # exact product, one rounding (to 53 bits and then 24)
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(f32)


def _sums(p, q):
    """Squared distance of two poses of 64 atoms, over the atoms in order and over the
    lanes of a wave."""
    d = p - q
    in_order = f32(0)
    for i in range(64):
        for k in (2, 1, 0):
            in_order = _fma(d[i, k], d[i, k], in_order)
    v = np.zeros(64, f32)
    for k in (2, 1, 0):
        v = _fma(d[:, k], d[:, k], v)
    rows = v.reshape(4, 16)
    for s in (1, 2, 4, 8):
        rows[:, s:] = rows[:, s:] + rows[:, :-s].copy()
    top = rows[:, 15]
    return in_order, (top[3] + top[2]) + (top[1] + top[0])


def _threshold(a, b):
    """dedup_rmsd whose square, times 64 atoms, lies above one of a < b and not above the
    other, or None."""
    r = f32(np.sqrt(np.float64(b) / 64))
    for _ in range(8):
        lim = f32(np.float64(r) ** 2) * f32(64)
        if a < lim <= b:
            return float(r)
        r = np.nextafter(r, f32(0))
    return None


def test_selection_does_not_depend_on_tile_or_library_size(D, ctx):  # noqa: F811
    pk = synth.pocket_gaussians(61, 4, 40, 0.5, 60, 4.0)
    sizes = {n: synth.library_from_sizes(62, [64] * n, [3] * n) for n in (2, 600, 1100)}
    q = synth.start_quats(63, 48)
    pid = D.dock_pocket_load(ctx, pk.values, pk.spacing, pk.origin)
    kw = dict(torsion_steps=16, sweep_passes=1, align_steps=6, top_k=48, final_align=0)

    def dock(lib, rmsd, waves=0):
        params = D.SearchParams(q, dedup_rmsd=rmsd, **kw)
        dl = D.DeviceLibrary(lib)
        res = D.DeviceResults(lib.n_ligands, dl.n_atoms_total, dl.n_rot_total, params)
        tile = dict(ligands=1, dock_waves=4, select_waves=waves, falign_waves=4)
        D.dock_set_tuning(ctx, params, [tile] * D.NUM_BINS if waves else None)
        D.dock_ligands_batch(ctx, pid, dl, params, res)
        torch.cuda.synchronize()
        h = res.to_host()
        return h["n_poses"][:2], h["pose_restart"][:2 * 48], h["pose_xyz"][:2 * 48 * 64 * 3]

    _, _, xyz = dock(sizes[2], 0.0)  # every pose, in order of rank (no final step)
    poses = xyz.reshape(2, 48, 64, 3)
    tried = 0
    for l in range(2):
        for i in range(1, 48):
            for j in range(i):
                if tried >= 24 or i // 16 != j // 16 or i // 4 == j // 4 and (i + j) % 3:
                    continue
                a, b = _sums(poses[l, i], poses[l, j])
                rmsd = _threshold(min(a, b), max(a, b)) if a != b else None
                if rmsd is None:
                    continue
                tried += 1
                ref = dock(sizes[2], rmsd, 4)
                for waves in (1, 2, 3, 6, 8, 16, 0):
                    for x, y in zip(ref, dock(sizes[2], rmsd, waves)):
                        np.testing.assert_array_equal(x, y, err_msg=f"{i} {j} {waves}")
                if tried % 8 == 1:
                    print(f"[case] select order, pair {i} {j}", flush=True)
                    for n in (600, 1100):
                        for x, y in zip(ref, dock(sizes[n], rmsd)):
                            np.testing.assert_array_equal(x, y, err_msg=f"{i} {j} {n}")
    assert tried >= 8
    D.dock_pocket_unload(ctx, pid)


@pytest.mark.parametrize("atoms,restarts,top_k", [((3, 64), 40, 30), ((60, 256), 40, 30),
                                                  ((250, 256), 70, 1), ((3, 256), 64, 64)])
def test_plain_poses_as_found_are_the_poses_replayed(D, ctx, atoms, restarts, top_k):  # noqa: F811
    # (a context with a memory budget keeps no poses of the restarts: they are replayed)
    pk = synth.pocket_gaussians(9, 4, 32, 0.5, 40, 4.0)
    lib = synth.library_uniform(9, 12, atoms, (0, 4))
    params = D.SearchParams(synth.start_quats(9, restarts), torsion_steps=16, sweep_passes=2,
                            align_steps=12, top_k=top_k, dedup_rmsd=2.0, mode=1)
    print(f"[case] plain poses {atoms} R={restarts} K={top_k}", flush=True)
    tight = D.dock_create(0, hbm_budget_bytes=1 << 30)
    got = []
    for c in (ctx, tight):
        pid = D.dock_pocket_load(c, pk.values, pk.spacing, pk.origin)
        dl = D.DeviceLibrary(lib)
        res = D.DeviceResults(12, dl.n_atoms_total, dl.n_rot_total, params)
        D.dock_ligands_batch(c, pid, dl, params, res)
        torch.cuda.synchronize()
        got.append(res.to_host())
        D.dock_pocket_unload(c, pid)
    D.dock_destroy(tight)
    for k in ("best_score", "n_poses", "status", "pose_score", "pose_restart", "pose_xyz"):
        np.testing.assert_array_equal(got[0][k], got[1][k], err_msg=k)
