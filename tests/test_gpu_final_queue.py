"""The final step's queue: items taken several at a time where they are small, no more
of them than a ligand can keep poses, and none where there is no alignment to balance."""
import time

import numpy as np
import pytest

import synth
from tests.test_gpu_parity import D, ctx  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
KEYS = ("best_score", "n_poses", "status", "pose_score", "pose_restart", "pose_xyz")


def _setup(D, ctx, L, atoms, restarts, **kw):  # noqa: F811
    pk = synth.pocket_gaussians(5, 4, 32, 0.5, 40, 4.0)
    lib = synth.library_uniform(5, L, atoms, (0, 2))
    params = D.SearchParams(synth.start_quats(5, restarts), torsion_steps=8, sweep_passes=1,
                            dedup_rmsd=0.0, **kw)
    dl = D.DeviceLibrary(lib)
    return (D.dock_pocket_load(ctx, pk.values, pk.spacing, pk.origin), dl, params,
            [D.DeviceResults(L, dl.n_atoms_total, dl.n_rot_total, params) for _ in range(2)])


@pytest.mark.parametrize("atoms,restarts,top_k,kw", [
    ((3, 32), 40, 64, dict(align_steps=5)),    # 16 items at a time
    ((3, 32), 40, 63, dict(align_steps=12)),   # 8
    ((3, 32), 33, 33, dict(align_steps=30)),   # 2
    ((33, 64), 40, 40, dict(align_steps=12)),  # 4 of the next bin
    ((3, 32), 40, 40, dict(align_steps=36)),   # 1, without strips
    ((3, 32), 40, 64, dict(align_steps=5, final_align=0)),
    ((3, 32), 3, 64, dict(align_steps=5))])
def test_items_from_the_queue_are_the_items_in_turn(D, ctx, atoms, restarts, top_k, kw):  # noqa: F811
    # (the split over XCDs takes its items in turn)
    pid, dl, params, (ref, got) = _setup(D, ctx, 2040, atoms, restarts, top_k=top_k, **kw)
    print(f"[case] final queue {atoms} R={restarts} K={top_k} {kw}", flush=True)
    tile = dict(ligands=1, dock_waves=4, select_waves=4, falign_waves=4, falign_xcd=1)
    D.dock_set_tuning(ctx, params, [tile] * D.NUM_BINS)
    D.dock_ligands_batch(ctx, pid, dl, params, ref)
    D.dock_set_tuning(ctx, params, None)
    D.dock_ligands_batch(ctx, pid, dl, params, got)
    torch.cuda.synchronize()
    for k in KEYS:
        np.testing.assert_array_equal(getattr(ref, k).cpu().numpy(), getattr(got, k).cpu().numpy(),
                                      err_msg=k)
    D.dock_pocket_unload(ctx, pid)


def test_poses_that_cannot_be_kept_cost_nothing(D, ctx):  # noqa: F811
    # one restart: a single pose a ligand, whatever the limit
    def best(top_k):
        pid, dl, params, (res, _) = _setup(D, ctx, 2040, (6, 6), 1, top_k=top_k, align_steps=5)
        t = []
        for _ in range(12):
            torch.cuda.synchronize()
            a = time.perf_counter()
            D.dock_ligands_batch(ctx, pid, dl, params, res)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
        D.dock_pocket_unload(ctx, pid)
        return min(t)

    print("[case] final queue, one restart", flush=True)
    one, many = best(1), best(64)
    assert many < 2.0 * one, (one, many)
