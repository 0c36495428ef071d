"""The alignment by score bounds (30 alignment steps) against the FP64 oracle, at the
sizes and pockets where a bound, a list or a record could go wrong."""
import numpy as np
import pytest

import synth
from tests.test_gpu_parity import D, check_all, ctx, run_batch  # noqa: F401

pytestmark = pytest.mark.gpu


def _pocket(kind, seed):
    pk = synth.pocket_gaussians(seed, 4, 32, 0.5, 40, 4.0)
    if kind == "flat":  # every orientation ties: all of them are scored
        pk.values[:] = 0.25
    elif kind == "walls":  # forbidden regions
        pk.values[pk.values < -0.2] = -1e6
    elif kind == "peak":  # one value far above the others: few bins keep the bounds
        pk.values[2, 16, 17, 15] = 60.0 * pk.values.max()
    elif kind == "negative":  # no positive value
        pk.values -= 3.0
    elif kind == "far":  # coordinates far from the origin
        o = tuple(x + s for x, s in zip(pk.origin, (310.0, -145.0, 78.0)))
        pk = synth.Pocket(pk.values, pk.spacing, o)
    return pk


@pytest.mark.parametrize("kind,atoms,restarts", [
    ("plain", [1, 2, 3, 31, 32, 33], 1),
    ("plain", [63, 64, 65, 127, 128], 3),
    ("plain", [129, 192, 193, 256], 21),
    ("plain", [20, 40], 17),
    ("flat", [7, 40], 3),
    ("walls", [12, 66], 9),
    ("walls", [130, 200, 256], 5),
    ("peak", [12, 40, 66, 130, 200, 256], 5),
    ("negative", [12, 66], 8),
])
def test_bounded_alignment_is_the_oracles(D, ctx, kind, atoms, restarts):  # noqa: F811
    pk = _pocket(kind, 71)
    lib = synth.library_from_sizes(72, atoms, [0] * len(atoms))
    q = synth.start_quats(73, restarts)
    print(f"[case] bounds {kind} {atoms} R={restarts}", flush=True)
    h, params = run_batch(D, ctx, pk, lib, q, torsion_steps=16, sweep_passes=1, top_k=2,
                          dedup_rmsd=0.0)
    check_all(D, pk, lib, q, h, params, label=f"bounds-{kind}")


@pytest.mark.parametrize("kind,atoms,rot,restarts", [
    ("plain", [5, 33, 70], [1, 3, 5], 11),
    # FP32 coordinates this far from the origin are off by more than the oracle's
    # tolerance on either path
    ("far", [12, 66], [0, 0], 7),
])
def test_pocket_without_bounds_takes_the_same_orientations(D, ctx, kind, atoms, rot,  # noqa: F811
                                                           restarts):
    # one value beyond the range the bounds are kept for, in a corner no ligand
    # reaches: every decision is that of the pocket with bounds
    pk = _pocket(kind, 71)
    lib = synth.library_from_sizes(72, atoms, rot)
    q = synth.start_quats(73, restarts)
    kw = dict(torsion_steps=32, sweep_passes=1, top_k=4, dedup_rmsd=0.0)
    print(f"[case] bounds on and off, {kind}", flush=True)
    a, _ = run_batch(D, ctx, pk, lib, q, **kw)
    off = pk.values.copy()
    off[:, 0, 0, 0] = 2e30
    b, _ = run_batch(D, ctx, synth.Pocket(off, pk.spacing, pk.origin), lib, q, **kw)
    for k in ("trace", "restart_score", "pose_score", "pose_xyz", "final_trace"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("align_steps", [30, 20])
@pytest.mark.parametrize("shift", [300.0, 6e4, 1e6, 4e6, 2e7])
def test_ligands_far_from_their_origin(D, ctx, shift, align_steps):  # noqa: F811
    # a ligand's coordinates round in its own frame, and the centroid of its start pose
    # misses the grid centre by that much: the batched alignment takes the orientations
    # of the plain form, which samples every one from global memory
    pk = synth.pocket_gaussians(74, 4, 48, 0.25, 60, 4.0)
    lib = synth.library_from_sizes(75, [9, 31, 40, 66, 100, 150], [0] * 6)
    lib.xyz = (lib.xyz + np.array([shift, -0.7 * shift, 0.4 * shift])).astype(np.float32)
    q = synth.start_quats(76, 19)
    kw = dict(torsion_steps=16, sweep_passes=1, align_steps=align_steps, top_k=4, dedup_rmsd=0.0)
    print(f"[case] far ligands {shift} A={align_steps}", flush=True)
    a, _ = run_batch(D, ctx, pk, lib, q, **kw)
    b, _ = run_batch(D, ctx, pk, lib, q, mode=D.DOCK_MODE_PLAIN, **kw)
    for k in ("trace", "restart_score", "pose_score", "pose_xyz"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("align_steps", [30, 20])
@pytest.mark.parametrize("shift", [300.0, 4e3, 6e4, 1e6])
def test_pockets_far_from_the_origin(D, ctx, shift, align_steps):  # noqa: F811
    pk = synth.pocket_gaussians(74, 4, 48, 0.25, 60, 4.0)
    o = tuple(float(np.float32(x + s * shift)) for x, s in zip(pk.origin, (1.0, -0.7, 0.4)))
    pk = synth.Pocket(pk.values, pk.spacing, o)
    lib = synth.library_from_sizes(75, [9, 31, 40, 66, 100, 150], [0] * 6)
    q = synth.start_quats(76, 19)
    kw = dict(torsion_steps=16, sweep_passes=1, align_steps=align_steps, top_k=4, dedup_rmsd=0.0)
    print(f"[case] far pocket {shift} A={align_steps}", flush=True)
    a, _ = run_batch(D, ctx, pk, lib, q, **kw)
    b, _ = run_batch(D, ctx, pk, lib, q, mode=D.DOCK_MODE_PLAIN, **kw)
    for k in ("trace", "restart_score", "pose_score", "pose_xyz"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("box", [(48, 30, 21), (20, 48, 33), (17, 24, 48), (3, 40, 40)])
def test_bounds_of_a_box_that_is_no_cube(D, ctx, box):  # noqa: F811
    # (nz, ny, nx): the bins' spheres leave the grid at different radii on each axis
    pk = synth.pocket_gaussians(77, 4, 48, 0.5, 60, 5.0)
    v = np.ascontiguousarray(pk.values[:, :box[0], :box[1], :box[2]])
    pk = synth.Pocket(v, pk.spacing, pk.origin)
    lib = synth.library_from_sizes(78, [4, 20, 33, 64, 90, 130], [0] * 6)
    q = synth.start_quats(79, 18)
    kw = dict(torsion_steps=16, sweep_passes=1, top_k=4, dedup_rmsd=0.0)
    print(f"[case] bounds, box {box}", flush=True)
    a, _ = run_batch(D, ctx, pk, lib, q, **kw)
    b, _ = run_batch(D, ctx, pk, lib, q, mode=D.DOCK_MODE_PLAIN, **kw)
    for k in ("trace", "restart_score", "pose_score", "pose_xyz"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
