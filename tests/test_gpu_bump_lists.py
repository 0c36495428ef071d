"""The listed bump check of a torsion decision, at the list, slot and arc edges: the
pruned decisions are those of the exhaustive check, and the oracle's."""
import numpy as np
import pytest

import synth
from tests.test_gpu_parity import D, check_all, ctx, run_batch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,bump_dist", [
    (16, 2.0), (128, 2.0), (129, 2.0), (132, 3.0), (192, 1.0), (256, 0.0), (256, 2.0),
    (256, 4.0), (600, 2.5), (1024, 2.0)])
def test_pruned_decisions_are_the_exhaustive_ones(D, ctx, T, bump_dist):  # noqa: F811
    # 16 to 200 atoms: decisions with a few moving atoms (tested row by row), with many
    # (listed, several batches of 64 pairs at the larger distances) and with every slot
    # count; T at and around whole slots and where arcs are first told apart
    pk = synth.pocket_gaussians(81, 4, 40, 0.5, 40, 4.0)
    lib = synth.library_from_sizes(82, [16, 40, 64, 65, 129, 200], [4, 9, 12, 14, 20, 24])
    q = synth.start_quats(83, 3)
    kw = dict(torsion_steps=T, sweep_passes=2, align_steps=6, top_k=3, bump_dist=bump_dist)
    print(f"[case] bump lists T={T} dist={bump_dist}", flush=True)
    a, _ = run_batch(D, ctx, pk, lib, q, bump_prune=1, **kw)
    b, _ = run_batch(D, ctx, pk, lib, q, bump_prune=0, **kw)
    for k in ("trace", "restart_score", "pose_score", "pose_xyz"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("bump_dist", [1.0, 3.5])
def test_listed_bump_check_is_the_oracles(D, ctx, bump_dist):  # noqa: F811
    pk = synth.pocket_gaussians(84, 4, 40, 0.5, 40, 4.0)
    lib = synth.library_from_sizes(85, [24, 70, 140], [6, 10, 8])
    q = synth.start_quats(86, 2)
    print(f"[case] bump lists, oracle, dist={bump_dist}", flush=True)
    h, params = run_batch(D, ctx, pk, lib, q, torsion_steps=256, sweep_passes=1, align_steps=6,
                          top_k=2, bump_dist=bump_dist)
    check_all(D, pk, lib, q, h, params, label=f"bump-{bump_dist}")


@pytest.mark.parametrize("plain", [True, False])
@pytest.mark.parametrize("shift,bump_dist", [(3e3, 2.0), (3e5, 2.0), (2e6, 1.0), (2e6, 4.0), (8e6, 3.0)])
def test_pruned_decisions_of_a_pocket_far_from_the_origin(D, ctx, shift, bump_dist, plain):  # noqa: F811
    # coordinates round by up to half an Angstrom there: a pair that the tested form of the distance
    # calls a bump is listed although its axial distance is a little above
    pk = synth.pocket_gaussians(87, 4, 40, 0.25, 40, 4.0)
    o = tuple(float(np.float32(x + s * shift)) for x, s in zip(pk.origin, (1.0, -0.7, 0.4)))
    pk = synth.Pocket(pk.values, pk.spacing, o)
    lib = synth.library_from_sizes(88, [40, 64, 65, 129], [9, 12, 14, 20])
    q = synth.start_quats(89, 8)
    kw = dict(torsion_steps=256, sweep_passes=2, align_steps=6, top_k=3, bump_dist=bump_dist,
              mode=D.DOCK_MODE_PLAIN if plain else D.DOCK_MODE_BATCHED)
    print(f"[case] bump lists, far pocket {shift} dist={bump_dist}", flush=True)
    a, _ = run_batch(D, ctx, pk, lib, q, bump_prune=1, **kw)
    b, _ = run_batch(D, ctx, pk, lib, q, bump_prune=0, **kw)
    for k in ("trace", "restart_score", "pose_score", "pose_xyz"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
