"""Performance cases of the docking library: what a screening program has it do.

Every case goes through the public entry points of `paper_2209_05069_amd.dock`:
the batched form on device-resident libraries (`dock_ligands_batch`), its form
without device allocations (`dock_ligands_batch_noalloc`), the plain per-ligand
form (mode DOCK_MODE_PLAIN) and the asynchronous form on host memory
(`dock_submit` / `dock_wait`).  Sizes and search settings are those of the
workload recipes, the size grid, the serving mix and the tests; launch tiles are
the defaults, as in a program that does not autotune.

A case names its ligand mix and search settings:
  mix      uniform sizes (atoms_lo..hi, rot_lo..hi) or "lognormal" (serving)
  form     "batch", "noalloc", "plain" or "submit"
  grid     vertices per axis of the 4-type pocket (spacing and Gaussians follow)
`draw` spreads the number of ligands, their sizes and the search settings over
the ranges of the listed cases.
"""
import math

import numpy as np
import torch

import synth
from paper_2209_05069_amd import dock as D

# Search settings of the workload recipes.
PRODUCTION = dict(restarts=256, torsion_steps=256, sweep_passes=3, align_steps=30, top_k=30,
                  dedup_rmsd=2.0, bump_prune=1, bin_mode=0, outputs="poses")


def _case(form, ligands, atoms, rot, mix="uniform", grid=96, **kw):
    c = dict(form=form, mix=mix, ligands=ligands, atoms_lo=atoms[0], atoms_hi=atoms[1],
             rot_lo=rot[0], rot_hi=rot[1], grid=grid)
    c.update(PRODUCTION)
    c.update(kw)
    return c


def listed():
    return [
        # a program's first call: a handful of small ligands, a small search (recipe 1)
        dict(_case("batch", 8, (20, 20), (3, 3), grid=32, restarts=16, torsion_steps=64,
                   sweep_passes=2, top_k=16, outputs="all"), name="small_batch"),
        # interactive docking: one ligand now, the whole GPU on it
        dict(_case("plain", 1, (20, 80), (2, 12)), name="one_ligand_plain"),
        # the per-ligand form over a short list (recipe 2's mix)
        dict(_case("plain", 96, (20, 80), (2, 12)), name="plain_list"),
        # serving at low load: a short batch from host memory, scores only
        dict(_case("submit", 32, (12, 150), (0, 30), mix="lognormal", outputs="scores"),
             name="serve_short_batch"),
        # serving at saturation: a full bucket from host memory, scores only
        dict(_case("submit", 4096, (12, 150), (0, 30), mix="lognormal", outputs="scores"),
             name="serve_full_batch"),
        # a medium library at the paper's scale (recipe 2's mix)
        dict(_case("batch", 2500, (20, 80), (2, 12)), name="paper_scale"),
        # the paper's search and buckets: 36-degree torsion steps, lists per size and bonds
        dict(_case("batch", 2500, (20, 80), (2, 12), torsion_steps=10, bin_mode=1),
             name="paper_search_buckets"),
        # a screening library (recipe 3's mix)
        dict(_case("batch", 16000, (20, 100), (0, 20)), name="large_library"),
        # the largest ligands the library takes, with every restart's score and trace
        dict(_case("batch", 200, (100, 256), (8, 30), outputs="all"), name="largest_ligands"),
        # fragments: the size grid's small cell
        dict(_case("batch", 6000, (16, 16), (4, 4), restarts=128), name="fragments"),
        # a serving loop that may not allocate, with contact scores of every pose
        dict(_case("noalloc", 300, (20, 80), (2, 12), outputs="contacts"), name="rescored_noalloc"),
        # the no-early-exit ablation (size grid's 64 atoms x 24 bonds)
        dict(_case("batch", 300, (64, 64), (24, 24), restarts=128, bump_prune=0), name="no_pruning"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    # sizes are redrawn until the case costs no more than the largest listed one
    top = work(_case("batch", 16000, (20, 100), (0, 20)))["flops"]
    while True:
        c = _draw(rng)
        if work(c)["flops"] <= top:
            return c


def _draw(rng):
    kind = rng.choice(["small", "plain", "submit", "mix", "mix", "buckets", "cell", "large",
                       "noalloc", "no_prune"])
    lo = rng.randint(12, 60)
    atoms = (lo, rng.randint(lo, 100))
    blo = rng.randint(0, 8)
    rot = (blo, rng.randint(blo, 20))
    if kind == "small":
        return _case("batch", _log_int(rng, 1, 64), atoms, rot, grid=rng.randint(32, 64),
                     restarts=rng.randint(8, 64), torsion_steps=rng.choice([10, 36, 64, 100]),
                     sweep_passes=rng.randint(1, 3), align_steps=rng.choice([12, 20, 30, 36]),
                     top_k=rng.randint(1, 16), outputs="all")
    if kind == "plain":
        return _case("plain", _log_int(rng, 1, 128), atoms, rot)
    if kind == "submit":
        return _case("submit", _log_int(rng, 16, 4096), (12, 150), (0, 30), mix="lognormal",
                     outputs=rng.choice(["scores", "poses"]))
    if kind == "mix":
        return _case("batch", _log_int(rng, 100, 12000), atoms, rot, grid=rng.randint(72, 96),
                     restarts=rng.choice([64, 128, 200, 256]),
                     torsion_steps=rng.choice([36, 72, 128, 256]), sweep_passes=rng.randint(1, 3))
    if kind == "buckets":
        return _case("batch", _log_int(rng, 200, 4000), atoms, rot, torsion_steps=10, bin_mode=1)
    if kind == "cell":
        n = rng.choice([16, 24, 32, 48, 64, 128])
        b = min(rng.choice([0, 4, 8, 16, 24]), n - 8)
        return _case("batch", _log_int(rng, 200, 6000), (n, n), (b, b), restarts=128)
    if kind == "large":
        lo = rng.randint(90, 200)
        return _case("batch", _log_int(rng, 8, 200), (lo, rng.randint(lo, 256)),
                     (rng.randint(0, 8), rng.randint(8, 30)), outputs=rng.choice(["all", "poses"]))
    if kind == "noalloc":
        return _case("noalloc", _log_int(rng, 4, 300), (20, 80), (2, 12),
                     outputs=rng.choice(["contacts", "poses"]))
    return _case("batch", _log_int(rng, 50, 600), (64, 64), (rng.randint(0, 24), 24), restarts=128,
                 bump_prune=0)


# ---------------------------------------------------------------------------
# Inputs


def _pocket(seed, n):
    """Values of a 4-type pocket (the recipes' Gaussian mixtures: 40 within 4 A on a
    grid of 0.5 A up to 64 vertices, else 160 within 9 A on one of 0.375 A)."""
    spacing, count, half = (0.5, 40, 4.0) if n <= 64 else (0.375, 160, 9.0)
    rng = np.random.default_rng([int(seed), 1])
    origin = -spacing * (n - 1) / 2.0
    x = torch.from_numpy(origin + spacing * np.arange(n)).cuda()
    values = torch.empty((4, n, n, n), dtype=torch.float32, device="cuda")
    for t in range(4):
        centre = torch.from_numpy(rng.uniform(-half, half, (count, 3))).cuda()
        sigma = torch.from_numpy(rng.uniform(1.0, 2.0, count)).cuda()
        amp = torch.from_numpy(rng.uniform(-1.0, 1.0, count)).cuda()
        e = torch.exp(-(x[None, None, :] - centre[:, :, None]) ** 2 / (2 * sigma ** 2)[:, None, None])
        zy = (e[:, 2, :, None] * e[:, 1, None, :]).reshape(count, n * n)
        values[t] = (zy.t().contiguous() @ (amp[:, None] * e[:, 0])).reshape(n, n, n).float()
    return synth.Pocket(values.cpu().numpy(), spacing, (origin, origin, origin))


def _inputs(case, seed):
    """(pocket, library, start orientations, search settings) of a case."""
    seed = int(seed) & 0x7FFFFFFF
    pk = _pocket(seed, case["grid"])
    # sizes belong to the case (the seed changes trees, coordinates, types and bonds)
    L, rng = case["ligands"], np.random.default_rng(2209)
    if case["mix"] == "lognormal":
        n = np.clip(np.rint(40.0 * np.exp(0.5 * rng.standard_normal(L))), 12, 150)
        b = np.clip(rng.poisson(6.0, L), 0, 30)
    else:
        n = rng.integers(case["atoms_lo"], case["atoms_hi"] + 1, L)
        b = rng.integers(case["rot_lo"], case["rot_hi"] + 1, L)
    if case["outputs"] == "all":
        b = np.minimum(b, n // 4)  # every tree has as many: the trace's length is fixed
    lib = synth.library_from_sizes(seed, n.astype(np.int32), b.astype(np.int32))
    q = synth.start_quats(seed, case["restarts"])
    s = {k: case[k] for k in ("torsion_steps", "sweep_passes", "align_steps", "top_k",
                              "dedup_rmsd", "bump_prune", "bin_mode")}
    return pk, lib, q, s


_ctx = None


def _context():
    """The program's one context, kept until it ends."""
    global _ctx
    if _ctx is None:
        _ctx = D.dock_create(0)
    return _ctx


class _State:
    def __del__(self):
        try:
            D.dock_pocket_unload(_context(), self.pocket)
        except Exception:  # the interpreter is ending
            pass


def prepare(case, seed):
    pk, lib, q, s = _inputs(case, seed)
    ctx = _context()
    st = _State()
    st.form = case["form"]
    st.pocket = D.dock_pocket_load(ctx, pk.values, pk.spacing, pk.origin)
    st.params = D.SearchParams(
        q, mode=D.DOCK_MODE_PLAIN if st.form == "plain" else D.DOCK_MODE_BATCHED, **s)
    want = case["outputs"]
    if want == "contacts":
        pa = synth.pocket_atoms(int(seed) & 0x7FFFFFFF, pk)
        D.dock_pocket_set_atoms(ctx, st.pocket, pa.xyz, pa.type, pa.ntypes, pa.weight,
                                pa.contact_dist)
    kw = dict(poses=want != "scores", contacts=want == "contacts", restart_scores=want == "all",
              trace=want == "all", final_trace=want == "all")
    sizes = (lib.n_ligands, int(lib.atom_off[-1]), int(lib.rot_off[-1]))
    if st.form == "submit":
        st.library = lib
        st.results = D.HostResults(*sizes, st.params, **kw)
    else:
        st.library = D.DeviceLibrary(lib)
        st.results = D.DeviceResults(*sizes, st.params, **kw)
    return st


_FIELDS = ("best_score", "n_poses", "status", "pose_score", "pose_restart", "pose_xyz",
           "restart_score", "trace", "final_trace", "pose_contacts")


def run(state):
    ctx, r = _context(), state.results
    if state.form == "submit":
        D.dock_wait(ctx, D.dock_submit(ctx, state.pocket, state.library, state.params, r))
    elif state.form == "noalloc":
        D.dock_ligands_batch_noalloc(ctx, state.pocket, state.library, state.params, r)
    else:
        D.dock_ligands_batch(ctx, state.pocket, state.library, state.params, r)
    return {k: getattr(r, k) for k in _FIELDS if getattr(r, k) is not None}


def work(case):
    """Bytes of the pocket, the library and the results; FP32 operations of the
    rigid steps (49 per atom sample: placed, interpolated, summed) of every
    restart and kept pose, and of the torsion samples: a moving fragment holds about
    7 atoms in these trees, and a quarter of the candidates pass the bump check
    (all are scored without pruning)."""
    L, R, K, A = case["ligands"], case["restarts"], case["top_k"], case["align_steps"]
    if case["mix"] == "lognormal":
        n, b = 45.0, 6.0
    else:
        n = (case["atoms_lo"] + case["atoms_hi"]) / 2.0
        b = min((case["rot_lo"] + case["rot_hi"]) / 2.0, 0.5 * n)
    nbytes = 16.0 * case["grid"] ** 3 + L * (13 * n + 8 * n + 24 * b + 12 + 12 + 8 * K)
    if case["outputs"] != "scores":
        nbytes += L * n * K * 12.0
    if case["outputs"] == "all":
        nbytes += L * R * (4.0 + 2.0 * (1 + case["sweep_passes"] * b))
    samples = L * n * A * A * (R + min(K, R))
    samples += L * b * min(7.0, n / 3) * R * case["sweep_passes"] * case["torsion_steps"] * (
        0.25 if case["bump_prune"] else 1.0)
    return {"bytes": nbytes, "flops": 49.0 * samples}


# ---------------------------------------------------------------------------
# The same search in float64, in plain torch


def _rotations(q):
    q = q / q.norm(dim=1, keepdim=True)
    w, x, y, z = q.unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)],
                       1).reshape(-1, 3, 3)


class _Grid:
    def __init__(self, pk, dev):
        self.v = torch.from_numpy(pk.values).to(dev).double()
        self.h, self.origin = float(np.float32(pk.spacing)), torch.tensor(
            np.asarray(pk.origin, np.float32).astype(np.float64), device=dev)
        self.n = self.v.shape[1]
        self.centre = self.origin + self.h * (self.n - 1) / 2.0

    def samples(self, p, types):
        """Interpolated values at p[..., atoms, 3] for atoms of `types`."""
        n = self.n
        g = ((p - self.origin) / self.h).clamp(0, n - 1)
        c = g.floor().clamp(max=n - 2)
        fx, fy, fz = (g - c).unbind(-1)
        ix, iy, iz = c.long().unbind(-1)
        at = ((types * n + iz) * n + iy) * n + ix
        v = self.v.reshape(-1)

        def row(o):
            a = v[at + o]
            return a + fx * (v[at + o + 1] - a)

        lo = row(0) + fy * (row(n) - row(0))
        hi = row(n * n) + fy * (row(n * n + n) - row(n * n))
        return lo + fz * (hi - lo)


def _align(grid, Y, types, A):
    """(best orientation index, its pose) of every pose in Y [R, n, 3]."""
    c = Y.mean(1, keepdim=True)
    d = Y - c
    ang = 2 * math.pi * torch.arange(A, dtype=torch.float64, device=Y.device) / A
    cb, sb = ang.cos()[None, :, None], ang.sin()[None, :, None]

    def turned(i):
        y = math.cos(2 * math.pi * i / A) * d[..., 1] - math.sin(2 * math.pi * i / A) * d[..., 2]
        z = math.sin(2 * math.pi * i / A) * d[..., 1] + math.cos(2 * math.pi * i / A) * d[..., 2]
        x, y, z = d[:, None, :, 0], y[:, None, :], z[:, None, :]
        return torch.stack([cb * x + sb * z, y.expand(-1, A, -1), cb * z - sb * x],
                           -1) + c[:, None]

    S = torch.cat([grid.samples(turned(i), types).sum(-1) for i in range(A)], 1)
    o = S.argmax(1)
    out = torch.empty_like(Y)
    for i in range(A):
        r = torch.nonzero(o // A == i).flatten()
        if len(r):
            out[r] = turned(i)[r, o[r] % A]
    return o, out


def _sweep(grid, Y, types, far, a, b, mask, T, bump2):
    """One decision of every pose in Y: the best bump-free turn of the fragment `mask`."""
    u = Y[:, b] - Y[:, a]
    u = u / u.norm(dim=1, keepdim=True)
    mv, st = torch.nonzero(mask).flatten(), torch.nonzero(~mask).flatten()
    d = Y[:, mv] - Y[:, a, None]
    along = (d * u[:, None]).sum(-1, keepdim=True) * u[:, None]
    v = d - along
    w = torch.cross(u[:, None].expand_as(d), d, dim=-1)
    ang = 2 * math.pi * torch.arange(T, dtype=torch.float64, device=Y.device) / T
    p = (Y[:, a, None] + along)[:, None] + ang.cos()[None, :, None, None] * v[:, None] \
        + ang.sin()[None, :, None, None] * w[:, None]
    fm, fs = torch.nonzero(far[mv][:, st], as_tuple=True)
    bump = torch.zeros(p.shape[:2], dtype=torch.bool, device=Y.device)
    step = max(1, (1 << 25) // (p.shape[0] * T))
    for k in range(0, len(fm), step):
        d2 = (p[:, :, fm[k:k + step]] - Y[:, None, st[fs[k:k + step]]]).square().sum(-1)
        bump |= (d2 < bump2).any(-1)
    S = grid.samples(p, types[mv]).sum(-1).masked_fill(bump, -math.inf)
    best = S.argmax(1)
    turned = p[torch.arange(len(Y), device=Y.device), best]
    keep = bump.all(1)
    Y[:, mv] = torch.where(keep[:, None, None], Y[:, mv], turned)
    return torch.where(keep, torch.full_like(best, 0xFFFF), best)


def _dock(grid, rot, lib, l, s, dev):
    x, t, bonds, rb, rm = lib.ligand(l)
    n, K = len(x), s["top_k"]
    X = torch.from_numpy(x.astype(np.float64)).to(dev)
    types = torch.from_numpy(t.astype(np.int64)).to(dev)
    near = np.eye(n, dtype=bool)
    adj = np.eye(n, dtype=bool)
    adj[bonds[:, 0], bonds[:, 1]] = adj[bonds[:, 1], bonds[:, 0]] = True
    for _ in range(D.DEFAULT_PARAMS["bump_min_bonds"] - 1):
        near = (near.astype(int) @ adj.astype(int)) > 0
    far = torch.from_numpy(~near).to(dev)
    Y = (X - X.mean(0)) @ rot.transpose(1, 2) + grid.centre
    o, Y = _align(grid, Y, types, s["align_steps"])
    bits = (rm[:, np.arange(n) // 64] >> (np.arange(n) % 64).astype(np.uint64)) & np.uint64(1)
    masks = torch.from_numpy(bits.astype(bool)).to(dev)
    for _ in range(s["sweep_passes"]):
        for b in range(len(rb)):
            _sweep(grid, Y, types, far, int(rb[b, 0]), int(rb[b, 1]), masks[b],
                   s["torsion_steps"], float(np.float32(D.DEFAULT_PARAMS["bump_dist"])) ** 2)
    S = grid.samples(Y, types).sum(-1)
    kept = []
    for r in torch.sort(-S, stable=True).indices.tolist():
        if len(kept) == K:
            break
        if all(float((Y[r] - Y[q]).square().sum(-1).mean().sqrt()) >= s["dedup_rmsd"]
               for q in kept):
            kept.append(r)
    kept = torch.tensor(kept, device=dev)
    _, F = _align(grid, Y[kept], types, s["align_steps"])
    fs = grid.samples(F, types).sum(-1)
    order = sorted(range(len(kept)), key=lambda q: (-float(fs[q]), int(kept[q])))
    ps = np.full(K, -np.inf)
    ps[:len(order)] = fs[order].cpu().numpy()
    xyz = np.zeros((K, n, 3))
    xyz[:len(order)] = F[order].cpu().numpy()
    return ps, xyz.reshape(-1), S.cpu().numpy()


def exact(case, seed):
    # about a quarter of a second for a ligand of the production search
    if work(case)["flops"] > 40 * work(_case("plain", 1, (20, 80), (2, 12)))["flops"] \
            or case["ligands"] > 40:
        return None
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    pk, lib, q, s = _inputs(case, seed)
    grid = _Grid(pk, dev)
    rot = _rotations(torch.from_numpy(q.astype(np.float64)).to(dev))
    got = [_dock(grid, rot, lib, l, s, dev) for l in range(lib.n_ligands)]
    out = dict.fromkeys(_FIELDS[:5])
    out["best_score"] = np.array([g[0][0] for g in got])
    out["pose_score"] = np.concatenate([g[0] for g in got])
    if case["outputs"] != "scores":
        out["pose_xyz"] = np.concatenate([g[1] for g in got])
    if case["outputs"] == "all":
        out.update(restart_score=np.concatenate([g[2] for g in got]), trace=None, final_trace=None)
    if case["outputs"] == "contacts":
        out["pose_contacts"] = None
    return out
