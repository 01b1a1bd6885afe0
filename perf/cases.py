"""Performance cases of the docking library: the calls its users make, over
the sizes they make them at.

A case is a dict of plain values with a "kind":

  sample   dock_sample (or, with keep, dock_run_restart of a run made once),
           the run's state, dock_best_poses: one docking or one screening batch
  score    dock_score_grad of caller poses (grid maps, the direct pair sum, or
           grid maps + E_MDN)
  maps     a pocket's grid maps: dock_pocket_rebuild of a kept handle, or
           dock_load_pocket of a new receptor (load)
  diff     forward and backward through the autograd function (caller maps,
           weights and DOFs)
  adjoint  dock_score_adjoint, deterministic, into every pocket's maps
  recgrad  the same for one pocket, chained to the receptor's coordinates and
           the term constants (dock_pocket_map_adjoint)
  hits     dock_best_poses of a finished screen's candidates and
           dock_screen_rank of the ligands by their best E_screen

Receptors are random atom clouds of protein density around a cavity, ligands
random drug-like trees, poses uniform over each ligand's box.  Everything is
drawn on the GPU from the seed.
"""
import math

import numpy as np
import torch

import paper_2510_24186_amd as D

DEV = "cuda" if torch.cuda.is_available() else "cpu"
H = 0.375                  # grid spacing, Angstrom
N_LOCAL = 10               # Adam steps per MC step
TOP_N = 8
CLOUD_P = (0.35, 0.25, 0.05, 0.08, 0.05, 0.12, 0.07, 0.03)   # receptor types
ELEMENT_P = (0.70, 0.12, 0.14, 0.04)                         # C N O Cl
VALENCE = (4, 3, 2, 1)


def listed():
    def case(name, kind, **kw):
        return dict(name=name, kind=kind, **kw)

    one = dict(pockets=1)
    return [
        # one complex, one small ligand: the smallest docking a user runs
        # (64 trajectories x 100 MC steps), bound by latency
        case("dock_one", "sample", rec=600, grid=40, lig=1, lo=24, hi=24, tors=4, T=64, S=100, keep=False, **one),
        # one docking in the paper's sampling shape: 1,024 copies x 8 MC steps
        case("dock_paper", "sample", rec=2000, grid=64, lig=1, lo=35, hi=35, tors=8, T=1024, S=8, keep=False, **one),
        # the screening batch: 256 ligands of every size against one pocket
        case("screen", "sample", rec=2000, grid=64, lig=256, lo=10, hi=60, tors=15, T=128, S=100, keep=False, **one),
        # multi-target screening: 16 pockets of mixed sizes, larger ligands
        # too, a kept run started over with a new seed (the largest case)
        case("screen_mixed", "sample", rec=1900, grid=72, lig=2048, lo=10, hi=70, tors=15, T=64, S=30, keep=True,
             pockets=16),
        # scoring one ligand's poses: the smallest call, launch latency
        case("score_one", "score", mode="grid", preset=0, rec=600, grid=40, lig=1, lo=24, hi=24, tors=4, poses=64, **one),
        # rescoring a screen: 256 ligands x 128 poses, energies and gradients
        case("score_screen", "score", mode="grid", preset=0, rec=2000, grid=64, lig=256, lo=10, hi=60, tors=15,
             poses=128, **one),
        # the paper's own pairwise form (no maps) over a shortlist
        case("score_direct", "score", mode="direct", preset=0, rec=2000, grid=64, lig=64, lo=10, hi=60, tors=12,
             poses=32, **one),
        # the map build of one pocket, per-term maps kept for the adjoint
        case("maps", "maps", preset=0, rec=2000, grid=64, terms=True, load=False),
        # one training step on maps, weights and poses: 64 ligands x 32 poses,
        # Vina-form terms
        case("diff", "diff", preset=1, rec=2000, grid=64, lig=64, lo=10, hi=60, tors=15, poses=32, **one),
        # the adjoint of a multi-target screen's best poses, bitwise repeatable
        case("adjoint_mixed", "adjoint", preset=0, rec=1900, grid=72, lig=4096, lo=10, hi=70, tors=15, poses=1,
             pockets=16),
        # gradient of docked energies with respect to the receptor
        case("receptor_grad", "recgrad", preset=0, rec=2000, grid=64, lig=64, lo=10, hi=60, tors=12, poses=4, **one),
        # a finished screen: top poses of every ligand, then the ligand ranking
        case("hits", "hits", lig=4096, lo=10, hi=70, tors=15, T=64, top_k=1000),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["sample"] * 4 + ["score"] * 3 + ["maps", "diff", "adjoint", "recgrad", "hits"])
    lo = rng.randint(8, 30)
    hi = lo + rng.randint(0, 40)
    c = dict(kind=kind, lo=lo, hi=hi, tors=rng.randint(0, min(15, hi - 4)))
    if kind == "sample":
        # ligand evaluations stay below the largest listed case's
        pockets = rng.choice([1, 1, 1, 3, 16])
        lig = max(pockets, log(1, 1500))
        T = log(8, 1100)
        S = max(1, min(log(2, 120), int(30e6 / (lig * T * (N_LOCAL + 1)))))
        T = max(8, min(T, int(30e6 / (lig * S * (N_LOCAL + 1)))))
        return dict(c, rec=log(300, 2400), grid=rng.randint(32, 80), pockets=pockets, lig=lig, T=T, S=S,
                    keep=rng.random() < 0.5)
    if kind == "maps":
        return dict(kind=kind, preset=rng.randint(0, 1), rec=log(200, 3000), grid=rng.randint(32, 88),
                    terms=rng.random() < 0.5, load=rng.random() < 0.5)
    if kind == "hits":
        lig = log(1, 4096)
        T = min(log(4, 1000), 260000 // lig)
        return dict(c, lig=lig, T=T, top_k=min(1024, log(1, lig)) if lig > 1 else 1)
    c.update(preset=rng.randint(0, 1), rec=log(300, 2400), grid=rng.randint(32, 72), lig=log(1, 256),
             poses=log(1, 128), pockets=1)
    if kind == "score":
        c["mode"] = rng.choice(["grid", "grid", "grid", "direct", "mdn"])
        if c["mode"] != "grid":
            c.update(preset=0, lig=min(c["lig"], 64), poses=min(c["poses"], 32))
    elif kind == "adjoint":
        p = rng.choice([1, 2, 16])
        c.update(lig=max(c["lig"], p), pockets=p)
    elif kind == "recgrad":
        c.update(preset=0, poses=min(c["poses"], 8))
    elif kind == "diff":
        c.update(poses=min(c["poses"], 64))
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed, *path):
    s = int(seed)
    for p in path:
        s = (s * 1000003 + int(p) + 12345) % (1 << 62)
    return torch.Generator(device=DEV).manual_seed(s)


def receptor(seed, n, grid):
    """n atoms at random in a ball of protein density around an empty cavity,
    no two closer than 2.2 A (the candidates are taken in their order, each
    unless an earlier one that was taken is too near)."""
    g = _gen(seed, 1, n, grid)
    R = 15.0 * (n / 600.0) ** (1.0 / 3.0)
    m = 12 * n + 64
    v = torch.randn((m, 3), generator=g, device=DEV, dtype=torch.float64)
    u = torch.rand((m, 1), generator=g, device=DEV, dtype=torch.float64)
    r_in = 0.4 * R
    x = v / v.norm(dim=1, keepdim=True) * (r_in ** 3 + u * (R ** 3 - r_in ** 3)) ** (1.0 / 3.0)
    x = x.float()
    near = torch.zeros((m, m), dtype=torch.bool, device=DEV)
    for i in range(0, m, 1024):
        near[i:i + 1024] = sum((x[i:i + 1024, None, c] - x[None, :, c]) ** 2 for c in range(3)) < 2.2 ** 2
    near &= torch.ones_like(near).tril(-1)            # earlier candidates only
    undecided = torch.ones(m, dtype=torch.bool, device=DEV)
    taken = torch.zeros_like(undecided)
    while bool(undecided.any()):
        undecided &= ~(near & taken).any(1)
        new = undecided & ~(near & undecided).any(1)
        taken |= new
        undecided &= ~new
    at = torch.nonzero(taken)[:n, 0]
    assert len(at) == n, "too few places for the receptor's atoms"
    types = torch.multinomial(torch.tensor(CLOUD_P, device=DEV), n, replacement=True, generator=g)
    o = np.float32(-(grid - 1) * H / 2.0)
    return dict(xyz=x[at].cpu().numpy(), type=types.cpu().numpy().astype(np.uint8),
                origin=np.array([o, o, o], np.float32), spacing=H, dims=(grid, grid, grid))


def receptors(case, seed):
    """Pocket p of several: sizes spread around the case's."""
    P = case.get("pockets", 1)
    out = []
    for p in range(P):
        f = 1.0 if P == 1 else 0.6 + 0.8 * ((5 * p) % P) / (P - 1)
        out.append(receptor(seed * 31 + p, int(case["rec"] * f), 8 * int(round(case["grid"] * (0.5 + 0.5 * f) / 8)) if P > 1
                            else case["grid"]))
    return out


def ligands(case, seed):
    """Random trees of single bonds: every atom is bonded to a random earlier
    one with a free valence, 1.3-1.6 A away, no other atom nearer than 2 A;
    up to `tors` of the bonds between inner atoms turn."""
    B, lo, hi = case["lig"], case["lo"], case["hi"]
    g = _gen(seed, 2, B, lo, hi)
    K = 16
    n = torch.randint(lo, hi + 1, (B,), generator=g, device=DEV)
    nt = torch.randint(0, case["tors"] + 1, (B,), generator=g, device=DEV)
    # ligand 0 is of the largest size and begins as a chain, so that `tors`
    # of its bonds can turn: pose arrays are as wide for every seed
    n[0], nt[0] = hi, case["tors"]
    val = torch.tensor(VALENCE, device=DEV)
    pe = torch.tensor(ELEMENT_P, device=DEV)
    pos = torch.zeros((B, hi, 3), device=DEV)
    elem = torch.zeros((B, hi), dtype=torch.long, device=DEV)
    free = torch.zeros((B, hi), dtype=torch.long, device=DEV)
    parent = torch.zeros((B, hi), dtype=torch.long, device=DEV)
    free[:, 0] = val[0]
    rows = torch.arange(B, device=DEV)
    for a in range(1, hi):
        todo = n > a
        for attempt in range(60):
            e = torch.multinomial(pe, B, replacement=True, generator=g)
            if attempt > 20:
                e = torch.zeros_like(e)
            w = (free[:, :a] > 0).float()
            if a < case["tors"] + 4:
                e[0] = 0
                w[0, :a - 1] = 0.0
            p = torch.multinomial(w + 1e-30, K, replacement=True, generator=g)
            d = torch.randn((B, K, 3), generator=g, device=DEV)
            d = d / d.norm(dim=-1, keepdim=True) * (1.3 + 0.3 * torch.rand((B, K, 1), generator=g, device=DEV))
            x = pos.gather(1, p[..., None].expand(-1, -1, 3)) + d
            far = ((x[:, :, None] - pos[:, None, :a]) ** 2).sum(-1).scatter(2, p[..., None], 1e9).min(-1).values
            if attempt == 59:
                far = far + 1e6                     # crowded: the place with the most room
            good = (far >= 4.0) & (w.gather(1, p) > 0)
            good &= ~((val[e] == 1) & (a < n - 1) & (w.sum(1) <= 1))[:, None]
            pick = torch.where(good, far, torch.full_like(far, -1.0))
            k = pick.argmax(1) if attempt == 59 else good.float().argmax(1)
            put = todo & good.any(1)
            i = rows[put]
            kk = k[put]
            pos[i, a] = x[i, kk]
            parent[i, a] = p[i, kk]
            elem[i, a] = e[put]
            free[i, a] = val[e[put]] - 1
            free[i, p[i, kk]] -= 1
            todo = todo & ~put
            if not bool(todo.any()):
                break
        assert not bool(todo.any()), "a ligand has no place for its next atom"
    deg = val[elem] - free
    at = torch.arange(hi, device=DEV)[None] < n[:, None]
    inner = at & (deg >= 2) & (deg.gather(1, parent) >= 2)
    inner[:, 0] = False
    score = torch.where(inner, torch.rand((B, hi), generator=g, device=DEV), torch.full_like(pos[..., 0], -1.0))
    rank = score.argsort(dim=1, descending=True, stable=True).argsort(dim=1, stable=True)
    rot = inner & (rank < nt[:, None])
    # centred near the cavity's middle, turned at random
    mean = (pos * at[..., None]).sum(1) / n[:, None]
    q = torch.randn((B, 4), generator=g, device=DEV)
    q = q / q.norm(dim=1, keepdim=True)
    w_, x_, y_, z_ = q.unbind(1)
    Rm = torch.stack([1 - 2 * (y_ * y_ + z_ * z_), 2 * (x_ * y_ - z_ * w_), 2 * (x_ * z_ + y_ * w_),
                      2 * (x_ * y_ + z_ * w_), 1 - 2 * (x_ * x_ + z_ * z_), 2 * (y_ * z_ - x_ * w_),
                      2 * (x_ * z_ - y_ * w_), 2 * (y_ * z_ + x_ * w_), 1 - 2 * (x_ * x_ + y_ * y_)], 1).view(B, 3, 3)
    c = torch.randn((B, 1, 3), generator=g, device=DEV)
    pos = ((pos - mean[:, None])[:, :, None, :] * Rm[:, None]).sum(-1) + c
    at, nn = at.cpu().numpy(), n.cpu().numpy()
    par, bond = parent.cpu().numpy(), at.copy()
    bond[:, 0] = False
    idx = np.broadcast_to(np.arange(hi), (B, hi))
    off = np.concatenate([[0], np.cumsum(nn)]).astype(np.int32)
    boff = np.concatenate([[0], np.cumsum(nn - 1)]).astype(np.int32)
    P = case.get("pockets", 1)
    return dict(atom_off=off, element=elem.cpu().numpy()[at].astype(np.uint8), n_h=free.cpu().numpy()[at].astype(np.uint8),
                xyz=pos.cpu().numpy()[at].astype(np.float32), bond_off=boff,
                bonds=np.stack([par[bond], idx[bond]], 1).astype(np.int32),
                rotatable=rot.cpu().numpy()[bond].astype(np.uint8), pocket_index=(np.arange(B) % P).astype(np.int32))


def n_dofs(L):
    c = np.concatenate([[0], np.cumsum(L["rotatable"])])
    return 6 + c[L["bond_off"][1:]] - c[L["bond_off"][:-1]]


def boxes(L):
    at = L["atom_off"][:-1]
    return np.minimum.reduceat(L["xyz"], at, axis=0), np.maximum.reduceat(L["xyz"], at, axis=0)


def poses(case, L, seed):
    """(ligand of each pose, q): translation uniform in the ligand's box,
    angles uniform; a ligand's poses one after the other."""
    g = _gen(seed, 3)
    nd = n_dofs(L)
    qs = int(nd.max())
    lo, hi = (torch.tensor(v, device=DEV) for v in boxes(L))
    lig = torch.arange(case["lig"], device=DEV).repeat_interleave(case["poses"])
    q = torch.rand((len(lig), qs), generator=g, device=DEV)
    q[:, :3] = lo[lig] + (hi - lo)[lig] * q[:, :3]
    q[:, 3:] = -math.pi + 2 * math.pi * q[:, 3:]
    q *= torch.arange(qs, device=DEV)[None] < torch.tensor(nd, device=DEV)[lig][:, None]
    return lig.int(), q.contiguous()


def candidates(case, L, seed):
    """E [lig, T] and q [lig, T, qs] as a sampling run leaves them: some
    trajectories in common basins, the others alone."""
    g = _gen(seed, 4)
    B, T = case["lig"], case["T"]
    nd = n_dofs(L)
    qs = int(nd.max())
    lo, hi = (torch.tensor(v, device=DEV) for v in boxes(L))
    C = 12
    q = torch.rand((B, C, qs), generator=g, device=DEV)
    q[..., :3] = lo[:, None] + (hi - lo)[:, None] * q[..., :3]
    q[..., 3:] = -math.pi + 2 * math.pi * q[..., 3:]
    Ec = 10.0 * torch.rand((B, C), generator=g, device=DEV) - 8.0
    which = (C * torch.rand((B, T), generator=g, device=DEV) ** 1.5).long().clamp_(max=C - 1)
    wide = torch.where(torch.rand((B, T, 1), generator=g, device=DEV) < 0.3, 1.0, 0.04)
    q = q.gather(1, which[..., None].expand(-1, -1, qs)) + wide * torch.randn((B, T, qs), generator=g, device=DEV)
    E = Ec.gather(1, which) + 3.0 * wide[..., 0] * torch.rand((B, T), generator=g, device=DEV)
    q *= (torch.arange(qs, device=DEV)[None] < torch.tensor(nd, device=DEV)[:, None])[:, None]
    return E.contiguous(), q.contiguous()


def residues(pk):
    """About eight neighbouring atoms each: 6 A cells of the receptor."""
    cell = np.floor((pk["xyz"] - pk["xyz"].min(0)) / 6.0).astype(np.int64)
    return np.unique(cell @ np.array([1, 1000, 1000000]), return_inverse=True)[1].astype(np.int32)


def mixtures(n_atoms, n_res, seed):
    g = _gen(seed, 5)
    pi = torch.rand((n_atoms, n_res, 4), generator=g, device=DEV)
    pi = pi / pi.sum(-1, keepdim=True)
    mu = 2.5 + 3.0 * torch.rand((n_atoms, n_res, 4), generator=g, device=DEV)
    sig = 0.3 + 0.7 * torch.rand((n_atoms, n_res, 4), generator=g, device=DEV)
    return torch.stack([pi, mu, sig], -1).cpu().numpy()


def weights(case, seed):
    """Term weights on their way through a fit: near the preset's."""
    w0 = torch.tensor((0.2, 10.0, 0.6) if case["preset"] == 0 else (-0.0356, -0.00516, 0.840, -0.0351, -0.587), device=DEV)
    g = _gen(seed, 6)
    return (w0 + 0.1 * w0.abs() * torch.randn((case.get("pockets", 1), len(w0)), generator=g, device=DEV)).contiguous()


def dLdE_of(n, seed):
    return 0.5 + torch.rand(n, generator=_gen(seed, 7), device=DEV)


# ------------------------------------------------------------------ the calls

def _load(pk, case, keep=False):
    kw = {}
    if case.get("mode") == "direct":
        kw["inter_mode"] = D.INTER_DIRECT
    if case.get("mode") == "mdn":
        kw["residue"] = residues(pk)
    return D.dock_load_pocket(pk["xyz"], pk["type"], pk["origin"], pk["spacing"], pk["dims"],
                              preset=case.get("preset", 0), keep_per_term=keep, **kw)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, seed=seed & 0x7FFFFFFF)
    if kind == "maps":
        s["pk"] = receptor(seed, case["rec"], case["grid"])
        if not case["load"]:
            s["pocket"] = _load(s["pk"], case, case["terms"])
        return s
    L = ligands(case, seed)
    s["L"] = D.dock_load_ligands(**L)
    if kind == "hits":
        s["E"], s["q"] = candidates(case, L, seed)
        return s
    pks = receptors(case, seed)
    s["pockets"] = [_load(pk, case, kind in ("diff", "adjoint", "recgrad")) for pk in pks]
    if kind == "sample":
        if case["keep"]:
            s["run"] = D.dock_sample(s["pockets"], s["L"], n_traj=case["T"], n_steps=case["S"], n_local=N_LOCAL,
                                     seed=s["seed"] ^ 1)
        return s
    s["lig"], s["q"] = poses(case, L, seed)
    if kind == "score":
        if case["mode"] == "mdn":
            res = residues(pks[0])
            D.dock_ligands_set_mdn(s["L"], mixtures(len(L["element"]), int(res.max()) + 1, seed))
        return s
    s["w"] = weights(case, seed)
    s["dLdE"] = dLdE_of(len(s["lig"]), seed)
    if kind == "diff":
        s["G"] = D.dock_pocket_maps(s["pockets"][0], per_term=True).requires_grad_()
        s["w"].requires_grad_()
        s["q"].requires_grad_()
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "sample":
        r = s.get("run")
        if r is None:
            r = D.dock_sample(s["pockets"], s["L"], n_traj=case["T"], n_steps=case["S"], n_local=N_LOCAL, seed=s["seed"])
        else:
            D.dock_run_restart(r, s["seed"])
        st = D.dock_run_state(r)
        best = D.dock_best_poses(s["L"], case["T"], st["E_best"], st["q_best"], top_n=TOP_N)
        return dict(st, best=best)
    if kind == "score":
        return D.dock_score_grad(s["pockets"], s["L"], s["lig"], s["q"])[:2]
    if kind == "maps":
        p = s.get("pocket")
        if p is None:
            p = _load(s["pk"], case, case["terms"])
        else:
            D.dock_pocket_rebuild(p)
        return [D.dock_pocket_maps(p, per_term=t) for t in ((False, True) if case["terms"] else (False,))]
    if kind == "diff":
        s["G"].grad = s["w"].grad = s["q"].grad = None
        E = D.dock_score(s["pockets"], s["L"], s["lig"], s["w"], s["G"], q=s["q"])
        (E * s["dLdE"]).sum().backward()
        return E.detach(), s["G"].grad, s["w"].grad, s["q"].grad
    if kind in ("adjoint", "recgrad"):
        dG = [torch.zeros((8, p.n_terms, p.dims[2], p.dims[1], p.dims[0]), device=DEV) for p in s["pockets"]]
        dw, dq = torch.zeros_like(s["w"]), torch.zeros_like(s["q"])
        D.dock_score_adjoint(s["pockets"], s["L"], s["lig"], s["w"], s["dLdE"], q=s["q"], dLdG=dG, dLdw=dw, dLdq=dq,
                             deterministic=True)
        if kind == "adjoint":
            return dG, dw, dq
        dx = torch.zeros((case["rec"], 3), device=DEV)
        dth = torch.zeros(13, dtype=torch.float64, device=DEV)
        D.dock_pocket_map_adjoint(s["pockets"][0], dG[0], dx, dth)
        return dG[0], dw, dq, dx, dth
    best = D.dock_best_poses(s["L"], case["T"], s["E"], s["q"], top_n=TOP_N)
    score, lig = D.dock_screen_rank(best["E_screen"], case["top_k"], stride=TOP_N)
    return dict(best, score=score, lig=lig)


# ------------------------------------------------------------------ work

def work(case):
    """Operations of the path itself: 105 per atom (placement, trilinear value
    and gradient, chain rule), 50 per intra-ligand pair, 60 per torsion and
    evaluation; 20 per receptor pair inside a cutoff; maps: per node and
    neighbour inside the cutoff.  Bytes: maps, ligands, poses and candidates
    read once, results written once."""
    kind, P = case["kind"], case.get("pockets", 1)
    K = 3 if case.get("preset", 0) == 0 else 5
    N = 0.5 * (case.get("lo", 0) + case.get("hi", 0))
    qs = 6 + case.get("tors", 0)
    nodes = case.get("grid", 0) ** 3
    pairs = 0.42 * N * N * min(1.0, case.get("tors", 0) / 6.0)
    ev = 105 * N + 50 * pairs + 30 * case.get("tors", 0)
    near = 0.042 * 4.19 * 1000 if K == 3 else 0.042 * 4.19 * 512     # receptor atoms inside the cutoff
    best = 4 * TOP_N * (3 + qs + 3 * case.get("hi", 0))
    if kind == "sample":
        n = case["lig"] * case["T"]
        return dict(flops=ev * n * (1 + case["S"] * (N_LOCAL + 1)),
                    bytes=P * nodes * 32.0 + n * 4 * (4 * qs + 6) + case["lig"] * (16 * N + 8 * pairs + best))
    if kind == "maps":
        return dict(flops=nodes * near * 8 * K * 5.0, bytes=nodes * 32.0 * (1 + (K if case["terms"] else 0)) + 16 * case["rec"])
    if kind == "hits":
        n = case["lig"] * case["T"]
        return dict(flops=case["lig"] * 3 * TOP_N * (15 * N + 60 * case["tors"] / 2 + 4 * TOP_N * N),
                    bytes=n * 4.0 + case["lig"] * (best + TOP_N * 4 * qs + 16 * N))
    n = case["lig"] * case["poses"]
    rw = n * 4.0 * (2 + 2 * qs) + case["lig"] * (16 * N + 8 * pairs)
    if kind == "score":
        if case["mode"] == "direct":
            return dict(flops=n * (ev + N * near * 20), bytes=rw + 16.0 * case["rec"])
        return dict(flops=n * ev, bytes=rw + min(nodes * 32.0, n * N * 32.0))
    touched = min(nodes * 8.0 * K, n * N * 8.0 * K)
    flops = n * (ev + 40 * N * 8 * K)
    if kind == "diff":
        return dict(flops=2 * flops, bytes=rw + 4.0 * (touched + nodes * 8 * K))
    if kind == "recgrad":
        flops += min(nodes, n * N * 8) * near * 8 * 20.0
    return dict(flops=flops, bytes=rw + 4.0 * (P * touched + P * nodes * 8 * K))


# ------------------------------------------------------------------ 64 bits

RAD = (1.9, 1.9, 1.8, 1.8, 1.8, 1.7, 1.7, 1.8)
DON, ACC, HYD = (3, 6), (4, 5, 6), (0, 7)
F64 = torch.float64


def _t(v, dtype=F64):
    return torch.as_tensor(np.asarray(v), device=DEV).to(dtype)


def _pair_tables(a, b):
    """(radius sum, hydrogen bond, hydrophobic) of type arrays a [..] and b [..]."""
    rad = torch.tensor(RAD, dtype=F64, device=DEV)
    is_ = lambda t, s: sum((t == v) for v in s).bool()  # noqa: E731
    hb = (is_(a, DON) & is_(b, ACC)) | (is_(a, ACC) & is_(b, DON))
    return rad[a] + rad[b], hb, is_(a, HYD) & is_(b, HYD)


def _terms(preset, d2, d, rs, hb, hyd):
    """Unweighted terms of a pair; d2 decides the cutoffs."""
    z = torch.zeros_like(d)
    if preset == 0:
        s = d - rs - 3.0
        dc = torch.where(hb, torch.full_like(rs, 2.6), rs)
        dc2 = (dc.float() * dc.float()).to(d2.dtype)
        safe = d.clamp(min=0.1)
        return [torch.where(d2 < 100.0, -torch.exp(-0.25 * s * s), z), torch.where(d2 < dc2, -torch.log(safe / dc), z),
                torch.where(hb & (d2 < float(np.float32(3.4) * np.float32(3.4))), -torch.exp(-(d - 2.88) ** 2 / 0.18), z)]
    s = d - rs
    t = s - 3.0
    inside = d2 < 64.0
    v = [torch.exp(-4.0 * s * s), torch.exp(-0.25 * t * t), torch.where(s < 0, s * s, z),
         torch.where(hyd, (1.5 - s).clamp(0.0, 1.0), z), torch.where(hb, (-s / 0.7).clamp(0.0, 1.0), z)]
    return [torch.where(inside, x, z) for x in v]


def _node_axes(pk):
    return [torch.tensor(np.float64(pk["origin"][c]) + H * np.arange(pk["dims"][c]), device=DEV).float() for c in range(3)]


def maps64(pk, preset):
    """G [8, K, nz, ny, nx] in 64 bits; cutoffs decided on the 32-bit squared
    distance ((dx dx + dy dy) + dz dz), as the maps are specified."""
    X, Y, Z = _node_axes(pk)
    nx, ny, nz = pk["dims"]
    K = 3 if preset == 0 else 5
    rec, tr = _t(pk["xyz"], torch.float32), _t(pk["type"], torch.long)
    n = nx * ny * nz
    G = torch.zeros((8, K, n), dtype=F64, device=DEV)
    step = max(1, 24_000_000 // len(rec))
    node = torch.stack([t.reshape(-1) for t in torch.meshgrid(Z, Y, X, indexing="ij")], 1).flip(1)
    for i in range(0, n, step):
        dx = [node[i:i + step, c, None] - rec[None, :, c] for c in range(3)]
        d2 = (dx[0] * dx[0] + dx[1] * dx[1]) + dx[2] * dx[2]
        d = sum((node[i:i + step, c, None].double() - rec[None, :, c].double()) ** 2 for c in range(3)).sqrt()
        for r in sorted(set(RAD)):
            ts = [t for t in range(8) if RAD[t] == r]
            rs = (torch.tensor(RAD, dtype=F64, device=DEV)[tr] + r)[None].expand_as(d)
            off, on = torch.zeros_like(rs, dtype=torch.bool), torch.ones_like(rs, dtype=torch.bool)
            plain, bonded = _terms(preset, d2, d, rs, off, on), _terms(preset, d2, d, rs, on, on)
            for t in ts:
                _, hb, hyd = _pair_tables(torch.full_like(tr, t), tr)
                h, y = hb.double(), hyd.double()
                for k in range(K):
                    if preset == 0:
                        G[t, k, i:i + step] = plain[k] @ (1 - h) + bonded[k] @ h
                    else:
                        sel = y if k == 3 else (h if k == 4 else torch.ones_like(h))
                        G[t, k, i:i + step] = bonded[k] @ sel
    return G.view(8, K, nz, ny, nx)


class Topo:
    """Types, torsions and intra-ligand pairs of the ligands, padded."""

    def __init__(self, L):
        B = len(L["atom_off"]) - 1
        per = [self._one(L, i) for i in range(B)]
        N = max(len(p["x"]) for p in per)
        nt = max([len(p["tors"]) for p in per] + [1])
        npair = max([len(p["pairs"]) for p in per] + [1])
        x, typ, live = np.zeros((B, N, 3)), np.zeros((B, N), np.int64), np.zeros((B, N), bool)
        c0, u, xb, mask = np.zeros((B, 3)), np.zeros((B, nt, 3)), np.zeros((B, nt, 3)), np.zeros((B, nt, N), bool)
        pr, pl = np.zeros((B, npair, 2), np.int64), np.zeros((B, npair), bool)
        for i, p in enumerate(per):
            n, k, m = len(p["x"]), len(p["tors"]), len(p["pairs"])
            x[i, :n], typ[i, :n], live[i, :n], c0[i] = p["x"], p["type"], True, p["c0"]
            for j, (a, b, mv) in enumerate(p["tors"]):
                v = p["x"][b] - p["x"][a]
                u[i, j], xb[i, j], mask[i, j, :n] = v / np.linalg.norm(v), p["x"][b], mv
            pr[i, :m], pl[i, :m] = p["pairs"], True
        self.x, self.type, self.live, self.c0 = _t(x), _t(typ, torch.long), _t(live, torch.bool), _t(c0)
        self.u, self.xb, self.mask, self.nt = _t(u), _t(xb), _t(mask), nt
        self.pairs, self.pair_live = _t(pr, torch.long), _t(pl, torch.bool)
        self.pocket = _t(L["pocket_index"], torch.long)
        self.n_tors = _t(n_dofs(L) - 6)
        self.n_atoms = _t(np.diff(L["atom_off"]))

    @staticmethod
    def _one(L, i):
        a0, a1, b0, b1 = (int(L[k][j]) for k, j in (("atom_off", i), ("atom_off", i + 1), ("bond_off", i), ("bond_off", i + 1)))
        el, nh, x = L["element"][a0:a1], L["n_h"][a0:a1], L["xyz"][a0:a1].astype(np.float64)
        bonds, rot = L["bonds"][b0:b1], L["rotatable"][b0:b1]
        n = a1 - a0
        dist, frag, fpar = np.zeros((n, n), np.int64), np.zeros(n, np.int64), [-1]
        link = [None]
        deg, polar = np.zeros(n, np.int64), np.zeros(n, bool)
        for (p, a), r in zip(bonds.tolist(), rot.tolist()):      # bond k attaches atom k + 1
            dist[a, :a] = dist[:a, a] = dist[p, :a] + 1
            dist[a, a] = 0
            deg[p] += 1
            deg[a] += 1
            polar[a] |= el[p] in (1, 2)
            polar[p] |= el[a] in (1, 2)
            frag[a] = frag[p]
            if r:
                frag[a] = len(fpar)
                fpar.append(int(frag[p]))
                link.append((p, a))
        F = len(fpar)
        fd = np.zeros((F, F), np.int64)
        adj = [[] for _ in range(F)]
        for f in range(1, F):
            fd[f, :f] = fd[:f, f] = fd[fpar[f], :f] + 1
            adj[f].append(fpar[f])
            adj[fpar[f]].append(f)
        root = int(fd.max(1).argmin())
        order, seen, tors = [root], {root}, []
        for f in order:
            for h in sorted(adj[f]):
                if h not in seen:
                    seen.add(h)
                    order.append(h)
                    a, b = link[h] if fpar[h] == f else link[f][::-1]
                    tors.append((a, b, dist[b] < dist[a]))
        typ = np.where(el == 0, np.where(polar, 1, 0),
                       np.where(el == 1, np.where(nh >= 1, 3, np.where(deg <= 2, 4, 2)),
                                np.where(el == 2, np.where(nh >= 1, 6, 5), 7)))
        ii, jj = np.nonzero(np.triu((dist >= 4) & (frag[:, None] != frag[None]), 1))
        return dict(x=x, type=typ, tors=tors, pairs=np.stack([ii, jj], 1), c0=x[frag == root].mean(0))

    def place(self, lig, q):
        """World coordinates [P, N, 3] of poses q (differentiable)."""
        x = self.x[lig]
        for k in range(self.nt - 1, -1, -1):          # innermost axes last
            u, xb, m = self.u[lig, k][:, None], self.xb[lig, k][:, None], self.mask[lig, k][..., None]
            if 6 + k >= q.shape[1]:
                continue
            th = q[:, 6 + k, None, None]
            v = x - xb
            turned = xb + v * th.cos() + torch.linalg.cross(u.expand_as(v), v) * th.sin() + u * (u * v).sum(-1, keepdim=True) * (1 - th.cos())
            x = x + m * (turned - x)
        a, b, g = q[:, 3], q[:, 4], q[:, 5]
        ca, sa, cb, sb, cg, sg = a.cos(), a.sin(), b.cos(), b.sin(), g.cos(), g.sin()
        R = torch.stack([ca * cb, ca * sb * sg - sa * cg, ca * sb * cg + sa * sg, sa * cb, sa * sb * sg + ca * cg,
                         sa * sb * cg - ca * sg, -sb, cb * sg, cb * cg], 1).view(-1, 3, 3)
        return q[:, None, :3] + ((x - self.c0[lig][:, None])[:, :, None, :] * R[:, None]).sum(-1)


def _cells(pk, x):
    """Lower corner (flat index), fractions and the out-of-box penalty."""
    o = _t(pk["origin"].astype(np.float64))
    n = torch.tensor(pk["dims"], device=DEV)
    top = (o + H * (n - 1)).float().double()
    xc = torch.minimum(torch.maximum(x, o), top)
    u = (xc - o) / H
    c = torch.minimum(u.detach().floor().long(), n - 2).clamp(min=0)
    flat = (c[..., 2] * n[1] + c[..., 1]) * n[0] + c[..., 0]
    return flat, u - c, 10.0 * (x - xc).abs().sum(-1)


def _corners(pk, f):
    nx, nxy = pk["dims"][0], pk["dims"][0] * pk["dims"][1]
    for dz in (0, 1):
        for dy in (0, 1):
            for dx in (0, 1):
                w = (f[..., 0] if dx else 1 - f[..., 0]) * (f[..., 1] if dy else 1 - f[..., 1]) * (f[..., 2] if dz else 1 - f[..., 2])
                yield dx + dy * nx + dz * nxy, w


def _intra(T, lig, x, preset):
    """Per-term sums [P, K] of the intra-ligand pairs."""
    i, j = T.pairs[lig, :, 0], T.pairs[lig, :, 1]
    d2 = ((x.gather(1, i[..., None].expand(-1, -1, 3)) - x.gather(1, j[..., None].expand(-1, -1, 3))) ** 2).sum(-1)
    live = T.pair_live[lig]
    d2 = torch.where(live, d2, torch.ones_like(d2))
    rs, hb, hyd = _pair_tables(T.type[lig].gather(1, i), T.type[lig].gather(1, j))
    return torch.stack([(v * live).sum(1) for v in _terms(preset, d2.detach(), d2.sqrt(), rs, hb, hyd)], 1)


def _inter_direct(pk, T, lig, x, preset, w):
    rec, tr = _t(pk["xyz"].astype(np.float64)), _t(pk["type"], torch.long)
    d2 = ((x[:, :, None] - rec) ** 2).sum(-1)
    rs, hb, hyd = _pair_tables(T.type[lig][..., None], tr)
    v = _terms(preset, d2.detach(), d2.sqrt(), rs.expand_as(d2), hb.expand_as(d2), hyd.expand_as(d2))
    return sum(w[k] * v[k] for k in range(len(v))).sum(-1)


def _inter_mdn(pk, T, lig, x, par):
    """par: [ligand, atom, residue, gaussian, 3]"""
    rec, res = _t(pk["xyz"].astype(np.float64)), _t(residues(pk), torch.long)
    d = ((x[:, :, None] - rec) ** 2).sum(-1).sqrt()
    near = torch.full(d.shape[:2] + (int(res.max()) + 1,), math.inf, dtype=F64, device=DEV)
    near = near.scatter_reduce(2, res.expand_as(d), d, "amin")
    g = par[lig]
    P = (g[..., 0] * torch.exp(-(near[..., None] - g[..., 1]) ** 2 / (2 * g[..., 2] ** 2))).sum(-1)
    return -torch.where(near.detach() < 5.0, P, torch.zeros_like(P)).sum(-1)


def _w32(preset):
    return _t(np.asarray((0.2, 10.0, 0.6) if preset == 0 else (-0.0356, -0.00516, 0.840, -0.0351, -0.587), np.float32))


def _score64(case, seed):
    pk, L = receptors(case, seed)[0], ligands(case, seed)
    T = Topo(L)
    lig, q = poses(case, L, seed)
    lig = lig.long()
    w, preset, mode = _w32(case["preset"]), case["preset"], case["mode"]
    M = None if mode == "direct" else (maps64(pk, preset) * w[None, :, None, None, None]).sum(1).reshape(8, -1)
    par = None
    if mode == "mdn":
        flat = _t(mixtures(len(L["element"]), int(residues(pk).max()) + 1, seed))
        par = torch.zeros(T.live.shape + flat.shape[1:], dtype=F64, device=DEV)
        par[..., 2] = 1.0
        par[T.live] = flat
    E, g = [], []
    step = max(1, (2048 if mode == "grid" else 16) * 35 // max(1, case["hi"]))
    for i in range(0, len(lig), step):
        li, qi = lig[i:i + step], q[i:i + step].double().requires_grad_()
        x = T.place(li, qi)
        if mode == "direct":
            e = _inter_direct(pk, T, li, x, preset, w)
        else:
            c, f, out = _cells(pk, x)
            e = sum(wt * M[T.type[li], c + o] for o, wt in _corners(pk, f)) + out
            if par is not None:
                e = e + _inter_mdn(pk, T, li, x, par)
        e = (e * T.live[li]).sum(1) + (_intra(T, li, x, preset) * w).sum(1)
        g.append(torch.autograd.grad(e.sum(), qi)[0])
        E.append(e.detach())
    return torch.cat(E), torch.cat(g)


def _diff64(case, seed):
    """(E, [dL/dG], dL/dw, dL/dq) of sum(dLdE E) in 64 bits."""
    pks, L = receptors(case, seed), ligands(case, seed)
    T = Topo(L)
    lig, q = poses(case, L, seed)
    lig = lig.long()
    preset, w = case["preset"], weights(case, seed).double()
    c_all = dLdE_of(len(lig), seed).double()
    K = w.shape[1]
    E, dq = torch.zeros(len(lig), dtype=F64, device=DEV), torch.zeros(q.shape, dtype=F64, device=DEV)
    dw, dG = torch.zeros_like(w), []
    for p, pk in enumerate(pks):
        G = maps64(pk, preset).reshape(8, K, -1)
        d = torch.zeros_like(G)
        mine = torch.nonzero(T.pocket[lig] == p)[:, 0]
        for at in mine.split(512):
            li, qi, c = lig[at], q[at].double().requires_grad_(), c_all[at]
            x = T.place(li, qi)
            cell, f, out = _cells(pk, x)
            live, typ = T.live[li], T.type[li]
            per = _intra(T, li, x, preset)
            for o, wt in _corners(pk, f):
                idx = (cell + o)
                per = per + ((wt * live)[..., None] * G[typ, :, idx]).sum(1)
                add = ((wt * live).detach() * c[:, None])[..., None] * w[p]
                for k in range(K):
                    d.view(-1).index_add_(0, ((typ * K + k) * G.shape[2] + idx).reshape(-1), add[..., k].reshape(-1))
            e = (per * w[p]).sum(1) + (out * live).sum(1)
            dq[at] = torch.autograd.grad((e * c).sum(), qi)[0]
            E[at] = e.detach()
            dw[p] += (per.detach() * c[:, None]).sum(0)
        dG.append(d.view(8, K, *pk["dims"][::-1]))
    return E, dG, dw, dq


def _receptor64(pk, lam):
    """dL/d(receptor xyz) and dL/d(term constants) for lam = dL/dG."""
    rec, tr = _t(pk["xyz"], torch.float32), _t(pk["type"], torch.long)
    X, Y, Z = _node_axes(pk)
    node = torch.stack([t.reshape(-1) for t in torch.meshgrid(Z, Y, X, indexing="ij")], 1).flip(1)
    lam = lam.reshape(8, 3, -1)
    at = torch.nonzero((lam != 0).any(0).any(0))[:, 0]
    dx, dth = torch.zeros((len(rec), 3), dtype=F64, device=DEV), torch.zeros(13, dtype=F64, device=DEV)
    for ids in at.split(max(1, 8_000_000 // len(rec))):
        e32 = [node[ids, c, None] - rec[None, :, c] for c in range(3)]
        d2 = (e32[0] * e32[0] + e32[1] * e32[1]) + e32[2] * e32[2]
        e = rec.double()[None] - node[ids].double()[:, None]
        d = (e ** 2).sum(-1).sqrt()
        dphi = torch.zeros_like(d)
        for t in range(8):
            rs, hb, _ = _pair_tables(torch.full_like(tr, t), tr)
            l0, l1, l2 = (lam[t, k, ids][:, None] for k in range(3))
            s = d - rs - 3.0
            a = torch.where(d2 < 100.0, l0 * torch.exp(-0.25 * s * s), torch.zeros_like(d))
            dphi += a * s / 2.0
            dth[0] -= (a * s / 2.0).sum()
            dth[1] -= (a * s * s / (2.0 * math.sqrt(2.0))).sum()
            per_atom = -(a * s / 2.0).sum(0)
            dc = torch.where(hb, torch.full_like(rs, 2.6), rs)
            inside = d2 < (dc.float() * dc.float())
            dphi -= torch.where(inside & (d > 0.1), l1 / d, torch.zeros_like(d))
            cl = torch.where(inside, l1 / dc, torch.zeros_like(d)).sum(0)
            dth[4] += cl[hb].sum()
            per_atom = per_atom + torch.where(hb, torch.zeros_like(cl), cl)
            dth[5 + t] += per_atom.sum()
            dth[5:].index_add_(0, tr, per_atom)
            y = d - 2.88
            b = torch.where(hb & (d2 < float(np.float32(3.4) * np.float32(3.4))), l2 * torch.exp(-y * y / 0.18), torch.zeros_like(d))
            dphi += b * y / 0.09
            dth[2] -= (b * y / 0.09).sum()
            dth[3] -= (b * y * y / 0.027).sum()
        dx += (dphi / d.clamp(min=1e-300))[..., None].mul(e).sum(0)
    return dx, dth


def _hits64(case, seed):
    """Ranking, clustering (1 A, no superposition) and placement."""
    L = ligands(case, seed)
    T = Topo(L)
    E, q = candidates(case, L, seed)
    B, n_t = E.shape
    order = torch.sort(E, dim=1, stable=True)
    dev = dict(dtype=F64, device=DEV)
    kept = torch.zeros((B, TOP_N, T.x.shape[1], 3), **dev)
    out_E, out_q = torch.full((B, TOP_N), math.inf, **dev), torch.zeros((B, TOP_N, q.shape[2]), **dev)
    n = torch.zeros(B, dtype=torch.long, device=DEV)
    rows = torch.arange(B, device=DEV)
    for c in range(n_t):
        qc = q[rows, order.indices[:, c]]
        x = T.place(rows, qc.double()) * T.live[..., None]
        rmsd = ((((kept - x[:, None]) ** 2).sum((2, 3))) / T.n_atoms[:, None]).sqrt()
        near = ((rmsd < 1.0) & (torch.arange(TOP_N, device=DEV)[None] < n[:, None])).any(1)
        put = torch.nonzero(~near & (n < TOP_N))[:, 0]
        kept[put, n[put]] = x[put]
        out_E[put, n[put]] = order.values[put, c].double()
        out_q[put, n[put]] = qc[put].double()
        n[put] += 1
    screen = out_E / (1.0 + 0.01 * T.n_tors[:, None])
    rank = torch.sort(screen[:, 0], stable=True)
    return dict(E=out_E, E_screen=screen, q=out_q, idx=None, xyz=kept, n=None, score=rank.values[:case["top_k"]], lig=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "sample":
        return None                      # a chain of accept/reject decisions
    if kind == "maps":
        G = maps64(receptor(seed, case["rec"], case["grid"]), case["preset"])
        M = (G * _w32(case["preset"])[None, :, None, None, None]).sum(1)
        return [M, G] if case["terms"] else [M]
    if kind == "score":
        return _score64(case, seed)
    if kind == "hits":
        return _hits64(case, seed) if case["lig"] * case["T"] <= 1 << 18 else None
    E, dG, dw, dq = _diff64(case, seed)
    if kind == "diff":
        return E, dG[0], dw, dq
    if kind == "adjoint":
        return dG, dw, dq
    pk = receptors(case, seed)[0]
    return (dG[0], dw, dq) + _receptor64(pk, dG[0])
