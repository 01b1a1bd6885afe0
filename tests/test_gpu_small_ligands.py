"""Handles whose ligands all take 16 lanes are scored by kernels of that form
alone, other handles by kernels that choose the form per pose: the same poses of
the same ligands get the same bits from either, in every mode of the score and
in the differentiable form.  Run on an MI355X."""
import numpy as np
import pytest

import synth
from oracle import params as P
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SPEC = [(2, 0), (10, 4), (16, 8), (9, 2), (12, 1)]


def _handles(n_poses):
    ligs = [synth.make_ligand(n, t, np.random.default_rng(500 + n)) for n, t in SPEC]
    out = []
    for more in ([], [synth.make_ligand(70, 8, np.random.default_rng(9))]):
        L = synth.pack_ligands(ligs + more)
        L.pocket_index = np.zeros(L.n_ligands, np.int32)
        out.append((G.load_ligands(L), int(L.atom_off[-1])))
    rng = np.random.default_rng(n_poses)
    lig = rng.integers(0, len(SPEC), n_poses).astype(np.int32)
    if n_poses > 8:
        lig[rng.choice(n_poses, 2, replace=False)] = -1
    (H, _), (B, _) = out
    assert H.q_stride == B.q_stride
    q = np.zeros((n_poses, H.q_stride), np.float32)
    q[:, :3] = rng.uniform(-3, 3, (n_poses, 3))
    q[:, 3:] = rng.uniform(-np.pi, np.pi, (n_poses, H.q_stride - 3))
    return out, torch.tensor(lig, device="cuda"), torch.tensor(q, device="cuda"), rng


def _same(a, b):
    return torch.equal(torch.nan_to_num(a, nan=123.0), torch.nan_to_num(b, nan=123.0))


@pytest.mark.parametrize("n_poses", [1, 3, 5, 1023, 9001])
@pytest.mark.parametrize("mode", ["grid", "direct", "mdn"])
def test_score(n_poses, mode):
    D = G.lib()
    G.say("small ligands", mode, n_poses)
    pk = synth.make_pocket(600, grid=40, seed=6)
    res = synth.make_residues(pk) if mode == "mdn" else None
    p = G.load_pocket(pk, direct=mode == "direct", residue=res)
    handles, lig, q, _ = _handles(n_poses)
    got = []
    for H, atoms in handles:
        if mode == "mdn":
            par = synth.make_mdn_params(handles[1][1], int(res.max()) + 1, 4, seed=5)
            D.dock_ligands_set_mdn(H, par[:atoms])
        E, g, xyz = D.dock_score_grad(p, H, lig, q, want_xyz=True)
        got.append((E, g, xyz[:, :16]))
    for a, b in zip(*got):
        assert _same(a, b)


@pytest.mark.parametrize("n_poses", [1, 3, 5, 1023, 9001])
@pytest.mark.parametrize("preset", [P.PRESET_TRIDS, P.PRESET_VINA])
def test_differentiable_form(n_poses, preset):
    D = G.lib()
    G.say("small ligands, differentiable", preset, n_poses)
    p = G.load_pocket(synth.make_pocket(600, grid=40, seed=6), preset, keep=True)
    handles, lig, q, rng = _handles(n_poses)
    w = torch.tensor(G.weights32(preset)[None], device="cuda")
    c = torch.tensor(rng.normal(size=n_poses).astype(np.float32), device="cuda")
    got = []
    for H, _ in handles:
        xyz = D.dock_score_grad(p, H, lig, q, want_grad=False, want_xyz=True)[2]
        out = [D.dock_score_terms(p, H, lig, w, q=q), D.dock_score_terms(p, H, lig, w, xyz=xyz)]
        for kw in (dict(q=q, dLdq=torch.zeros_like(q)), dict(xyz=xyz, dLdx=torch.zeros_like(xyz))):
            dG, dw = torch.zeros((8, p.n_terms) + p.dims[::-1], device="cuda"), torch.zeros_like(w)
            D.dock_score_adjoint(p, H, lig, w, c, dLdG=[dG], dLdw=dw, deterministic=True, **kw)
            # (the fixed-point unit of dL/dG follows the largest |dL/dE| * atoms of the
            # poses, the same in both)
            out += [dG, dw, kw["dLdq"] if "dLdq" in kw else kw["dLdx"][:, :16]]
        got.append(out)
    for k, (a, b) in enumerate(zip(*got)):
        assert _same(a, b), k
