"""The adjoint's per-pocket sums (dL/dG through marked bricks of nodes) against
its float atomics: a call of 768 or more poses goes through the sums, the same
poses in calls of fewer go straight into the maps.  Poses inside, on the faces
of and outside the grid, grids that do not fill their last bricks, pockets
without dL/dG, a dL/dG that two pockets share, repeated accumulation, invalid
ligands and non-finite dL/dE.  Run on an MI355X.

Tolerance: both add the same products of FP32 corner weights; they differ in
the order of FP32 additions and in whether the weight w_k multiplies each
contribution or their sum, so an entry agrees to a few FP32 roundings of the
sum of the magnitudes added to it (at most 1,024 poses' here: 2^-23 * 1024 of
the largest entry bounds it, 1e-4 of it in practice is never reached)."""
import numpy as np
import pytest

import synth
from oracle import params as P
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SPEC = [(3, 0), (16, 5), (17, 3), (33, 5), (40, 9), (64, 12), (66, 6), (100, 8)]
TOL = 2.0 ** -23 * 1024


def _setup(preset, small_grid):
    D = G.lib()
    pks = [synth.make_pocket(300, grid=g, seed=20 + g) for g in ((9, 6) if small_grid else (33, 41))]
    ps = [G.load_pocket(pk, preset, keep=True) for pk in pks]
    L = synth.pack_ligands([synth.make_ligand(n, t, np.random.default_rng(900 + n)) for n, t in SPEC])
    L.pocket_index = (np.arange(L.n_ligands) % 2).astype(np.int32)
    return D, ps, G.load_ligands(L)


def _poses(H, n, seed):
    rng = np.random.default_rng(seed)
    lig = rng.integers(0, H.n, n).astype(np.int32)
    q = np.zeros((n, H.q_stride), np.float32)
    q[:, :3] = rng.uniform(-9, 9, (n, 3))   # many atoms outside the grid
    q[:, 3:] = rng.uniform(-np.pi, np.pi, (n, H.q_stride - 3))
    lig[rng.choice(n, 2, replace=False)] = [-1, H.n]
    dev = lambda a: torch.tensor(a, device="cuda")  # noqa: E731
    return dev(lig), dev(q), dev(rng.normal(size=n).astype(np.float32))


def _zeros(ps, w, q):
    return ([torch.zeros((8, p.n_terms) + p.dims[::-1], device="cuda") for p in ps], torch.zeros_like(w), torch.zeros_like(q))


def _close(a, b, tag):
    s = float(b.abs().max())
    assert float((a - b).abs().max()) <= TOL * s, (tag, float((a - b).abs().max()), s)


@pytest.mark.parametrize("preset", [P.PRESET_TRIDS, P.PRESET_VINA])
@pytest.mark.parametrize("n", [256, 768, 1021])
@pytest.mark.parametrize("small_grid", [False, True])
def test_sums_equal_atomics(preset, n, small_grid):
    D, ps, H = _setup(preset, small_grid)
    lig, q, c = _poses(H, n, n)
    G.say("adjoint sums", preset, n, small_grid)
    w = torch.tensor(np.stack([G.weights32(preset)] * 2), device="cuda") * torch.tensor([[1.0], [0.7]], device="cuda")
    dG, dw, dq = _zeros(ps, w, q)
    D.dock_score_adjoint(ps, H, lig, w, c, q=q, dLdG=dG, dLdw=dw, dLdq=dq)
    rG, rw, rq = _zeros(ps, w, q)
    tq = torch.zeros_like(q)
    for at in torch.arange(n, device="cuda").split(200):   # below the sums' threshold
        part = torch.zeros_like(q[at])
        D.dock_score_adjoint(ps, H, lig[at], w, c[at], q=q[at].contiguous(), dLdG=rG, dLdw=rw, dLdq=part)
        tq[at] = part
    for a, b in zip(dG, rG):
        assert float(b.abs().max()) > 0
        _close(a, b, "dG")
        assert torch.equal(a == 0, b == 0) or float((a[b == 0]).abs().max()) <= TOL * float(b.abs().max())
    _close(dw, rw, "dw")
    assert torch.equal(dq, tq)
    # the repeatable mode: the same again, bit for bit, and close to both
    eG, ew, eq = _zeros(ps, w, q)
    fG, fw, fq = _zeros(ps, w, q)
    for out in ((eG, ew, eq), (fG, fw, fq)):
        D.dock_score_adjoint(ps, H, lig, w, c, q=q, dLdG=out[0], dLdw=out[1], dLdq=out[2], deterministic=True)
    for a, b, r in zip(eG, fG, rG):
        assert torch.equal(a, b)
        _close(a, r, "fixed dG")
    assert torch.equal(ew, fw) and torch.equal(eq, dq)
    # accumulation, one pocket without dL/dG
    D.dock_score_adjoint(ps, H, lig, w, c, q=q, dLdG=[None, eG[1]], deterministic=True)
    _close(eG[1], 2 * fG[1], "accumulated")
    assert torch.equal(eG[0], fG[0])


@pytest.mark.parametrize("det", [False, True])
def test_a_buffer_two_pockets_share_and_coordinate_poses(det):
    D, ps, H = _setup(P.PRESET_TRIDS, False)
    ps = [ps[0], ps[0]]
    lig, q, c = _poses(H, 800, 5)
    w = torch.tensor(np.stack([G.weights32(P.PRESET_TRIDS)] * 2), device="cuda")
    _, _, xyz = D.dock_score_grad(ps, H, lig, q, want_grad=False, want_xyz=True)
    G.say("adjoint sums: shared buffer", det)
    two, dw, _ = _zeros(ps, w, q)
    D.dock_score_adjoint(ps, H, lig, w, c, xyz=xyz, dLdG=two, dLdw=dw, deterministic=det)
    one = torch.zeros_like(two[0])
    D.dock_score_adjoint(ps, H, lig, w, c, xyz=xyz, dLdG=[one, one], deterministic=det)
    _close(one, two[0] + two[1], "shared")


def test_a_bound_that_is_not_finite_makes_its_pocket_nan():
    D, ps, H = _setup(P.PRESET_TRIDS, False)
    lig, q, c = _poses(H, 800, 6)
    w = torch.tensor(np.stack([G.weights32(P.PRESET_TRIDS)] * 2), device="cuda")
    c[int((lig == 1).nonzero()[0])] = float("nan")   # a ligand of pocket 1
    G.say("adjoint sums: non-finite")
    dG, _, _ = _zeros(ps, w, q)
    D.dock_score_adjoint(ps, H, lig, w, c, q=q, dLdG=dG, deterministic=True)
    assert torch.isnan(dG[1]).all() and torch.isfinite(dG[0]).all()
    fG, _, _ = _zeros(ps, w, q)
    D.dock_score_adjoint(ps, H, lig, w, c, q=q, dLdG=fG)   # float sums: the nodes that pose reaches
    assert torch.isnan(fG[1]).any() and not torch.isnan(fG[1]).all() and torch.isfinite(fG[0]).all()
