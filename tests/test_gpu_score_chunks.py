"""dock_score_grad and the differentiable form give a pose the same values
however its call groups poses into wavefronts: calls large enough to take two
or four poses per wavefront against the same poses a few at a time, ligands of
every lane configuration next to each other, invalid ligand indices among
them.  (Few poses at a time are what the parity tests compare with the
oracle.)  Run on an MI355X."""
import numpy as np
import pytest

import synth
from oracle import params as P
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SPEC = [(2, 0), (10, 4), (16, 8), (17, 3), (9, 2), (32, 9), (33, 5), (64, 12), (12, 1), (65, 6), (70, 15), (100, 8)]


def _inputs(n_poses, small_only=False):
    spec = [s for s in SPEC if s[0] <= 16] if small_only else SPEC
    L = synth.pack_ligands([synth.make_ligand(n, t, np.random.default_rng(500 + n)) for n, t in spec])
    L.pocket_index = np.zeros(L.n_ligands, np.int32)
    H = G.load_ligands(L)
    rng = np.random.default_rng(n_poses)
    # runs of one ligand, of neighbours and single poses
    lig = rng.integers(0, L.n_ligands, n_poses).astype(np.int32)
    lig[: n_poses // 3] = np.sort(lig[: n_poses // 3])
    q = np.zeros((n_poses, H.q_stride), np.float32)
    q[:, :3] = rng.uniform(-3, 3, (n_poses, 3))
    q[:, 3:] = rng.uniform(-np.pi, np.pi, (n_poses, H.q_stride - 3))
    bad = rng.choice(n_poses, 5, replace=False)
    lig[bad[:3]], lig[bad[3:]] = -1, L.n_ligands
    return H, torch.tensor(lig, device="cuda"), torch.tensor(q, device="cuda"), bad


@pytest.mark.parametrize("n_poses", [4096, 4097, 8191, 8193, 8195])
@pytest.mark.parametrize("small_only", [False, True])
def test_score_does_not_depend_on_the_grouping(n_poses, small_only):
    D = G.lib()
    pk = synth.make_pocket(600, grid=40, seed=6)
    p = G.load_pocket(pk)
    H, lig, q, bad = _inputs(n_poses, small_only)
    G.say("score chunks", n_poses, small_only)
    E, g, xyz = D.dock_score_grad(p, H, lig, q, want_xyz=True)
    at = np.unique(np.concatenate([bad, [0, 1, 2, 3, n_poses - 1], np.random.default_rng(1).choice(n_poses, 500)]))
    idx = torch.tensor(at, device="cuda")
    e1, g1, x1 = D.dock_score_grad(p, H, lig[idx].contiguous(), q[idx].contiguous(), want_xyz=True)
    assert torch.isnan(E[torch.tensor(bad, device="cuda")]).all()
    ok = ~torch.isnan(e1)
    assert ok.sum() == len(at) - len(bad)
    assert torch.equal(E[idx][ok], e1[ok]) and torch.equal(g[idx], g1) and torch.equal(xyz[idx], x1)
