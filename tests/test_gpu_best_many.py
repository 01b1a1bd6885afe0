"""Best poses and the screening rank at the sizes where their kernels change:
candidate counts around a power of two and up to thousands (sorted by one or
four waves, compared four at a time), clusters that fill, undershoot and
overflow top_n inside one turn of four candidates, energies that are NaN,
infinite, equal and signed zero; rank blocks around 2,048.  Against the oracle
(selection is compared for ligands without an RMSD within 1e-4 A of the
cutoff, as FP32 and FP64 coordinates may decide it differently).  Run on an
MI355X."""
import numpy as np
import pytest

import synth
from oracle import best as BEST, topology
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,top_n", [(1, 1), (3, 2), (4, 8), (5, 3), (63, 8), (65, 8), (257, 28), (1000, 8)])
def test_best_poses_around_their_turns(T, top_n):
    D = G.lib()
    L = synth.pack_ligands([synth.make_ligand(n, t, np.random.default_rng(n)) for n, t in [(2, 0), (17, 3), (40, 8), (70, 12)]])
    L.pocket_index = np.zeros(4, np.int32)
    H = G.load_ligands(L)
    rng = np.random.default_rng(T)
    E = np.round(rng.normal(size=(4, T)) * 4).astype(np.float32) / 4          # many ties
    E[0, rng.integers(0, T)] = np.nan
    E[1, rng.integers(0, T)] = np.inf
    E[2, :] = np.where(E[2] == 0, -0.0, E[2])
    q = np.zeros((4, T, H.q_stride), np.float32)
    centres = rng.integers(0, 5, (4, T))
    base = rng.normal(size=(4, 5, H.q_stride)) * 2
    for i in range(4):
        q[i] = base[i, centres[i]] + rng.normal(size=(T, H.q_stride)) * np.where(rng.random((T, 1)) < 0.5, 0.02, 0.6)
    G.say("best poses", T, top_n)
    got = D.dock_best_poses(H, T, torch.tensor(E, device="cuda"), torch.tensor(q, device="cuda"), top_n=top_n)
    got = {k: v.cpu().numpy() for k, v in got.items()}
    compared = 0
    for i in range(4):
        t = topology.from_ligands(L, i)
        ref = BEST.best_poses(t, np.where(np.isnan(E[i]), np.inf, E[i]).astype(np.float64),
                              q[i, :, :t.n_dof].astype(np.float64), top_n=top_n, rmsd_cut=1.0, margins=True)
        if not ref["rmsd_margin"] > 1e-4:
            continue
        compared += 1
        n, kept = int(got["n"][i]), list(ref["idx"])
        assert n == len(kept) and got["idx"][i, :n].tolist() == kept
        assert np.array_equal(got["E"][i, :n].view(np.uint32), E[i, kept].view(np.uint32))
        assert np.all(got["idx"][i, n:] == -1) and np.all(np.isposinf(got["E"][i, n:]))
        np.testing.assert_allclose(got["xyz"][i, :n, :t.n_atoms], ref["xyz"], atol=2e-5)
    assert compared >= 2


@pytest.mark.parametrize("n,k", [(1, 1), (2047, 1024), (2048, 3), (2049, 1024), (4097, 100), (300001, 1024)])
def test_rank_around_its_blocks(n, k):
    D = G.lib()
    rng = np.random.default_rng(n)
    s = np.round(rng.normal(size=n) * 50).astype(np.float32) / 8
    s[rng.integers(0, n, n // 7)] = 0.0
    s[rng.integers(0, n, n // 9)] = -0.0
    s[rng.integers(0, n, n // 20)] = np.nan
    s[rng.integers(0, n, n // 30)] = -np.inf
    G.say("rank", n, k)
    val, idx = D.dock_screen_rank(torch.tensor(s, device="cuda"), k)
    ref = BEST.screen_rank(s, k)
    assert np.array_equal(idx.cpu().numpy(), np.asarray(ref[1], np.int32))
    m = min(n, k)
    got = val.cpu().numpy()
    assert np.array_equal(got[:m].view(np.uint32), s[idx.cpu().numpy()[:m]].view(np.uint32))
    assert np.all(np.isposinf(got[m:]))
