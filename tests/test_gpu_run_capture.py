"""dock_run_restart and dock_run_advance on a capturing stream: every replay
gives what the same calls give eagerly, with eager work of the same run and
synchronisations between the replays.  Run on an MI355X."""
import numpy as np
import pytest

import synth
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SPEC = [(10, 4), (17, 3), (33, 5), (65, 6)]
KEYS = ("q_cur", "E_cur", "q_best", "E_best", "n_evals")


def _setup():
    D = G.lib()
    L = synth.pack_ligands([synth.make_ligand(n, t, np.random.default_rng(300 + n)) for n, t in SPEC])
    L.pocket_index = np.zeros(L.n_ligands, np.int32)
    return D, G.load_pocket(synth.make_pocket(600, grid=40, seed=4)), G.load_ligands(L)


def _state(D, run):
    st = D.dock_run_state(run)
    torch.cuda.synchronize()
    return {k: st[k].clone() for k in KEYS}


def _same(a, b, what):
    for k in KEYS:
        assert torch.equal(a[k], b[k]), (what, k)


@pytest.mark.parametrize("use_graph", [0, 1])
@pytest.mark.parametrize("warm", [0, 1])
def test_a_captured_restart_and_advance(use_graph, warm):
    D, p, H = _setup()
    kw = dict(n_traj=21, n_steps=3, n_local=3)
    ref = D.dock_sample(p, H, seed=9, use_graph=0, **kw)
    D.dock_run_advance(ref, 2)
    ref = _state(D, ref)
    run = D.dock_sample(p, H, seed=5, use_graph=use_graph, **kw)
    for k in range(warm):
        D.dock_run_restart(run, 20 + k)
    G.say("captured restart and advance, graph", use_graph, "warm", warm)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        D.dock_run_restart(run, 9)
        D.dock_run_advance(run, 2)
    for rep in range(4):
        g.replay()
        torch.cuda.synchronize()
        _same(_state(D, run), ref, rep)
        D.dock_run_advance(run, 1)   # eager work of the same run between the replays
        torch.cuda.synchronize()
