"""With use_graph = 1 an MC-step phase is launched as it is the first time and
captured when one of as many steps comes again (abi.cpp, run_phase): the
states equal those of a run without graphs through every order of phases,
with other work of the stream between the replays.  Run on an MI355X."""
import numpy as np
import pytest

import synth
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SPEC = [(10, 4), (17, 3), (33, 5), (65, 6)]


@pytest.mark.parametrize("phases", [(3, 3, 3, 3), (2, 3, 3, 2, 3), (0, 1, 1, 4, 1)])
@pytest.mark.parametrize("chunk", [0, 1])
def test_phases_with_and_without_graph(phases, chunk):
    D = G.lib()
    G.say("phase graph:", phases, "chunk", chunk)
    pk = synth.make_pocket(600, grid=40, seed=4)
    L = synth.pack_ligands([synth.make_ligand(n, t, np.random.default_rng(300 + n)) for n, t in SPEC])
    L.pocket_index = np.zeros(L.n_ligands, np.int32)
    p, H = G.load_pocket(pk), G.load_ligands(L)
    runs = [D.dock_sample(p, H, n_traj=21, n_steps=phases[0], n_local=3, seed=5, steps_per_launch=chunk, use_graph=g)
            for g in (0, 1)]

    def check(what):
        a, b = (D.dock_run_state(r) for r in runs)
        torch.cuda.synchronize()
        assert a["step"] == b["step"]
        for k in ("q_cur", "E_cur", "q_best", "E_best", "n_evals"):
            assert torch.equal(a[k], b[k]), (what, k)

    check("created")
    for n in phases[1:]:
        for r in runs:
            D.dock_run_advance(r, n)
        check(n)
    for seed in (5, 6, 7):
        for r in runs:
            D.dock_run_restart(r, seed)
        check(("restart", seed))
