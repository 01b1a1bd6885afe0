"""A run of no more trajectories than the device has SIMDs takes workgroups of
one wavefront, a larger one of four (abi.cpp, create_run).  A trajectory's
draws depend on its number alone, so the same trajectories on both sides of
the line have the same bits.  Run on an MI355X."""
import numpy as np
import pytest

import synth
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SPEC = [(1, 0), (16, 8), (17, 3), (33, 5), (65, 6)]


@pytest.mark.parametrize("form", ["BATCHED", "PLAIN"])
def test_same_trajectories_on_both_sides_of_the_line(form):
    D = G.lib()
    pk = synth.make_pocket(600, grid=40, seed=4)
    L = synth.pack_ligands([synth.make_ligand(n, t, np.random.default_rng(300 + n)) for n, t in SPEC])
    L.pocket_index = np.zeros(L.n_ligands, np.int32)
    p, H = G.load_pocket(pk), G.load_ligands(L)
    line = 4 * torch.cuda.get_device_properties(0).multi_processor_count // L.n_ligands
    G.say("small runs:", form, "line at", line)
    run = lambda T: D.dock_run_state(D.dock_sample(p, H, n_traj=T, n_steps=3, n_local=4, seed=5,
                                                   form=getattr(D, "FORM_" + form)))
    over = run(line + 1)
    for T in (1, 63, line):
        small = run(T)
        for k in ("q_cur", "E_cur", "q_best", "E_best"):
            assert torch.equal(small[k], over[k][:, :T]), (k, T)
