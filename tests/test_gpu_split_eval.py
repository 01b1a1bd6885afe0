"""A run that logs its trajectories evaluates the energy and the gradient of
every pose; a run that does not computes in each evaluation only the one its
rule uses (kernels.hip, run_traj).  Both reach the same state bit for bit:
every local rule, preset and receptor mode, ligands at the edges of the lane
configurations, one and two atoms per lane.  Run on an MI355X."""
import numpy as np
import pytest

import synth
from oracle import params as P
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SPEC = [(2, 0), (10, 4), (16, 8), (17, 3), (32, 9), (33, 5), (64, 12), (65, 6), (70, 15), (100, 8)]
STATE = ("q_cur", "E_cur", "q_best", "E_best", "n_evals")


@pytest.fixture(scope="module")
def inputs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pk = synth.make_pocket(600, grid=40, seed=4)
    L = synth.pack_ligands([synth.make_ligand(n, t, np.random.default_rng(300 + n)) for n, t in SPEC])
    L.pocket_index = np.zeros(L.n_ligands, np.int32)
    return G.lib(), pk, L


def _both(D, p, H, **kw):
    plain = D.dock_run_state(D.dock_sample(p, H, use_graph=0, **kw))
    logged = D.dock_run_state(D.dock_sample(p, H, use_graph=0, record_trace=1, trace_lig_stride=3, trace_traj=1, **kw))
    for k in STATE:
        assert torch.equal(plain[k], logged[k]), k


@pytest.mark.parametrize("rule", ["ADAM", "SGD", "RMSPROP", "ADAGRAD", "ADAMW", "LINESEARCH"])
def test_logged_and_unlogged_runs_agree(inputs, rule):
    D, pk, L = inputs
    G.say("split evaluations:", rule)
    lr = 1e-3 if rule == "SGD" else 0.1
    _both(D, G.load_pocket(pk), G.load_ligands(L), n_traj=9, n_steps=4, n_local=5, lr=lr, seed=7,
          local_opt=getattr(D, "LOCAL_" + rule))


@pytest.mark.parametrize("mode", ["vina", "direct", "mdn", "no local steps"])
def test_logged_and_unlogged_runs_agree_in_every_mode(inputs, mode):
    D, pk, L = inputs
    G.say("split evaluations:", mode)
    H = G.load_ligands(L)
    residue = None
    if mode == "mdn":
        residue = synth.make_residues(pk)
        D.dock_ligands_set_mdn(H, synth.make_mdn_params(int(L.atom_off[-1]), int(residue.max()) + 1, 4, seed=2))
    p = G.load_pocket(pk, P.PRESET_VINA if mode == "vina" else P.PRESET_TRIDS, direct=mode == "direct", residue=residue)
    _both(D, p, H, n_traj=9, n_steps=3, n_local=0 if mode.startswith("no") else 4, seed=8)


def test_logged_and_unlogged_runs_agree_two_atoms_per_lane(inputs):
    D, pk, L = inputs
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    mid = sum(32 < n <= 64 for n, _ in SPEC)
    T = -(-4 * 12 * n_cu // mid) + 1   # two poses per wavefront fill two waves per wave slot
    p, H = G.load_pocket(pk), G.load_ligands(L)
    G.say("split evaluations: two atoms per lane, T =", T)
    kw = dict(n_traj=T, n_steps=1, n_local=3, seed=9)
    plan = D.dock_run_plan(D.dock_sample(p, H, **kw))
    assert (32, 2) in set(zip(plan["lanes"], plan["apl"]))
    _both(D, p, H, **kw)
