"""dock_best_poses with the energies' own buffer as E_out or E_screen (as many
slots as candidates, so a ligand's outputs take the place of its energies):
the same bits as with separate outputs, -0.0, ties, infinities and NaN among
the energies.  Run on an MI355X."""
import numpy as np
import pytest

import synth
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_lig, T", [(1, 24), (3, 7), (300, 16), (2100, 4)])
@pytest.mark.parametrize("which", ["E_out", "E_screen"])
def test_outputs_over_the_energies(n_lig, T, which):
    D = G.lib()
    G.say("best in place", n_lig, T, which)
    base = synth.pack_ligands([synth.make_ligand(n, t, np.random.default_rng(n)) for n, t in ((9, 1), (30, 6), (70, 8))])
    L = base.subset(np.arange(n_lig) % 3)
    L.pocket_index = np.zeros(n_lig, np.int32)
    H = G.load_ligands(L)
    rng = np.random.default_rng(T)
    E = rng.normal(size=(n_lig, T)).astype(np.float32)
    special = rng.choice(np.array([-0.0, 0.0, 0.25, np.inf, -np.inf, np.nan], np.float32), size=E.shape)
    E = np.where(rng.random(E.shape) < 0.3, special, E).astype(np.float32)
    E = torch.tensor(E, device="cuda")
    q = torch.tensor(rng.normal(size=(n_lig, T, H.q_stride)).astype(np.float32) * 2, device="cuda")
    ref = D.dock_best_poses(H, T, E, q, top_n=T, want_xyz=False)
    b = D.binding
    own, other = E.clone(), torch.empty_like(E)
    out = (own, other) if which == "E_out" else (other, own)
    idx = torch.empty((n_lig, T), dtype=torch.int32, device="cuda")
    b._check(D.lib.dock_best_poses(H.handle, T, b._dptr(own), b._dptr(q), H.q_stride, T, 1.0, 0.01, b._dptr(out[0]),
                                   b._dptr(out[1]), None, b._dptr(idx), None, 0, None, b._stream(None)))
    bits = lambda t: t.view(torch.int32)  # noqa: E731
    assert torch.equal(idx, ref["idx"])
    assert torch.equal(bits(out[0]), bits(ref["E"])) and torch.equal(bits(out[1]), bits(ref["E_screen"]))
    # separate outputs keep the energies' own bits
    kept = ref["idx"] >= 0
    took = torch.gather(E, 1, ref["idx"].clamp_min(0).long())
    assert torch.equal(bits(ref["E"])[kept], bits(took)[kept])
