"""dL/dG entry by entry.  A call of many poses collects its contributions in
bricks of nodes that the poses' atoms mark first; a brick that was not marked
or not cleared would show in small entries too.  So each entry is held to the
roundings of its own contributions, in both modes and in a captured call
(which adds without the bricks), with a pocket's frame at the origin and far
from it; and where no pose reaches, nothing is added.  Run on an MI355X.

Tolerance: an entry is an FP32 sum, in any order, of at most 64 n products of
FP32 factors (64: atoms of a ligand), so it differs from the exact sum of the
same contributions by at most (n + 8) 2^-24 times the sum of their magnitudes
where at most n of them meet (poses this far apart); the deterministic mode
rounds each to a multiple of 2^(e - 62), 2^e at most twice
n max |dL/dE| 64 max |w|.  The magnitudes come from the same poses with
|dL/dE| and |w| in small calls, the reference from calls of 100 poses summed
in 64 bits."""
import numpy as np
import pytest

import synth
from oracle import params as P
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SPEC = ((12, 2), (30, 6), (50, 9), (64, 12))


@pytest.mark.parametrize("preset", [P.PRESET_TRIDS, P.PRESET_VINA])
@pytest.mark.parametrize("offset", [0.0, 4000.0])
@pytest.mark.parametrize("n", [300, 800, 3000])
def test_every_entry(preset, offset, n):
    D = G.lib()
    G.say("adjoint entries", preset, offset, n)
    pk = synth.make_pocket(300, grid=33, seed=9)
    o = np.array([offset, -offset / 2, offset / 4], np.float32)
    p = D.dock_load_pocket(pk.xyz + o, pk.type, np.asarray(pk.origin, np.float32) + o, pk.spacing, pk.dims, preset=preset,
                           keep_per_term=True)
    L = synth.pack_ligands([synth.make_ligand(k, t, np.random.default_rng(40 + k)) for k, t in SPEC])
    L.pocket_index = np.zeros(L.n_ligands, np.int32)
    H = G.load_ligands(L)
    rng = np.random.default_rng(n)
    q = np.zeros((n, H.q_stride), np.float32)
    q[:, :3] = rng.uniform(-3, 3, (n, 3)) + o
    q[:, 3:] = rng.uniform(-np.pi, np.pi, (n, H.q_stride - 3))
    lig = torch.tensor(rng.integers(0, len(SPEC), n).astype(np.int32), device="cuda")
    q = torch.tensor(q, device="cuda")
    c = torch.tensor(rng.normal(size=n).astype(np.float32), device="cuda")
    w = torch.tensor(G.weights32(preset)[None], device="cuda")
    shape = (8, p.n_terms) + p.dims[::-1]

    def call(c, w, det=False, at=slice(None)):
        out = torch.zeros(shape, device="cuda")
        D.dock_score_adjoint(p, H, lig[at].contiguous(), w, c[at].contiguous(), q=q[at].contiguous(), dLdG=[out],
                             deterministic=det)
        return out

    parts = [slice(k, k + 100) for k in range(0, n, 100)]
    ref = sum(call(c, w, at=s).double() for s in parts)
    mag = sum(call(c.abs(), w.abs(), at=s).double().abs() for s in parts)
    unit = 2 * n * 64 * float(c.abs().max()) * float(w.abs().max()) * 2.0 ** -62
    held = torch.zeros(shape, device="cuda")   # captured: outputs allocated beforehand
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        D.dock_score_adjoint(p, H, lig, w, c, q=q, dLdG=[held])
    g.replay()
    for what, got, extra in (("float", call(c, w), 0.0), ("fixed", call(c, w, det=True), 64 * n * unit / 2),
                             ("captured", held, 0.0)):
        over = (got.double() - ref).abs() - ((n + 8) * 2.0 ** -24 * mag + extra)
        assert float(over.max()) <= 0, (what, float(over.max()))
        assert bool((got[mag == 0] == 0).all()), what
    held.zero_()
    g.replay()
    assert float(((held.double() - ref).abs() - (n + 8) * 2.0 ** -24 * mag).max()) <= 0


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_a_weight_that_is_not_finite_meets_every_contribution(bad):
    """deterministic = 0: the entries that a non-finite weight reaches are the
    same in one call as in small ones, poses with dL/dE = 0 included."""
    D = G.lib()
    G.say("adjoint entries: weight", bad)
    pk = synth.make_pocket(300, grid=33, seed=9)
    p = G.load_pocket(pk, P.PRESET_TRIDS, keep=True)
    L = synth.pack_ligands([synth.make_ligand(30, 6, np.random.default_rng(70))])
    L.pocket_index = np.zeros(1, np.int32)
    H = G.load_ligands(L)
    rng = np.random.default_rng(5)
    n = 1500
    q = np.zeros((n, H.q_stride), np.float32)
    q[:, :3] = rng.uniform(-3, 3, (n, 3))
    q[:, 3:] = rng.uniform(-np.pi, np.pi, (n, H.q_stride - 3))
    lig, q = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.tensor(q, device="cuda")
    c = torch.tensor(np.where(rng.random(n) < 0.9, 0.0, 1.0).astype(np.float32), device="cuda")
    w = torch.tensor(G.weights32(P.PRESET_TRIDS)[None], device="cuda")
    w[0, 1] = bad
    one, parts = (torch.zeros((8, p.n_terms) + p.dims[::-1], device="cuda") for _ in range(2))
    D.dock_score_adjoint(p, H, lig, w, c, q=q, dLdG=[one])
    for k in range(0, n, 100):
        D.dock_score_adjoint(p, H, lig[k:k + 100], w, c[k:k + 100], q=q[k:k + 100], dLdG=[parts])
    assert torch.equal(torch.isnan(one), torch.isnan(parts)) and torch.equal(torch.isinf(one), torch.isinf(parts))
    assert bool(torch.isnan(one).any())
