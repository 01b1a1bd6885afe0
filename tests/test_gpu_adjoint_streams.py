"""Adjoints with float atomics (deterministic = 0) that overlap on two streams
and add to one dL/dG and dL/dw lose nothing, below and from the number of
poses where the sums of a call are collected first (adj_expand_kernel and
adj_wreduce_kernel then do the adding).  Run on an MI355X.

Tolerance: every call adds FP32 sums of at most n poses' contributions to an
entry, in any order, then one addend per call: (n + calls) roundings of
2^-24 of the sum of the magnitudes, which a call with |dL/dE| and |w| gives (in
absolute value: a node of a face gets the corner weight 1 - f of the atoms
clamped to the opposite side, which rounds to -2^-24 or so).  The reference is
the deterministic mode, whose contributions (at most 64 atoms' of n poses to an
entry) are each rounded to a multiple of 2^(e - 62), 2^e at most twice
n max |dL/dE| 64 max |w|."""
import numpy as np
import pytest

import synth
from oracle import params as P
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CALLS = 16


@pytest.mark.parametrize("preset", [P.PRESET_TRIDS, P.PRESET_VINA])
@pytest.mark.parametrize("n", [300, 1500, 4000])
def test_calls_on_two_streams_add_to_one_gradient(preset, n):
    D = G.lib()
    G.say("adjoint streams", preset, n)
    p = G.load_pocket(synth.make_pocket(300, grid=33, seed=9), preset, keep=True)
    L = synth.pack_ligands([synth.make_ligand(k, t, np.random.default_rng(40 + k)) for k, t in ((12, 2), (30, 6), (50, 9))])
    L.pocket_index = np.zeros(L.n_ligands, np.int32)
    H = G.load_ligands(L)
    rng = np.random.default_rng(n)
    q = np.zeros((n, H.q_stride), np.float32)
    q[:, :3] = rng.uniform(-2, 2, (n, 3))   # close together: many poses per node
    q[:, 3:] = rng.uniform(-np.pi, np.pi, (n, H.q_stride - 3))
    lig = torch.tensor(rng.integers(0, 3, n).astype(np.int32), device="cuda")
    q = torch.tensor(q, device="cuda")
    c = torch.tensor(rng.normal(size=n).astype(np.float32), device="cuda")
    w = torch.tensor(G.weights32(preset)[None], device="cuda")
    new = lambda: (torch.zeros((8, p.n_terms) + p.dims[::-1], device="cuda"), torch.zeros_like(w))  # noqa: E731

    def call(out, w, c, stream=None, det=False):
        D.dock_score_adjoint(p, H, lig, w, c, q=q, dLdG=[out[0]], dLdw=out[1], deterministic=det, stream=stream)

    one, mag, both = new(), new(), new()
    call(one, w, c, det=True)
    call(mag, w.abs(), c.abs(), det=True)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k in range(CALLS):
        call(both, w, c, streams[k % 2])
    torch.cuda.synchronize()
    unit = 2 * n * 64 * float(c.abs().max()) * float(w.abs().max()) * 2.0 ** -62
    bound = CALLS * ((n + CALLS) * 2.0 ** -24 * mag[0].double().abs() + 64 * n * unit / 2)
    diff = (both[0].double() - CALLS * one[0].double()).abs()
    assert bool((diff <= bound).all()), float((diff - bound).max())
    # dL/dw: the magnitude of a pose's contribution is not known from mag (the
    # terms' sums cancel): a lost call is 1 / CALLS of the entry
    assert torch.allclose(both[1], CALLS * one[1], rtol=1e-3, atol=1e-3 * float(one[1].abs().max()))
