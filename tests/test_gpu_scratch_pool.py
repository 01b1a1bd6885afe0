"""The adjoints' scratch comes from a pool that outlives a call (abi.cpp,
scratch_alloc): calls of different sizes enqueued on two streams without a
synchronisation between them, before and after a handle was freed (which
returns the pool's memory), give the bits each gives alone.  Run on an
MI355X."""
import numpy as np
import pytest

import synth
from oracle import params as P
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_two_streams_share_the_pool():
    D = G.lib()
    G.say("scratch pool: two streams")
    pk = synth.make_pocket(300, grid=33, seed=9)
    L = synth.pack_ligands([synth.make_ligand(n, t, np.random.default_rng(40 + n)) for n, t in ((12, 2), (30, 6), (50, 9))])
    L.pocket_index = np.zeros(L.n_ligands, np.int32)
    p, H = G.load_pocket(pk, P.PRESET_TRIDS, keep=True), G.load_ligands(L)
    w = torch.tensor(G.weights32(P.PRESET_TRIDS)[None], device="cuda")
    rng = np.random.default_rng(1)
    calls = []
    for n in (7, 300, 1500):
        q = np.zeros((n, H.q_stride), np.float32)
        q[:, :3] = rng.uniform(-5, 5, (n, 3))
        q[:, 3:] = rng.uniform(-np.pi, np.pi, (n, H.q_stride - 3))
        calls.append((torch.tensor(rng.integers(0, 3, n).astype(np.int32), device="cuda"), torch.tensor(q, device="cuda"),
                      torch.tensor(rng.normal(size=n).astype(np.float32), device="cuda")))
    new = lambda: (torch.zeros((8, p.n_terms) + p.dims[::-1], device="cuda"), torch.zeros_like(w))  # noqa: E731

    def call(k, out, stream=None):
        lig, q, c = calls[k]
        D.dock_score_adjoint(p, H, lig, w, c, q=q, dLdG=[out[0]], dLdw=out[1], deterministic=True, stream=stream)

    ref = [new() for _ in calls]
    for k, out in enumerate(ref):
        call(k, out)
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(2):
        jobs = [(k, streams[i % 2], new()) for i, k in enumerate((2, 0, 1, 2, 2, 1, 0, 2, 1, 1))]
        torch.cuda.synchronize()
        for k, s, out in jobs:
            call(k, out, s)
        torch.cuda.synchronize()
        for k, _, out in jobs:
            assert torch.equal(out[0], ref[k][0]) and torch.equal(out[1], ref[k][1]), (rep, k)
        G.load_ligands(L).free()   # the pool gives its memory back
