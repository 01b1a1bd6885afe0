"""The adjoints' scratch between calls (abi.cpp, scratch_take): calls of
different sizes that take turns, on the null stream and on others, find their
blocks again instead of mapping memory anew after every synchronisation; at
most 128 MiB are kept; the last handle's end returns them; and the results are
those of each call alone.  Run on an MI355X."""
import gc

import numpy as np
import pytest

import synth
from oracle import params as P
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MIB = 2 ** 20


def _free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _inputs(D, grid, n):
    p = G.load_pocket(synth.make_pocket(300, grid=grid, seed=9), P.PRESET_VINA, keep=True)
    L = synth.pack_ligands([synth.make_ligand(k, t, np.random.default_rng(40 + k)) for k, t in ((12, 2), (30, 6), (50, 9))])
    L.pocket_index = np.zeros(L.n_ligands, np.int32)
    H = G.load_ligands(L)
    rng = np.random.default_rng(n)
    q = np.zeros((n, H.q_stride), np.float32)
    q[:, :3] = rng.uniform(-5, 5, (n, 3))
    q[:, 3:] = rng.uniform(-np.pi, np.pi, (n, H.q_stride - 3))
    return (p, H, torch.tensor(rng.integers(0, 3, n).astype(np.int32), device="cuda"), torch.tensor(q, device="cuda"),
            torch.tensor(rng.normal(size=n).astype(np.float32), device="cuda"),
            torch.tensor(G.weights32(P.PRESET_VINA)[None], device="cuda"))


def test_turns_keep_their_blocks_and_the_last_handle_returns_them():
    D = G.lib()
    G.say("scratch kept: turns")
    gc.collect()
    p, H, lig, q, c, w = _inputs(D, 64, 2000)   # deterministic 80 MiB, float 8 MiB of sums
    dG = torch.zeros((8, p.n_terms) + p.dims[::-1], device="cuda")
    dw = torch.zeros_like(w)

    def call(det, stream=None):
        D.dock_score_adjoint(p, H, lig, w, c, q=q, dLdG=[dG], dLdw=dw, deterministic=det, stream=stream)

    before = _free_bytes()
    for det in (True, False):
        call(det)
        _free_bytes()
    kept = before - _free_bytes()
    assert 80 * MIB <= kept <= 132 * MIB, kept / MIB
    for det in (True, False, True, False, False, True):
        call(det)
        assert before - _free_bytes() == kept, det
    side = torch.cuda.Stream()
    for k in range(6):
        call(k % 2 == 0, side)
        assert before - _free_bytes() <= 132 * MIB
    p2, H2 = _inputs(D, 9, 1)[:2]
    del p, H, p2, H2
    gc.collect()
    assert before - _free_bytes() <= 2 * MIB


def test_results_do_not_depend_on_whose_block_it_was():
    D = G.lib()
    G.say("scratch kept: streams")
    sets = [_inputs(D, g, n) for g, n in ((33, 900), (40, 2500), (48, 1500), (64, 800))]

    def call(k, stream=None):
        p, H, lig, q, c, w = sets[k]
        out = torch.zeros((8, p.n_terms) + p.dims[::-1], device="cuda"), torch.zeros_like(w)
        torch.cuda.synchronize()
        D.dock_score_adjoint(p, H, lig, w, c, q=q, dLdG=[out[0]], dLdw=out[1], deterministic=True, stream=stream)
        return out

    ref = []
    for k in range(4):
        ref.append(call(k))
        torch.cuda.synchronize()
    streams = [None, torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(3):
        # outputs first, so that the calls themselves are enqueued back to back
        jobs = [(k, streams[(k + j + rep) % 3]) for j in range(4) for k in range(4)]
        outs = [(torch.zeros_like(ref[k][0]), torch.zeros_like(ref[k][1])) for k, _ in jobs]
        torch.cuda.synchronize()
        for (k, s), out in zip(jobs, outs):
            p, H, lig, q, c, w = sets[k]
            D.dock_score_adjoint(p, H, lig, w, c, q=q, dLdG=[out[0]], dLdw=out[1], deterministic=True, stream=s)
        torch.cuda.synchronize()
        for (k, _), out in zip(jobs, outs):
            assert torch.equal(out[0], ref[k][0]) and torch.equal(out[1], ref[k][1]), (rep, k)
        streams[1 + rep % 2] = torch.cuda.Stream()   # a stream of another name, or of an old one's
