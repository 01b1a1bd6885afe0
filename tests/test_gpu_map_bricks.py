"""The map build and its adjoint at the edges of their bricks of nodes: grids
that do not fill the last brick, receptors of one atom, around a multiple of
the 256 atoms tested at a time, and with more atoms near one brick than its
list holds; lambda that is zero but for a few nodes.  Run on an MI355X.

Tolerances: the maps are FP64 sums rounded once to FP32 (one FP32 ulp of the
oracle's FP64 value, plus 1e-12 of the absolute sum for the order of the FP64
additions); dL/dr is an FP64 sum rounded once and added in FP32 (1e-6),
dL/dtheta FP64 (1e-9)."""
import numpy as np
import pytest

import synth
from oracle import maps as MAPS, params as P
from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pocket(n, dims, radius, seed):
    rng = np.random.default_rng(seed)
    x = rng.normal(size=(n, 3))
    x *= (radius * rng.random((n, 1)) ** (1 / 3)) / np.linalg.norm(x, axis=1, keepdims=True)
    origin = np.array([-(d - 1) * 0.375 / 2 for d in dims], np.float32)
    return synth.Pocket(xyz=x.astype(np.float32), type=rng.integers(0, 8, n).astype(np.uint8), origin=origin,
                        spacing=0.375, dims=dims, radius=radius)


CASES = [((2, 2, 2), 1, 4.0), ((9, 8, 5), 255, 14.0), ((8, 9, 4), 257, 14.0), ((17, 5, 3), 1500, 9.0), ((40, 33, 7), 512, 16.0)]


@pytest.mark.parametrize("preset", [P.PRESET_TRIDS, P.PRESET_VINA])
@pytest.mark.parametrize("dims,n,radius", CASES)
def test_maps_at_brick_edges(dims, n, radius, preset):
    D = G.lib()
    G.say("map bricks", dims, n, preset)
    pk = _pocket(n, dims, radius, seed=n)
    w, K = G.weights32(preset), P.n_terms(preset)
    p = G.load_pocket(pk, preset, w, keep=True)
    ref = MAPS.build_maps(pk, preset).reshape(8, K, -1)
    got = D.dock_pocket_maps(p, per_term=True).cpu().numpy().reshape(8, K, -1)
    tol = np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64) + 1e-12 * np.maximum(np.abs(ref), 1.0)
    assert np.all(np.abs(got - ref) <= tol)
    M = np.einsum("k,tkn->tn", w.astype(np.float64), ref)
    S = np.einsum("k,tkn->tn", np.abs(w.astype(np.float64)), np.abs(ref))
    got = D.dock_pocket_maps(p).cpu().numpy().reshape(8, -1)
    assert np.all(np.abs(got - M) <= np.spacing(np.abs(M).astype(np.float32)) + 1e-12 * np.maximum(S, 1.0))


@pytest.mark.parametrize("dims,n,radius", CASES[1:])
@pytest.mark.parametrize("some", [0, 1, 5, None])
def test_map_adjoint_of_sparse_lambda(dims, n, radius, some):
    from oracle import map_adjoint as MA
    D = G.lib()
    G.say("map adjoint bricks", dims, n, some)
    pk = _pocket(n, dims, radius, seed=n + 1)
    p = G.load_pocket(pk)
    rng = np.random.default_rng(n)
    lam = rng.normal(size=(8, 3, int(np.prod(dims)))).astype(np.float32)
    if some is not None:   # the first and last node among the few
        keep = np.zeros(lam.shape[2], bool)
        keep[rng.choice(lam.shape[2], some, replace=False)] = True
        if some > 1:
            keep[[0, -1]] = True
        lam[:, :, ~keep] = 0.0
    dx = torch.zeros((n, 3), device="cuda")
    dth = torch.zeros(13, dtype=torch.float64, device="cuda")
    D.dock_pocket_map_adjoint(p, torch.tensor(lam.reshape((8, 3) + dims[::-1]), device="cuda"), dx, dth)
    ref_x, ref_t = MA.map_adjoint(pk, lam.astype(np.float64))
    assert np.abs(dx.cpu().numpy() - ref_x).max() <= 1e-6 * max(1.0, np.abs(ref_x).max())
    assert np.all(np.abs(dth.cpu().numpy() - ref_t) <= 1e-9 * np.maximum(1.0, np.abs(ref_t).max()))


def test_map_adjoint_under_capture():
    """A captured call goes without the node masks (their scratch cannot be
    allocated there): the same sums in another order."""
    D = G.lib()
    G.say("map adjoint bricks, captured")
    dims, n = (17, 9, 6), 300
    pk = _pocket(n, dims, 12.0, seed=3)
    p = G.load_pocket(pk)
    lam = np.random.default_rng(4).normal(size=(8, 3) + dims[::-1]).astype(np.float32)
    lam[..., ::3] = 0.0
    lam = torch.tensor(lam, device="cuda")
    new = lambda: (torch.zeros((n, 3), device="cuda"), torch.zeros(13, dtype=torch.float64, device="cuda"))
    ref_x, ref_t = new()
    D.dock_pocket_map_adjoint(p, lam, ref_x, ref_t)
    dx, dth = new()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        D.dock_pocket_map_adjoint(p, lam, dx, dth)
    for _ in range(3):
        dx.zero_()
        dth.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert (dx - ref_x).abs().max() <= 1e-6 * max(1.0, float(ref_x.abs().max()))
        assert (dth - ref_t).abs().max() <= 1e-9 * max(1.0, float(ref_t.abs().max()))
