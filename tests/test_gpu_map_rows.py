"""Maps of grids with enough rows of bricks to be dealt to the XCDs row by row
(launch_map_build), rows that do and do not come out even over the eight, bricks
that are not full: every node against the oracle, with the tolerance of FP64 sums
rounded once to FP32 (one ulp, plus 1e-12 for the order of the additions).  Run
on an MI355X."""
import numpy as np
import pytest

import synth
from oracle import maps as MAPS, params as P
from tests import _gpu as G

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("preset", [P.PRESET_TRIDS, P.PRESET_VINA])
@pytest.mark.parametrize("dims", [(9, 97, 121), (2, 128, 95), (17, 128, 96)])   # 403, 384 and 384 rows
def test_every_node(dims, preset):
    D = G.lib()
    G.say("map rows", dims, preset)
    n = 40
    rng = np.random.default_rng(n + dims[0])
    x = rng.uniform(-0.5, 0.5, (n, 3)) * (np.array(dims) - 1) * 0.375 * 1.1
    pk = synth.Pocket(xyz=x.astype(np.float32), type=rng.integers(0, 8, n).astype(np.uint8),
                      origin=np.array([-(d - 1) * 0.375 / 2 for d in dims], np.float32), spacing=0.375, dims=dims, radius=20.0)
    K = P.n_terms(preset)
    p = G.load_pocket(pk, preset, G.weights32(preset), keep=True)
    ref = MAPS.build_maps(pk, preset).reshape(8, K, -1)
    got = D.dock_pocket_maps(p, per_term=True).cpu().numpy().reshape(8, K, -1)
    tol = np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64) + 1e-12 * np.maximum(np.abs(ref), 1.0)
    assert np.all(np.abs(got - ref) <= tol)
