"""The clash term is flat below 0.1 Angstrom: there its lambda, however large,
gives no force on the receptor atom (map_adjoint_kernel).  Run on an MI355X."""
import numpy as np
import pytest

from tests import _gpu as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [1.0, 3e38, float("inf")])
def test_no_force_from_the_flat_part(value):
    D = G.lib()
    G.say("map adjoint: flat part", value)
    n, h = 17, 0.375
    node = (8, 7, 9)
    xyz = (np.array([node], np.float32) * h + np.float32(0.03)).astype(np.float32)
    p = D.dock_load_pocket(xyz, np.array([1], np.uint8), np.zeros(3, np.float32), h, (n, n, n), keep_per_term=True)
    lam = torch.zeros((8, 3, n, n, n), device="cuda")
    lam[1, 1, node[2], node[1], node[0]] = value
    dx, dth = torch.zeros((1, 3), device="cuda"), torch.zeros(13, dtype=torch.float64, device="cuda")
    D.dock_pocket_map_adjoint(p, lam, dx, dth)
    assert torch.equal(dx, torch.zeros_like(dx)), dx
    assert float(dth[5 + 1]) > 0   # the radius takes lambda / d_clash from either atom
