"""Equilibrium initialisation against the oracle at widths where the split of a
cell number into row and column can go wrong (1, powers of two and their
neighbours, one long row or column), and the storage scale that 16-bit
lattices choose from the largest population."""
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 777), (2, 9), (63, 5), (64, 3), (65, 7), (127, 4), (1023, 3), (1025, 3),
                                   (100003, 1), (4097, 130)])
def test_init_matches_the_oracle(nx, ny):
    from paper_1107_4543_amd import Lattice
    rng = np.random.default_rng(nx + ny)
    r = lambda: 1e-3 * rng.standard_normal((ny, nx))
    rho, ux, uy = 1.0 + r(), 0.03 + r(), r()
    ref = oracle.init(rho, ux, uy)
    # sums of about ten terms below 1/2, each rounded: 1e-14 is 45 such roundings
    lat = Lattice(nx, ny, 1.3, 1.2, 1.7, 1.85, storage="f64", u0=(0.03, 0.0), device="cuda:0").init(rho, ux, uy)
    assert np.max(np.abs(lat.populations().cpu().numpy() - ref)) <= 1e-14
    base = oracle.init(np.ones((1, 1)), np.full((1, 1), 0.03), np.zeros((1, 1)))
    largest = np.max(np.abs(ref - base))
    half = Lattice(nx, ny, 1.3, 1.2, 1.7, 1.85, storage="f16", u0=(0.03, 0.0), device="cuda:0").init(rho, ux, uy)
    want = math.log2(8192.0 / largest)
    assert half.scale_exp == math.floor(want) or abs(want - round(want)) < 1e-9


def test_non_finite_fields_are_reported():
    from paper_1107_4543_amd import Lattice, _lib
    rho = torch.ones((40, 70), dtype=torch.float64, device="cuda:0")
    rho[17, 69] = float("inf")
    z = torch.zeros_like(rho)
    for storage in ("f64", "f32", "f16"):
        lat = Lattice(70, 40, 1.3, 1.2, 1.7, 1.85, storage=storage, scale_exp=10, device="cuda:0").init(rho, z, z)
        status, d = lat.diagnostics()
        assert status == _lib.LBM_E_NONFINITE and 1 <= d[3] <= 9
