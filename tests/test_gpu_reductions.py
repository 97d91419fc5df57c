"""Global reductions against numpy on the lattice's own populations, at the
shapes where their work split can go wrong: one cell, rows narrower than a
wave, widths around and beyond a block's 256 and 1024 threads, more rows than
one table of row phases holds, ragged last bands."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (3, 700), (1, 5000), (2, 66000), (700, 3), (64, 64), (255, 33), (257, 70), (1025, 41), (40000, 2), (1300, 1100)]
MODES = [(0, 0), (1, 0), (3, -2), (-7, 11), (70001, -65539)]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_projection_and_diagnostics_match_numpy(nx, ny, storage):
    from paper_1107_4543_amd import Lattice
    g = torch.Generator(device="cuda:0").manual_seed(nx + 3 * ny)
    r = lambda: 1e-3 * torch.randn((ny, nx), dtype=torch.float64, device="cuda:0", generator=g)
    lat = Lattice(nx, ny, 1.3, 1.2, 1.7, 1.85, storage=storage, u0=(0.02, 0.0), device="cuda:0")
    lat.init(1.0 + r(), 0.025 + r(), 0.01 + r())
    base = Lattice(1, 1, 1.3, 1.2, 1.7, 1.85, storage="f64", u0=(0.02, 0.0), device="cuda:0")
    one = torch.ones((1, 1), dtype=torch.float64)
    f0 = base.init(one, 0.02 * one, 0.0 * one).populations().cpu().numpy()[:, 0, 0]
    f = lat.populations().cpu().numpy()
    d = f - f0[:, None, None]
    # a sum of n values about f0, each stored to a rounding of its size
    tol = nx * ny * np.spacing(np.max(np.abs(f)))
    x, y = np.arange(nx)[None, :], np.arange(ny)[:, None]
    for mx, my in MODES:
        ph = np.exp(-2j * np.pi * (((mx * x) % nx) / nx + ((my * y) % ny) / ny))
        want = (d * ph[None]).sum(axis=(1, 2))
        got = lat.project(mx, my).cpu().numpy()
        got = got[0::2] + 1j * got[1::2]
        assert np.max(np.abs(got - want)) <= 1e-12 * np.max(np.abs(want)) + tol, (mx, my)
    st, got = lat.diagnostics()
    cx, cy = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1]), np.array([0, 0, 1, 0, -1, 1, 1, -1, -1])
    per = d.sum(axis=(1, 2))
    want = [per.sum(), (cx * per).sum(), (cy * per).sum()]
    assert st == 0 and got[3] == 0
    assert np.max(np.abs(np.array(got[:3]) - want)) <= 9 * tol


def test_non_finite_values_are_counted():
    from paper_1107_4543_amd import Lattice, _lib
    lat = Lattice(300, 41, 1.3, 1.2, 1.7, 1.85, storage="f32", device="cuda:0")
    f = torch.zeros((9, 41, 300), dtype=torch.float64, device="cuda:0") + 0.1
    f[3, 40, 299] = float("nan")
    f[8, 0, 0] = float("inf")
    f[0, 20, 128] = -float("inf")
    status, d = lat.set_populations(f).diagnostics()
    assert status == _lib.LBM_E_NONFINITE and d[3] == 3
