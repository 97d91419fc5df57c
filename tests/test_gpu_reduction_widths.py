"""Projections at widths and heights between 46342 and 65535, where a product of
two coordinates passes 2^31 but not 2^32, on modes near the largest, against
numpy on the lattice's own populations."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(65535, 2), (2, 60000), (46342, 3), (65536, 1)])
def test_modes_near_the_largest(nx, ny):
    from paper_1107_4543_amd import Lattice
    g = torch.Generator(device="cuda:0").manual_seed(nx + ny)
    r = lambda: 1e-3 * torch.randn((ny, nx), dtype=torch.float64, device="cuda:0", generator=g)
    lat = Lattice(nx, ny, 1.3, 1.2, 1.7, 1.85, storage="f64", device="cuda:0").init(1.0 + r(), r(), r())
    f = lat.populations().cpu().numpy()
    # the populations of the base state, rho = 1 at rest
    d = f - np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None, None]
    # a sum of n values, each within an ulp of f of its own
    tol = nx * ny * np.spacing(np.max(np.abs(f)))
    x, y = np.arange(nx, dtype=np.int64)[None, :], np.arange(ny, dtype=np.int64)[:, None]
    for mx, my in [(nx - 1, ny - 1), (nx - 2, 1), (nx // 2 + 1, ny - 1), (-1, -1)]:
        ph = np.exp(-2j * np.pi * (((mx * x) % nx) / nx + ((my * y) % ny) / ny))
        want = (d * ph[None]).sum(axis=(1, 2))
        got = lat.project(mx, my).cpu().numpy()
        got = got[0::2] + 1j * got[1::2]
        assert np.max(np.abs(got - want)) <= 1e-12 * np.max(np.abs(want)) + tol, (mx, my)


@pytest.mark.parametrize("nx,mode", [(1200000000, 1000000000), (2147400000, 1500000000)])
def test_lattices_of_more_than_2_to_30_columns(nx, mode):
    # one plane wave at rest, whose populations are w_i a cos(k x): the mode's sum
    # is w_i a n / 2 however it is numbered, every other mode's and the mass are 0
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 130e9:
        pytest.skip("needs 130 GB of device memory")
    from paper_1107_4543_amd import Lattice
    a = 1e-3
    q = torch.arange(nx, dtype=torch.int64, device="cuda:0")
    q *= mode
    q %= nx
    rho = q.to(torch.float64)
    del q
    rho *= 2 * np.pi / nx
    rho.cos_()
    rho *= a
    rho += 1.0
    rho = rho.view(1, nx)
    z = torch.zeros_like(rho)
    lat = Lattice(nx, 1, 1.3, 1.2, 1.7, 1.85, storage="f16", device="cuda:0").init(rho, z, z)
    get = lambda m: lat.project(m, 0).cpu().numpy().view(np.complex128)
    want = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4) * a * nx / 2
    # each stored value is within 2^-11 of its own
    assert np.all(np.abs(get(mode) - want) <= 2.0 ** -11 * want)
    assert np.array_equal(get(mode - nx), get(mode))
    assert np.max(np.abs(get(7))) <= 2.0 ** -11 * np.max(want)
    status, d = lat.diagnostics()
    assert status == 0 and d[3] == 0 and abs(d[0]) <= 2.0 ** -11 * a * nx and d[1] == d[2] == 0
    del lat, rho, z
    torch.cuda.empty_cache()
