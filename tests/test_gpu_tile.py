"""The register-tile step kernel that lattices of up to some million cells take
by default: bitwise equal to one-step launches at the sizes where tiles can go
wrong (one cell, widths and heights around a tile's 64 columns and 12, 16, 24,
32, 48 or 64 rows less its halo, several ragged tiles, lattices narrower than
the halo, the largest size of the default) and for step counts that fill,
overfill and split its launches."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

RATES = (1.3, 1.2, 1.7, 1.85)
SIZES = [(1, 1), (2, 5), (3, 130), (200, 1), (46, 30), (50, 2), (51, 3), (63, 65), (64, 64), (65, 17), (131, 49),
         (181, 147), (333, 215), (600, 430), (1000, 760)]


def pair(nx, ny, storage, compute=None, seed=0):
    from paper_1107_4543_amd import Lattice
    g = torch.Generator(device="cuda:0").manual_seed(seed + 1000 * nx + ny)
    r = lambda: 1e-3 * torch.randn((ny, nx), dtype=torch.float64, device="cuda:0", generator=g)
    fields = (1.0 + r(), 0.02 + r(), r())
    kw = dict(storage=storage, compute=compute, u0=(0.02, 0.0), device="cuda:0")
    tiled = Lattice(nx, ny, *RATES, **kw).init(*fields)
    single = Lattice(nx, ny, *RATES, **kw).set_launch(variant=0).init(*fields)
    return tiled, single


@pytest.mark.parametrize("storage,compute", [("f64", None), ("f64", "f32"), ("f32", None), ("f16", None),
                                             ("bf16", None)])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_tiles_equal_single_steps(nx, ny, storage, compute):
    tiled, single = pair(nx, ny, storage, compute)
    for n in (2, 3, 9, 1, 10, 23):
        assert tiled.launches_for(n) < n or n == 1
        tiled.step(n)
        single.step(n)
        assert tiled.t == single.t
        assert torch.equal(tiled.populations(), single.populations()), (n, tiled.t)


@pytest.mark.parametrize("storage,nx,ny", [("f64", 2048, 1792), ("f32", 3072, 2048), ("f16", 2048, 2048), ("bf16", 2048, 2048),
                                           ("bf16", 2560, 2048)])
def test_largest_tiled_size_equals_single_steps(storage, nx, ny):
    # the storage type's most cells, and one row more (back to strips)
    for rows in (ny, ny + 1):
        tiled, single = pair(nx, rows, storage)
        assert torch.equal(tiled.step(16).populations(), single.step(16).populations())
        del tiled, single


def test_setting_a_shape_replaces_the_tiles():
    tiled, single = pair(96, 80, "f32")
    assert tiled.launches_for(16) < 16 and single.launches_for(16) == 16
    shape = tiled.launch
    tiled.set_launch(**shape)
    assert tiled.launch == shape and tiled.launches_for(16) == 16
    assert torch.equal(tiled.step(16).populations(), single.step(16).populations())


def test_tuning_keeps_the_state_and_the_values():
    tiled, single = pair(130, 70, "f32")
    before = tiled.populations()
    shape, us = tiled.tune(2)
    assert us > 0 and tiled.launch == shape
    assert torch.equal(before, tiled.populations())
    assert torch.equal(tiled.step(13).populations(), single.step(13).populations())


def test_non_finite_values_spread_as_with_single_steps():
    # a NaN and an infinity cross tile edges exactly as one-step launches carry them
    tiled, single = pair(140, 75, "f32")
    f = single.populations()
    f[1, 40, 60] = float("nan")
    f[7, 10, 0] = float("inf")
    for lat in (tiled, single):
        lat.set_populations(f).step(11)
    a, b = tiled.populations(), single.populations()
    assert torch.equal(torch.isnan(a), torch.isnan(b)) and int(torch.isnan(a).sum()) > 0
    fin = ~torch.isnan(a)
    assert torch.equal(a[fin], b[fin])


def test_tiles_under_graph_capture():
    from paper_1107_4543_amd import Lattice
    side = torch.cuda.Stream()
    rho = 1.0 + 1e-3 * torch.rand((70, 130), dtype=torch.float64, device="cuda:0")
    z = torch.zeros_like(rho)
    torch.cuda.synchronize()
    lat = Lattice(130, 70, *RATES, storage="f32", device="cuda:0", stream=side).init(rho, z, z)
    ref = Lattice(130, 70, *RATES, storage="f32", device="cuda:0").set_launch(variant=0).init(rho, z, z)
    lat.step(4)                        # an even number of launches returns to the same buffer
    side.synchronize()
    n = next(k for k in range(8, 40) if lat.launches_for(k) % 2 == 0)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        lat.step(n)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
    assert torch.equal(lat.populations(), ref.step(4 + 3 * n).populations())
