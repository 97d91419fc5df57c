"""What the launch queries say of a lattice on register tiles: the tuner's shape
and time belong together."""
import pytest
import torch

pytestmark = pytest.mark.gpu

RATES = (1.64, 1.54, 1.9, 1.98)


def lattice(nx, ny, storage):
    from paper_1107_4543_amd import Lattice
    x = torch.arange(nx, dtype=torch.float64, device="cuda:0")[None, :]
    rho = 1.0 + 1e-3 * torch.cos(0.1 * x).expand(ny, nx).contiguous()
    z = torch.zeros_like(rho)
    return Lattice(nx, ny, *RATES, storage=storage, device="cuda:0").init(rho, z, z)


def test_tuned_shape_takes_the_time_reported_with_it():
    # one-step launches of this lattice take almost three times as long per step
    # as its tiles; either figure repeats to well within a factor of two
    lat = lattice(64, 64, "f32")
    shape, us = lat.tune(20)
    assert lat.launches_for(64) < 64                    # the tiles stay in use
    lat.set_launch(**shape)
    own = lat.time_launches(200) / lat.steps_per_launch
    assert own / 2 <= us <= own * 2, (us, own)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
def test_timed_launches_are_those_that_step_takes(storage):
    # 64 columns: no padding between rows, so a buffer is compared as it is
    lat, ref = lattice(64, 48, storage), lattice(64, 48, storage)
    T = lat.steps_per_launch
    assert lat.tiles["steps"] == T > 1 and lat.launches_for(3 * T) == 3
    lat.time_launches(3)
    now, n = lat.save_state()[0], lat.save_state()[0].numel()
    half = (n + 255) // 256 * 256
    bufs = [lat._ws[:n], lat._ws[half:half + n]]
    # the launches leave the state and put the one T steps on in the other buffer
    other = bufs[1] if torch.equal(bufs[0], now) else bufs[0]
    assert torch.equal(now, ref.save_state()[0]) and torch.equal(other, ref.step(T).save_state()[0])
    # by hand: one step per launch, and the tiles are out of use
    lat.set_launch(**lat.launch)
    assert lat.tiles is None and lat.steps_per_launch == 1
