"""A pool's tables over the life of its members: one-step tiles are in them while
launches need them and leave with the next change of members."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

RANGES = 16          # table ranges: 4 storage types x 2 compute types x 2 chains


def counts(pool):
    """(one-step tiles, T-step tasks) in the tables on the device: the header at
    the start of the workspace holds the first and one past the last of each
    range, for one-step tiles, T-step tasks and two-wave tasks."""
    torch.cuda.synchronize()
    h = pool._ws[:6 * RANGES * 4].cpu().numpy().view(np.int32).reshape(3, 2, RANGES)
    n = (h[:, 1] - h[:, 0]).sum(axis=1)
    return int(n[0]), int(n[1] + n[2])


def lattice(nx, ny, seed):
    from paper_1107_4543_amd import Lattice
    rng = np.random.default_rng(seed)
    r = lambda: 1e-3 * rng.standard_normal((ny, nx))
    f = (1.0 + r(), r(), r())
    a = Lattice(nx, ny, 1.3, 1.1, 1.7, 1.85, storage="f32", device="cuda:0").init(*f)
    return a, Lattice(nx, ny, 1.3, 1.1, 1.7, 1.85, storage="f32", device="cuda:0").set_launch(variant=0).init(*f)


@pytest.mark.parametrize("flags", [0, 32, 96])
def test_one_step_tiles_leave_with_the_next_change_of_members(flags):
    from paper_1107_4543_amd.pool import Pool
    pool = Pool(max_members=4, max_tiles=1 << 12)
    pool.set_shape(tile_cells=512, block=256, grid=64, graph_steps=28, steps_per_launch=7, seg_rows=32, flags=flags)
    (a, ra), (b, rb), (c, rc) = (lattice(130 + 9 * i, 70 + i, i) for i in range(3))
    pool.add(a, 15)                                    # 14 steps in launches of seven and one left over
    pool.step(14)
    one, tasks = counts(pool)
    assert one == 0 and tasks > 0
    pool.step(1)
    assert counts(pool)[0] > 0
    assert pool.poll(wait=True) == [a]
    pool.add(b, 21)
    pool.step(14)
    one, tasks = counts(pool)
    assert one == 0 and tasks > 0
    pool.add(c, 8)                                     # one step left over beside b's last seven
    pool.step(8)
    out = []
    while pool.members:
        out += pool.poll(wait=True)
    assert len(out) == 2
    for lat, ref, n in ((a, ra, 15), (b, rb, 21), (c, rc, 8)):
        assert lat.t == n and torch.equal(lat.populations(), ref.step(n).populations())
    pool.close()
