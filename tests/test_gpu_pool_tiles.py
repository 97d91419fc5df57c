"""A pool's register tiles (few cells) and shared-halo strips (large members): members
equal the same lattice advanced alone by one-step launches, bitwise, for sizes
around a tile's edges, every storage type, chunks of fewer steps than T, members
that join and leave on the way; and strips once a large member fills the device
with them, or where the tile table has no room for tiles."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SETS = [[1.64, 1.54, 1.9, 1.98], [1.3, 1.1, 1.7, 1.85], [1.2, 1.5, 1.4, 1.6]]
SIZES = [(1, 1), (1, 60), (52, 36), (53, 37), (64, 64), (257, 21), (104, 130), (333, 75)]
STEPS = [40, 23, 37, 64, 5, 44, 71, 30]
# steps per launch, flags
SHAPES = [(7, 32), (7, 98), (6, 34), (4, 32), (2, 32)]


def make(nx, ny, s, storage, seed):
    from paper_1107_4543_amd import Lattice
    rng = np.random.default_rng(seed)
    r = lambda: 1e-3 * rng.standard_normal((ny, nx))
    f = (1.0 + r(), 0.02 + r(), r())
    a = Lattice(nx, ny, *s, storage=storage, u0=(0.02, 0.0), device="cuda:0").init(*f)
    b = Lattice(nx, ny, *s, storage=storage, u0=(0.02, 0.0), device="cuda:0").set_launch(variant=0).init(*f)
    return a, b


def run(pool, sizes, storages, steps, join):
    """Adds the members from `join` on only after the others have run 9 steps."""
    pairs = [make(nx, ny, SETS[i % 3], storages[i % len(storages)], 70 + i) for i, (nx, ny) in enumerate(sizes)]
    for i, (a, _) in enumerate(pairs):
        if i == join:
            pool.step(9)
        pool.add(a, steps[i])
    pool.step(25)
    pool.step(1000)
    out = []
    while pool.members:
        out += pool.poll(wait=True)
    assert len(out) == len(pairs)
    for (a, b), n in zip(pairs, steps):
        assert a.t == n
        assert torch.equal(a.populations(), b.step(n).populations()), (a.nx, a.ny, a.storage)


@pytest.mark.parametrize("storages", [["f64"], ["f32"], ["f16"], ["bf16"], ["f32", "f64", "f16"]])
@pytest.mark.parametrize("T,flags", SHAPES)
def test_tile_tables_match_single_steps(T, flags, storages):
    from paper_1107_4543_amd.pool import Pool
    pool = Pool(max_members=16, max_tiles=1 << 14)
    # grid 16: a workgroup walks several tiles in turn
    pool.set_shape(tile_cells=512, block=256, grid=16, graph_steps=28, steps_per_launch=T, flags=flags)
    run(pool, SIZES, storages, STEPS, 5)
    pool.close()


@pytest.mark.parametrize("storage,big", [("f64", (4000, 4096)), ("f32", (4096, 4003)), ("bf16", (4096, 3500))])
@pytest.mark.parametrize("T,flags", SHAPES[:3])
def test_strips_of_large_members_match_single_steps(T, flags, storage, big):
    from paper_1107_4543_amd.pool import Pool
    pool = Pool(max_members=16, max_tiles=1 << 17)
    pool.set_shape(tile_cells=512, block=256, grid=64, graph_steps=28, steps_per_launch=T, flags=flags)
    # the large member leaves first: the others go on with tiles
    run(pool, SIZES[1:] + [(600, 70), big], [storage], STEPS[1:] + [50, 16], 4)
    pool.close()


def test_a_full_tile_table_keeps_strips():
    # 64 x 64 at 512 cells a tile: 8 one-step tiles and one strip of one segment
    from paper_1107_4543_amd.pool import Pool
    pool = Pool(max_members=2, max_tiles=9)
    pool.set_shape(tile_cells=512, block=256, grid=16, graph_steps=28, steps_per_launch=7, seg_rows=64, flags=32)
    a, b = make(64, 64, SETS[0], "f32", 3)
    pool.add(a, 33)
    pool.step(33)
    assert pool.poll(wait=True) == [a]
    assert torch.equal(a.populations(), b.step(33).populations())
    pool.close()


def test_timing_and_tuning_leave_tiled_members_as_they_are():
    from paper_1107_4543_amd.pool import Pool
    pool = Pool(max_members=4, max_tiles=1 << 12)
    a, b = make(130, 70, SETS[1], "f32", 4)
    pool.add(a, 40)
    pool.step(14)
    assert pool.time_launches(2) > 0
    pool.step(40)
    assert pool.poll(wait=True) == [a]
    assert torch.equal(a.populations(), b.step(40).populations())
    pool.close()


@pytest.mark.parametrize("storage", ["f16", "bf16"])
def test_tall_16_bit_tiles_match_single_steps(storage):
    # members large enough for the shape of four rows per lane and sixteen waves
    from paper_1107_4543_amd.pool import Pool
    pool = Pool(max_members=16, max_tiles=1 << 14)
    pool.set_shape(tile_cells=512, block=256, graph_steps=28, steps_per_launch=6, flags=34)
    run(pool, [(1024, 1000), (777, 1021), (53, 37), (901, 640)], [storage], [40, 23, 64, 31], 3)
    pool.close()
