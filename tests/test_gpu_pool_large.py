"""A pool member whose nine planes exceed the 4 GiB that one buffer resource
reaches: it has no register tiles, so the pool takes strips, bitwise equal to
one-step launches."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_a_member_beyond_one_buffer_resource_takes_strips():
    from paper_1107_4543_amd import Lattice
    from paper_1107_4543_amd.pool import Pool
    nx, ny = 7744, 7745                                # 4.32e9 bytes of FP64 populations
    assert nx * ny * 9 * 8 > 1 << 32
    x = torch.arange(nx, dtype=torch.float64, device="cuda:0")[None, :]
    y = torch.arange(ny, dtype=torch.float64, device="cuda:0")[:, None]
    rho = 1.0 + 1e-3 * torch.cos(0.01 * x) * torch.cos(0.02 * y)
    u = 1e-3 * torch.sin(0.013 * x + 0.004 * y)
    pair = [Lattice(nx, ny, 1.3, 1.1, 1.7, 1.85, storage="f64", device="cuda:0").init(rho, u, u) for _ in range(2)]
    a, b = pair[0], pair[1].set_launch(variant=0)
    small = Lattice(64, 64, 1.3, 1.1, 1.7, 1.85, storage="f64", device="cuda:0")
    small.init(rho[:64, :64].contiguous(), u[:64, :64].contiguous(), u[:64, :64].contiguous())
    pool = Pool(max_members=2, max_tiles=1 << 19)
    pool.add(a, 9)
    pool.add(small, 9)
    pool.step(9)
    done = 0
    while done < 2:
        done += len(pool.poll(wait=True))
    assert torch.equal(a.populations(), b.step(9).populations())
    pool.close()
