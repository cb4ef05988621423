"""A blocked FP32 state whose single plane exceeds 4 GiB.

The initial fields repeat a small lattice along x and y, so every step must
repeat the small lattice's, bit for bit; the small lattice takes other tiles
and offsets.  The march and the two-pass step both run, and a copy out and in.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu

SMALL, COPIES = (64, 52, 1), (118, 144)        # 7552 x 7488 x 1: 4.3 GB a distribution


@pytest.mark.parametrize("step,coll", [(1, 0), (1, 2), (2, 0)])
def test_repeats_the_small_lattice(lbgpu, step, coll):
    nx, ny = SMALL[0] * COPIES[0], SMALL[1] * COPIES[1]
    print("case plane beyond 4 GiB %dx%dx1 FP32 step %d collision %d" % (nx, ny, step, coll), flush=True)
    assert nx * ny * 19 * 4 >= 2 ** 32
    shape, rep = (1, SMALL[1], SMALL[0]), (1, COPIES[1], COPIES[0])
    kw = dict(generator=torch.Generator().manual_seed(9), dtype=torch.float64)
    rho = (1 + 0.1 * torch.rand(shape, **kw)).cuda()
    u = (0.05 * (2 * torch.rand((3,) + shape, **kw) - 1)).cuda()
    phi = (0.2 * torch.rand(shape, **kw) - 0.1).cuda()
    par = dict(model=lbgpu.LB_BINARY, storage=lbgpu.LB_F32, collision=coll, binary_step=step, tau_f=0.8, tau_minus=1.1,
               tau_bulk=1.3, tau_ghost_even=0.9, tau_ghost_odd=1.2)
    a = lbgpu.Lattice(*SMALL, **par)
    b = lbgpu.Lattice(nx, ny, 1, **par)
    a.init_equilibrium(rho, u, phi)
    b.init_equilibrium(rho.repeat(rep), u.repeat((1,) + rep), phi.repeat(rep))
    del rho, u, phi

    def same(x, y):
        """y is x repeated."""
        x = x.reshape(19, 1, SMALL[1], 1, SMALL[0])
        return bool((y.reshape(19, COPIES[1], SMALL[1], COPIES[0], SMALL[0]) == x).all())

    for n in (1, 2):
        a.step(n)
        b.step(n)
    f, g = b.get_state()
    for x, y in zip(a.get_state(), (f, g)):
        assert same(x, y)
    b.set_state(f, g)
    del f, g
    a.step(2)
    b.step(2)
    for x, y in zip(a.get_state(), b.get_state()):
        assert same(x, y)
    a.close()
    b.close()
