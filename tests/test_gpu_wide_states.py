"""Blocked states of 4 GiB and more a buffer, which take wide offsets: binary16
states, and records from FP64 ones.

The initial fields repeat a small lattice along every axis, so every step and
record must repeat the small lattice's bits.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu

SMALL = (64, 40, 37)


def _pair(lbgpu, copies, model, storage, coll, step):
    rep, shape = copies[::-1], SMALL[::-1]
    kw = dict(generator=torch.Generator().manual_seed(8), dtype=torch.float64)
    rho = (1 + 0.1 * torch.rand(shape, **kw)).cuda()
    u = (0.05 * (2 * torch.rand((3,) + shape, **kw) - 1)).cuda()
    phi = (0.2 * torch.rand(shape, **kw) - 0.1).cuda() if model else None
    par = dict(model=model, storage=storage, collision=coll, binary_step=step, tau_f=0.8, tau_minus=1.1, tau_bulk=1.3,
               tau_ghost_even=0.9, tau_ghost_odd=1.2)
    a = lbgpu.Lattice(*SMALL, **par)
    b = lbgpu.Lattice(*[n * k for n, k in zip(SMALL, copies)], **par)
    a.init_equilibrium(rho, u, phi)
    b.init_equilibrium(rho.repeat(rep), u.repeat((1,) + rep), None if phi is None else phi.repeat(rep))
    return a, b


def _same(x, y, copies):
    """y, any leading dimensions and then the lattice, is x repeated."""
    shape, rep = SMALL[::-1], copies[::-1]
    lead = tuple(y.shape[:-3])
    blocks = y.reshape(lead + tuple(v for k, n in zip(rep, shape) for v in (k, n)))
    return all(bool((blocks[i] == x[i].reshape(1, shape[0], 1, shape[1], 1, shape[2])).all()) for i in range(lead[0]))


@pytest.mark.parametrize("model,coll,step", [(0, 0, 0), (0, 2, 0), (1, 0, 1), (1, 2, 1), (1, 0, 2)])
def test_binary16(lbgpu, model, coll, step):
    copies = (8, 12, 14)                   # 512 x 480 x 518: 4.8 GB a buffer
    print("case wide FP16 model %d collision %d step %d" % (model, coll, step), flush=True)
    a, b = _pair(lbgpu, copies, model, lbgpu.LB_F16, coll, step)
    assert b.nsite * 19 * 2 >= 2 ** 32
    for n in (1, 3):
        a.step(n)
        b.step(n)
        sa, sb = a.get_state(), b.get_state()
        for x, y in zip(sa, sb):
            assert x is None or _same(x, y, copies)
    b.set_state(*sb)
    a.set_state(*sa)
    del sa, sb
    last = torch.arange(b.nsite - 100, b.nsite, dtype=torch.int32, device="cuda")
    got = b.get_sites(last)
    b.set_sites(last, *got)
    for x, y in zip(got, b.get_sites(last)):
        assert x is None or torch.equal(x, y)
    a.step(1)
    b.step(1)
    for x, y in zip(a.get_state(), b.get_state()):
        assert x is None or _same(x, y, copies)
    a.close()
    b.close()


@pytest.mark.parametrize("model,coll", [(0, 0), (0, 1), (1, 0), (1, 2)])
@pytest.mark.parametrize("pending", [False, True])
def test_records(lbgpu, model, coll, pending):
    copies = (5, 8, 8)                     # 320 x 320 x 296 FP64: 4.6 GB a buffer
    print("case wide record model %d collision %d pending %d" % (model, coll, pending), flush=True)
    a, b = _pair(lbgpu, copies, model, lbgpu.LB_F64, coll, 0)
    assert b.nsite * 19 * 8 >= 2 ** 32
    if pending:
        a.step(1)
        b.step(1)
    n = 2 if model else 3                  # binary: the second step marches; single: a pair follows the first step
    posts = []
    for lat in (a, b):
        post = torch.empty((n * (38 if model else 19),) + lat.shape, dtype=torch.float64, device="cuda")
        phi = torch.empty((n,) + lat.shape, dtype=torch.float64, device="cuda") if model else None
        lbgpu.lb_step_record(lat.ctx, n, post, phi)
        posts.append((post, phi))
    for x, y in zip(*posts):
        assert x is None or _same(x, y, copies)
    del posts, post, phi
    for x, y in zip(a.get_state(), b.get_state()):
        assert x is None or _same(x, y, copies)
    a.close()
    b.close()
