"""States of 4 GiB and more a buffer, whose blocked layout takes wide offsets
where nx is a multiple of 64 and which are a structure of arrays otherwise.

The initial fields repeat a small lattice along every axis, so every step and
report must repeat the small lattice's, with the same bits (each site's
arithmetic is the same); the small lattice, under 4 GiB, is the reference.
A sum over the lattice is the small one's times the number of copies, within
the roundings of its additions: at most 256 a value in either, 512 x 2^-53
relative to the sum of absolute values.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu

# small lattice, copies along x, y and z; 30.3e6 sites: 4.6 GB a buffer
CASES = [((64, 40, 37), (5, 8, 8)), ((66, 40, 36), (5, 8, 8))]


@pytest.mark.parametrize("model,coll", [(0, 0), (0, 2), (1, 0), (1, 1)])
@pytest.mark.parametrize("small,copies", CASES)
def test_repeats_the_small_lattice(lbgpu, small, copies, model, coll):
    print("case beyond 4 GiB %s x %s model %d collision %d" % (small, copies, model, coll), flush=True)
    rep = (copies[2], copies[1], copies[0])
    shape = small[::-1]
    gen = torch.Generator().manual_seed(7)
    kw = dict(generator=gen, dtype=torch.float64)
    rho = (1 + 0.1 * torch.rand(shape, **kw)).cuda()
    u = (0.05 * (2 * torch.rand((3,) + shape, **kw) - 1)).cuda()
    phi = (0.2 * torch.rand(shape, **kw) - 0.1).cuda() if model else None
    par = dict(model=model, collision=coll, tau_f=0.8, tau_minus=1.1, tau_bulk=1.3, tau_ghost_even=0.9,
               tau_ghost_odd=1.2)
    a = lbgpu.Lattice(*small, **par)
    b = lbgpu.Lattice(*[n * k for n, k in zip(small, copies)], **par)
    a.init_equilibrium(rho, u, phi)
    b.init_equilibrium(rho.repeat(rep), u.repeat((1,) + rep), None if phi is None else phi.repeat(rep))

    def same(x, y):
        """y is x repeated."""
        lead = y.dim() - 3
        blocks = y.reshape(y.shape[:lead] + tuple(v for k, n in zip(rep, shape) for v in (k, n)))
        return bool((blocks == x.reshape(x.shape[:lead] + (1, shape[0], 1, shape[1], 1, shape[2]))).all())

    def check():
        for x, y in zip(a.moments(), b.moments()):
            assert (x is None) == (y is None)
            assert x is None or same(x, y)
        scale = float(a.conserved_sums()[0]) * copies[0] * copies[1] * copies[2]
        for x, y in ((a.conserved_sums(), b.conserved_sums()), (a.field_stats()[:6], b.field_stats()[:6])):
            assert float((y - x * (copies[0] * copies[1] * copies[2])).abs().max()) <= 2 * 512 * 2.0 ** -53 * scale
        assert torch.equal(a.field_stats()[6:8], b.field_stats()[6:8])

    check()                              # direct
    for n in (1, 4):                     # then pending
        a.step(n)
        b.step(n)
        check()
    # the last sites, which lie beyond 4 GiB: out, doubled, and in again
    for lat in (a, b):
        last = torch.arange(lat.nsite - 100, lat.nsite, dtype=torch.int32, device="cuda")
        got = lat.get_sites(last)
        lat.set_sites(last, *[None if t is None else 2 * t for t in got])
        again = lat.get_sites(last)
        for t, s in zip(got, again):
            assert t is None or torch.equal(2 * t, s)
        lat.set_sites(last, *got)
    sa, sb = a.get_state(), b.get_state()
    for x, y in zip(sa, sb):
        assert x is None or same(x, y)
    b.set_state(*sb)
    del sb
    a.propagate()
    b.propagate()
    a.collide()
    b.collide()
    for x, y in zip(a.get_state(), b.get_state()):
        assert x is None or same(x, y)
    a.close()
    b.close()
