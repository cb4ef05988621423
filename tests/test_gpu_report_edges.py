"""Reductions over the lattice and mask compaction at the edges of their
blocking: more 64 x 4 tiles than the reductions have blocks and fewer, ragged
tiles, one site; masks whose length is no multiple of 16 sites or of a block's
4096, at any alignment, full and empty.  The reference is torch on the state
handed out.

Tolerance of a sum: every value passes through at most 256 additions here (19
directions, a few tiles a block, two block-wide reductions) and torch's own
pairwise sum through fewer, so each is within 512 x 2^-53 = 5.7e-14 of the
exact sum, relative to the sum of absolute values.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu

# 64 x 4 tiles: 1, 18, 2048, 2049, 3672
SHAPES = [(1, 1, 1), (65, 9, 3), (64, 32, 256), (64, 4, 2049), (130, 69, 68)]
REL = 512 * 2.0 ** -53


def _lattice(lbgpu, shape, model):
    nx, ny, nz = shape
    gen = torch.Generator().manual_seed(nx + ny + nz)
    rho = 1 + 0.1 * torch.rand(nz, ny, nx, generator=gen, dtype=torch.float64)
    u = 0.05 * (2 * torch.rand(3, nz, ny, nx, generator=gen, dtype=torch.float64) - 1)
    phi = torch.rand(nz, ny, nx, generator=gen, dtype=torch.float64) - 0.5 if model else None
    lat = lbgpu.Lattice(nx, ny, nz, model=model)
    lat.init_equilibrium(rho, u, phi)
    return lat


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_sums_and_stats(lbgpu, shape, model):
    from paper_1405_6162_amd import adjoint
    print("case sums %s model %d" % (shape, model), flush=True)
    lat = _lattice(lbgpu, shape, model)
    for pending in (False, True):
        if pending:
            lat.step(1)
        f, g = lat.get_state()
        c = adjoint.velocity_table(f.device).t()
        want = [f.sum()] + [(c[a].reshape(19, 1, 1, 1) * f).sum() for a in range(3)]
        size = f.abs().sum()
        sums, stats = lat.conserved_sums(), lat.field_stats()
        for k in range(4):
            for got in (sums[k], stats[k]):
                assert abs(float(got - want[k])) <= 2 * REL * float(size)
        if model:
            phi = g.sum(0)
            for got in (sums[4], stats[4]):
                assert abs(float(got - phi.sum())) <= 2 * REL * float(g.abs().sum())
            # a site's phi is itself a sum of 19 values; both are rounded
            near = 64 * 2.0 ** -53 * float(g.abs().sum(0).max())
            assert abs(float(stats[6] - phi.min())) <= near and abs(float(stats[7] - phi.max())) <= near
    f[(0,) + tuple(n - 1 for n in f.shape[1:])] = float("nan")
    lat.set_state(f, g)
    assert torch.isnan(lat.conserved_sums()[0]) and torch.isnan(lat.field_stats()[0])


@pytest.mark.parametrize("shape", [(1, 1, 1), (15, 1, 1), (16, 16, 16), (4097, 1, 1), (63, 65, 33), (130, 69, 68)])
def test_mask_compaction(lbgpu, shape):
    nx, ny, nz = shape
    n = nx * ny * nz
    print("case mask %s" % (shape,), flush=True)
    lat = lbgpu.Lattice(nx, ny, nz)
    gen = torch.Generator().manual_seed(n)
    for share in (0.0, 0.3, 1.0):
        for shift in (0, 1, 8, 13):
            buf = torch.full((n + 16,), 255, dtype=torch.uint8)       # what lies around the mask must not count
            buf[shift:shift + n] = (torch.rand(n, generator=gen) < share) * torch.randint(1, 256, (n,), generator=gen)
            mask = buf.cuda()[shift:shift + n].reshape(nz, ny, nx)
            got = lat.mask_index(mask)
            assert torch.equal(got.long(), mask.reshape(-1).nonzero().reshape(-1))
