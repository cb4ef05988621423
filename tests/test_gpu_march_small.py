"""The single-pass binary step where LB_STEP_AUTO takes it on small lattices.

Its blocks then march chunks of one or a few planes, the grid is rounded up
to a multiple of 8 with surplus blocks that leave, and the stores are ordinary
ones.  Extents of one and two sites, one site over and short of a tile (64 x 8
and 128 x 4 columns) and of a chunk, each against the two-pass step, which
sums phi in the same order and shares the collision: the same bits in every
storage and collision.  On either side of the size from which FP64 takes the
march, the result is also held to the C oracle (1e-12 relative to the largest
value, the bound of every FP64 path).
"""

import numpy as np
import pytest
import torch

from oracle import c_backend as C
from paper_1405_6162_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (2, 3, 1), (1, 7, 5), (65, 1, 2), (130, 5, 3), (33, 40, 1), (63, 9, 4), (64, 8, 2), (129, 4, 9),
          (127, 3, 130)]


def _fields(nx, ny, nz):
    rho, _u, phi = inputs.spinodal_quench(nx, ny, nz, seed=51, phi_max=0.3)
    _r, u = inputs.single_fluid_random(nx, ny, nz, seed=52, u_max=0.01)
    return rho, u, phi


@pytest.mark.parametrize("nx,ny,nz", SHAPES)
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("collision", [0, 1, 2])
def test_small_march_equals_two_pass(lbgpu, storage, collision, nx, ny, nz):
    print("case binary %dx%dx%d %s collision %d, march vs two-pass" % (nx, ny, nz, storage, collision), flush=True)
    code = {"f64": lbgpu.LB_F64, "f32": lbgpu.LB_F32, "f16": lbgpu.LB_F16}[storage]
    rho, u, phi = _fields(nx, ny, nz)
    states = []
    for step in (lbgpu.LB_STEP_AUTO, lbgpu.LB_STEP_MARCH, lbgpu.LB_STEP_TWO_PASS):
        lat = lbgpu.Lattice(nx, ny, nz, model=lbgpu.LB_BINARY, storage=code, phi0=float(phi.mean()), binary_step=step,
                            collision=collision, tau_minus=1.25, tau_bulk=1.4, tau_ghost_even=0.9, tau_ghost_odd=1.2)
        lat.init_equilibrium(rho, u, phi)
        lat.step(5)
        states.append(lat.get_state())
        lat.close()
    for other in states[:2]:
        for a, b in zip(other, states[2]):
            assert bool(torch.isfinite(b).all()) and torch.equal(a, b)


@pytest.mark.parametrize("nx,ny,nz", [(57, 58, 60), (59, 60, 60)])
def test_step_choice_boundary_against_oracle(lbgpu, nx, ny, nz):
    print("case binary %dx%dx%d FP64 x3 vs C oracle" % (nx, ny, nz), flush=True)
    rho, u, phi = _fields(nx, ny, nz)
    C.set_threads(0)
    ref = C.CLattice(nx, ny, nz, model=1)
    ref.init_equilibrium(rho, u, phi)
    ref.step(3)
    want = ref.state()
    ref.close()
    lat = lbgpu.Lattice(nx, ny, nz, model=lbgpu.LB_BINARY)
    lat.init_equilibrium(rho, u, phi)
    lat.step(3)
    got = [a.cpu().numpy() for a in lat.get_state()]
    lat.close()
    for a, b in zip(got, want):
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
