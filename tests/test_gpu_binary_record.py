"""lb_step_record of the binary fluid: step 0 collides from the state's own
layout straight into the canonical record.

Every recorded post-collision f and g, phi of every state collided and the
state afterwards have the bits of collide and propagate calls, from a direct
state and from pending ones, with the march and the two-pass step, for records
of one and more steps, with phi asked for and not, on lattices whose rows fill
no whole 64-site block and whose tiles are ragged.
"""

import pytest
import torch

from paper_1405_6162_amd import inputs

pytestmark = pytest.mark.gpu

COLL = {"bgk": {}, "trt": dict(collision=1, tau_minus=1.25),
        "mrt": dict(collision=2, tau_minus=1.25, tau_bulk=1.4, tau_ghost_even=0.9, tau_ghost_odd=1.2)}


@pytest.mark.parametrize("coll", ["bgk", "trt", "mrt"])
@pytest.mark.parametrize("vvl", [0, 4])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx,ny,nz", [(3, 2, 1), (65, 9, 7), (64, 64, 52)])
def test_records_equal_single_calls(lbgpu, nx, ny, nz, storage, vvl, coll):
    print("case record binary %dx%dx%d %s vvl %d %s" % (nx, ny, nz, storage, vvl, coll), flush=True)
    code = {"f64": lbgpu.LB_F64, "f32": lbgpu.LB_F32, "f16": lbgpu.LB_F16}[storage]
    fields = inputs.spinodal_quench(nx, ny, nz, seed=3)
    a, b = (lbgpu.Lattice(nx, ny, nz, model=lbgpu.LB_BINARY, storage=code, vvl=vvl, tau_f=0.8, **COLL[coll])
            for _ in range(2))
    for lat in (a, b):
        lat.init_equilibrium(*fields)
    ph_type = torch.float64 if storage == "f64" else torch.float32
    for n, with_phi in ((1, True), (2, False), (3, True), (1, False)):
        post = torch.full((n, 38, nz, ny, nx), float("nan"), dtype=lbgpu.STORAGE_DTYPE[code], device="cuda")
        phi = torch.full((n, nz, ny, nx), float("nan"), dtype=ph_type, device="cuda") if with_phi else None
        lbgpu.lb_step_record(a.ctx, n, post, phi)
        for k in range(n):
            if with_phi:
                # phi0 is 0 and both are sums of the same 19 values
                want = b.moments()[2]
                size = float(b.get_state()[1].abs().double().sum(0).max())
                tol = 40 * (2.0 ** -53 if storage == "f64" else 2.0 ** -24) * size
                assert float((phi[k].double() - want).abs().max()) <= tol
            b.collide()
            f, g = b.get_state()
            assert torch.equal(post[k, :19], f) and torch.equal(post[k, 19:], g)
            b.propagate()
        for x, y in zip(a.get_state(), b.get_state()):
            assert torch.equal(x, y)
    a.close()
    b.close()
