"""How many launches single-fluid steps take: five for steps of 2, 3 and 4 that
run two to a launch, nine for steps taken alone, exactly, for every storage and
collision, so that a comparison of pairs with single steps compares the two.
A record of five steps takes its first alone and the others in pairs.  The
bits are those of single calls either way."""

import pytest
import torch

from paper_1405_6162_amd import inputs

pytestmark = pytest.mark.gpu

COLL = {"bgk": {}, "trt": dict(collision=1, tau_minus=1.25),
        "mrt": dict(collision=2, tau_minus=1.25, tau_bulk=1.4, tau_ghost_even=0.9, tau_ghost_odd=1.2)}


@pytest.mark.parametrize("storage,coll,nx,ny,nz,paired", [
    ("f64", "bgk", 67, 9, 216, True), ("f64", "trt", 63, 7, 297, True), ("f64", "trt", 130, 91, 89, True),
    ("f64", "mrt", 128, 128, 32, True), ("f64", "mrt", 130, 91, 89, True), ("f64", "mrt", 64, 64, 64, False),
    ("f64", "bgk", 40, 40, 40, False), ("f64", "bgk", 300, 2, 300, False), ("f64", "bgk", 1100, 1000, 1, False),
    ("f32", "bgk", 127, 33, 49, True), ("f32", "trt", 67, 45, 67, False), ("f32", "trt", 88, 88, 88, True),
    ("f32", "trt", 200, 97, 101, True), ("f32", "mrt", 150, 70, 90, True),
    ("f32", "mrt", 200, 97, 101, True), ("f32", "mrt", 128, 40, 40, False),
    ("f16", "bgk", 192, 104, 101, True), ("f16", "bgk", 128, 128, 123, True), ("f16", "trt", 256, 256, 192, True),
    ("f16", "trt", 128, 128, 123, False), ("f16", "mrt", 128, 128, 123, False)])
def test_launches(lbgpu, storage, coll, nx, ny, nz, paired):
    print("case launches single %dx%dx%d %s %s" % (nx, ny, nz, storage, coll), flush=True)
    code = {"f64": lbgpu.LB_F64, "f32": lbgpu.LB_F32, "f16": lbgpu.LB_F16}[storage]
    rho, u = inputs.single_fluid_random(nx, ny, nz, seed=nx)
    a, b = (lbgpu.Lattice(nx, ny, nz, storage=code, tau_f=0.8, **COLL[coll]) for _ in range(2))
    for lat in (a, b):
        lat.init_equilibrium(rho, u)
    lbgpu.lb_profile(a.ctx, True)
    for n in (2, 3, 4):
        a.step(n)
        for _ in range(n):
            b.step(1)
    lbgpu.lb_profile(a.ctx, False)
    assert lbgpu.lb_kernel_times(a.ctx, lbgpu.LB_K_COLLIDE)[1] == (5 if paired else 9)
    assert torch.equal(a.get_state()[0], b.get_state()[0])
    post = torch.empty((5, 19, nz, ny, nx), dtype=lbgpu.STORAGE_DTYPE[code], device="cuda")
    lbgpu.lb_profile(a.ctx, True)
    lbgpu.lb_step_record(a.ctx, 5, post)
    lbgpu.lb_profile(a.ctx, False)
    assert lbgpu.lb_kernel_times(a.ctx, lbgpu.LB_K_COLLIDE)[1] == (3 if paired else 5)
    for k in range(5):
        b.collide()
        assert torch.equal(post[k], b.get_state()[0])
        b.propagate()
    a.close()
    b.close()
