"""Steps captured into a graph and replayed.

A graph's kernels work on fixed buffers.  An even number of steps captured on
a pending state must end in the buffer it began in, so every replay advances
the state; lattices whose steps run two to a launch are no exception, whatever
the parity of the number of pairs.  The reference is the same number of steps
taken eagerly, one call each, from the same state, with eager work and a
synchronisation between the replays; the bits are the same.
"""

import pytest
import torch

from paper_1405_6162_amd import inputs

pytestmark = pytest.mark.gpu


def _capture(fn):
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fn()
    return graph


# every total is even; single 64x64x32 FP64 and 128x40x40 FP32 pair their steps
@pytest.mark.parametrize("calls", [(2,), (4,), (6,), (3, 1), (5, 2, 3)])
@pytest.mark.parametrize("model,storage,nx,ny,nz", [
    ("single", "f64", 64, 64, 32), ("single", "f32", 128, 40, 40), ("single", "f64", 16, 8, 4),
    ("binary", "f64", 32, 16, 8), ("binary", "f32", 65, 9, 17)])
def test_replays_advance_the_state(lbgpu, model, storage, nx, ny, nz, calls):
    print("case graph %s %dx%dx%d %s, calls %s" % (model, nx, ny, nz, storage, calls), flush=True)
    code = {"f64": lbgpu.LB_F64, "f32": lbgpu.LB_F32}[storage]
    make = inputs.spinodal_quench if model == "binary" else inputs.single_fluid_random
    kind = lbgpu.LB_BINARY if model == "binary" else lbgpu.LB_SINGLE
    a, b = (lbgpu.Lattice(nx, ny, nz, model=kind, storage=code, tau_f=0.8) for _ in range(2))
    for lat in (a, b):
        lat.init_equilibrium(*make(nx, ny, nz, seed=5))
        lat.step(1)
    torch.cuda.synchronize()
    graph = _capture(lambda: [a.step(n) for n in calls])
    for _ in range(3):
        graph.replay()
        for _ in range(sum(calls)):
            b.step(1)
        torch.cuda.synchronize()
        for x, y in zip(a.get_state(), b.get_state()):
            assert x is None or torch.equal(x, y)
    a.step(3)                                  # the context knows where the state is
    for _ in range(3):
        b.step(1)
    for x, y in zip(a.get_state(), b.get_state()):
        assert x is None or torch.equal(x, y)
    a.close()
    b.close()


@pytest.mark.parametrize("n", [2, 5])
def test_capture_from_a_direct_state(lbgpu, n):
    """set_state and steps captured together: every replay starts from the
    array's values at that time."""
    nx, ny, nz = 64, 64, 32
    print("case graph single %dx%dx%d, set_state and %d steps" % (nx, ny, nz, n), flush=True)
    a, b = (lbgpu.Lattice(nx, ny, nz, tau_f=0.8) for _ in range(2))
    b.init_equilibrium(*inputs.single_fluid_random(nx, ny, nz, seed=6))
    f = b.get_state()[0].clone()
    out = torch.empty_like(f)

    def work():
        a.set_state(f)
        a.step(n)
        lbgpu.lb_get_state(a.ctx, out)
    graph = _capture(work)
    for _ in range(3):
        graph.replay()
        b.set_state(f)
        for _ in range(n):
            b.step(1)
        want = b.get_state()[0]
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        f.copy_(want)
    a.close()
    b.close()
