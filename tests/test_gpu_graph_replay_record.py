"""A binary record captured into a graph and replayed, with eager work and a
synchronisation between the replays."""

import pytest
import torch

from paper_1405_6162_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3])
def test_replayed_binary_record_repeats_its_segment(lbgpu, n):
    """A record of the binary fluid captured on a pending state leaves that
    state's buffer alone: a replay records the same steps again."""
    nx, ny, nz = 65, 9, 17
    print("case graph binary record %dx%dx%d n %d" % (nx, ny, nz, n), flush=True)
    a, b = (lbgpu.Lattice(nx, ny, nz, model=lbgpu.LB_BINARY, tau_f=0.8) for _ in range(2))
    for lat in (a, b):
        lat.init_equilibrium(*inputs.spinodal_quench(nx, ny, nz, seed=7))
        lat.step(1)
    post = torch.zeros((n, 38, nz, ny, nx), dtype=torch.float64, device="cuda")
    want = torch.zeros_like(post)
    lbgpu.lb_step_record(b.ctx, n, want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lbgpu.lb_set_stream(a.ctx, torch.cuda.current_stream().cuda_stream)
        lbgpu.lb_step_record(a.ctx, n, post)
    for _ in range(3):
        post.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(post, want)
    for x, y in zip(a.get_state(), b.get_state()):
        assert torch.equal(x, y)
    a.close()
    b.close()
