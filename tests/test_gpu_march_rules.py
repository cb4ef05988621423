"""The march where its launch rules turn: the same bits as the two-pass step.

Chunks are chosen by rounds x (depth + 3), blocks go in XCD or launch order, and
what is loaded ahead depends on storage, tile and depth; each case names the
turn it stands at, and the grid is computed here as the rules state it.
"""

import pytest
import torch

from paper_1405_6162_amd import inputs

pytestmark = pytest.mark.gpu


def _grid(storage, nx, ny, nz):
    """Columns, chunks, depth and whether tiles are 128 wide."""
    wide = storage != "f64" and -(-nx // 128) * 2 == -(-nx // 64)
    cols = -(-nx // (128 if wide else 64)) * -(-ny // (4 if wide else 8))
    slots = 512 if storage == "f16" else 256
    cost = [(-(-cols * c // slots) * (-(-nz // c) + 3), c) for c in range(-(-nz // 128), nz + 1)]
    chunks = min(cost)[1]
    return cols * chunks, -(-nz // chunks), wide, slots


CASES = [
    # (storage, shape, what): blocks, depth, width asserted below
    ("f64", (512, 260, 4), "short chunks, two rounds"), ("f32", (512, 512, 5), "short chunks, two rounds"),
    ("f32", (320, 840, 5), "short chunks, 64 wide"), ("f64", (65, 544, 48), "launch order, blocks a multiple of 8"),
    ("f64", (65, 520, 48), "launch order, blocks no multiple of 8"), ("f64", (100, 50, 30), "one round"),
    ("f64", (512, 256, 126), "one deep chunk"), ("f64", (130, 9, 257), "many chunks"),
    ("f32", (192, 192, 164), "64 wide, the ring loaded ahead"), ("f32", (256, 520, 9), "XCD order, two rounds"),
    ("f64", (512, 520, 2), "two planes"), ("f32", (512, 1030, 2), "two planes"), ("f32", (512, 300, 1), "one plane"),
    ("f16", (200, 136, 70), "128 wide"), ("f16", (150, 97, 41), "64 wide"), ("f16", (512, 900, 6), "two rounds")]


@pytest.mark.parametrize("storage,shape,what", CASES)
def test_march_equals_two_pass(lbgpu, storage, shape, what):
    nx, ny, nz = shape
    blocks, depth, wide, slots = _grid(storage, nx, ny, nz)
    print("case march %s %dx%dx%d: %s; %d blocks, depth %d" % (storage, nx, ny, nz, what, blocks, depth), flush=True)
    if "short" in what:
        assert 4 <= depth < 8 and blocks > slots
    if "launch order" in what:
        assert depth > 15 and blocks > slots and (blocks % 8 == 0) == ("a multiple" in what)
    if "XCD" in what or "two rounds" in what:
        assert depth < 16 and slots < blocks <= 2 * slots
    if "one round" in what or "deep" in what:
        assert blocks <= slots
    if "deep" in what:
        assert depth > 120
    if "wide" in what:
        assert wide == ("128" in what)
    if "ring" in what:
        assert not wide and nx * ny * nz >= 6000000
    code = {"f64": lbgpu.LB_F64, "f32": lbgpu.LB_F32, "f16": lbgpu.LB_F16}[storage]
    fields = inputs.spinodal_quench(nx, ny, nz, seed=4)
    got = []
    for step in (lbgpu.LB_STEP_MARCH, lbgpu.LB_STEP_TWO_PASS):
        lat = lbgpu.Lattice(nx, ny, nz, model=lbgpu.LB_BINARY, storage=code, binary_step=step, tau_f=0.8)
        lat.init_equilibrium(*fields)
        lat.step(3)
        got.append(lat.get_state())
        lat.close()
    for a, b in zip(*got):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)
