"""The library's launch rules, asked on the host (tests/c/launch_rules.cpp,
compiled against the library's own header; nothing is launched)."""

import os
import random
import subprocess

import pytest

from paper_1405_6162_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.run([build.hipcc(), "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-x", "hip",
                    os.path.join(ROOT, "tests", "c", "launch_rules.cpp"), "-o", out], check=True,
                   capture_output=True, text=True)

    def call(lines, timeout=60):
        res = subprocess.run([out], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True,
                             timeout=timeout)
        return res.stdout.split("\n")[:len(lines)]
    return call


def test_chunks_are_the_best_of_all_counts(ask):
    """The chunk count is the one that trying every count gives."""
    rng = random.Random(3)
    cases = [(c, n, s) for c in (1, 2, 3, 31, 32, 255, 256, 257, 512, 4000) for n in (1, 2, 3, 127, 128, 129, 257)
             for s in (256, 512, 1024)]
    cases += [(int(2 ** rng.uniform(0, 12)), int(2 ** rng.uniform(0, 14)), rng.choice((256, 512, 1024)))
              for _ in range(1500)]
    got = ask(["chunks %d %d %d" % c for c in cases])
    assert got == ask(["tried %d %d %d" % c for c in cases])


def test_chunks_of_a_long_lattice_take_no_time(ask):
    """The count is looked for at every launch: 300 launches on lattices of up
    to 5e8 planes within 10 s (trying every count takes about 1 s each)."""
    ask(["chunks %d %d 256" % (1 + k % 3, 500000000 // (1 + k % 7)) for k in range(300)], timeout=10)


F64, F32, F16 = 0, 1, 2


@pytest.mark.parametrize("storage,vvl,shape,march", [
    # small FP64 lattices take the two-pass step, others march
    (F64, 0, (56, 56, 56), 0), (F64, 1, (64, 64, 64), 1), (F64, 0, (256, 256, 256), 1), (F64, 0, (512, 512, 1), 1),
    (F32, 0, (8, 8, 8), 1), (F16, 0, (24, 24, 24), 1), (F16, 0, (384, 384, 384), 1),
    # few rows: the two-pass step in FP64, and beyond the cache in the others
    (F64, 0, (700, 3, 300), 0), (F64, 0, (700, 5, 200), 0), (F64, 0, (2048, 1, 256), 0), (F64, 0, (700, 6, 200), 1),
    (F32, 0, (700, 3, 300), 1), (F32, 0, (4, 4, 16384), 0), (F16, 0, (2, 2, 4000000), 0), (F32, 0, (4, 6, 16384), 1),
    # more than one site per lane: from 256 blocks of at most 16 planes
    (F64, 2, (512, 512, 4), 1), (F32, 4, (512, 512, 4), 1), (F64, 4, (64, 64, 64), 0), (F16, 2, (112, 112, 112), 0),
    (F32, 2, (128, 128, 128), 1), (F64, 2, (2048, 1, 256), 1)])
def test_binary_step_taken(ask, storage, vvl, shape, march):
    assert ask(["march %d 0 %d %d %d %d" % ((storage, vvl) + shape)]) == [str(march)]


BGK, TRT, MRT = 0, 1, 2


@pytest.mark.parametrize("storage,coll,shape,pair", [
    # few planes: a pair's chunks lead in and out over more than they keep
    (F64, BGK, (2048, 2048, 1), 0), (F64, BGK, (2048, 2048, 2), 1), (F64, MRT, (2048, 2048, 1), 0),
    (F64, MRT, (2048, 2048, 2), 1), (F32, BGK, (2048, 2048, 1), 1), (F32, TRT, (2048, 2048, 1), 0),
    (F32, MRT, (2048, 2048, 1), 0), (F16, BGK, (2048, 2048, 4), 0), (F16, BGK, (1024, 1024, 8), 1),
    (F16, TRT, (1024, 1024, 8), 0), (F64, BGK, (512, 512, 1), 0), (F64, TRT, (1024, 512, 1), 0),
    # few rows, and rows shorter than a wavefront
    (F64, BGK, (2048, 1, 256), 0), (F64, BGK, (2048, 2, 256), 0), (F64, BGK, (2048, 3, 256), 1),
    (F64, MRT, (2048, 3, 256), 0), (F64, BGK, (64, 2, 2000), 0), (F64, BGK, (64, 3, 2000), 1),
    (F32, BGK, (300, 2, 400), 0), (F64, BGK, (4, 4, 16384), 0), (F64, BGK, (4, 8, 16384), 1),
    (F64, BGK, (2, 2, 50000), 0), (F32, BGK, (2, 2, 4000000), 0), (F64, BGK, (16, 16, 2048), 1),
    (F32, TRT, (4, 8, 16384), 1), (F32, BGK, (60, 2, 40000), 1), (F64, MRT, (65, 130, 70), 1),
    # in the cache, all blocks at once
    (F64, BGK, (64, 8, 255), 1), (F64, TRT, (256, 256, 2), 0), (F64, TRT, (64, 64, 64), 1),
    (F64, MRT, (64, 64, 32), 0), (F64, MRT, (64, 64, 64), 0), (F64, MRT, (128, 128, 32), 1),
    (F32, TRT, (80, 80, 80), 0), (F32, TRT, (88, 88, 88), 1), (F32, MRT, (64, 64, 64), 0), (F32, MRT, (104, 104, 104), 0),
    # the cubes
    (F64, BGK, (48, 48, 48), 0), (F64, BGK, (256, 256, 256), 1), (F64, MRT, (256, 256, 256), 1),
    (F32, MRT, (128, 128, 128), 1), (F32, MRT, (150, 70, 90), 1), (F16, BGK, (128, 128, 128), 1),
    (F16, TRT, (128, 128, 128), 0), (F16, TRT, (256, 256, 256), 1), (F16, MRT, (256, 256, 256), 0),
    (F16, BGK, (200, 204, 100), 0)])
def test_pairs_taken(ask, storage, coll, shape, pair):
    assert ask(["pair %d %d 0 %d %d %d" % ((storage, coll) + shape)]) == [str(pair)]


def test_no_pairs_with_more_than_one_site_per_lane(ask):
    assert ask(["pair 0 0 2 256 256 256"]) == ["0"]


SINGLE, BINARY = 0, 1


@pytest.mark.parametrize("model,storage,vvl,shape,layout", [
    # below 4 GiB a buffer: blocked (FP32, addressed by element, below 2^32 values)
    (BINARY, F64, 0, (256, 256, 256), "1 0 0"), (BINARY, F32, 0, (384, 384, 384), "1 0 0"),
    (SINGLE, F16, 4, (100, 90, 77), "1 0 0"),
    # from 4 GiB: blocked with wide offsets where that needs no more room, which the workspace size (that of the
    # structure of arrays) does not show; else the structure of arrays
    (BINARY, F64, 0, (320, 320, 320), "1 1 0"), (SINGLE, F64, 1, (320, 320, 320), "1 1 0"),
    (BINARY, F64, 2, (320, 320, 320), "0 0 0"), (BINARY, F64, 0, (330, 300, 310), "0 0 0"),
    (BINARY, F16, 0, (512, 512, 440), "1 1 0"), (BINARY, F16, 0, (500, 500, 460), "0 0 0"),
    (BINARY, F32, 0, (640, 640, 560), "0 0 0"),
    # planes of 4 GiB
    (BINARY, F32, 0, (8192, 8192, 1), "1 0 1"), (BINARY, F32, 4, (8192, 8192, 3), "1 0 1"),
    (SINGLE, F32, 0, (8192, 8192, 1), "0 0 0"), (BINARY, F32, 0, (8192, 8192, 4), "0 0 0"),
    (BINARY, F64, 0, (8192, 8192, 1), "0 0 0")])
def test_state_layout(ask, model, storage, vvl, shape, layout):
    assert ask(["layout %d %d 0 %d %d %d %d" % ((model, storage, vvl) + shape)]) == [layout]
