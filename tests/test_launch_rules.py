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
