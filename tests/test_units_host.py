"""The persistent kernel's cut of a work entry into units (csrc/tpmc_units.hpp),
built for the host: over sizes at the edges of batches, shares and caps, part
counts and grids, the units cover every particle exactly once.  No GPU."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1312_3691_amd", "csrc")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("units") / "harness")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I", CSRC,
                    os.path.join(ROOT, "tests", "units_harness.cpp"), "-o", exe], check=True, capture_output=True)
    return exe


def test_units_cover_every_particle_once(harness):
    rng = random.Random(3)
    sizes = [1, 63, 64, 65, 127, 128, 129, 1000, 4096, 16384, 16385, 100_000, 262_143, 262_144, 262_145, 1_000_003]
    lines = []
    for n in sizes + [int(10 ** rng.uniform(0, 8)) for _ in range(200)] + [3_000_000_019]:
        for sub, grid in ((0, 1), (0, 1024), (4, 1024), (4, 7), (3, 391), (0, 0), (4, 0), (2, 3)):
            waves = max(1, grid * 4)
            share = 6
            while waves << (share + 1) <= n:
                share += 1
            for share_used in {share, max(6, share - 2), share + 3}:
                cap = rng.randint(0, 8) if n < 10_000_000 else rng.randint(5, 8)
                lines.append((64 * rng.randint(0, 1000), n, sub, grid, share_used, cap))
    out = subprocess.run([harness], input="\n".join(" ".join(map(str, ln)) for ln in lines), check=True,
                         capture_output=True, text=True).stdout.splitlines()
    assert len(out) == len(lines)
    bad = [(ln, o) for ln, o in zip(lines, out) if o != "ok"]
    assert not bad, bad[:5]
