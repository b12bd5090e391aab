"""How the workgroups of a persistent launch start (csrc/tpmc_units.hpp), built for
the host: every part has its own workgroups, also where there are more parts than
workgroups (left without, all waves of a launch went for the same part), and the
units of a part cover it with any bound on its starting units.  No GPU."""
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
    exe = str(tmp_path_factory.mktemp("start") / "harness")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I", CSRC,
                    os.path.join(ROOT, "tests", "start_harness.cpp"), "-o", exe], check=True, capture_output=True)
    return exe


def test_every_part_has_its_own_workgroups(harness):
    rng = random.Random(2)
    lines = [(g, p) for g in (1, 2, 3, 79, 256, 1023, 1024) for p in (1, 2, 16, 60, 200, 1023, 1024, 1025, 1500, 20_000)]
    lines += [(rng.randint(1, 1024), rng.randint(1, 5000)) for _ in range(300)] + [(1024, 1_000_003)]
    lines = [ln + (int(10 ** rng.uniform(0, 6.5)), rng.randint(6, 20), rng.randint(0, 8), rng.randint(0, 10)) for ln in lines]
    out = subprocess.run([harness], input="\n".join(" ".join(map(str, ln)) for ln in lines), check=True, capture_output=True,
                         text=True).stdout.splitlines()
    assert len(out) == len(lines)
    bad = [(ln, o) for ln, o in zip(lines, out) if o != "ok"]
    assert not bad, bad[:5]
