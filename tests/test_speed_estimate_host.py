"""The seeding estimate's normal speed (speed_estimate32, csrc/tpmc_math.hpp), built
for the host: wherever it does not give up, its error stays below 1e-4, for s over
the whole range of its table and draws from the middle to both ends; it gives up
for few draws where particles are.  The bound is that of its comment: F rounded by
up to 1e-6 of max(chi, exp(-s^2)), F' at least a hundredth of that.  No GPU."""
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1312_3691_amd", "csrc")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("speed") / "harness")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I", CSRC,
                    os.path.join(ROOT, "tests", "speed_estimate_harness.cpp"), "-o", exe],
                   check=True, capture_output=True)
    return exe


def test_speed_error_is_bounded_where_the_estimate_is_kept(harness):
    rng = random.Random(11)
    rows = []
    for s in [-4.0, -3.97, -3.5, -3.0, -2.53, -2.0, -1.5, -1.0, -0.5, -0.2, 0.0, 0.3, 1.0, 2.5, 5.0, 9.0, 9.99]:
        s = float(np.float32(s))
        ks = [rng.getrandbits(32) for _ in range(600)]
        for _ in range(300):  # towards both ends
            k = int(2.0 ** rng.uniform(0, 32)) - 1
            ks += [k, 2 ** 32 - 1 - k]
        rows += [(s, k) for k in ks]
    out = subprocess.run([harness], input="\n".join("%s %d" % (s.hex(), k) for s, k in rows), capture_output=True,
                         text=True, check=True).stdout.split("\n")[:-1]
    assert len(out) == len(rows)
    worst, kept = {}, {}
    for i, ((s, k), line) in enumerate(zip(rows, out)):
        keep, err = line.split()
        if keep == "1":
            worst[s] = max(worst.get(s, 0.0), float(err))
        if i % 1200 < 600:  # the uniform draws
            kept[s] = kept.get(s, 0) + int(keep)
    print(worst)
    assert max(worst.values()) <= 1e-4, worst
    assert all(n >= 0.95 * 600 for s, n in kept.items()), kept
