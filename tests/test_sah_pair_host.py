"""The plane of a node of two triangles in the SAH build's wave stage
(csrc/tpmc_sah.hpp), built for the host: over centres that coincide, are equal on
some axes, next to each other, denormally close, or further apart than FP32 can
hold, the plane is the lowest one with a triangle on either side (every such plane
of a pair costs the same), and where there is none the range is halved.  No GPU."""
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1312_3691_amd", "csrc")
BINS, MAX_LEVEL = 32, 32


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("sah") / "harness")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I", CSRC,
                    os.path.join(ROOT, "tests", "sah_harness.cpp"), "-o", exe], check=True, capture_output=True)
    return exe


def _lowest_plane(level, a, b):
    """(plane or -1, triangles on its left) by trying every plane of every axis."""
    with np.errstate(all="ignore"):
        for k in range(3):
            lo, hi = min(a[k], b[k]), max(a[k], b[k])
            ext = np.float32(hi) - np.float32(lo)
            scale = np.float32(BINS) / ext
            if not (level < MAX_LEVEL and ext > 0 and scale < np.inf):
                continue
            at = [(np.float32(c) - np.float32(lo)) * scale for c in (a[k], b[k])]
            bins = [0 if np.isnan(v) else min(BINS - 1, int(v)) for v in at]  # an infinite extent: scale 0
            for plane in range(1, BINS):
                left = sum(x < plane for x in bins)
                if left == 1:
                    return k * BINS + plane, 1
    return -1, 1


def test_pair_is_always_split_in_two(harness):
    rng = random.Random(5)
    big = float(np.finfo(np.float32).max)
    values = [0.0, 1.0, -1.0, 1e-30, 1e-42, 0.75 * big, -0.75 * big, big, -big, 0.4 * big, float(np.float32(0.1))]
    pairs = [(0, (0.75 * big, 0.0, 0.0), (-0.75 * big, 1.0, 0.0)),  # wider than FP32 on the first axis
             (0, (0.75 * big, 0.75 * big, 0.75 * big), (-0.75 * big, -0.75 * big, -0.75 * big)),  # on every axis
             (0, (1.0, 2.0, 3.0), (1.0, 2.0, 3.0)), (32, (0.0, 0.0, 0.0), (1.0, 0.0, 0.0))]
    for _ in range(3000):
        pick = lambda: rng.choice(values) if rng.random() < 0.6 else rng.uniform(-2.0, 2.0)
        a = [pick() for _ in range(3)]
        b = [x if rng.random() < 0.3 else float(np.nextafter(np.float32(x), np.float32(3))) if rng.random() < 0.2
             else pick() for x in a]
        pairs.append((rng.choice((0, 1, 31, 32, 40)), a, b))
    pairs = [(lv, np.float32(a), np.float32(b)) for lv, a, b in pairs]
    lines = [" ".join([str(lv)] + [float(x).hex() for x in (*a, *b)]) for lv, a, b in pairs]
    out = subprocess.run([harness], input="\n".join(lines), check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(out) == len(pairs)
    for (lv, a, b), o in zip(pairs, out):
        assert tuple(map(int, o.split())) == _lowest_plane(lv, a, b), (lv, a, b, o)
