"""What the persistent launches' grid rests on, from the compiled code objects'
metadata: every instance of the batched kernel, the mixed one of serving steps
among them, has at most 128 VGPRs without spilling (four workgroups of four waves per
compute unit), its static LDS stays within what the launch reckons with, and the
instances of 32-slot stacks fit four times into a compute unit's 160 KB.  No GPU."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1312_3691_amd", "csrc")


@pytest.fixture(scope="module")
def instances(tmp_path_factory):
    """(stack slots, mode) -> metadata of batch_kernel's instances."""
    from paper_1312_3691_amd import build as B
    if not os.path.exists("/opt/rocm/bin/hipcc") and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("limits") / "k.s")
    cmd = B.compile_command(os.path.join(CSRC, "tpmc_kernels.hip"), out)
    cmd[cmd.index("-c")] = "-S"
    subprocess.run(cmd[:1] + ["--cuda-device-only"] + cmd[1:], check=True, capture_output=True)
    meta = {}
    # one list item per kernel; its fields are in alphabetical order, some before the name
    for item in re.split(r"\n  - (?=\.)", open(out).read().split("amdhsa.kernels:", 1)[1])[1:]:
        m = re.search(r"\.name:\s+\S*batch_kernelILi(\d+)ELN\S*?(\d)E|\.name:\s+\S*batch_kernelILi(\d+)ELi(\d+)E", item)
        if m:
            key = tuple(int(v) for v in m.groups() if v is not None)
            meta[key] = {k: int(re.search(r"\." + k + r":\s+(\d+)", item).group(1))
                         for k in ("vgpr_count", "vgpr_spill_count", "group_segment_fixed_size")}
    assert len(meta) == 25, sorted(meta)
    return meta


def _constant(name):
    text = open(os.path.join(CSRC, "tpmc_launch.h")).read()
    return int(re.search(name + r" = (\d+)", text).group(1))


def test_every_instance_leaves_four_waves_per_simd(instances):
    for k, v in instances.items():
        assert v["vgpr_count"] <= 128 and v["vgpr_spill_count"] == 0, (k, v)


def test_static_lds_is_what_the_launch_reckons_with(instances):
    for (stack, mode), v in instances.items():
        beside = v["group_segment_fixed_size"] - stack * 256 * 4
        bound = _constant("kBatchLdsPrecull" if stack <= 32 else "kBatchLds")
        assert 0 < beside <= bound, (stack, mode, v, bound)


def test_lds_of_four_workgroups(instances):
    totals = 7 * 4 * 8
    dynamic = {(4, 2): 2 * 7 * 256 * 8, (16, 1): 256 * 7 * 8, (32, 0): 0, (32, 3): totals, (32, 4): totals}
    for key, dyn in dynamic.items():
        assert instances[key]["group_segment_fixed_size"] + dyn <= 160 * 1024 // 4, (key, instances[key])
