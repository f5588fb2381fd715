"""Which kernel runs a step without a fixed-N kernel (CPU): the choice on the
host, natively, and that builds whose load window leaves a worker count
without a fixed-N kernel still hold one that takes it."""

import os
import re
import subprocess

from paper_1805_07891_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_choice_on_the_host(tmp_path):
    exe = tmp_path / "check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           f"-I{build.CSRC}",
                           os.path.join(HERE, "native", "any_kernel_check.cpp"),
                           os.path.join(build.CSRC, "plan.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr


def test_the_shared_stash_leaves_room_for_a_second_launch(tmp_path):
    asm = open(build.device_assembly(str(tmp_path / "shared.s"), "fused_many_shared.hip")).read()
    blocks = asm.split("  - .agpr_count:")[1:]
    assert len(blocks) == 4
    for block in blocks:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        opt = int(re.search(r"fused_step_many_sharedILi(\d)E", name).group(1))

        def field(key):
            return int(re.search(rf"\.{key}:\s+(\d+)", block).group(1))

        states = {0: 2, 1: 2, 2: 1, 3: 3}[opt]
        lds = field("group_segment_fixed_size")
        assert lds == 4 * (4 // states) * states * 4096 <= 80 * 1024
        # the registers that the launch claims leave room for as many waves
        claimed = re.search(rf"\.amdhsa_kernel {name}\n(?:.*\n)*?.*\.amdhsa_next_free_vgpr (\d+)", asm)
        assert 512 // (-(-int(claimed.group(1)) // 8) * 8) >= 160 * 1024 // lds
        assert field("private_segment_fixed_size") == 0 and field("vgpr_spill_count") == 0


def test_a_window_without_fixed_kernels_keeps_one_for_few_workers(tmp_path):
    """A ring of 7 loads takes seven phases for most worker counts (plain SGD
    here): those run the batched any-N kernel, which takes every count."""
    asm = open(build.device_assembly(str(tmp_path / "ring7.s"),
                                     defines=["PHUB_LOADS_AHEAD=6", "PHUB_STEP_PART=4"])).read()
    names = re.findall(r"^\s+\.name:\s+(\S+)", asm, re.M)
    fixed = {int(m.group(1)) for m in (re.search(r"fused_step_fixedILi(\d+)ELi2ELb0E", n) for n in names) if m}
    assert {n for n in range(1, 17) if 4 * (n + 1) % 7 == 0} <= fixed and not fixed & {1, 2, 3, 4, 5}
    assert any("fused_step_anyILi2ELb0E" in n for n in names)
