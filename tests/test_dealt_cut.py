"""Which jobs cut the tiles left over from the last whole round of their
schedule (CPU: the rule and the plans, natively; GPU: the segments of jobs on
either side of it)."""

import os
import subprocess

import pytest

from paper_1805_07891_amd.build import CSRC
from paper_1805_07891_amd.workloads import Job

HERE = os.path.dirname(os.path.abspath(__file__))


def test_rule_and_plans(tmp_path):
    exe = tmp_path / "check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           f"-I{CSRC}", os.path.join(HERE, "native", "dealt_cut_check.cpp"),
                           os.path.join(CSRC, "plan.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("n,opt,kw,rounds", [
    (8, None, {}, 0), (6, "sgd", {}, 0), (14, "adam", {}, 0), (32, None, {}, 0),
    (1, "adam", {}, None), (4, None, {}, None), (8, "adam", {}, None),
    (17, None, {"resident_bytes": 0}, 8), (21, "adam", {"resident_bytes": 0}, 8),
    (8, None, {"resident_bytes": 1 << 28}, None), (8, None, {"unfused": True}, None)])
def test_segments_of_jobs(n, opt, kw, rounds):
    from paper_1805_07891_amd.job import TorchJob
    print("segments", n, opt, kw, flush=True)
    for tiles in (4, 20, 68):  # on 8 waves: none, two and eight whole rounds, four tiles left over
        job = TorchJob(Job("cut", n, (tiles * 1024 + 3,)), "cuda:0", workgroups=2, optimizer=opt, **kw)
        assert (job.info()[2] > tiles + 1) == (rounds is not None and tiles // 8 >= rounds), tiles
        job.destroy()
