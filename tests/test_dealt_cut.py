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


# below one whole round on 8 waves, by the tiles left over: a piece is 3/7 and
# 4/7 of a tile (to 64 elements); then 2, 4, 8 and 16 whole rounds and four tiles
LEFT = (3, 4, 20, 36, 68, 132)
BURST, CACHED, PIECEWISE, ANY = (3, 4, 20, 36, 68, 132), (3, 4, 36, 68, 132), (3, 132), (3, 68, 132)


@pytest.mark.gpu
@pytest.mark.parametrize("n,opt,kw,cut", [
    (8, None, {}, BURST), (6, "sgd", {}, BURST), (14, "adam", {}, BURST), (32, None, {}, BURST),
    (1, "adam", {}, PIECEWISE), (4, None, {}, PIECEWISE), (8, "adam", {}, PIECEWISE),
    (8, "adam", {"resident_bytes": 0}, (3, 20, 36, 68, 132)),
    (17, None, {"resident_bytes": 0}, ANY), (21, "adam", {"resident_bytes": 0}, ANY),
    (8, None, {"resident_bytes": 1 << 28}, CACHED), (8, None, {"unfused": True}, PIECEWISE)])
def test_segments_of_jobs(n, opt, kw, cut):
    from paper_1805_07891_amd.job import TorchJob
    print("segments", n, opt, kw, flush=True)
    for tiles in LEFT:
        job = TorchJob(Job("cut", n, (tiles * 1024 + 3,)), "cuda:0", workgroups=2, optimizer=opt, **kw)
        assert (job.info()[2] > tiles + 1) == (tiles in cut), tiles
        job.destroy()
