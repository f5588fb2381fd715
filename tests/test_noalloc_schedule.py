"""The schedule that phub_step_noalloc builds on the device: its size limit is
the host-built schedule's (CPU), and every shape it can take gives the
oracle's bits (GPU): fewer tiles than waves, exact multiples, more
remainders than waves, more keys than its LDS copy holds, tables too large
for kernel arguments, empty keys, several calls in a row without a wait."""

import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_1805_07891_amd import phub
from paper_1805_07891_amd.build import CSRC
from paper_1805_07891_amd.workloads import key_offsets

HERE = os.path.dirname(os.path.abspath(__file__))


def test_lpt_counts_match_the_schedule(tmp_path):
    exe = tmp_path / "check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", f"-I{CSRC}",
                           os.path.join(HERE, "native", "lpt_counts_check.cpp"),
                           os.path.join(CSRC, "plan.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    assert int(out.stdout.split()[0]) == 306 * 6 * 4


def _bits(a):
    return np.ascontiguousarray(a, np.float32).view(np.uint32)


def _sizes(count, most, seed):
    return tuple(int(n) for n in np.random.default_rng(seed).integers(0, most, count))


@pytest.mark.gpu
@pytest.mark.parametrize("n,keys,chunk", [
    (1, (3,), 32768), (2, (1024,), 32768), (3, (0, 1023, 0, 1025, 0), 16),
    (8, (1024 * 1024,), 32768),                    # one tile a wave, no remainder
    (8, (1024 * 1024 + 1024, 7), 4096),            # one wave with two tiles
    (4, (1024 * 1023, 5, 6), 32768),               # the remainders' first wave is the last
    (2, _sizes(1500, 60, 1), 32768),               # more remainders than waves
    (1, _sizes(2500, 3000, 2), 32768),             # more keys than the LDS copy
    (16, _sizes(700, 2000, 3), 32768),             # more words than the arguments take
    (17, _sizes(90, 5000, 4), 32768), (40, (5, 70001, 0, 12), 32768)])
def test_noalloc_matches_the_oracle(n, keys, chunk):
    import torch
    from paper_1805_07891_amd.job import load_library
    lib = load_library()
    print("noalloc", n, len(keys), sum(keys), flush=True)
    sys.stdout.flush()
    offs, total = key_offsets(keys)
    rng = np.random.default_rng(len(keys) + n)
    host = [rng.standard_normal(max(total, 1), dtype=np.float32) * np.float32(1e-2) for _ in range(n)]
    w0 = rng.standard_normal(max(total, 1), dtype=np.float32) * np.float32(0.05)
    dev = [torch.from_numpy(h).cuda() for h in host]
    W = torch.from_numpy(w0).cuda()
    M = torch.full_like(W, 7.0)
    for o, m in zip(offs, keys):
        M[o:o + m] = 0
    ptrs = phub.pointer_array([d.data_ptr() + 4 * o for d in dev for o in offs])
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(3):  # nothing waits between the calls
        lib.phub_step_noalloc(n, keys, chunk, 0.05, 0.9, 1e-3, True, ptrs, W.data_ptr(),
                              M.data_ptr(), st.cuda_stream)
    torch.cuda.synchronize()
    Wo = [w0[o:o + m].copy() for o, m in zip(offs, keys)]
    Mo = [np.zeros(m, np.float32) for m in keys]
    g = [[h[o:o + m] for o, m in zip(offs, keys)] for h in host]
    for _ in range(3):
        oracle.step(g, Wo, Mo, 0.05, 0.9, 1e-3, True)
    wantW, wantM = w0.copy(), np.full_like(w0, 7.0)  # the padding keeps its values
    for k, (o, m) in enumerate(zip(offs, keys)):
        wantW[o:o + m], wantM[o:o + m] = Wo[k], Mo[k]
    assert np.array_equal(_bits(W.cpu().numpy()), _bits(wantW))
    assert np.array_equal(_bits(M.cpu().numpy()), _bits(wantM))


@pytest.mark.gpu
def test_noalloc_is_refused_under_capture():
    import torch
    from paper_1805_07891_amd.job import load_library
    lib = load_library()
    g, W, M = (torch.zeros(64, device="cuda") for _ in range(3))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rc = lib.phub_step_noalloc(1, (64,), 32768, 0.05, 0.9, 1e-3, True, [g.data_ptr()],
                                   W.data_ptr(), M.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream, check=False)
        W.add_(1.0)
    assert rc == phub.PHUB_EHIP and "captured" in lib.last_error()
    graph.replay()
    torch.cuda.synchronize()
    assert float(W[0]) == 1.0
