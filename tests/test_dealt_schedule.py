"""The schedule phub_init deals for the LPT option (CPU: coverage, order and
balance of every plan, natively; GPU: jobs around one tile per wave, where
leftover tiles are cut into pieces, against the oracle bit for bit)."""

import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_1805_07891_amd.build import CSRC
from paper_1805_07891_amd.workloads import Job, key_offsets

HERE = os.path.dirname(os.path.abspath(__file__))


def test_dealt_plans(tmp_path):
    exe = tmp_path / "check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", f"-I{CSRC}",
                           os.path.join(HERE, "native", "dealt_check.cpp"),
                           os.path.join(CSRC, "plan.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=600)
    assert out.returncode == 0, out.stderr
    assert int(out.stdout.split()[0]) == 157 * 5


@pytest.mark.gpu
@pytest.mark.parametrize("n,opt,tiles,resident", [
    # on 8 waves: no whole round, one leftover tile (cut to 256 elements),
    # pieces of 320 and 640, too many leftover tiles to cut, two bins' state;
    # above one round 2 to 4 workers and any-N jobs leave theirs whole
    (8, None, 1, 0), (2, None, 9, 0), (8, None, 10, 0), (3, "adam", 13, 0), (16, "sgd", 15, 0),
    (4, None, 29, 8 * 9000), (20, None, 9, 0), (24, "adam", 11, 0), (33, None, 10, 0),
    (17, "sgd", 5, 4 * 3000)])
def test_leftover_tiles(n, opt, tiles, resident):
    import torch
    from paper_1805_07891_amd.job import TorchJob
    print("leftover", n, opt, tiles, resident, flush=True)
    for keys in ((tiles * 1024,), (1024 * (tiles - tiles // 2), 1024 * (tiles // 2), 5),
                 (tiles * 1024 + 1, 77, 3, 300)):
        spec = Job("left", n, keys, lr=0.05)
        job = TorchJob(spec, "cuda:0", workgroups=2, optimizer=opt, resident_bytes=resident)
        offs, total = key_offsets(keys)
        rng = np.random.default_rng(n + tiles)
        host = [rng.standard_normal(total, dtype=np.float32) * np.float32(1e-2) for _ in range(n)]
        w0 = rng.standard_normal(total, dtype=np.float32) * np.float32(0.05)
        job.set_weights(torch.from_numpy(w0).cuda())
        dev = [torch.from_numpy(h).cuda() for h in host]
        for w, d in enumerate(dev):
            job.attach_grads(w, d)
        torch.cuda.synchronize()
        job.push_and_step()
        g = [[h[o:o + m] for o, m in zip(offs, keys)] for h in host]
        W = [w0[o:o + m].copy() for o, m in zip(offs, keys)]
        M, V = ([np.zeros(m, np.float32) for m in keys] for _ in range(2))
        if opt == "sgd":
            oracle.step_sgd(g, W, spec.lr, spec.weight_decay)
        elif opt == "adam":
            oracle.step_adam(g, W, M, V, spec.lr, 0.9, 0.999, 1e-8, spec.weight_decay, 1)
        else:
            oracle.step(g, W, M, spec.lr, spec.momentum, spec.weight_decay, True)
        Wg, Mg = job.state_arenas()
        for k, (o, m) in enumerate(zip(offs, keys)):
            assert np.array_equal(Wg[o:o + m].view(np.uint32), W[k].view(np.uint32)), (keys, k)
            if opt != "sgd":
                assert np.array_equal(Mg[o:o + m].view(np.uint32), M[k].view(np.uint32)), (keys, k)
        job.destroy()
