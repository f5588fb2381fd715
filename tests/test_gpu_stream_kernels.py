"""GPU parity of every stream-walk kernel of a fixed worker count (all of
kStreamBlock's counts and optimizers, and 20, 24 and 32 workers), on a grid
small enough that a wave walks many tiles, nothing cached and with a budget
cut inside a key; and of the fixed-N kernels' own bursts at the few tiles a
wave where they still run.  Bit-exact against the CPU oracle over two steps."""

import os
import re

import numpy as np
import pytest

import oracle
from paper_1805_07891_amd.build import CSRC
from paper_1805_07891_amd.job import TorchJob
from paper_1805_07891_amd.workloads import Job, key_offsets

# 126 full tiles and ragged ends: 31 tiles a wave on one workgroup
KEYS = (5, 1024 * 37 + 3, 70001, 1024 * 11, 4097, 1, 1024 * 6)
LR, MU, WD, B1, B2, EPS = 0.05, 0.9, 1e-3, 0.9, 0.999, 1e-8


def _stream_kernels():
    """(workers, optimizer) of every stream kernel, read from the table."""
    text = open(os.path.join(CSRC, "kernels.hpp")).read()
    table = text[text.index("kStreamBlock[3]"):]
    rows = re.findall(r"\{([\d, ]+)\},", table[:table.index("};")])
    blocks = [[int(x) for x in row.split(",")] for row in rows]
    assert [len(b) for b in blocks] == [16, 16, 16]
    kernels = []
    for opt, states in (("sgd", 1), ("momentum", 2), ("nesterov", 2), ("adam", 3)):
        counts = [n for n in range(1, 17) if blocks[states - 1][n - 1]] + [20, 24, 32]
        kernels += [(n, opt) for n in counts]
    return kernels


BURSTS = [(n, opt) for opt, least in (("sgd", 6), ("momentum", 6), ("nesterov", 6), ("adam", 14))
          for n in [*range(least, 17), 20, 24, 32]]


def test_the_table_names_every_compiled_kernel():
    assert len(_stream_kernels()) == 41


def _run(n, opt, workgroups, resident):
    import torch
    states = {"sgd": 1, "adam": 3}.get(opt, 2)
    print("stream kernel", n, opt, workgroups, resident, flush=True)
    spec = Job("stream", n, KEYS, lr=LR, momentum=MU, weight_decay=WD, nesterov=opt == "nesterov")
    job = TorchJob(spec, "cuda:0", resident_bytes=4 * states * resident, workgroups=workgroups,
                   optimizer={"momentum": None, "nesterov": None}.get(opt, opt), betas=(B1, B2), eps=EPS)
    offs, total = key_offsets(KEYS)
    rng = np.random.default_rng(100 * n + states)
    w0 = rng.standard_normal(total, dtype=np.float32) * np.float32(0.05)
    job.set_weights(torch.from_numpy(w0).cuda())
    W = [w0[o:o + m].copy() for o, m in zip(offs, KEYS)]
    M, V = ([np.zeros(m, np.float32) for m in KEYS] for _ in range(2))
    for t in range(2):
        host = [rng.random(total, dtype=np.float32) - np.float32(0.5) for _ in range(n)]
        dev = [torch.from_numpy(h).cuda() for h in host]
        for w, d in enumerate(dev):
            job.attach_grads(w, d)
        torch.cuda.synchronize()
        job.push_and_step()
        g = [[h[o:o + m] for o, m in zip(offs, KEYS)] for h in host]
        if opt == "sgd":
            oracle.step_sgd(g, W, LR, WD)
        elif opt == "adam":
            oracle.step_adam(g, W, M, V, LR, B1, B2, EPS, WD, t + 1)
        else:
            oracle.step(g, W, M, LR, MU, WD, opt == "nesterov")
        Wg, Mg = job.state_arenas()
        Vg = job.second_moment_arena()
        for k, (o, m) in enumerate(zip(offs, KEYS)):
            assert np.array_equal(Wg[o:o + m].view(np.uint32), W[k].view(np.uint32)), (t, k)
            if opt != "sgd":
                assert np.array_equal(Mg[o:o + m].view(np.uint32), M[k].view(np.uint32)), (t, k)
            if opt == "adam":
                assert np.array_equal(Vg[o:o + m].view(np.uint32), V[k].view(np.uint32)), (t, k)
    job.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("n,opt", _stream_kernels())
@pytest.mark.parametrize("resident", [0, 50000])
def test_stream_kernels(n, opt, resident):
    _run(n, opt, 1, resident)


@pytest.mark.gpu
@pytest.mark.parametrize("n,opt", BURSTS)
def test_bursts_over_few_tiles(n, opt):
    # 3.2 tiles a wave on average, Adam 1.97: below kStreamMinTiles
    _run(n, opt, 16 if opt == "adam" else 10, 0)
