"""GPU parity of the any-N kernels on the device's whole grid with two and more
full tiles a wave: the stream walk at every filling of its last block of
loads, every optimizer, state streamed and partly cached, and a key beyond
the 2^20 float4 that are folded into the gradients' bases (a wave walks tiles
on both sides of the fold, then another key's); cached state up to three
tiles a wave (the shared stash) and beyond (batches); bit-exact against the
CPU oracle."""

import numpy as np
import pytest

import oracle
from paper_1805_07891_amd.job import TorchJob
from paper_1805_07891_amd.workloads import Job, key_offsets

pytestmark = pytest.mark.gpu

KEYS = (5, 1024 * 1024 * 2 + 3, 0, 700001, 1024 * 500, 4097, 1)
MID = (1024 * 1024 * 2 + 3, 300001, 0, 5)
FOLD = (4300003, 1300001, 5, 0, 1023)


@pytest.mark.parametrize("n,opt,keys,resident", [
    (17, "nesterov", FOLD, 0), (17, "adam", FOLD, 0), (23, "sgd", FOLD, 0), (18, "momentum", KEYS, 0),
    (19, "nesterov", KEYS, 0), (21, "nesterov", KEYS, None), (22, "sgd", KEYS, None),
    (25, "adam", KEYS, 0), (17, "momentum", FOLD, 8 * 1000000), (33, "adam", KEYS, 12 * 1000000),
    (40, "nesterov", KEYS, None), (65, "momentum", KEYS, None),
    (17, "momentum", MID, 1 << 28), (22, "sgd", MID, 1 << 28), (33, "adam", MID, 1 << 28),
    (19, "nesterov", KEYS, 1 << 28), (25, "adam", KEYS, 1 << 28), (17, "sgd", FOLD, 1 << 28)])
def test_whole_grid(n, opt, keys, resident):
    import torch
    print("stream", n, opt, sum(keys), resident, flush=True)
    spec = Job("stream", n, keys, lr=0.05, weight_decay=1e-3, nesterov=opt == "nesterov")
    job = TorchJob(spec, "cuda:0", resident_bytes=resident,
                   optimizer={"momentum": None, "nesterov": None}.get(opt, opt))
    offs, total = key_offsets(keys)
    rng = np.random.default_rng(n)
    host = [(rng.random(total, dtype=np.float32) - np.float32(0.5)) for _ in range(n)]
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
        oracle.step(g, W, M, spec.lr, spec.momentum, spec.weight_decay, opt == "nesterov")
    Wg, Mg = job.state_arenas()
    Vg = job.second_moment_arena()
    for k, (o, m) in enumerate(zip(offs, keys)):
        assert np.array_equal(Wg[o:o + m].view(np.uint32), W[k].view(np.uint32)), f"W key {k}"
        if opt != "sgd":
            assert np.array_equal(Mg[o:o + m].view(np.uint32), M[k].view(np.uint32)), f"M key {k}"
        if opt == "adam":
            assert np.array_equal(Vg[o:o + m].view(np.uint32), V[k].view(np.uint32)), f"V key {k}"
    job.destroy()
