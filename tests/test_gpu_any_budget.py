"""The default cache budget of jobs without a fixed-N kernel: their pushpull
steps cache the state, so they take their share of the budget whatever their
size, also where their other steps stream all of it; both kinds of step in
turn over one job against the CPU oracle, bit for bit, with the budget whole
and with what another job leaves of it (cut inside a key)."""

import numpy as np
import pytest

import oracle
from paper_1805_07891_amd.job import TorchJob
from paper_1805_07891_amd.workloads import Job, key_offsets

pytestmark = pytest.mark.gpu

MiB = 1 << 20
# 64 workers over these: gradients and state 277 MiB, the state 8.4
KEYS = (700001, 5, 0, 1024 * 300, 90000)


@pytest.mark.parametrize("n,opt,elems", [(17, None, 1 << 22), (17, "sgd", 1 << 22), (33, "adam", 1 << 21),
                                         (17, None, 1 << 20), (64, None, 1 << 19)])
def test_the_state_is_scheduled_as_cached(n, opt, elems):
    states = {"sgd": 1, "adam": 3}.get(opt, 2)
    for unfused in (False, True):
        job = TorchJob(Job("any", n, (elems,)), "cuda:0", optimizer=opt, unfused=unfused)
        assert job.info()[4] == 4 * states * elems
        job.destroy()


def test_the_share_is_the_device_budgets():
    a = TorchJob(Job("any.a", 17, (1 << 24,)), "cuda:0")  # 128 MiB of state
    b = TorchJob(Job("any.b", 64, (1 << 25,)), "cuda:0")  # what is left
    c = TorchJob(Job("any.c", 1, (1 << 20,)), "cuda:0")
    assert [j.info()[4] // MiB for j in (a, b, c)] == [128, 128, 0]
    a.destroy()
    d = TorchJob(Job("any.d", 1, (1 << 20,)), "cuda:0")
    assert d.info()[4] == 8 * MiB
    for j in (b, c, d):
        j.destroy()


@pytest.mark.parametrize("opt,left,groups", [("nesterov", 256, 1), ("nesterov", 5, 1), ("momentum", 3, 2),
                                             ("sgd", 1, 1), ("adam", 6, 1)])
def test_both_kinds_of_step(opt, left, groups):
    import torch
    n = 64
    states = {"sgd": 1, "adam": 3}.get(opt, 2)
    print("budget", opt, left, groups, flush=True)
    other = TorchJob(Job("other", 1, ((256 - left) * MiB // 8,)), "cuda:0") if left < 256 else None
    spec = Job("any.both", n, KEYS, lr=0.05, weight_decay=1e-3, nesterov=opt == "nesterov")
    job = TorchJob(spec, "cuda:0", optimizer={"momentum": None, "nesterov": None}.get(opt, opt),
                   key_group=[k % groups for k in range(len(KEYS))] if groups > 1 else None)
    offs, total = key_offsets(KEYS)
    assert 0 < job.info()[4] <= left * MiB
    assert (job.info()[4] < 4 * states * sum(KEYS)) == (left < 256)
    rng = np.random.default_rng(left)
    host = [rng.random(total, dtype=np.float32) - np.float32(0.5) for _ in range(n)]
    w0 = rng.standard_normal(total, dtype=np.float32) * np.float32(0.05)
    job.set_weights(torch.from_numpy(w0).cuda())
    dev = [torch.from_numpy(h).cuda() for h in host]
    models = [torch.zeros(total, device="cuda") for _ in range(n)]
    for w, d in enumerate(dev):
        job.attach_grads(w, d)
        job.attach_models(w, models[w])
    torch.cuda.synchronize()
    g = [[h[o:o + m] for o, m in zip(offs, KEYS)] for h in host]
    W = [w0[o:o + m].copy() for o, m in zip(offs, KEYS)]
    M, V = ([np.zeros(m, np.float32) for m in KEYS] for _ in range(2))
    for t, pull in enumerate((False, True, False)):
        job.pushpull_all() if pull else job.push_all()
        job.step()
        if opt == "sgd":
            oracle.step_sgd(g, W, spec.lr, spec.weight_decay)
        elif opt == "adam":
            oracle.step_adam(g, W, M, V, spec.lr, 0.9, 0.999, 1e-8, spec.weight_decay, t + 1)
        else:
            oracle.step(g, W, M, spec.lr, spec.momentum, spec.weight_decay, opt == "nesterov")
        Wg, Mg = job.state_arenas()
        out = models[n - 1].cpu().numpy() if pull else Wg
        for k, (o, m) in enumerate(zip(offs, KEYS)):
            assert np.array_equal(Wg[o:o + m].view(np.uint32), W[k].view(np.uint32)), (t, k)
            assert np.array_equal(out[o:o + m].view(np.uint32), W[k].view(np.uint32)), (t, k)
            if opt != "sgd":
                assert np.array_equal(Mg[o:o + m].view(np.uint32), M[k].view(np.uint32)), (t, k)
    job.destroy()
    if other:
        other.destroy()
