"""The exchange steps whose speed counts, each through the public entry points.

A case is one call of a training program's server side: N workers' gradients
are pushed and one step aggregates and optimizes every key.  ``listed`` holds
the cases that stand for real use, ``draw`` gives others of the same ranges:
1 to 64 workers, 10^5 to 2 * 10^8 parameters, all three optimizers, key lists
of real models and ragged ones, and the ways a program can drive a step:

  step      every worker pushes every key from buffers that stay registered
            (TorchJob.push_and_step)
  fresh     the same with gradients in other buffers than the last step's (a
            backward pass that alternates between two sets of buffers)
  groups    readiness groups of 25 MB, keys pushed in backward order
  pushpull  the step also writes the new weights into every worker's model
            buffer, with the cache budget that phub.h recommends for it
  noalloc   phub_step_noalloc over the caller's own W and M
  tenants   several jobs, each on a stream of its own, stepped concurrently

Results are defined bit for bit (the sum in worker order, every operation
rounded once), so outputs are compared exactly.
"""

import math

import numpy as np
import torch

from paper_1805_07891_amd import phub
from paper_1805_07891_amd import workloads as wl
from paper_1805_07891_amd.job import TorchJob, load_library

DEVICE = "cuda:0"
GROUP_BYTES = 25e6  # a readiness group: the gradient bucket of data-parallel training
PUSHPULL_BUDGET = 256 << 20
STATES = {"momentum": 2, "sgd": 1, "adam": 3}
BETAS, EPS = (0.9, 0.999), 1e-8


def listed():
    return [
        # the smallest call: a small model's step, 26 MB, bound by the launch
        _case("tiny_4", "step", 4, "tiny"),
        # a small model of many ragged keys whose backward pass alternates
        # between two sets of gradient buffers: new pointers every step
        _case("ragged_8_fresh", "fresh", 8, "ragged", params=2_000_003, num_keys=64, shape=11),
        # the ordinary call: a 25.6 M-parameter network, 8 workers
        _case("resnet50_8", "step", 8, "resnet50"),
        # the same, its keys arriving in backward order in 25 MB buckets
        _case("resnet50_8_groups", "groups", 8, "resnet50"),
        # the same, every worker's model buffer filled by the step
        _case("resnet50_8_pushpull", "pushpull", 8, "resnet50"),
        # the same from a caller that cannot allocate device memory
        _case("resnet50_8_noalloc", "noalloc", 8, "resnet50"),
        # the same network with a rack's worth of workers
        _case("resnet50_64", "step", 64, "resnet50"),
        # few large keys, the other two optimizers
        _case("alexnet_8_adam", "step", 8, "alexnet", optimizer="adam"),
        _case("alexnet_8_sgd", "step", 8, "alexnet", optimizer="sgd"),
        # few workers, a large model: more state than gradients, plain momentum
        _case("vgg19_2", "step", 2, "vgg19", nesterov=False),
        # the largest single job: 818 keys, 16 workers, 8.2 GB
        _case("resnet269_16", "step", 16, "resnet269"),
        # the largest call: four tenants of 8 workers, 10.5 GB
        _case("tenants_8", "tenants", 8, "multitenant"),
    ]


def _case(name, call, workers, keys, optimizer="momentum", nesterov=True, params=0, num_keys=0,
          shape=0):
    return {"name": name, "call": call, "workers": workers, "keys": keys, "optimizer": optimizer,
            "nesterov": nesterov, "params": params, "num_keys": num_keys, "shape": shape}


def draw(rng):
    call = rng.choice(["step", "step", "step", "step", "fresh", "groups", "pushpull", "noalloc"])
    top = 16 if call == "pushpull" else 64
    workers = min(top, int(2.0 ** rng.uniform(0.0, math.log2(top + 1))))
    optimizer = "momentum" if call == "noalloc" else rng.choice(["momentum", "momentum", "sgd", "adam"])
    streams = (2 if call == "pushpull" else 1) * workers + 2 * STATES[optimizer]
    most = min(1.5e8, 8e9 / (4 * streams))  # no dearer than the listed ones
    params = int(math.exp(rng.uniform(math.log(1e5), math.log(most))))
    case = _case("", call, workers, "ragged", optimizer, rng.random() < 0.75, params,
                 int(math.exp(rng.uniform(math.log(8), math.log(800)))), rng.randrange(1 << 30))
    del case["name"]
    return case


# ---------------------------------------------------------------- the keys

MODELS = {"tiny": wl.tiny_keys, "resnet50": wl.resnet50_keys, "alexnet": wl.alexnet_keys,
          "vgg19": wl.vgg19_keys, "resnet269": wl.resnet269_keys}


def _ragged(params, num_keys, seed):
    """num_keys sizes spread over the logarithm of three decades, about
    params in all; few are multiples of 4."""
    r = np.random.default_rng(seed)
    size = 10.0 ** (3.0 * r.random(num_keys))
    return [max(1, int(n)) for n in size * (params / size.sum())]


def _jobs(case):
    """(name, key sizes) of the case's jobs: one, or the tenants'."""
    if case["keys"] == "multitenant":
        return [(j.name, j.key_elems) for j in wl.workload("multitenant").jobs]
    if case["keys"] == "ragged":
        return [("ragged", tuple(_ragged(case["params"], case["num_keys"], case["shape"])))]
    return [(case["keys"], tuple(MODELS[case["keys"]]()))]


def _spec(case, name, keys):
    return wl.Job(name, case["workers"], keys, nesterov=case["nesterov"],
                  lr=1e-3 if case["optimizer"] == "adam" else 0.1)


# -------------------------------------------------------------- the inputs

_streams = []


def _stream(i):
    """The program's i-th exchange stream: one per tenant, made once."""
    while len(_streams) <= i:
        _streams.append(torch.cuda.Stream(device=DEVICE))
    return _streams[i]


def _normal(seed, job, which, total, sigma):
    return wl.device_normal_arena(torch, DEVICE, seed * 1000003 + job * 1009 + which, total, sigma)


def _grads(spec, seed, job, total, second=False):
    return [_normal(seed, job, w + (500 if second else 0), total, spec.sigma_g)
            for w in range(spec.num_workers)]


def _mask(keys):
    """Which elements of an arena belong to a key (the rest is padding)."""
    offs, total = wl.key_offsets(keys)
    edge = torch.zeros(total + 1, dtype=torch.int32)
    offs = torch.tensor(offs)
    # empty keys and keys that end where the next begins cancel out
    edge.index_add_(0, offs, torch.ones(len(keys), dtype=torch.int32))
    edge.index_add_(0, offs + torch.tensor(keys), -torch.ones(len(keys), dtype=torch.int32))
    return torch.cumsum(edge[:total].to(DEVICE), 0) > 0


def _weights(spec, seed, job, total):
    w = _normal(seed, job, 999, total, spec.sigma_w)
    return w * _mask(spec.key_elems)


class _DeviceArray:
    """The job's own device memory as torch sees it (it keeps the job)."""

    def __init__(self, job, ptr, n):
        self.job = job
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<f4", "data": (ptr, False),
                                         "strides": None, "version": 2}


def _state_tensors(job):
    n, dev = job.arena_elems, torch.device(DEVICE)
    w, m = job.lib.phub_get_state(job.handle, 0)
    v = job.lib.phub_get_second_moment(job.handle, 0)
    return {k: torch.as_tensor(_DeviceArray(job, p, n), device=dev)
            for k, p in (("W", w), ("M", m), ("V", v)) if p}


def _readiness_groups(spec):
    """Keys in backward order, in runs of at least GROUP_BYTES."""
    group, g, acc = [0] * spec.num_keys, 0, 0
    for k in reversed(range(spec.num_keys)):
        group[k] = g
        acc += 4 * spec.key_elems[k]
        if acc >= GROUP_BYTES and k > 0:
            g, acc = g + 1, 0
    return group


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.call, s.jobs, s.out = case["call"], [], []
    for ji, (name, keys) in enumerate(_jobs(case)):
        spec = _spec(case, name, keys)
        total = wl.key_offsets(keys)[1]
        grads = _grads(spec, seed, ji, total)
        w0 = _weights(spec, seed, ji, total)
        if s.call == "noalloc":
            s.lib, s.spec, s.grads = load_library(), spec, grads
            s.W, s.M = w0, torch.zeros_like(w0)
            offs = wl.key_offsets(keys)[0]
            s.ptrs = phub.pointer_array([g.data_ptr() + 4 * o for g in grads for o in offs])
            s.stream = _stream(0)
            s.out.append({"W": s.W, "M": s.M})
            continue
        job = TorchJob(spec, DEVICE, stream=_stream(ji), optimizer=case["optimizer"], betas=BETAS,
                       eps=EPS, key_group=_readiness_groups(spec) if s.call == "groups" else None,
                       resident_bytes=PUSHPULL_BUDGET if s.call == "pushpull" else None)
        job.set_weights(w0)
        for w, g in enumerate(grads):
            job.attach_grads(w, g)
        out = _state_tensors(job)
        if s.call == "pushpull":
            s.models = [torch.zeros(total, device=DEVICE) for _ in grads]
            for w, m in enumerate(s.models):
                job.attach_models(w, m)
            out["models"] = s.models
        if s.call == "groups":
            order = range(max(job.key_group) + 1)
            members = [[k for k in range(spec.num_keys) if job.key_group[k] == g] for g in order]
            s.buckets = [(w, job.bucket(w, ks)) for ks in members for w in range(len(grads))]
        if s.call == "fresh":
            s.both = [grads, _grads(spec, seed, ji, total, second=True)]
            s.tables = [phub.pointer_array([g.data_ptr() + 4 * o for g in gs for o in job.offsets])
                        for gs in s.both]
            s.turn = 0
        s.jobs.append(job)
        s.out.append(out)
    return s


def run(s):
    if s.call == "noalloc":
        p = s.spec
        s.lib.phub_step_noalloc(p.num_workers, p.key_elems, p.chunk_bytes, p.lr, p.momentum,
                                p.weight_decay, p.nesterov, s.ptrs, s.W.data_ptr(),
                                s.M.data_ptr(), s.stream.cuda_stream)
        return s.out
    for job in s.jobs:
        if s.call == "fresh":
            job.lib.phub_push_all(job.handle, s.tables[s.turn])
            s.turn ^= 1
        elif s.call == "groups":
            for w, bucket in s.buckets:
                job.push_bucket(w, bucket)
        elif s.call == "pushpull":
            job.pushpull_all()
        else:
            job.push_all()
        job.step()
    return s.out


# ------------------------------------------------- what a pass cannot avoid

def work(case):
    states, n = STATES[case["optimizer"]], case["workers"]
    streams = n + 2 * states + (n if case["call"] == "pushpull" else 0)
    params = sum(sum(keys) for _, keys in _jobs(case))
    flops = n - 1 + {"momentum": 8, "sgd": 4, "adam": 14}[case["optimizer"]]
    return {"bytes": 4 * params * streams, "flops": params * flops}


def tolerance(case):
    return "exact"


# ------------------------------------------------------- the step in 64 bits

def exact(case, seed):
    out = []
    for ji, (name, keys) in enumerate(_jobs(case)):
        spec = _spec(case, name, keys)
        total = wl.key_offsets(keys)[1]
        s = torch.zeros(total, dtype=torch.float64, device=DEVICE)
        for w in range(spec.num_workers):
            s += _normal(seed, ji, w, total, spec.sigma_g)
        w0 = _weights(spec, seed, ji, total).double()
        lr, mu, wd, b1, b2, eps = (float(np.float32(v)) for v in (
            spec.lr, spec.momentum, spec.weight_decay, *BETAS, EPS))
        d = (s + wd * w0) * _mask(keys)
        if case["optimizer"] == "sgd":
            got = {"W": w0 - lr * d}
        elif case["optimizer"] == "adam":
            m, v = (1.0 - b1) * d, (1.0 - b2) * d * d
            step = lr / (1.0 - b1) * m / (torch.sqrt(v / (1.0 - b2)) + eps)
            got = {"W": w0 - step, "M": m, "V": v}
        else:
            got = {"W": w0 - lr * (d + mu * d if spec.nesterov else d), "M": d}
        if case["call"] == "pushpull":
            got["models"] = [got["W"]] * spec.num_workers
        out.append(got)
    return out
