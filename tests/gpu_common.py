"""Helpers of the GPU parity tests: config-1 data built by the oracle, host<->device copies."""

import functools

import numpy as np


@functools.lru_cache(maxsize=None)
def config1(n=100_000, m=16, d=128, nq=16, train_n=20_000, iters=10):
    """Config 1: mixture data, PQ m x 16 trained by 10 k-means iterations on 20k vectors."""
    from oracle import qadc_oracle as O, cref
    from workloads import (MixtureSpec, mixture_vectors, kmeans_init_rows,
                           SEED_TRAIN, SEED_BASE, SEED_QUERY)
    spec = MixtureSpec(d=d)
    train = mixture_vectors(spec, SEED_TRAIN, 0, train_n)
    cb = O.pq_train(train, m, 16, iters, kmeans_init_rows(train_n, 16))
    base = mixture_vectors(spec, SEED_BASE, 0, n)
    codes = cref.pq_encode(base, cb)
    queries = mixture_vectors(spec, SEED_QUERY, 0, nq)
    return dict(spec=spec, codebooks=cb, base=base, codes=codes, queries=queries)


def to_gpu(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def idx_np(t):
    return t.cpu().numpy().view(np.uint32)


def gpu_us(f, reps=20, rounds=3):
    """Microseconds of one call of f among others, the fastest of a few rounds."""
    import torch
    f()
    best = float("inf")
    for _ in range(rounds):
        a, b = torch.cuda.Event(True), torch.cuda.Event(True)
        torch.cuda.synchronize()
        a.record()
        for _ in range(reps):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / reps)
    return best


def smallest_workspace(Q, call):
    """call(workspace) with the least bytes it takes, one byte less having been refused; that number and its result."""
    import re
    import torch
    buf = lambda nbytes: Q.qadc_workspace_init(torch.empty((nbytes,), dtype=torch.uint8, device="cuda:0"))
    try:
        call(buf(256))
        raise AssertionError("256 bytes were enough")
    except Q.QadcError as e:
        assert e.code == Q.QADC_ENOMEM
        least = max(int(v) for v in re.findall(r"\b\d+\b", Q.qadc_last_error()))
    try:
        call(buf(least)[:least - 1])
        raise AssertionError("a byte less was enough")
    except Q.QadcError as e:
        assert e.code == Q.QADC_ENOMEM
    return least, call(buf(least))
