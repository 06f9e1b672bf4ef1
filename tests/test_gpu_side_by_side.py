"""Filters of four contexts at once (a thread and a stream each, chains whose
teams fill an XCD) take no longer than one after the other; with teams that went
on with a quarter of their members they took two to three times as long."""
import threading
import time

import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_parity import dev, host, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_four_contexts(pk):
    say("four contexts, L=18")
    L, K, reps = 18, 1500, 6
    a, dE = np.full(K + 1, 1e-3), 60.0
    sides = []
    for i in range(4):
        ctx = pk.Context(0, torch.cuda.Stream())
        op = pk.Operator.xxz(ctx, L, L // 2, 1.0, 1.0, wl.xxz_fields(L, 3.0, i), True)
        sides.append((op, dev(np.random.default_rng(i).standard_normal(op.D))))
    torch.cuda.synchronize()
    out = [None] * 4

    def work(i):
        for _ in range(reps):
            out[i] = pk.filter_apply(sides[i][0], 0.0, dE, a, sides[i][1])

    for i in range(4):
        work(i)  # tables and kernel choices
    ref = [host(w) for w in out]
    t0 = time.perf_counter()
    for i in range(4):
        work(i)
    one_by_one = time.perf_counter() - t0
    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    t0 = time.perf_counter()
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    together = time.perf_counter() - t0
    say(f"   one by one {1e3 * one_by_one:.1f} ms, together {1e3 * together:.1f} ms")
    assert all(np.array_equal(host(w), r) for w, r in zip(out, ref))
    assert together <= one_by_one
