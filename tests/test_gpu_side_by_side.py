"""Calls of four contexts at once (a thread and a stream each, chains whose teams
fill an XCD) take no longer than one after the other: filters of a column and of
a batch; with teams that went on with a part of their members they took two to
six times as long."""
import threading
import time

import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_parity import dev, host, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("what,B,K,reps", [("column", 1, 1500, 10), ("batch", 13, 400, 6)])
def test_four_contexts(pk, what, B, K, reps):
    L, a, dE = 18, np.full(K + 1, 1e-3), 60.0
    sides = []
    for i in range(4):
        ctx = pk.Context(0, torch.cuda.Stream())
        ops = [pk.Operator.xxz(ctx, L, L // 2, 1.0, 1.0, wl.xxz_fields(L, 3.0, 20 * i + c), True)
               for c in range(B)]
        sides.append((ops, dev(np.random.default_rng(i).standard_normal((B, ops[0].D)))))
    torch.cuda.synchronize()
    out = [None] * 4

    def work(i):
        for _ in range(reps):
            ops, v = sides[i]
            if what == "column":
                out[i] = pk.filter_apply(ops[0], 0.0, dE, a, v)
            else:
                out[i] = pk.filter_apply_batch(ops, [0.0] * B, [dE] * B, [a] * B, v)

    for i in range(4):
        work(i)  # tables and kernel choices
    ref = [host(w) for w in out]

    def timed(together):
        t0 = time.perf_counter()
        ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
        for t in ts:
            t.start()
            if not together:
                t.join()
        for t in ts:
            t.join()
        return time.perf_counter() - t0

    one_by_one = np.median([timed(False) for _ in range(5)])
    together = np.median([timed(True) for _ in range(5)])
    say(f"   {what}: one by one {1e3 * one_by_one:.1f} ms, together {1e3 * together:.1f} ms")
    assert all(np.array_equal(host(w), r) for w, r in zip(out, ref))
    # columns run side by side, batches one after the other
    assert together <= (1.0 if what == "column" else 1.3) * one_by_one
