"""Allocation-free filters that overlap on one GPU (two contexts): their vectors
lie in one array, so what they return is not defined, but the teams of each have
a state of their own and every launch ends; a call by itself is right again."""
import numpy as np
import pytest

import workloads as wl
from oracle import filter as flt
from tests.test_gpu_parity import dev, host, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_overlapping_calls_end(pk):
    say("noalloc filters on two streams at once")
    K, sides = 200, []
    a = flt.coefficients(0.1, K)
    for i, L in enumerate((15, 16)):
        ctx = pk.Context(0, torch.cuda.Stream())
        op = pk.Operator.xxz(ctx, L, L // 2, 1.0, 1.0, wl.xxz_fields(L, 3.0, i), True)
        v = dev(np.random.default_rng(i).standard_normal(op.D))
        torch.cuda.synchronize()
        sides.append((ctx, op, v, torch.empty_like(v), host(pk.filter_apply(op, 0.0, 2.6 * L, a, v)),
                      2.6 * L))
    for _ in range(10):
        for ctx, op, v, w, _, dE in sides:
            pk.filter_apply_noalloc(op, 0.0, dE, a, v, w)
    for ctx, *_ in sides:
        ctx.sync()
    for ctx, op, v, w, ref, dE in sides:
        pk.filter_apply_noalloc(op, 0.0, dE, a, v, w)
        ctx.sync()
        assert np.array_equal(host(w), ref)
