"""A single column and a few of them in one workgroup each, two rows a thread
(513 to 1,024 rows), against the oracle's filter."""
import numpy as np
import pytest

import workloads as wl
from oracle import filter as flt
from oracle import models
from tests.test_gpu_batch import filter_tol
from tests.test_gpu_parity import ctx, dev, host, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,N,periodic", [(16, 3, True), (12, 5, False), (14, 4, True)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_two_rows_a_thread(pk, ctx, L, N, periodic, prec):
    say(f"resident, one workgroup, L={L} N={N} {prec}")
    p, dt = (pk.FP64, torch.float64) if prec == "fp64" else (pk.FP32, torch.float32)
    ops, Hs = [], []
    for c in range(3):
        h = wl.xxz_fields(L, 3.0, 20 + c)
        ops.append(pk.Operator.xxz(ctx, L, N, 1.0, 0.7, h, periodic))
        Hs.append(models.xxz(L, N, 1.0, 0.7, h, periodic)[0])
    ops[0].set_batch_kernel(3, p, 5)
    V = np.random.default_rng(4).standard_normal((3, ops[0].D))
    for K in (16, 131):
        a = flt.coefficients(0.15, K)
        ref = [flt.apply_filter(H, 0.3, 2.5 * L, a, v) for H, v in zip(Hs, V)]
        got = [host(pk.filter_apply(ops[0], 0.3, 2.5 * L, a, dev(V[0], dt), p))]
        got += list(host(pk.filter_apply_batch(ops, [0.3] * 3, [2.5 * L] * 3, [a] * 3, dev(V, dt), p)))
        for g, r in zip(got, [ref[0]] + ref):
            assert np.max(np.abs(g.astype(np.float64) - r)) <= filter_tol(K, prec) * np.max(np.abs(r))
