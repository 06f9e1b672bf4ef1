"""The step kernel of a fresh operator is chosen by the first call that applies
H, also where that call runs another kernel (the extraction's H on a block, the
moments' resident recurrence): the allocation-free filter accepts it then."""
import numpy as np
import pytest

import workloads as wl
from oracle import filter as flt
from tests.test_gpu_parity import dev, host, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

L = 14


def extract(pk, op):
    V = np.linalg.qr(np.random.default_rng(1).standard_normal((op.D, 12)))[0]
    T = np.linalg.qr(np.random.default_rng(2).standard_normal((12, 5)))[0]
    pk.extract(op, dev(np.ascontiguousarray(V.T)), dev(np.ascontiguousarray(T.T)))


def moments(pk, op):
    pk.kpm_moments(op, 0.0, 2.6 * L, 40, 3)


@pytest.mark.parametrize("call", [extract, moments])
def test_noalloc_filter_after(pk, call):
    say(f"first call {call.__name__}")
    op = pk.Operator.xxz(pk.Context(0), L, L // 2, 1.0, 1.0, wl.xxz_fields(L, 3.0, 1), True)
    call(pk, op)
    assert op.set_kernel(pk.FP64, -2) >= 0
    v = dev(np.random.default_rng(3).standard_normal(op.D))
    a, w = flt.coefficients(0.1, 60), torch.empty_like(v)
    pk.filter_apply_noalloc(op, 0.0, 2.6 * L, a, v, w)
    torch.cuda.synchronize()
    assert np.array_equal(host(w), host(pk.filter_apply(op, 0.0, 2.6 * L, a, v)))
