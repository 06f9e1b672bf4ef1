"""KPM moments of more vectors than one launch takes, where a shorter group's
own best shape would have more slabs than the full group's (D = 5,005, 4,368
and 4,845: 4 slabs for 64 vectors, 16 for 17 to 32)."""
import numpy as np
import pytest

import workloads as wl
from oracle import kpm, models
from tests.test_gpu_parity import ctx, dev, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,N,R", [(15, 6, 96), (16, 5, 85), (20, 4, 81)])
def test_last_group_of_vectors(pk, ctx, L, N, R):
    say(f"kpm groups L={L} N={N} R={R}")
    h = wl.xxz_fields(L, 3.0, 4)
    op = pk.Operator.xxz(ctx, L, N, 1.0, 0.7, h, True)
    H = models.xxz(L, N, 1.0, 0.7, h, True)[0]
    v = np.random.default_rng(6).standard_normal((R, op.D))
    E_c, dE = 0.2, 2.6 * L
    got = pk.kpm_moments(op, E_c, dE, 100, R, dev(v))
    assert np.max(np.abs(got - kpm.moments(H, E_c, dE, v.T, 100))) <= 1e-11 * op.D


# the resident recurrence sums its products every 256 steps, the launches every
# 8,192 partial sums (170 moments at D = 48,620)
@pytest.mark.parametrize("L,N,R,variant,counts", [
    (12, 6, 3, -1, (256, 257, 258, 513, 600)), (16, 8, 20, -1, (257, 300)),
    (18, 9, 2, 0, (169, 170, 171, 345))])
def test_more_moments_than_one_sum(pk, ctx, L, N, R, variant, counts):
    say(f"kpm moments L={L} variant={variant} {counts}")
    h = wl.xxz_fields(L, 3.0, 8)
    op = pk.Operator.xxz(ctx, L, N, 1.0, 0.7, h, True)
    op.set_kernel(pk.FP64, variant)
    H = models.xxz(L, N, 1.0, 0.7, h, True)[0]
    v = np.random.default_rng(9).standard_normal((R, op.D))
    E_c, dE = 0.2, 2.6 * L
    ref = kpm.moments(H, E_c, dE, v.T, max(counts))
    for n in counts:
        got = pk.kpm_moments(op, E_c, dE, n, R, dev(v))
        assert np.max(np.abs(got - ref[:n])) <= 1e-11 * op.D, n
