"""A barrier of the resident kernels that gives up (its bounded wait set to
zero, so that every member runs on to its end at once): the call returns no
numbers, also where the failure lies launches before the last one, and with
the wait as in a new context the same operator is right again."""
import numpy as np
import pytest

import workloads as wl
from oracle import filter as flt
from oracle import models
from tests.test_gpu_batch import filter_tol
from tests.test_gpu_parity import dev, host, pk, qsun_case, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture
def own(pk):
    return pk.Context(0)


def filter_gives_up(pk, ctx, op, H, dE, K):
    a = flt.coefficients(0.1, K)
    v = np.random.default_rng(1).standard_normal(op.D)
    ref = flt.apply_filter(H, 0.0, dE, a, v)
    tol = filter_tol(K, "fp64") * np.max(np.abs(ref))
    assert np.max(np.abs(host(pk.filter_apply(op, 0.0, dE, a, dev(v))) - ref)) <= tol
    ctx.set_team_wait(0)
    w = host(pk.filter_apply(op, 0.0, dE, a, dev(v)))
    assert np.isnan(w).any()
    ctx.set_team_wait(30)
    assert np.max(np.abs(host(pk.filter_apply(op, 0.0, dE, a, dev(v))) - ref)) <= tol


@pytest.mark.parametrize("K", [60, 8200])
def test_filter_of_a_chain(pk, own, K):
    say(f"team wait 0, chain, K={K}")
    L = 14
    h = wl.xxz_fields(L, 3.0, 5)
    op = pk.Operator.xxz(own, L, 7, 1.0, 0.7, h, True)
    filter_gives_up(pk, own, op, models.xxz(L, 7, 1.0, 0.7, h, True)[0], 2.5 * L, K)


def test_filter_of_a_quantum_sun(pk, own):
    say("team wait 0, quantum sun")
    N, L = 3, 10
    q, H = qsun_case(N, L, 3)
    op = pk.Operator.qsun(own, N, L, q["A"], 1.0, 1.0, 0.75, q["u"], q["n_of_j"], q["h"])
    filter_gives_up(pk, own, op, H, 1.2 * L + 8.0, 47)


@pytest.mark.parametrize("L,N,R", [(14, 7, 5), (16, 8, 40)])
def test_kpm_moments(pk, own, L, N, R):
    say(f"team wait 0, kpm L={L} R={R}")
    op = pk.Operator.xxz(own, L, N, 1.0, 0.7, wl.xxz_fields(L, 3.0, 5), True)
    good = pk.kpm_moments(op, 0.0, 2.6 * L, 60, R, seed=3)
    own.set_team_wait(0)
    with pytest.raises(pk.PolfedError) as e:
        pk.kpm_moments(op, 0.0, 2.6 * L, 60, R, seed=3)
    assert "gave up" in str(e.value)
    own.set_team_wait(30)
    assert np.array_equal(pk.kpm_moments(op, 0.0, 2.6 * L, 60, R, seed=3), good)
