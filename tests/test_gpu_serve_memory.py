"""What a served solve reserves at admission covers what its buffers hold
(mem_peak <= mem_reserved), and a density of states from KPM moments raises
neither: a request that was admitted without it is admitted with it."""
import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_parity import dev, host, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture
def own(pk):
    return pk.Context(0)


def served(pk, ctx, op, budget, n_ev, **kw):
    x0 = dev(wl.start_vector(op.D, 3))
    with pk.Server(ctx, budget, max_cols=2) as srv:
        ev, _, res, rep, status = srv.submit(op, x0, n_ev, 0.5, "normalized", **kw).wait()
    assert status == "OK" and host(res).max() <= 1e-8
    assert 0 < rep["mem_peak"] <= rep["mem_reserved"], (rep["mem_peak"], rep["mem_reserved"])
    return host(ev), rep


# the moments of 64 vectors at once would take 20 MB, the solve 12
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_kpm_moments_in_the_room_of_the_solve(pk, own, prec):
    say(f"served kpm {prec}")
    p = pk.FP64 if prec == "fp64" else pk.FP32
    op = pk.Operator.xxz(own, 16, 8, 1.0, 1.0, wl.xxz_fields(16, 1.0, 2), True)
    lo, hi = pk.bounds(op, dev(wl.start_vector(op.D, 3)))
    kw = dict(E_min=lo, E_max=hi, precision=p)
    plain, rep = served(pk, own, op, 1 << 30, 2, **kw)
    budget = int(1.1 * rep["mem_reserved"])
    say(f"   reserved {budget / 1e6:.2f} MB, peak {rep['mem_peak'] / 1e6:.2f} MB")
    got, rep = served(pk, own, op, budget, 2, kpm_moments=64, kpm_vectors=64, **kw)
    say(f"   with moments: peak {rep['mem_peak'] / 1e6:.2f} MB")
    assert np.max(np.abs(got - plain)) <= 1e-9


# few pairs: the bounds before the iteration hold the most, up to 300 vectors
# and a partial sum of every column for each of up to 768 workgroups
@pytest.mark.parametrize("L,N", [(12, 6), (16, 7), (16, 8), (18, 9)])
def test_bounds_within_the_reservation(pk, own, L, N):
    say(f"served bounds L={L} N={N}")
    op = pk.Operator.xxz(own, L, N, 1.0, 1.0, wl.xxz_fields(L, 1.0, 2), True)
    _, rep = served(pk, own, op, 1 << 30, 2)
    say(f"   reserved {rep['mem_reserved'] / 1e6:.2f} MB, peak {rep['mem_peak'] / 1e6:.2f} MB")
