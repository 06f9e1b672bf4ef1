"""What a solve reports about its filter is what ran: K steps an application, or,
where a short chain's filter is computed as a matrix, K steps of each of its
columns once and the matrix's bytes an application."""
import pytest

import workloads as wl
from tests.test_gpu_parity import ctx, dev, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,n_ev,matrix", [(12, 20, True), (14, 12, False)])
def test_filter_steps_and_bytes(pk, ctx, L, n_ev, matrix):
    say(f"report L={L}")
    op = pk.Operator.xxz(ctx, L, L // 2, 1.0, 1.0, wl.xxz_fields(L, 1.0, 0), True)
    D, x0 = op.D, dev(wl.start_vector(op.D, 0))
    for graph in (0, 2):  # 2: the caller's launches, never a matrix
        rep, status = pk.solve(op, x0, n_ev, 0.5, "normalized", graph=graph)[3:]
        assert status == "OK" and rep["restarts"] == 0
        K, n = rep["K"], rep["iters"]
        steps = K * D if matrix and graph == 0 else K * n
        assert rep["filter_steps"] == steps
        products = n * (8 * D * D + 16 * D) if matrix and graph == 0 else 0
        assert rep["filter_bytes"] == pytest.approx(32.0 * D * steps + products, rel=1e-12)
