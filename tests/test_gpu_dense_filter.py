"""Solves of short chains, whose filter is applied as a matrix, at the sizes
where that begins and ends: one workgroup a column (D <= 1,024) and several,
D odd, a periodic hop of its own sign, open chains, the largest D of the rule
and the first beyond; against dense diagonalization and against the solve with
the recurrence (direct launches)."""
import sys

import numpy as np
import pytest

import workloads as wl
from oracle import models

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_10191_amd as pk
    pk.load_library()
    return pk


@pytest.fixture(scope="module")
def ctx(pk):
    c = pk.Context(0)
    yield c
    c.sync()


@pytest.mark.parametrize("model,L,N,periodic,n_ev", [
    ("xxz", 8, 4, True, 5), ("xxz", 11, 5, False, 12), ("tv", 11, 4, True, 10),
    ("xxz", 12, 6, True, 30), ("tv", 12, 6, True, 8), ("xxz", 13, 4, True, 15),
    ("xxz", 13, 6, False, 20), ("tv", 14, 4, True, 20), ("xxz", 14, 5, True, 10),
    ("xxz", 14, 6, True, 10)])
def test_solve(pk, ctx, model, L, N, periodic, n_ev):
    print(f"dense filter {model} L={L} N={N} periodic={periodic}")
    sys.stdout.flush()
    if model == "xxz":
        f = wl.xxz_fields(L, 2.0, 6)
        H, _ = models.xxz(L, N, 1.0, 1.0, f, periodic)
        op = pk.Operator.xxz(ctx, L, N, 1.0, 1.0, f, periodic)
    else:
        f = wl.tv_onsite(L, 6)
        H, _ = models.tv(L, N, 1.0, 1.0, f, periodic)
        op = pk.Operator.tv(ctx, L, N, 1.0, 1.0, f, periodic)
    x0 = torch.as_tensor(np.random.default_rng(3).standard_normal(op.D), device="cuda:0")
    E, U, res, rep, _ = pk.solve(op, x0, n_ev, 0.5, "normalized")
    E2, _, _, rep2, _ = pk.solve(op, x0, n_ev, 0.5, "normalized", graph=2)
    E, E2 = (np.sort(np.asarray(e.cpu() if hasattr(e, "cpu") else e)) for e in (E, E2))
    ref = np.linalg.eigvalsh(H.toarray())
    span = ref[-1] - ref[0]
    near = np.array([ref[np.argmin(abs(ref - e))] for e in E])
    # the solver accepts pairs with residuals of 1e-8 and less; a Ritz value's
    # error is at most its residual, and of the order of its square
    assert len(E) == n_ev and np.max(abs(E - near)) <= 1e-10 * span
    assert len(np.unique(near)) == n_ev
    assert np.max(abs(E - E2)) <= 1e-10 * span
    assert rep["K"] == rep2["K"]
    res = np.asarray(res.cpu() if hasattr(res, "cpu") else res)
    assert np.max(res) <= 1e-8
