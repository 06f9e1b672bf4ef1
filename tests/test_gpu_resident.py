"""The resident recurrence (a short chain's whole filter in one launch by
teams of workgroups on one XCD) against the oracle's filter, element by
element, at the sizes where its shapes change: one workgroup up to 1,024
rows, 4 to 32 slabs of a column with a remainder of rows, one to three rows a
thread, pairs of columns, more columns than teams, orders around the smallest
one that goes this way and around the steps of one launch; and on several
streams at once, where teams form while other teams hold the compute units."""
import threading

import numpy as np
import pytest

import workloads as wl
from oracle import filter as flt
from oracle import kpm, models
from tests.test_gpu_batch import filter_tol
from tests.test_gpu_parity import ctx, dev, host, pk, qsun_case, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def chain(pk, ctx, kind, L, N, periodic, seed):
    if kind == "xxz":
        h = wl.xxz_fields(L, 3.0, seed)
        return (pk.Operator.xxz(ctx, L, N, 1.0, 0.7, h, periodic),
                models.xxz(L, N, 1.0, 0.7, h, periodic)[0])
    eps = wl.tv_onsite(L, seed)
    return (pk.Operator.tv(ctx, L, N, 1.0, 1.3, eps, periodic),
            models.tv(L, N, 1.0, 1.3, eps, periodic)[0])


def check(got, ref, K, prec):
    got = got.astype(np.float64)
    assert np.max(np.abs(got - ref)) <= filter_tol(K, prec) * np.max(np.abs(ref))


# D: 6, 1, 924, 1716 (4 slabs), 3003 (8), 6435 (16), 12870 (32), 48620 (three
# rows a thread), 43758; t-V with an even particle number flips the sign of
# the periodic hop
@pytest.mark.parametrize("kind,L,N,periodic", [
    ("xxz", 4, 2, True), ("xxz", 6, 6, True), ("xxz", 12, 6, True), ("xxz", 13, 6, False),
    ("tv", 14, 6, True), ("tv", 15, 7, True), ("tv", 16, 8, True), ("xxz", 16, 8, False),
    ("xxz", 18, 9, True), ("tv", 18, 8, True)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_single_column(pk, ctx, kind, L, N, periodic, prec):
    say(f"resident {kind} L={L} N={N} periodic={periodic} {prec}")
    op, H = chain(pk, ctx, kind, L, N, periodic, 5)
    p, dt = (pk.FP64, torch.float64) if prec == "fp64" else (pk.FP32, torch.float32)
    v = np.random.default_rng(1).standard_normal(op.D)
    E_c, dE = 0.3, 2.5 * L
    for K in (15, 16, 17, 65, 130):
        a = flt.coefficients(0.15, K)
        w = pk.filter_apply(op, E_c, dE, a, dev(v, dt), p)
        check(host(w), flt.apply_filter(H, E_c, dE, a, v), K, prec)


def test_more_steps_than_one_launch(pk, ctx):
    say("resident, K = 8192, 8193, 16500 at L = 8 and 12")
    for L, N in ((8, 4), (13, 6)):
        op, H = chain(pk, ctx, "xxz", L, N, True, 2)
        v = np.random.default_rng(3).standard_normal(op.D)
        for K in (8192, 8193, 16500):
            a = flt.coefficients(-0.1, K)
            w = pk.filter_apply(op, 0.0, 2.0 * L, a, dev(v))
            check(host(w), flt.apply_filter(H, 0.0, 2.0 * L, a, v), K, "fp64")


@pytest.mark.parametrize("L,B", [(14, 35), (16, 9), (18, 13), (19, 3)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_batch_of_ragged_width(pk, ctx, L, B, prec):
    """Whatever kernel the tuner picks, each column equals the oracle's
    filter of its own realization (orders differ, one of them 0)."""
    say(f"batch L={L} B={B} {prec}")
    made = [chain(pk, ctx, "xxz", L, L // 2, True, 40 + c) for c in range(B)]
    ops, Hs = [m[0] for m in made], [m[1] for m in made]
    p, dt = (pk.FP64, torch.float64) if prec == "fp64" else (pk.FP32, torch.float32)
    Ks = [40 - 3 * (c % 5) for c in range(B)]
    Ks[-1] = 0
    V = np.random.default_rng(7).standard_normal((B, ops[0].D))
    coefs = [flt.coefficients(0.02 * (c % 7), Ks[c]) for c in range(B)]
    E_c, dE = [0.01 * c for c in range(B)], [2.5 * L + 0.1 * c for c in range(B)]
    w = host(pk.filter_apply_batch(ops, E_c, dE, coefs, dev(V, dt), p))
    say(f"   variant {ops[0].set_batch_kernel(B, p, -2)}")
    for c in range(0, B, max(1, B // 6)):
        check(w[c], flt.apply_filter(Hs[c], E_c[c], dE[c], coefs[c], V[c]), max(Ks), prec)
    check(w[B - 1], coefs[-1][0] * V[B - 1], max(Ks), prec)


def test_streams_side_by_side(pk):
    """Filters on six streams at once give what each gives alone."""
    say("resident on six streams")
    L, N, K = 17, 8, 300
    a = flt.coefficients(0.1, K)
    ctxs = [pk.Context(0, torch.cuda.Stream()) for _ in range(6)]
    ops = [chain(pk, c, "xxz", L, N, True, 60 + i)[0] for i, c in enumerate(ctxs)]
    vs = [dev(np.random.default_rng(i).standard_normal(ops[0].D)) for i in range(6)]
    torch.cuda.synchronize()
    alone = [host(pk.filter_apply(o, 0.0, 50.0, a, v)) for o, v in zip(ops, vs)]
    got = [[] for _ in ops]

    def work(i):
        for _ in range(5):
            got[i].append(pk.filter_apply(ops[i], 0.0, 50.0, a, vs[i]))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(6)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    for i in range(6):
        for w in got[i]:
            assert np.array_equal(host(w), alone[i])


@pytest.mark.parametrize("L,N,periodic,R", [(12, 6, True, 3), (13, 6, False, 17), (16, 8, True, 9),
                                            (14, 5, True, 70)])
def test_kpm_moments(pk, ctx, L, N, periodic, R):
    """Moments from the resident recurrence (one workgroup, teams, pairs of
    vectors, more vectors than one launch takes) for odd, even and the
    smallest numbers of them."""
    say(f"kpm L={L} N={N} R={R}")
    op, H = chain(pk, ctx, "tv" if L == 16 else "xxz", L, N, periodic, 9)
    v = np.random.default_rng(2).standard_normal((R, op.D))
    E_c, dE = 0.2, 2.6 * L
    ref = kpm.moments(H, E_c, dE, v.T, 61)
    for n in (1, 2, 3, 7, 8, 9, 60, 61):
        got = pk.kpm_moments(op, E_c, dE, n, R, dev(v))
        assert np.max(np.abs(got - ref[:n])) <= 1e-11 * op.D, n


# rows 4 (below a wave), 256, 2048 (one workgroup), 4096 to 65536 (slabs of
# one item a thread), 131072 and 262144 (two and four items), every dot size
@pytest.mark.parametrize("N,L", [(1, 1), (2, 6), (3, 8), (1, 11), (2, 11), (4, 8), (3, 13), (5, 9),
                                 (6, 6), (1, 16), (3, 14), (5, 12), (2, 16), (3, 15)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_quantum_sun(pk, ctx, N, L, prec):
    say(f"resident quantum sun {N}+{L} {prec}")
    q, H = qsun_case(N, L, 3)
    op = pk.Operator.qsun(ctx, N, L, q["A"], 1.0, 1.0, 0.75, q["u"], q["n_of_j"], q["h"])
    p, dt = (pk.FP64, torch.float64) if prec == "fp64" else (pk.FP32, torch.float32)
    v = np.random.default_rng(1).standard_normal(op.D)
    E_c, dE = 0.1, 1.2 * L + 8.0
    for K in (16, 47):
        a = flt.coefficients(0.15, K)
        w = pk.filter_apply(op, E_c, dE, a, dev(v, dt), p)
        check(host(w), flt.apply_filter(H, E_c, dE, a, v), K, prec)
