"""The error of the KPM moments against 80-bit arithmetic: that of a plain FP64
evaluation of the definition (three-term recurrence, products <r|t_n>), on
chains that take the resident recurrence and, with a step kernel set, on the
launches.  One chain's error scatters, so the squares are summed over chains,
and the two are compared with a factor of 1.5: moments from the doubled products
<t_n|t_n> have 1.7 times the error of the definition's at L = 12 and 2.1 at
L = 16.  t-V chains, whose site terms and hops the library takes as they are
given (an XXZ chain's constant and site terms are sums that it rounds first,
which would be most of the difference)."""
import numpy as np
import pytest

import workloads as wl
from oracle import models
from tests.test_gpu_parity import ctx, dev, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LD = np.longdouble


def tree_sum(p):
    n = 1 << (len(p) - 1).bit_length()
    q = np.zeros(n, p.dtype)
    q[:len(p)] = p
    while len(q) > 1:
        q = q[:len(q) // 2] + q[len(q) // 2:]
    return q[0]


def off_diagonal(H):
    H = H.tocsr().copy()
    H.setdiag(0.0)
    H.eliminate_zeros()
    H.sort_indices()
    return H


def diagonal(L, N, V, eps, dtype):
    """V n_i n_{i+1} + eps_i n_i of the states in ascending order."""
    st = np.array([s for s in range(1 << L) if bin(s).count("1") == N])
    n = [((st >> i) & 1).astype(dtype) for i in range(L)]
    d = dtype(V) * sum(n[i] * n[(i + 1) % L] for i in range(L))
    for i in range(L):
        d = d + dtype(eps[i]) * n[i]
    return d


def moments(H, diag, E_c, dE, r, N):
    """sum_r <r|T_n(H~)|r> / R in the arithmetic of diag, the products by a tree."""
    dt = diag.dtype.type
    data = H.data.astype(dt)
    E_c, dE = dt(E_c), dt(dE)

    def scaled(f, x):
        hx = np.add.reduceat(data * x[H.indices], H.indptr[:-1]) + diag * x
        return (f / dE) * hx + (-f * E_c / dE) * x

    mu = np.zeros(N, dt)
    for x in r.astype(dt):
        t0, t1 = x, scaled(dt(1), x)
        mu[0] += tree_sum(x * x)
        for n in range(1, N):
            mu[n] += tree_sum(x * t1)
            t0, t1 = t1, scaled(dt(2), t1) - t0
    return mu / len(r)


@pytest.mark.parametrize("L,chains,N,variant", [(12, 24, 50, -1), (16, 8, 100, -1), (12, 24, 50, 0)])
def test_moments_error(pk, ctx, L, chains, N, variant):
    say(f"kpm error L={L} N={N} variant={variant}")
    err = np.zeros(2)
    for c in range(chains):
        L2, V, eps = L // 2, 1.3, wl.tv_onsite(L, 300 + c)
        op = pk.Operator.tv(ctx, L, L2, 1.0, V, eps, True)
        op.set_kernel(pk.FP64, variant)
        H = off_diagonal(models.tv(L, L2, 1.0, V, eps, True)[0])
        e = np.sort(eps)
        lo, hi = e[:L2].sum() - 2.0 * L2, e[L2:].sum() + (2.0 + V) * L2
        E_c, dE = 0.5 * (lo + hi), 0.505 * (hi - lo)
        r = np.random.default_rng(c).uniform(-3 ** 0.5, 3 ** 0.5, (2, op.D))
        exact = moments(H, diagonal(L, L2, V, eps, LD), E_c, dE, r, N)
        plain = moments(H, diagonal(L, L2, V, eps, np.float64), E_c, dE, r, N)
        for i, mu in enumerate((pk.kpm_moments(op, E_c, dE, N, 2, dev(r)), plain)):
            d = (mu.astype(LD) - exact).astype(np.float64)
            err[i] += (d @ d) / float(exact @ exact)
    err = np.sqrt(err / chains)
    say(f"   rms error {err[0]:.3g}, plain FP64 {err[1]:.3g}")
    assert err[0] <= 1.5 * err[1]
