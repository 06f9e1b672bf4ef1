"""The orthogonalization of a Lanczos step at the sizes where its one-launch
form begins, changes and ends: one basis vector, fewer rows than slabs, the
change from 16 to 32 members, the largest basis of the rule and the first
beyond it; of the pass that makes the two middle products at once, whose slabs
have 64, 32 and 16 rows; with the identity as the filter (order 0), so that the step is the
orthogonalization of v_k itself against a random basis whose v_k is not
orthogonal to the others."""
import sys

import numpy as np
import pytest

import workloads as wl

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


@pytest.mark.parametrize("L,N,k", [(4, 2, 0), (4, 2, 3), (6, 1, 4), (8, 4, 33), (12, 6, 0),
                                   (12, 6, 8), (12, 6, 107), (12, 6, 108), (14, 7, 581),
                                   (14, 7, 582), (16, 8, 33), (16, 8, 34), (14, 6, 198),
                                   (17, 8, 0), (17, 8, 6), (17, 8, 7), (17, 8, 40),
                                   (16, 8, 103), (16, 8, 104), (16, 8, 207), (16, 8, 208),
                                   (16, 8, 599), (16, 8, 600), (19, 9, 30)])
def test_lanczos_step(pk, ctx, L, N, k):
    op = pk.Operator.xxz(ctx, L, N, 1.0, 1.0, wl.xxz_fields(L, 1.0, 2), True)
    D = op.D
    print(f"orthogonalization D={D} k={k}")
    sys.stdout.flush()
    rng = np.random.default_rng(D + k)
    # k orthonormal columns, then v_k with a part along each and one across
    Q, _ = np.linalg.qr(rng.standard_normal((D, k + 1)))
    V = np.zeros((k + 2, D))
    V[:k] = Q[:, :k].T
    u = Q @ np.concatenate([rng.standard_normal(k), [0.8]])
    u /= np.linalg.norm(u)
    V[k] = u
    tV = torch.as_tensor(V.ravel(), device="cuda:0")
    al = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    be = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    g = 0.75  # the filter of order 0 is this multiple of the identity
    pk.lanczos_step(op, 0.0, 10.0, np.array([g]), tV, k, al, be)
    torch.cuda.synchronize()
    got, a, b = tV.cpu().numpy().reshape(k + 2, D), float(al[0]), float(be[0])
    assert np.array_equal(got[:k + 1], V[:k + 1])
    w, ref_a = g * u.astype(np.longdouble), np.longdouble(0)
    for _ in range(2):
        c = V[:k + 1].astype(np.longdouble) @ w
        ref_a += c[k]
        w = w - c @ V[:k + 1]
    # both passes' rounding: k + 1 products of D terms each, of vectors of
    # norm 1 or less
    tol = 4 * (k + 2) * np.sqrt(D) * 2.0 ** -53
    assert abs(a - float(ref_a)) <= tol
    assert abs(b - float(np.linalg.norm(w.astype(float)))) <= tol
    if b > 1e3 * tol:
        n = w / np.sqrt((w * w).sum())
        assert np.max(abs(got[k + 1] - n.astype(float))) <= 2 * tol / b
