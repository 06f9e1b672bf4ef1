"""Step kernels of chains with few particles or few holes: tiles with hardly
any segments, runs of a wrapped tile that are empty, workgroups without a
share of the tile table, and both policies of the streamed vectors.  Every row
against the CPU oracle's matrix."""
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


@pytest.mark.parametrize("L,N,periodic", [(22, 1, True), (22, 19, False), (23, 3, True),
                                          (24, 5, True), (25, 22, False), (26, 4, True)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_sparse_tiles(pk, ctx, L, N, periodic, prec):
    h = wl.xxz_fields(L, 3.0, 4)
    H, _ = models.xxz(L, N, 1.0, 1.0, h, periodic)
    op = pk.Operator.xxz(ctx, L, N, 1.0, 1.0, h, periodic)
    p, dt, u = ((pk.FP64, torch.float64, 2.0 ** -53) if prec == "fp64"
                else (pk.FP32, torch.float32, 2.0 ** -24))
    rng = np.random.default_rng(8)
    v, b1, b2 = (rng.standard_normal(op.D).astype(np.float32).astype(np.float64)
                 for _ in range(3))
    E_c, dE, a_i = 0.3, 21.0, 0.019
    ref = a_i * v + 2.0 * (H @ b1 - E_c * b1) / dE - b2
    # a row is a sum of at most L hops, L + 4 terms of the diagonal and the
    # last three, each with a few roundings of its own: L + 24 roundings of
    # the sum of the terms' magnitudes, which a low bond without a hop (added
    # and taken back) raises by L |b1|
    mag = (abs(a_i * v) + 2.0 * (abs(H) @ abs(b1) + (np.abs(h).sum() + 2 * L) * abs(b1)) / dE
           + 2.0 * abs(E_c * b1) / dE + abs(b2))
    tried = 0
    for variant in range(10):
        try:
            op.set_kernel(p, variant)
        except pk.PolfedError:
            continue
        print(f"L={L} N={N} {prec} variant {variant}")
        sys.stdout.flush()
        t = torch.as_tensor(b2, dtype=dt, device="cuda:0")
        pk.clenshaw_step(op, E_c, dE, a_i, torch.as_tensor(v, dtype=dt, device="cuda:0"),
                         torch.as_tensor(b1, dtype=dt, device="cuda:0"), t, p)
        torch.cuda.synchronize()
        got = t.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - ref) <= (L + 24) * u * mag), variant
        tried += 1
    assert tried >= 7


@pytest.mark.parametrize("model,L,N,periodic,n", [
    ("xxz", 4, 2, True, 3), ("tv", 9, 4, True, 2), ("xxz", 12, 6, True, 9),
    ("xxz", 16, 3, False, 17), ("tv", 20, 4, True, 8), ("xxz", 21, 19, True, 5),
    ("xxz", 22, 2, True, 4)])
def test_hamiltonian_on_a_block(pk, ctx, model, L, N, periodic, n):
    """Rayleigh-Ritz on a random orthonormal block: H applied to its columns
    in one launch (up to L = 21) and one by one, odd and even column counts on
    one, two, four and all XCDs a column."""
    print(f"H on a block {model} L={L} N={N} n={n}")
    sys.stdout.flush()
    if model == "xxz":
        f = wl.xxz_fields(L, 2.0, 5)
        H, _ = models.xxz(L, N, 1.0, 1.0, f, periodic)
        op = pk.Operator.xxz(ctx, L, N, 1.0, 1.0, f, periodic)
    else:
        f = wl.tv_onsite(L, 5)
        H, _ = models.tv(L, N, 1.0, 1.0, f, periodic)
        op = pk.Operator.tv(ctx, L, N, 1.0, 1.0, f, periodic)
    rng = np.random.default_rng(L + n)
    V, _ = np.linalg.qr(rng.standard_normal((op.D, n)))
    E, U, res = pk.extract(op, torch.as_tensor(np.ascontiguousarray(V.T), device="cuda:0"),
                           torch.as_tensor(np.eye(n), device="cuda:0"))[:3]
    torch.cuda.synchronize()
    ref, Z = np.linalg.eigh(V.T @ (H @ V))
    norm = abs(H).sum(axis=1).max()
    # a projected entry sums D products of rows of up to L + 5 terms
    tol = (op.D + L + 10) * 2.0 ** -53 * norm * n
    got = np.asarray(E.cpu()).ravel()
    assert np.max(abs(np.sort(got) - ref)) <= tol
    R = H @ (V @ Z) - (V @ Z) * ref
    order = np.argsort(got)
    have = np.asarray(res.cpu()).ravel()[order]
    assert np.max(abs(have - np.linalg.norm(R, axis=0))) <= tol
