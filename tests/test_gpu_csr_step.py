"""The step kernel of stored sparse matrices at the edges of its blocks: rows
of no entry, of one more or less than the gathers in flight, of exactly the
LDS stage and one more, blocks that begin off a dword of the code array, a
last block of a few rows; plain values, one value, and coded values.  The
kernel treats each row by itself, so the matrices are not symmetric."""
import sys

import numpy as np
import pytest

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


@pytest.mark.parametrize("D", [1, 127, 128, 129, 4000])
@pytest.mark.parametrize("values", ["plain", "one", "coded"])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_rows(pk, ctx, D, values, prec):
    print(f"csr step D={D} {values} {prec}")
    sys.stdout.flush()
    import scipy.sparse as sp
    rng = np.random.default_rng(D)
    lens = rng.choice([0, 1, 5, 7, 8, 9, 16, 17, 31, 60], D)
    if D == 4000:
        lens[[3, 4, 900, 3999]] = 3072, 3073, 3071, 3072
        lens[2000:2300] = 0
    lens = np.minimum(lens, D - 1)
    cols = [np.sort(rng.choice(np.delete(np.arange(D), r) if n > 100 else
                               np.setdiff1d(rng.integers(0, D, 4 * n + 8), [r]),
                               n if n > 100 else min(n, 1), replace=False))
            if n == 1 or n > 100 else
            np.setdiff1d(rng.integers(0, D, 2 * n), [r])[:n] for r, n in enumerate(lens)]
    indptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])])
    idx = np.concatenate(cols).astype(np.int32) if indptr[-1] else np.zeros(0, np.int32)
    val = {"plain": rng.standard_normal(len(idx)), "one": np.full(len(idx), 0.37),
           "coded": rng.choice([0.5, -0.25, 1.75, 0.1], len(idx))}[values]
    H = sp.csr_matrix((val, idx, indptr), shape=(D, D))
    diag = rng.standard_normal(D)
    H = (H + sp.diags(diag)).tocsr()
    H.sort_indices()
    op = pk.Operator.csr(ctx, D, H.indptr, H.indices, H.data)
    if values != "plain" and len(idx):
        assert op.optimize_mapping() == len(np.unique(val))
    p, dt, u = ((pk.FP64, torch.float64, 2.0 ** -53) if prec == "fp64"
                else (pk.FP32, torch.float32, 2.0 ** -24))
    v, b1, b2 = (rng.standard_normal(D).astype(np.float32).astype(np.float64)
                 for _ in range(3))
    E_c, dE, a_i = 0.2, 17.0, 0.023
    t = torch.as_tensor(b2, dtype=dt, device="cuda:0")
    pk.clenshaw_step(op, E_c, dE, a_i, torch.as_tensor(v, dtype=dt, device="cuda:0"),
                     torch.as_tensor(b1, dtype=dt, device="cuda:0"), t, p)
    torch.cuda.synchronize()
    got = t.cpu().numpy().astype(np.float64)
    ref = a_i * v + 2.0 * (H @ b1 - E_c * b1) / dE - b2
    # one rounding for each entry of a row and its value, and a few of the
    # scalars and the last three terms
    n = np.diff(H.indptr)
    mag = abs(a_i * v) + 2.0 * (abs(H) @ abs(b1) + abs(E_c * b1)) / dE + abs(b2)
    assert np.all(np.abs(got - ref) <= (n + 10) * u * mag)
