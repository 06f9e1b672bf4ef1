"""The products of tall matrices at the edges of the 128 x 128 tiles: one row
or column more and less than a tile, inner dimensions around the chunk of 16,
a side that fits the 64 x 64 tiles, rows that leave XCDs without a tile."""
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


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), device="cuda:0")


@pytest.mark.parametrize("D,m,n", [(1, 1, 65), (127, 15, 128), (128, 16, 129), (129, 17, 127),
                                   (1023, 33, 120), (1025, 1, 257), (3000, 231, 66)])
@pytest.mark.parametrize("subtract", [False, True])
def test_nn(pk, ctx, D, m, n, subtract):
    print(f"wide nn D={D} m={m} n={n} subtract={subtract}")
    sys.stdout.flush()
    rng = np.random.default_rng(D + m + n)
    A, B, C = (rng.standard_normal(s) for s in ((D, m), (m, n), (D, n)))
    t = dev(C.T)
    pk.gemm_nn(ctx, dev(A.T), dev(B.T), t, subtract)
    torch.cuda.synchronize()
    ref = (C if subtract else 0.0) + (-1 if subtract else 1) * (A @ B)
    # m products and sums of a row, and the last difference
    bound = (m + 2) * 2.0 ** -53 * (abs(A) @ abs(B) + abs(C))
    assert np.all(abs(t.cpu().numpy().T - ref) <= 2 * bound)


@pytest.mark.parametrize("D,n1,n2", [(1, 65, 65), (15, 128, 65), (17, 129, 120), (255, 66, 257),
                                     (256, 127, 128), (513, 70, 64), (4097, 64, 200),
                                     (70000, 120, 120)])
def test_tn(pk, ctx, D, n1, n2):
    print(f"wide tn D={D} n1={n1} n2={n2}")
    sys.stdout.flush()
    rng = np.random.default_rng(D + n1 + n2)
    A, B = rng.standard_normal((D, n1)), rng.standard_normal((D, n2))
    G, G2 = (torch.zeros((n2, n1), dtype=torch.float64, device="cuda:0") for _ in range(2))
    pk.gemm_tn(ctx, dev(A.T), dev(B.T), G)
    pk.gemm_tn(ctx, dev(A.T), dev(B.T), G2)
    torch.cuda.synchronize()
    assert torch.equal(G, G2)
    bound = (D + 2) * 2.0 ** -53 * (abs(A).T @ abs(B))
    assert np.all(abs(G.cpu().numpy().T - A.T @ B) <= 2 * bound)
