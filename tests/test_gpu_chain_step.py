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
