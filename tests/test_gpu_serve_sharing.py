"""A short request served beside long ones is not kept waiting by their filters:
a resident launch that fills an XCD would hold every other stream's launches for
its whole length (milliseconds), and did: the latency of L = 14 requests beside
L = 18 was ten times that of the same requests alone."""
import time

import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_parity import dev, host, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_short_requests_beside_long_ones(pk):
    say("served L=14 beside L=18")
    ctx, n_ev = pk.Context(0), 30

    def make(L, seed):
        op = pk.Operator.xxz(ctx, L, L // 2, 1.0, 1.0, wl.xxz_fields(L, 3.0, seed), True)
        return op, dev(wl.start_vector(op.D, seed))

    long_ones = [make(18, s) for s in range(2)]
    short = [make(14, 10 + s) for s in range(7)]

    def latencies(srv):
        out, energies = [], []
        for op, x0 in short:
            ev, _, _, rep, status = srv.submit(op, x0, n_ev, 0.5, "normalized").wait()
            assert status == "OK"
            out.append(rep["t_latency"])
            energies.append(host(ev))
        return np.median(out[2:]), energies  # the first ones time kernels

    with pk.Server(ctx, 8 << 30, max_cols=8) as srv:
        alone, ref = latencies(srv)
        running = [srv.submit(op, x0, n_ev, 0.5, "normalized") for op, x0 in long_ones]
        time.sleep(0.3)
        beside, got = latencies(srv)
        still = not all(r.poll() for r in running)
        for r in running:
            assert r.wait()[4] == "OK"
    say(f"   median latency alone {alone:.3f} s, beside L = 18 {beside:.3f} s")
    assert still, "the long requests ended before the short ones"
    assert max(np.max(np.abs(a - b)) for a, b in zip(ref, got)) <= 1e-9
    assert beside <= 4 * alone + 0.05
