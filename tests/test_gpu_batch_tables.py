"""Batched solves that replay a graph from the first application on, where the
resident recurrence was chosen before its tables were there: set by the caller
on fresh operators, and remembered for the pattern after the operators that
held the tables are gone (33 columns at L = 15 take 8 slabs, a single one 16; 9
columns at L = 16 take 16, a single one 32).  The pairs are those of direct
launches."""
import gc

import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_parity import dev, host, pk, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N_EV = 8


@pytest.fixture
def own(pk):
    return pk.Context(0)


def make(pk, ctx, L, B):
    return [pk.Operator.xxz(ctx, L, L // 2, 1.0, 1.0, wl.xxz_fields(L, 3.0, 70 + c), True)
            for c in range(B)]


def energies(pk, ops, graph, prec):
    x0s = [dev(wl.start_vector(ops[0].D, c)) for c in range(len(ops))]
    res, status = pk.solve_batch(ops, x0s, N_EV, 0.5, "normalized", graph=graph, precision=prec)
    assert status == "OK"
    return np.array([host(r[0]) for r in res])


def test_variant_set_on_fresh_operators(pk, own):
    say("batch variant 5 set, graph=1, no tables yet")
    L, B = 15, 33
    ops = make(pk, own, L, B)
    assert ops[0].set_batch_kernel(B, pk.FP32, 5) == 5
    got = energies(pk, ops, 1, pk.FP32)
    assert ops[0].set_batch_kernel(B, pk.FP32, -2) == 5
    assert np.max(np.abs(got - energies(pk, ops, 2, pk.FP32))) <= 1e-10 * L


def test_remembered_choice_after_its_operators(pk, own):
    say("batch variant remembered, operators made anew, graph=1")
    L, B = 16, 9
    ops = make(pk, own, L, B)
    ref = energies(pk, ops, 2, pk.FP64)
    say(f"   variant {ops[0].set_batch_kernel(B, pk.FP64, -2)}")
    del ops
    gc.collect()
    assert np.max(np.abs(energies(pk, make(pk, own, L, B), 1, pk.FP64) - ref)) <= 1e-10 * L
