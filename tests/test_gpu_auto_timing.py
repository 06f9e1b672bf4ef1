"""The automatic precision compares the filters that a solve would run: for
short chains and quantum suns the reported time of a step is that of the
resident recurrence (measured through a filter of 4,000 steps), not that of a
launch of the step kernel, which takes two to three times as long."""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import sys, time
import numpy as np, torch
import paper_2605_10191_amd as pk
import workloads as wl
ctx = pk.Context(0)
if sys.argv[1] == "chain":
    L = 12
    op = pk.Operator.xxz(ctx, L, 6, 1.0, 1.0, wl.xxz_fields(L, 1.0, 0), True)
else:
    N, L = 3, 9
    q = wl.qsun_draws(N, L, 0)
    op = pk.Operator.qsun(ctx, N, L, q["A"], 1.0, 1.0, 0.75, q["u"], q["n_of_j"], q["h"])
x0 = torch.tensor(wl.start_vector(op.D, 0), device="cuda:0")
pk.solve(op, x0, 8, 0.5, "normalized", precision=pk.AUTO, allow_partial=True)
K = 4000
for dt, p in ((torch.float64, pk.FP64), (torch.float32, pk.FP32)):
    v = torch.randn(op.D, device="cuda:0", dtype=dt)
    best = 1e9
    for _ in range(4):
        t = time.perf_counter()
        pk.filter_apply(op, 0.0, 40.0, np.full(K + 1, 1e-3), v, p)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    print("filter", 1e6 * best / K, flush=True)
"""


@pytest.mark.parametrize("model", ["chain", "qsun"])
def test_auto_times_the_resident_filter(model):
    r = subprocess.run([sys.executable, "-c", CHILD, model], cwd=ROOT, capture_output=True,
                       text=True, timeout=100, env=dict(os.environ, POLFED_VERBOSE="1"))
    assert r.returncode == 0, r.stderr[-2000:]
    m = re.search(r"precision auto: step ([0-9.]+) us FP64, ([0-9.]+) us FP32", r.stderr)
    timed = [float(x) for x in m.groups()]
    steps = [float(x) for x in re.findall(r"filter ([0-9.]+)", r.stdout)]
    print(model, "timed", timed, "filter", steps)
    for t, f in zip(timed, steps):
        assert 0.6 * f <= t <= 1.5 * f
