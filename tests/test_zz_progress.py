"""How a single-map solve is enqueued and its records are read does not change
what it computes: one or several chunks per graph, records in pinned or in
device memory, against the solve without a context, which enqueues every
kernel by itself and copies its records.  The same kernels run in the same
order, so every value is the same to the bit."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _args(prec):
    import torch
    dt = torch.float32 if prec == "f32" else torch.float64
    p = synth.make_problem(64, 64, 5, mask_frac=0.05)

    def t(a):
        return torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")

    mask = torch.tensor(np.ascontiguousarray(p.mask), dtype=torch.uint8, device="cuda")
    return t(p.d), t(p.s_k), t(p.n_pix), t(p.p_oof), t(p.p_stripe), mask


def _same(x, y):
    assert bool((x[0] == y[0]).all())
    assert x[1]["sweeps"] == y[1]["sweeps"] and x[1]["n_records"] == y[1]["n_records"]
    np.testing.assert_array_equal(x[2], y[2])


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("rtol", [0.0, 1e-30])
@pytest.mark.parametrize("every,sweeps", [(8, 24), (8, 32), (8, 33), (4, 28), (1, 9), (5, 42)])
def test_chunks_per_graph(gpu_lib, prec, rtol, every, sweeps):
    """Budgets below, at and past a whole number of graphs, with a part of a
    chunk left, twice in one context; a tolerance (never met here) keeps one
    chunk per graph."""
    print(f"chunks {prec} rtol={rtol} {every} {sweeps}", flush=True)
    args = _args(prec)
    sched = gpu_lib.Schedule(lambdas=[float(l) for l in np.geomspace(50, 1, sweeps)], rtol=rtol,
                             max_sweeps=sweeps, monitor_every=every)
    a, ra, ta = gpu_lib.solve_noalloc(*args, schedule=sched)
    ctx = gpu_lib.Context(64, 64, prec)
    for _ in range(2):
        _same((a, ra, ta), ctx.solve(*args, schedule=sched))
        assert ra["sweeps"] == sweeps
    ctx.close()


@pytest.mark.parametrize("budget", [4096, 4097])
def test_records_in_pinned_and_device_memory(gpu_lib, budget):
    """One record per sweep, for 4096 sweeps (pinned) and 4097 (device)."""
    print(f"records {budget}", flush=True)
    args = _args("f64")
    sched = gpu_lib.Schedule(lambdas=[20.0, 3.0, 1.0], rtol=0.0, max_sweeps=budget, monitor_every=1)
    a, ra, ta = gpu_lib.solve_noalloc(*args, schedule=sched)
    ctx = gpu_lib.Context(64, 64, "f64")
    _same((a, ra, ta), ctx.solve(*args, schedule=sched))
    ctx.close()
