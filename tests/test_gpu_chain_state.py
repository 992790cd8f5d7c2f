"""The three-level chain's data-like field d_0 is formed from the two stored
messengers instead of being stored.  Its weights are checked against the
oracle (which stores every field) where they are extreme: modes without signal
(S = 0), projected modes (infinite 1/f variance), a tiny lent floor, lambda
rising and falling from sweep to sweep, and warm starts, whose fields no sweep
has formed."""

import dataclasses

import numpy as np
import pytest

import oracle
import synth
from parity_checks import assert_parity

pytestmark = pytest.mark.gpu

JUMPS = [30.0, 2.0, 900.0, 1.0, 7.0, 7.0, 0.5, 1e4, 1.0, 1.0, 40.0, 3.0, 1.0]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("warm", [False, True])
@pytest.mark.parametrize("floor_frac", [0.5, 1e-3])
@pytest.mark.parametrize("every,shape", [(1, (64, 64)), (5, (64, 128)), (13, (384, 64))])
def test_extreme_weights(gpu_lib, prec, warm, floor_frac, every, shape):
    import torch
    print(f"chain state {prec} {shape} warm={warm} floor={floor_frac} K={every}", flush=True)
    p = synth.make_problem(*shape, 31, mask_frac=0.05)
    s_k, p_oof = np.array(p.s_k), np.array(p.p_oof)
    s_k[shape[0] // 4: shape[0] // 4 + 3] = 0.0
    s_k[shape[0] - shape[0] // 4 - 2: shape[0] - shape[0] // 4 + 1] = 0.0
    s_k[:, 9] = 0.0
    p_oof[2, 3] = np.inf
    p_oof[0, 9] = np.inf
    p = dataclasses.replace(p, s_k=s_k, p_oof=p_oof)
    dt = torch.float32 if prec == "f32" else torch.float64

    def t(a):
        return torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    start = np.float32(1.2 * p.s_true).astype(np.float64) if warm else None
    ctx = gpu_lib.Context(*shape, prec)
    sched = gpu_lib.Schedule(lambdas=JUMPS, rtol=0.0, max_sweeps=len(JUMPS), monitor_every=every,
                             floor_frac=floor_frac)
    s, rep, _ = ctx.solve(t(p.d), t(p.s_k), t(p.n_pix), t(p.p_oof), t(p.p_stripe),
                          torch.tensor(p.mask, device="cuda"), schedule=sched,
                          s_init=t(start) if warm else None)
    assert rep["sweeps"] == len(JUMPS)
    ref = oracle.solve(p, oracle.FixedSchedule(JUMPS),
                       settings=oracle.Settings(floor_frac=floor_frac), s_init=start,
                       max_sweeps=len(JUMPS), monitor_every=len(JUMPS))
    assert_parity(s.cpu().numpy().astype(np.float64), ref.s, prec)
