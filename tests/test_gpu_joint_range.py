"""The joint objective where its links' variances, or its partial sums, are at
the ends of their range: maps in units far from the data's own, extreme per-mode
weights, and the lengths whose row blocks hold two rows.

Tolerances are those of the ordinary maps, 1e-8 in float64 and 1e-4 in float32:
units do not change a term's relative error, and relative changes of every
Fourier value by 3e-16 and 3e-7 move the oracle's J of these weights by at most
4e-11 and 8e-8."""

import dataclasses

import numpy as np
import pytest

import oracle
import synth
from oracle.bases import full_from_half

pytestmark = pytest.mark.gpu

JTOL = {"f64": 1e-8, "f32": 1e-4}
BETA = (0.9, 0.9, 0.95)  # every Nbar_i > 0, so J is finite
JUMPS = [30.0, 2.0, 900.0, 1.0, 7.0, 7.0, 0.5, 1e4, 1.0, 1.0, 40.0, 3.0, 1.0]


def _tensors(p, prec):
    import torch
    dt = torch.float32 if prec == "f32" else torch.float64

    def t(a):
        return None if a is None else torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    mask = None if p.mask is None else torch.tensor(p.mask, dtype=torch.uint8, device="cuda")
    return dict(d=t(p.d), s_k=t(p.s_k), n_pix=t(p.n_pix), p_oof=t(p.p_oof), p_stripe=t(p.p_stripe),
                mask=mask)


def _scaled_solve(gpu_lib, args, power, chain):
    scaled = {k: v * 2.0 ** (power if k == "d" else 2 * power)
              if v is not None and k != "mask" else v for k, v in args.items()}
    sched = gpu_lib.Schedule(lambdas=[30.0, 5.0, 1.0], rtol=0.0, max_sweeps=12, monitor_every=4,
                             beta=BETA, chain=chain)
    return gpu_lib.solve(**scaled, schedule=sched)[1:]


@pytest.mark.parametrize("chain", ["three", "merged", "augmented"])
def test_units(gpu_lib, chain):
    """J has no units: fields times 2^power and variances times its square (an
    exact scaling in float64) leave it as it is, up to where the residual's
    squares leave the double range and the call says so."""
    args = _tensors(synth.make_problem(64, 64, 31, mask_frac=0.08), "f64")
    _, plain = _scaled_solve(gpu_lib, args, 0, chain)
    assert np.all(plain[:, 5] > 0)
    for power in (-200, 166):
        rep, trace = _scaled_solve(gpu_lib, args, power, chain)
        np.testing.assert_allclose(trace[:, 5], plain[:, 5], rtol=JTOL["f64"])
        assert rep["chi2_joint"] == trace[-1, 5]
    with pytest.raises(gpu_lib.WFError) as e:
        _scaled_solve(gpu_lib, args, 250, chain)
    assert e.value.status == -3  # WF_ENONFINITE


def _joint(st, x, lam):
    """The oracle's J with the signal's two terms combined in Fourier space,
    |t_0|^2 / (S + T_0): defined where S = 0."""
    lv = st.levels
    full = full_from_half(st.S_chain.eig, st.shape[1]) + lam * lv[0].tau
    total = float(np.sum(np.abs(np.fft.fft2(x.t[0], norm="ortho")) ** 2 / full))
    for i in range(len(lv)):
        if i > 0:
            dl = x.t[i] - x.dd[i - 1]
            total += float(np.sum(dl * dl)) / (lam * lv[i].tau)
        right = x.dd[i] if i < len(lv) - 1 else st.d
        total += lv[i].nbar.inv_quad(right - x.t[i])
    return total


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("floor_frac", [0.5, 1e-3])
@pytest.mark.parametrize("sweeps,every,shape", [(4, 1, (64, 64)), (9, 5, (64, 128)),
                                                (13, 13, (384, 64))])
def test_extreme_weights(gpu_lib, prec, floor_frac, sweeps, every, shape):
    """Modes without signal, projected modes (infinite 1/f variance), a tiny
    lent floor, lambda rising and falling."""
    p = synth.make_problem(*shape, 31, mask_frac=0.05)
    s_k, p_oof = np.array(p.s_k), np.array(p.p_oof)
    s_k[shape[0] // 4: shape[0] // 4 + 3] = 0.0
    s_k[shape[0] - shape[0] // 4 - 2: shape[0] - shape[0] // 4 + 1] = 0.0
    s_k[:, 9] = 0.0
    p_oof[2, 3] = np.inf
    p_oof[0, 9] = np.inf
    p = dataclasses.replace(p, s_k=s_k, p_oof=p_oof)
    lams = JUMPS[:sweeps]
    sched = gpu_lib.Schedule(lambdas=lams, rtol=0.0, max_sweeps=sweeps, monitor_every=every,
                             floor_frac=floor_frac, beta=BETA)
    _, rep, _ = gpu_lib.solve(**_tensors(p, prec), schedule=sched)
    settings = oracle.Settings(floor_frac=floor_frac, beta=BETA)
    ref = oracle.solve(p, oracle.FixedSchedule(lams), settings=settings, max_sweeps=sweeps,
                       monitor_every=sweeps)
    want = _joint(oracle.setup(p, settings), ref.state, lams[-1])
    print(f"J {rep['chi2_joint']:.8e}, oracle {want:.8e}", flush=True)
    assert rep["chi2_joint"] == pytest.approx(want, rel=JTOL[prec])


@pytest.mark.parametrize("prec,shape", [("f32", (64, 4096)), ("f64", (64, 2048))])
@pytest.mark.parametrize("chain", ["three", "augmented"])
def test_two_rows_per_block(gpu_lib, prec, shape, chain):
    """A band of two rows leaves twice the row blocks' partial sums, behind
    which the column blocks' lie."""
    p = synth.make_problem(*shape, 33, mask_frac=0.05)
    lams = list(oracle.cooling_ramp(5, 9, 300.0))
    sched = gpu_lib.Schedule(lambdas=lams, rtol=0.0, max_sweeps=9, monitor_every=4, beta=BETA,
                             chain=chain)
    _, _, trace = gpu_lib.solve(**_tensors(p, prec), schedule=sched)
    ref = oracle.solve(p, oracle.FixedSchedule(lams),
                       settings=oracle.Settings(beta=BETA, chain=chain), max_sweeps=9,
                       monitor_every=4, record_joint=True)
    assert trace.shape[0] == len(ref.trace) == 3
    np.testing.assert_allclose(trace[:, 5], [o[5] for o in ref.trace], rtol=JTOL[prec])
