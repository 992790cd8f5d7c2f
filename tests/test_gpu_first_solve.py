"""A context's first solve of a few chunks records the graph of one chunk and no
more, whether the solve can stop early (one chunk per graph throughout) or not
(several, recorded by a later solve, and only where chunks are short)."""

import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("every", [16, 256])
def test_first_solve_records_one_chunk(gpu_lib, every):
    """What the first solve takes over later ones, for a budget of four chunks:
    at most twice as much without a tolerance as with one (four chunks in a graph took
    2.6 times as long with 16 sweeps a chunk, 3.4 times with 256)."""
    import torch
    p = synth.make_problem(64, 64, 1)
    args = [torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")
            for a in (p.d, p.s_k, p.n_pix, p.p_oof, p.p_stripe)]
    extra = {}
    for _ in range(12):
        for rtol in (0.0, 1e-30):
            sched = gpu_lib.Schedule(lambdas=[1.0], rtol=rtol, max_sweeps=4 * every,
                                     monitor_every=every)
            ctx = gpu_lib.Context(64, 64, "f32")
            took = []
            for _ in range(5):
                t0 = time.perf_counter()
                ctx.solve(*args, schedule=sched)
                took.append(time.perf_counter() - t0)
            ctx.close()
            extra.setdefault(rtol, []).append(took[0] - min(took[1:]))
    full, stop = np.median(extra[0.0]), np.median(extra[1e-30])
    print(f"every {every}: first solve +{full * 1e6:.0f} us, with a tolerance +{stop * 1e6:.0f}",
          flush=True)
    assert full <= 2.0 * stop
