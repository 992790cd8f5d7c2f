"""Host memory that every thread of a program holds for solve_noalloc (read
from the built library's program headers), and the longest tables in it."""

import os
import struct

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1704_00865_amd", "libwf.so")


def _thread_local_bytes(path):
    """Size of an ELF64 file's thread-local segment."""
    with open(path, "rb") as f:
        head = f.read(64)
        assert head[:5] == b"\x7fELF\x02"
        off, = struct.unpack_from("<Q", head, 32)
        size, count = struct.unpack_from("<HH", head, 54)
        f.seek(off)
        table = f.read(size * count)
    total = 0
    for i in range(count):
        kind, = struct.unpack_from("<I", table, i * size)
        if kind == 7:  # PT_TLS
            total += struct.unpack_from("<Q", table, i * size + 40)[0]
    return total


@pytest.mark.skipif(not os.path.exists(LIB), reason="libwf.so not built")
def test_thread_local_tables():
    """The twiddle tables of a map's two sides, in whichever precision needs
    more room: one table of 4096 complex float32 values a side, or three of
    2048 complex float64 ones; and a kilobyte for whatever else there is."""
    tables = 2 * max(4096 * 2 * 4, 3 * 2048 * 2 * 8)
    assert _thread_local_bytes(LIB) <= tables + 1024


@pytest.mark.gpu
@pytest.mark.parametrize("prec,shape", [("f64", (64, 2048)), ("f32", (4096, 64)),
                                        ("f64", (1536, 64)), ("f32", (64, 64))])
def test_longest_tables(gpu_lib, prec, shape):
    """The longest sides one after the other on one thread: the same map to the
    bit as with a context."""
    import torch
    p = synth.make_problem(*shape, 45)
    args = [torch.tensor(np.ascontiguousarray(a), device="cuda",
                         dtype=torch.float32 if prec == "f32" else torch.float64)
            for a in (p.d, p.s_k, p.n_pix, p.p_oof, p.p_stripe)]
    sched = gpu_lib.Schedule(lambdas=[50.0, 5.0, 1.0], rtol=0.0, max_sweeps=6, monitor_every=4)
    a, _, ta = gpu_lib.solve_noalloc(*args, schedule=sched)
    b, _, tb = gpu_lib.solve(*args, schedule=sched)
    assert bool((a == b).all())
    np.testing.assert_array_equal(ta, tb)
