"""Memory of a context that has not solved a map by itself (one that serves
batches): the buffers of its shape, and no pinned room for a solve's records."""

import pytest

pytestmark = pytest.mark.gpu


def _mapped_kb():
    """GPU-visible memory mapped into this process, device and pinned host."""
    total = 0
    for line in open("/proc/self/maps"):
        if "/dev/dri/" in line:
            a, b = (int(x, 16) for x in line.split()[0].split("-"))
            total += b - a
    return total / 1024


def test_unused_context_pins_no_records(gpu_lib):
    """A 64^2 float32 context's buffers come to 266 KB, half of it the partial
    sums of the input checks; pinned room for 4096 records would be 192 KB more."""
    keep = [gpu_lib.Context(64, 64, "f32") for _ in range(8)]
    before = _mapped_kb()
    keep += [gpu_lib.Context(64, 64, "f32") for _ in range(32)]
    each = (_mapped_kb() - before) / 32
    print(f"{each:.0f} KB per context", flush=True)
    assert each <= 360
