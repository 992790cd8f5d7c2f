"""The convolution's tilings (8 x 8, 8 x 16 and 16 x 16 pixels; 16 to 96 output
channels; one, three or nine taps of weights staged at a time) against a plain
float64 sum over taps, at the image sizes where each is chosen.

Tolerance: products of bfloat16 values are exact in float32, sums of at most
1 152 of them err by 1e-6 of their size, and the result is rounded to the
nearest bfloat16, whose spacing at v is 2^(floor(log2 |v|) - 7): each value
within half that spacing of the reference, plus 1e-4 of the rms; relative L2
(the rounding errors' rms) <= 2^-9."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _ref(x, w, b):
    import torch
    x, w = x.double(), w.double()
    out = torch.zeros(x.shape[:3] + (w.shape[3],), dtype=torch.float64, device=x.device)
    if b is not None:
        out += b.double()
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            out += torch.roll(x, (-dy, -dx), (1, 2)) @ w[dy + 1, dx + 1]
    return out


@pytest.mark.parametrize("shape", [(1, 8, 8), (3, 8, 16), (2, 64, 8), (1, 16, 32), (2, 256, 256)])
@pytest.mark.parametrize("ci,co", [(32, 32), (32, 96), (64, 64), (64, 32), (96, 96), (96, 64),
                                   (128, 96), (128, 128)])
def test_conv_tilings(gpu_lib, shape, ci, co):
    import torch
    from paper_1704_00865_amd import nn
    print(f"conv tiles {shape} {ci}->{co}", flush=True)
    g = torch.Generator().manual_seed(sum(shape) + ci + 7 * co)
    x = torch.randn(shape + (ci,), generator=g).to(torch.bfloat16).cuda()
    w = (0.1 * torch.randn((3, 3, ci, co), generator=g)).to(torch.bfloat16).cuda()
    b = torch.randn(co, generator=g).cuda()
    fwd = nn.conv3x3(1, x, w, b, ci=ci, co=co).double()
    gy = torch.randn(shape + (co,), generator=g).to(torch.bfloat16).cuda()
    adj = nn.conv3x3(2, gy, w, ci=ci, co=co).double()
    wt = w.flip(0, 1).transpose(2, 3).contiguous()
    for got, ref in ((fwd, _ref(x, w, b).relu()), (adj, _ref(gy, wt, None))):
        err = (got - ref).abs()
        rms = ref.square().mean().sqrt()
        assert float(err.norm() / ref.norm()) <= 2.0 ** -9
        spacing = torch.exp2(torch.floor(torch.log2(ref.abs().clamp_min(1e-30))) - 7)
        assert bool((err <= 0.5 * spacing + 1e-4 * rms).all())


@pytest.mark.parametrize("shape", [(1, 8, 8), (3, 8, 16), (2, 64, 8), (1, 16, 32), (2, 8, 64),
                                   (1, 16, 256)])
@pytest.mark.parametrize("ci,co", [(32, 32), (96, 64), (128, 96)])
def test_weight_gradient_slabs(gpu_lib, shape, ci, co):
    """64-pixel slabs of one, two, four and eight image rows: float32 sums of
    exact products over at most 4 096 pixels, relative L2 <= 1e-5."""
    import torch
    from paper_1704_00865_amd import nn
    print(f"wgrad slabs {shape} {ci}x{co}", flush=True)
    g = torch.Generator().manual_seed(sum(shape) + ci + 7 * co)
    x = torch.randn(shape + (ci,), generator=g).to(torch.bfloat16).cuda()
    gy = torch.randn(shape + (co,), generator=g).to(torch.bfloat16).cuda()
    got = nn.conv3x3(3, x, g=gy, ci=ci, co=co).double()
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            sh = torch.roll(x.double(), (-dy, -dx), (1, 2)).reshape(-1, ci)
            ref = sh.t() @ gy.double().reshape(-1, co)
            assert float((got[dy + 1, dx + 1] - ref).norm() / ref.norm()) <= 1e-5


def test_nonfinite_inputs_reach_their_neighbours_only(gpu_lib):
    import torch
    from paper_1704_00865_amd import nn
    print("conv non-finite", flush=True)
    x = torch.ones((1, 16, 16, 32), dtype=torch.bfloat16, device="cuda")
    x[0, 4, 15, 3] = float("nan")
    x[0, 10, 5, 0] = float("inf")
    w = torch.full((3, 3, 32, 32), 0.5, dtype=torch.bfloat16, device="cuda")
    out = nn.conv3x3(0, x, w, ci=32, co=32).float().cpu().numpy()[0]
    nan = np.isnan(out).all(axis=2)
    inf = np.isposinf(out).all(axis=2)
    assert nan.sum() == 9 and inf.sum() == 9
    assert nan[3:6, [14, 15, 0]].all() and inf[9:12, 4:7].all()
    assert (out[~(nan | inf)] == 144.0).all()
