"""The per-group layer (G = 64) on the tiled kernel's forms: one wave set and
two (at most a workgroup per compute unit), reductions that leave the second
set a step fewer or half a step, the 4-bit form at its extremes (every
activation 15 or 0, every weight +1 or -1, where a group's sum reaches 64 * 15)
and with a random map, one-step fp32 outputs.  Within 1e-5 of the summand
magnitude of the oracle; codes and residual outputs bit for bit against the
fp32 output."""
import numpy as np
import pytest
import torch

import fgq_inputs as fi
import oracle

fgq = pytest.importorskip("paper_1705_01462_amd")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# B, H, W, C, O, R, all with more tiles of 32 rows than the kernel that divides
# K over a workgroup's waves takes
CASES = [
    (1, 47, 47, 128, 260, 3),    # two sets of 5 and 4 steps
    (1, 53, 52, 448, 200, 1),    # two sets, 3.5 steps
    (1, 66, 67, 192, 132, 1),    # one set, 1.5 steps
    (2, 97, 101, 64, 130, 1),    # one set, half a step: the one-step form
    (2, 97, 101, 128, 96, 3),    # one set, 9 steps
    (1, 66, 67, 192, 130, 1),    # single stores, residual values in batches
    (2, 97, 101, 192, 622, 1),   # two steps, single stores of 12 M values: the int8 form
    (2, 97, 101, 320, 820, 1),   # three steps, 16 M values: staged, the 4-bit form
    (2, 97, 101, 320, 818, 1),   # the same, single stores: the int8 form
]


@pytest.mark.parametrize("kind", ["random", "max"])
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("case", CASES)
def test_forms(case, bits, kind):
    B, H, W, C, O, R = case
    G, K, M, shape = 64, R * R * C, B * H * W, (B, H, W, C)
    w = fi.he_weights(O, C, R, R, "group-forms")
    x = fi.relu_gauss(shape, "group-forms")
    if kind == "max":  # equal magnitudes keep every weight; whole maps at the largest code, borders and a hole at 0
        w = np.sign(w) * np.float32(0.05)
        w[0] = np.float32(0.05)
        w[1] = -np.float32(0.05)
        x[:] = 1.0
        x[:, H // 2, :, :] = 0.0
    t, a, _ = oracle.ternarize(w, G)
    codes = oracle.pack_codes(t)
    q, s = oracle.quantize_act(x, bits)
    prep = fgq.fgq_prepare_weights(dev(codes), dev(a), O, K, G)
    args = (dev(q), bits, dev(np.array([s], np.float32)), shape, dev(codes), dev(a), O, R, R, 1, R // 2, G)
    y = fgq.fgq_conv2d(*args, prepared=prep)
    rows = np.unique(np.r_[0:64, M // 2:M // 2 + 8, M - 66:M, fi.rng("group-forms").integers(0, M, 64)])
    ref, mag = oracle.conv2d_rows(q, bits, s, shape, codes, a, O, R, R, (1, 1), (R // 2, R // 2), G, rows)
    err = np.abs(y.view(M, O).cpu().numpy()[rows].astype(np.float64) - ref)
    assert np.all(err <= 1e-5 * mag)
    so = torch.tensor([float(y.max()) / 200.0], device="cuda")
    want, _ = fgq.fgq_quantize_act(y, bits, scale_in=so)
    assert torch.equal(fgq.fgq_conv2d_q(*args, bits, so, prepared=prep).view(-1), want)
    res = torch.randn(y.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    yr, qr = fgq.fgq_conv2d_residual_q(*args, res, bits, so, prepared=prep)
    assert torch.equal(yr, (y + res).clamp_(min=0))
    want, _ = fgq.fgq_quantize_act(yr, bits, scale_in=so)
    assert torch.equal(qr.view(-1), want)
