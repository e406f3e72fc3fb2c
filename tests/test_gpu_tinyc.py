"""The first layer on four-channel 8-bit images: 8-bit weights and fixed-point
scales, bit for bit against the oracle.  Output widths on both sides of a
unit's 32, 64 and 128 pixels, rows that end inside a unit, filters that fill
their form's pieces and that do not, a scale outside fp32 (the fp64 scaling), output
channels that are not whole tiles, fp32, 8- and 4-bit outputs, and outputs the
form refuses (the tiled kernel).  Images hold 0 and 255 at their borders."""
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


# B, H, W, O, R, S, stride (h, w), pad (h, w)
CASES = [
    (2, 31, 45, 64, 7, 7, (2, 2), (3, 3)),      # 23 wide: four rows a unit
    (1, 20, 130, 64, 7, 7, (2, 2), (3, 3)),     # 65 wide
    (1, 9, 259, 32, 7, 7, (2, 2), (3, 3)),      # 130 wide: a second unit of two pixels
    (1, 12, 64, 96, 3, 3, (1, 1), (1, 1)),
    (1, 13, 33, 16, 4, 4, (1, 3), (2, 0)),
    (1, 11, 40, 80, 5, 5, (1, 1), (2, 2)),
    (2, 51, 63, 96, 11, 11, (4, 4), (0, 0)),
    (1, 30, 70, 32, 11, 12, (2, 1), (5, 6)),    # no form
    (2, 30, 250, 64, 7, 7, (2, 2), (3, 3)),     # 125 wide: a full unit
    (40, 21, 9, 48, 7, 8, (1, 2), (3, 4)),      # many images, units mostly empty
    (1, 16, 20, 100, 7, 7, (2, 2), (3, 3)),     # whole fp32 pieces, no whole code pieces
    (1, 16, 20, 34, 3, 3, (1, 1), (1, 1)),      # neither
    (1, 40, 20, 32, 13, 13, (1, 1), (6, 6)),    # no form
]


def image(case):
    B, H, W = case[:3]
    q = fi.rng("tinyc", *case[:6]).integers(0, 256, (B, H, W, 4)).astype(np.uint8)
    q[:, 0], q[:, -1], q[:, :, 0], q[:, :, -1] = 255, 0, 0, 255
    return q


def check(layer, ref, O, tag):
    y = layer(0, None)
    np.testing.assert_array_equal(y.cpu().numpy().reshape(ref.shape).view(np.uint32), ref.view(np.uint32), err_msg=tag)
    so = torch.tensor([float(np.abs(ref).max()) / 150.0], device="cuda")
    for bits in (8, 4):
        want, _ = fgq.fgq_quantize_act(y, bits, scale_in=so)
        assert torch.equal(layer(bits, so).view(-1), want), tag


@pytest.mark.parametrize("case", CASES)
def test_w8(case):
    B, H, W, O, R, S, st, pad = case
    w = fi.rng("tinyc-w", *case[:6]).standard_normal((O, 4, R, S)).astype(np.float32)
    w[0] = 1.0
    W8, fl = oracle.w8_quantize(w)
    q, sx = image(case), np.float32(0.0117)
    prep = fgq.fgq_prepare_weights_w8(dev(w))
    ref = oracle.conv2d_w8(q.reshape(-1), 8, sx, (B, H, W, 4), W8, fl, O, R, S, st, pad)
    check(lambda b, so: fgq.fgq_conv2d_w8(dev(q).view(-1), 8, dev(np.array([sx])), (B, H, W, 4), prep, O, R, S, st, pad,
                                          b, so), ref, O, "w8")


@pytest.mark.parametrize("case", CASES[:2] + CASES[8:9])
def test_fixed_point(case):
    B, H, W, O, R, S, st, pad = case
    w = fi.he_weights(O, 4, R, S, "tinyc")
    t, a, _ = oracle.ternarize(w, 4)
    A, fl = oracle.dfp_alpha(a, 8)
    codes = oracle.pack_codes(t)
    q, sx = image(case), np.float32(0.0117)
    prep = fgq.fgq_prepare_weights_dfp(dev(codes), dev(a), O, R * S * 4, 4, 8)
    ref = oracle.conv2d_dfp(q.reshape(-1), 8, sx, (B, H, W, 4), codes, A, fl, O, R, S, st, pad, 4)
    check(lambda b, so: fgq.fgq_conv2d_dfp(dev(q).view(-1), 8, dev(np.array([sx])), (B, H, W, 4), dev(codes), prep, O,
                                           R, S, st, pad, 4, b, so), ref, O, "dfp")


def test_scale_outside_fp32():
    # s_x 2^-fl below the fp32 range: the fp64 scaling decides the result
    case = CASES[0]
    B, H, W, O, R, S, st, pad = case
    w = fi.rng("tinyc-tiny", O, R).standard_normal((O, 4, R, S)).astype(np.float32) * np.float32(1e-30)
    W8, fl = oracle.w8_quantize(w)
    q, sx = image(case), np.float32(3e-17)
    ref = oracle.conv2d_w8(q.reshape(-1), 8, sx, (B, H, W, 4), W8, fl, O, R, S, st, pad)
    y = fgq.fgq_conv2d_w8(dev(q).view(-1), 8, dev(np.array([sx])), (B, H, W, 4), fgq.fgq_prepare_weights_w8(dev(w)), O,
                          R, S, st, pad)
    np.testing.assert_array_equal(y.cpu().numpy().reshape(ref.shape).view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("sx,so", [(-1e30, 1e-10), (1e30, 1e-10), (-0.0117, 0.02), (0.0117, 1e-37), (-0.0117, 1e-37)])
def test_codes_of_any_quotient(sx, so):
    # quotients y / so past fp32 on either side, also by a negative s_x:
    # saturated codes, as the quantization of the fp32 output gives
    case = CASES[8]
    B, H, W, O, R, S, st, pad = case
    w = fi.rng("tinyc-sign", O, R).standard_normal((O, 4, R, S)).astype(np.float32)
    q, prep = dev(image(case)).view(-1), fgq.fgq_prepare_weights_w8(dev(w))
    args = (q, 8, dev(np.array([sx], np.float32)), (B, H, W, 4), prep, O, R, S, st, pad)
    y = fgq.fgq_conv2d_w8(*args)
    scale = dev(np.array([so], np.float32))
    for bits in (8, 4):
        want, _ = fgq.fgq_quantize_act(y, bits, scale_in=scale)
        assert torch.equal(fgq.fgq_conv2d_w8(*args, bits, scale).view(-1), want), bits
