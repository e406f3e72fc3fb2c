"""The first layer on four-channel 8-bit images: 8-bit weights and fixed-point
scales, bit for bit against the oracle.  ROWS are layers the row-staging kernel
takes (its rule is repeated here, so a change of the rule shows): one, two and
four output rows a unit, several units a workgroup in uneven runs, several
units a row, rows that end inside a unit, filters that fill their form's pieces
and that do not, output channels that are not whole tiles.  TILED are layers it
leaves to the tiled kernel, for their filter, patch, fill or outputs.  fp32, 8-
and 4-bit outputs, scales outside fp32 (the fp64 scaling) and quotients outside
fp32.  Images hold 0 and 255 at their borders."""
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


# B, H, W, O, R, S, stride (h, w), pad (h, w); units and workgroups of them on
# 256 compute units
ROWS = [
    (1, 12, 64, 96, 3, 3, (1, 1), (1, 1)),      # two rows a unit
    (1, 13, 33, 16, 4, 4, (1, 3), (2, 0)),      # four; whole 8-bit pieces, no 4-bit ones
    (20, 30, 250, 64, 7, 7, (2, 2), (3, 3)),    # 125 wide: one row, 300 units
    (1, 9, 130, 64, 3, 3, (1, 1), (1, 1)),      # 130 wide: a second unit of two pixels
    (2, 9, 29, 32, 5, 5, (1, 1), (2, 2)),       # four rows of eight taps, 29 wide
    (1, 11, 57, 16, 5, 5, (1, 1), (2, 2)),      # two rows, 57 wide
    (1, 10, 243, 32, 7, 8, (1, 1), (3, 4)),     # the form's whole weights; 244 wide, two units
    (24, 81, 80, 32, 5, 5, (1, 1), (2, 2)),     # 80 wide, 1944 units on 768: runs of two and three
    (3, 41, 57, 1024, 3, 3, (1, 1), (1, 1)),    # 63 units on 48 workgroups
    (5, 61, 57, 1024, 3, 3, (1, 1), (1, 1)),    # 155: runs of three and four; fp32 tiled
    (1, 16, 28, 100, 3, 3, (1, 1), (1, 1)),     # whole fp32 pieces, no whole code pieces
]
TILED = [
    (2, 31, 45, 64, 7, 7, (2, 2), (3, 3)),      # a patch of 13 rows
    (1, 20, 130, 64, 7, 7, (2, 2), (3, 3)),     # 65 wide: units mostly empty
    (1, 9, 259, 32, 7, 7, (2, 2), (3, 3)),      # 130 wide, the same
    (1, 11, 40, 80, 5, 5, (1, 1), (2, 2)),      # 40 wide, the same
    (2, 51, 63, 96, 11, 11, (4, 4), (0, 0)),    # no form
    (1, 30, 70, 32, 11, 12, (2, 1), (5, 6)),    # no form
    (40, 21, 9, 48, 7, 8, (1, 2), (3, 4)),      # a patch of ten rows
    (1, 16, 20, 100, 7, 7, (2, 2), (3, 3)),     # a patch of 13 rows
    (1, 16, 20, 34, 3, 3, (1, 1), (1, 1)),      # no whole pieces of any kind
    (1, 40, 20, 32, 13, 13, (1, 1), (6, 6)),    # no form
    (2, 9, 29, 48, 5, 5, (1, 1), (2, 2)),       # one K step, few units
    (5, 21, 33, 256, 3, 3, (1, 1), (1, 1)),     # 33 wide, more than 64 channels
    (1, 30, 250, 128, 7, 7, (2, 2), (3, 3)),    # few units of 128 channels
]
CASES = ROWS + TILED


def takes(case, out_bits):
    """Whether the row-staging kernel takes the layer, and its workgroups'
    units as (units, workgroups)."""
    B, H, W, O, R, S, (sh, sw), (ph, pw) = case
    Ho, Wo = fgq.conv_out_hw(H, W, R, S, (sh, sw), (ph, pw))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    form = 1 if S <= 4 and R <= 4 else 2 if S <= 8 and R <= 7 else 0
    pxw = 1 if Wo <= 32 else 2 if Wo <= 64 else 4
    rows = 4 // pxw
    segs = -(-Wo // (32 * pxw))
    units = B * -(-Ho // rows) * segs
    tiles = units * -(-O // 64)
    fits = (rows - 1) * sh + R <= 8 and (pxw * 32 - 1) * sw + 4 * form <= 320
    whole = O % (4 if out_bits == 0 else 128 // out_bits) == 0
    full, f32, two_steps = 32 * pxw * segs, out_bits == 0, 4 * R * S > 128
    if O <= 64 and form == 1:
        pays = (O <= 32 and sh <= 3) or 16 * Wo >= 9 * full or units <= 3 * cus or units > 6 * cus
        pays &= not f32 or O <= 32 or units <= 16 * cus
    elif O <= 64 and two_steps:
        pays = (8 * Wo >= 7 * full and (not f32 or O <= 32 or units > cus)) or units > 5 * cus
    elif O <= 32 and units <= cus // 2:
        pays = 8 * Wo >= 7 * full
    elif O <= 64:
        pays = (O <= 32 or not f32) and units > 5 * cus and 8 * Wo >= 5 * full
    elif out_bits == 8 and O % 64 and units > 16 * cus:
        pays = False
    elif form == 1 and f32:
        pays = 8 * Wo >= 6 * full and tiles <= 6 * cus and (sh <= 3 or tiles > cus)
    elif form == 1:
        pays = (8 * Wo >= 6 * full or (8 * Wo >= 5 * full and units > 5 * cus)) and (sh <= 3 or tiles > cus)
    elif two_steps:
        pays = not f32 and 8 * Wo >= (5 if units > 5 * cus else 7) * full and tiles > 5 * cus
    else:
        pays = not f32 and 8 * Wo >= 7 * full and tiles > 12 * cus
    return form > 0 and fits and whole and pays, (units, min(units, 3 * cus // -(-O // 64)))


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


def test_which_kernel():
    for case in ROWS:
        assert any(takes(case, b)[0] for b in (0, 8, 4)), case
    for case in TILED:
        assert not any(takes(case, b)[0] for b in (0, 8, 4)), case
    for b in (0, 8, 4):  # workgroups of two and three units, either form
        for R in (3, 5):
            runs = [takes(c, b)[1] for c in ROWS if c[4] == R and takes(c, b)[0]]
            assert any(u > g and u % g for u, g in runs), (b, R)
    assert any(u > 3 * g for u, g in (takes(c, 8)[1] for c in ROWS))


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


@pytest.mark.parametrize("case", ROWS[:4] + ROWS[5:6] + TILED[:2])
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


@pytest.mark.parametrize("case", [ROWS[0], ROWS[2], TILED[0]])
def test_scale_outside_fp32(case):
    # s_x 2^-fl below the fp32 range: the fp64 scaling decides the result
    B, H, W, O, R, S, st, pad = case
    w = fi.rng("tinyc-tiny", O, R).standard_normal((O, 4, R, S)).astype(np.float32) * np.float32(1e-30)
    W8, fl = oracle.w8_quantize(w)
    q, sx = image(case), np.float32(3e-17)
    cd = np.float64(sx) * 2.0 ** -fl
    assert np.float64(np.float32(cd)) != cd
    ref = oracle.conv2d_w8(q.reshape(-1), 8, sx, (B, H, W, 4), W8, fl, O, R, S, st, pad)
    prep = fgq.fgq_prepare_weights_w8(dev(w))
    check(lambda b, so: fgq.fgq_conv2d_w8(dev(q).view(-1), 8, dev(np.array([sx])), (B, H, W, 4), prep, O, R, S, st, pad,
                                          b, so), ref, O, "tiny")


@pytest.mark.parametrize("sx,so", [(-1e30, 1e-10), (1e30, 1e-10), (-0.0117, 0.02), (0.0117, 1e-37), (-0.0117, 1e-37)])
def test_codes_of_any_quotient(sx, so):
    # quotients y / so past fp32 on either side, also by a negative s_x:
    # saturated codes, as the quantization of the fp32 output gives
    case = ROWS[2]
    B, H, W, O, R, S, st, pad = case
    w = fi.rng("tinyc-sign", O, R).standard_normal((O, 4, R, S)).astype(np.float32)
    q, prep = dev(image(case)).view(-1), fgq.fgq_prepare_weights_w8(dev(w))
    args = (q, 8, dev(np.array([sx], np.float32)), (B, H, W, 4), prep, O, R, S, st, pad)
    y = fgq.fgq_conv2d_w8(*args)
    scale = dev(np.array([so], np.float32))
    for bits in (8, 4):
        want, _ = fgq.fgq_quantize_act(y, bits, scale_in=scale)
        assert torch.equal(fgq.fgq_conv2d_w8(*args, bits, scale).view(-1), want), bits
