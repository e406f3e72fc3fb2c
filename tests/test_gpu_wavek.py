"""The layers at few rows, where a workgroup's waves divide K, and just past
the rule that picks them, where the tiled kernels run: row and channel
remainders, reductions that end inside a K step, four- and eight-way splits
with waves that get no step, every output kind, 8 and 4 bits.  Fixed-point
scales bit for bit against the oracle; fp32 scales within 1e-5 of the summand
magnitude; codes and residual outputs bit for bit against the fp32 output."""
import numpy as np
import pytest
import torch

import fgq_inputs as fi
import oracle

fgq = pytest.importorskip("paper_1705_01462_amd")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# B, H, W, C, O, R, stride.  K steps: 2, 4 (432: ends inside a step), 5, 9, 18
# (sixteen-channel taps) and 36; M from 1 to a few tiles, O around 32, 64, 128
SMALL = [
    (1, 1, 1, 256, 33, 1, 1),
    (1, 5, 7, 48, 30, 3, 1),
    (2, 9, 7, 64, 66, 3, 2),
    (1, 6, 11, 128, 36, 3, 1),
    (1, 8, 8, 256, 128, 3, 1),
    (1, 7, 7, 512, 34, 3, 1),
]
# more workgroups than compute units: the tiled kernels at the same remainders
TILED = [
    (1, 65, 67, 64, 66, 3, 1),
    (1, 61, 71, 48, 65, 3, 1),
    (3, 53, 57, 128, 36, 1, 1),
]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def setup(case, G, bits):
    B, H, W, C, O, R, st = case
    w = fi.he_weights(O, C, R, R, "wavek", G)
    t, a, _ = oracle.ternarize(w, G)
    q, s = oracle.quantize_act(fi.relu_gauss((B, H, W, C), "wavek"), bits)
    return t, a, oracle.pack_codes(t), q, s, (B, H, W, C), (O, R, R, st, R // 2, G)


def rows_of(M):
    return np.arange(M) if M <= 256 else np.unique(np.r_[0:64, M - 70:M, fi.rng("wavek-rows").integers(0, M, 64)])


def run_kinds(plain, fused, residual, O, n_rows, oshape):
    """fp32 output y; its codes at 8 (and 4) bits, and the residual forms,
    each against what the fp32 output gives."""
    y = plain()
    g = torch.Generator(device="cuda").manual_seed(1)
    res = torch.randn(oshape, device="cuda", generator=g)
    so = torch.tensor([0.013], device="cuda")
    yr = (y + res).clamp_(min=0)
    for bits in (8, 4) if O % 2 == 0 else (8,):
        want, _ = fgq.fgq_quantize_act(y, bits, scale_in=so)
        assert torch.equal(fused(bits, so).view(-1), want)
        wr, _ = fgq.fgq_quantize_act(yr, bits, scale_in=so)
        y2, q2 = residual(res, bits, so)
        assert torch.equal(y2, yr) and torch.equal(q2.view(-1), wr)
    inplace = res.clone()
    assert torch.equal(residual(inplace, 0, None, y=inplace), yr)
    return y.view(n_rows, O).cpu().numpy()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("case", SMALL + TILED)
def test_fixed_point(case, bits):
    t, a, codes, q, s, shape, (O, R, S, st, pad, G) = setup(case, 4, bits)
    A, fl = oracle.dfp_alpha(a, 8)
    K = R * S * shape[3]
    prep = fgq.fgq_prepare_weights_dfp(dev(codes), dev(a), O, K, G, 8)
    args = (dev(q), bits, dev(np.array([s], np.float32)), shape, dev(codes), prep, O, R, S, st, pad, G)
    Ho, Wo = fgq.conv_out_hw(shape[1], shape[2], R, S, (st, st), (pad, pad))
    M = shape[0] * Ho * Wo

    def residual(res, b, so, y=None):
        return fgq.fgq_conv2d_dfp_residual(*args, res, b, so, y=y)

    y = run_kinds(lambda: fgq.fgq_conv2d_dfp(*args), lambda b, so: fgq.fgq_conv2d_dfp(*args, b, so), residual, O, M,
                  (shape[0], Ho, Wo, O))
    ref = oracle.conv2d_dfp(q, bits, s, shape, codes, A, fl, O, R, S, (st, st), (pad, pad), G)
    np.testing.assert_array_equal(y.view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("G", [4, 8, 64])
@pytest.mark.parametrize("case", SMALL + TILED)
def test_fp32_scales(case, G, bits):
    if case[3] % G:
        pytest.skip("G divides C")
    t, a, codes, q, s, shape, (O, R, S, st, pad, G) = setup(case, G, bits)
    K = R * S * shape[3]
    prep = fgq.fgq_prepare_weights(dev(codes), dev(a), O, K, G, fallback=True)
    args = (dev(q), bits, dev(np.array([s], np.float32)), shape, dev(codes), dev(a), O, R, S, st, pad, G)
    Ho, Wo = fgq.conv_out_hw(shape[1], shape[2], R, S, (st, st), (pad, pad))
    M = shape[0] * Ho * Wo

    def residual(res, b, so, y=None):
        if b == 0:
            return fgq.fgq_conv2d_residual(*args, res, prepared=prep, y=y)
        return fgq.fgq_conv2d_residual_q(*args, res, b, so, prepared=prep, y=y)

    y = run_kinds(lambda: fgq.fgq_conv2d(*args, prepared=prep),
                  lambda b, so: fgq.fgq_conv2d_q(*args, b, so, prepared=prep), residual, O, M, (shape[0], Ho, Wo, O))
    rows = rows_of(M)
    ref, mag = oracle.conv2d_rows(q, bits, s, shape, codes, a, O, R, S, (st, st), (pad, pad), G, rows)
    assert np.all(np.abs(y[rows].astype(np.float64) - ref) <= 1e-5 * mag)


def test_one_unaligned_output():
    # an output that starts 4 bytes past a 16-byte boundary: single stores
    t, a, codes, q, s, shape, (O, R, S, st, pad, G) = setup(SMALL[4], 4, 8)
    prep = fgq.fgq_prepare_weights_dfp(dev(codes), dev(a), O, R * S * shape[3], G, 8)
    args = (dev(q), 8, dev(np.array([s], np.float32)), shape, dev(codes), prep, O, R, S, st, pad, G)
    y = fgq.fgq_conv2d_dfp(*args)
    buf = torch.zeros(y.numel() + 1, device="cuda")
    fgq.fgq_conv2d_dfp(*args, out=buf[1:])
    assert torch.equal(buf[1:].view_as(y), y) and buf[0] == 0


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("case", [
    (1, 47, 47, 128, 260, 3, 1),   # at most a tile per unit: two wave sets, 9 steps: 5 and 4
    (1, 53, 52, 448, 200, 1, 1),   # 3.5 steps: 2 and 2
    (1, 77, 75, 48, 200, 3, 1),    # C < 128: 4 steps, the last not whole; fp32 in one set
    (1, 90, 96, 144, 64, 3, 1),    # two channel waves: 11 steps: 6 and 5
    (1, 60, 60, 64, 200, 3, 1),    # 5 steps: two sets for codes and shortcuts, one for fp32
])
def test_fixed_point_two_sets(case, bits):
    test_fixed_point(case, bits)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("case", [
    (5, 57, 60, 2192, 68, 1, 1),   # 18 steps: the residual behind the last
    (5, 57, 60, 2192, 67, 1, 1),   # the same, single stores (no 4-bit codes)
    (5, 57, 60, 208, 72, 1, 1),    # two steps: ahead of it
    (5, 57, 60, 80, 30, 1, 1),     # one, single stores of one channel wave
])
def test_fixed_point_residual(case, bits):
    # tiled, one wave set: codes and residual outputs against the fp32 output
    B, H, W, C, O, R, st = case
    q = torch.randint(0, 256, (B * H * W * C * bits // 8,), dtype=torch.uint8, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(2))
    t, a, _ = oracle.ternarize(fi.he_weights(O, C, R, R, "wavek-res"), 4)
    codes = dev(oracle.pack_codes(t))
    prep = fgq.fgq_prepare_weights_dfp(codes, dev(a), O, C, 4, 8)
    args = (q, bits, torch.tensor([0.004], device="cuda"), (B, H, W, C), codes, prep, O, R, R, st, 0, 4)

    def residual(res, b, so, y=None):
        return fgq.fgq_conv2d_dfp_residual(*args, res, b, so, y=y)

    run_kinds(lambda: fgq.fgq_conv2d_dfp(*args), lambda b, so: fgq.fgq_conv2d_dfp(*args, b, so), residual, O,
              B * H * W, (B, H, W, O))
