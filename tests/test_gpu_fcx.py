"""The GEMM at few rows in one launch and just past the rule that picks it:
rows around 16, 32 and 64, channels that are not whole 16-channel tiles or
whole pieces, reductions that end inside a K step, an odd number of steps,
waves without a pair, the longest reductions of either side, every group size
of the layout, 8 and 4 bits, every output kind.  Fixed-point scales bit for bit
against the oracle, fp32 scales against the unsplit kernel (and that within
1e-5 of the summand magnitude)."""
import numpy as np
import pytest
import torch

import fgq_inputs as fi
import oracle

fgq = pytest.importorskip("paper_1705_01462_amd")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# M, K, O, G
CASES = [
    (1, 128, 16, 4),
    (16, 400, 33, 8),
    (17, 1168, 66, 16),
    (32, 2176, 130, 32),
    (33, 1024, 100, 64),
    (64, 1920, 36, 128),
    (48, 4096, 1000, 4),
    (1, 12288, 40, 4),     # 96 steps: the fixed-point rule's last
    (16, 12416, 40, 4),    # and past it
    (3, 16384, 18, 4),     # 128 steps: the fp32 rule's last
    (2, 16512, 18, 4),
    (20, 8192, 34, 4),     # 64 steps, more than 16 rows
    (20, 8320, 34, 4),
    (40, 256, 2080, 4),    # more workgroups than compute units
    (12, 10240, 40, 4),    # 80 and 81 steps at 12 rows, and 81 with many channels:
    (12, 10368, 40, 4),    #   the fixed-point rule's second line
    (13, 10368, 2052, 4),
    (33, 4224, 2080, 4),   # more than 32 rows, two rounds of workgroups, 33 steps:
    (40, 4224, 3280, 4),   #   few and many sums
    (20, 4224, 4112, 4),   # 20 rows, two rounds of workgroups, 33 steps and 64,
    (17, 8192, 4112, 4),   #   where the split form needs two rounds itself
]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def setup(M, K, O, G, bits):
    w = fi.gauss_weights(O, K, 0.02, "fcx", M, K)
    w = np.where(w < 0, -1.0, 1.0).astype(np.float32) * np.maximum(np.abs(w), np.float32(0.002))
    t, a, _ = oracle.ternarize(w, G)
    q, s = oracle.quantize_act(fi.relu_gauss((M, K), "fcx"), bits)
    return a, oracle.pack_codes(t), q, s


def outputs(call, O):
    """fp32 output; the code outputs against what it gives, aligned and not."""
    y = call(0, None, None)
    so = torch.tensor([float(y.abs().max()) / 200.0], device="cuda")
    for bits in (8, 4) if O % 2 == 0 else (8,):
        want, _ = fgq.fgq_quantize_act(y, bits, scale_in=so)
        assert torch.equal(call(bits, so, None).view(-1), want)
        buf = torch.zeros(want.numel() + 1, dtype=torch.uint8, device="cuda")
        assert torch.equal(call(bits, so, buf[1:]).view(-1), want) and buf[0] == 0
    buf = torch.zeros(y.numel() + 1, device="cuda")
    assert torch.equal(call(0, None, buf[1:]).view(-1), y.view(-1)) and buf[0] == 0
    return y.view(-1, O).cpu().numpy()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("case", CASES)
def test_fixed_point(case, bits):
    M, K, O, G = case
    a, codes, q, s = setup(*case, bits)
    A, fl = oracle.dfp_alpha(a, 8)
    prep = fgq.fgq_prepare_weights_dfp(dev(codes), dev(a), O, K, G, 8)
    args = (dev(q), bits, dev(np.array([s], np.float32)), M, K, dev(codes), prep, O, G)
    y = outputs(lambda b, so, out: fgq.fgq_gemm_dfp_ws(*args, b, so, out=out), O)
    ref = oracle.conv2d_dfp(q, bits, s, (1, M, 1, K), codes, A, fl, O, 1, 1, (1, 1), (0, 0), G).reshape(M, O)
    np.testing.assert_array_equal(y.view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("case", CASES)
def test_fp32_scales(case, bits):
    M, K, O, G = case
    a, codes, q, s = setup(*case, bits)
    prep = fgq.fgq_prepare_weights(dev(codes), dev(a), O, K, G, fallback=True)
    args = (dev(q), bits, dev(np.array([s], np.float32)), M, K, dev(codes), dev(a), O, G)
    y = outputs(lambda b, so, out: fgq.fgq_gemm_ws(*args, prepared=prep, out_bits=b, out_scale=so, out=out), O)
    unsplit = fgq.fgq_gemm(*args, prepared=prep).view(M, O).cpu().numpy()
    np.testing.assert_array_equal(y.view(np.uint32), unsplit.view(np.uint32))
    ref, mag = oracle.conv2d_rows(q, bits, s, (1, M, 1, K), codes, a, O, 1, 1, (1, 1), (0, 0), G, np.arange(M))
    assert np.all(np.abs(y.astype(np.float64) - ref) <= 1e-5 * mag)
