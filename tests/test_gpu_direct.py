"""The direct kernel (no prepared weights) where its chunked reduction can go
wrong: groups longer than a 64-wide chunk, groups that straddle chunks, one
weight per group, reductions that end inside a chunk, rows of codes that are
not whole words, and element offsets past 32 bits.  Bit for bit."""
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


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("C,G,R,O", [
    (160, 160, 1, 5),   # one group over two and a half chunks
    (40, 20, 3, 66),    # groups of 5 words straddle chunks
    (10, 5, 3, 65),     # no whole words: single weights, group ends inside words
    (6, 1, 3, 64),      # 64 group ends in a chunk
    (36, 12, 1, 1),     # one short chunk
])
def test_chunks_bit_exact(C, G, R, O, bits):
    B, H, W = 2, 7, 6
    w = fi.he_weights(O, C, R, R, "direct-chunks")
    t, a, _ = oracle.ternarize(w, G)
    codes = oracle.pack_codes(t)
    q, s = oracle.quantize_act(fi.relu_gauss((B, H, W, C), "direct-chunks"), bits)
    y = fgq.fgq_conv2d(dev(q), bits, dev(np.array([s], np.float32)), (B, H, W, C), dev(codes), dev(a), O, R, R, 2,
                       R // 2, G)
    ref = oracle.conv2d(q, bits, s, (B, H, W, C), codes, a, O, R, R, (2, 2), (R // 2, R // 2), G)
    np.testing.assert_array_equal(y.cpu().numpy().reshape(ref.shape).view(np.uint32), ref.view(np.uint32))


def test_offsets_past_32_bits():
    # 64 * 5800 * 5800 = 2.15e9 activations, every hundredth pixel of every
    # hundredth row read: the last reads are past 2^31
    C, O, H, st = 64, 8, 5800, 100
    g = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randint(0, 256, (H, H, C), dtype=torch.uint8, device="cuda", generator=g)
    w = fi.he_weights(O, C, 1, 1, "direct-64")
    t, a, _ = oracle.ternarize(w, 4)
    codes = oracle.pack_codes(t)
    y = fgq.fgq_conv2d(q.view(-1), 8, dev(np.array([0.01], np.float32)), (1, H, H, C), dev(codes), dev(a), O, 1, 1,
                       st, 0, 4)
    sub = q[::st, ::st].contiguous().cpu().numpy()
    n = sub.shape[0]
    ref = oracle.conv2d(sub.reshape(-1), 8, np.float32(0.01), (1, n, n, C), codes, a, O, 1, 1, (1, 1), (0, 0), 4)
    np.testing.assert_array_equal(y.cpu().numpy().reshape(ref.shape).view(np.uint32), ref.view(np.uint32))
