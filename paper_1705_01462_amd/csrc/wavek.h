// wavek.h -- the matrix-core layers where rows and channels give few tiles
// (a network at batch 1, small products): the K steps of one 32-row tile are
// divided among the waves of a workgroup.  Kernel template; the launchers are
// in wavek.hip (folded layouts) and group_wavek.hip (per-group layout).
//
// The tiled kernels (fold_kernel.h, group_kernel.h) walk K serially, a
// barrier and an exposed load per 128-wide step, and with fewer tiles than
// compute units that chain is the layer's time: 17.6 us (fixed-point scales)
// to 28.6 us (groups of 64) for the 3x3 layer of 512 channels at 7 x 7,
// batch 1 (4 tiles of 36 steps), 6.9 and 6.8 us here, and ResNet-50's whole
// forward pass at batch 1 594 -> 344 us (321 with later steps).  Here
//  * a wave takes every kWK-th step of the reduction and loads both operands
//    straight into matrix-instruction fragments, two steps ahead, with no LDS
//    and no barrier on the way: lane l holds row l % 32, k-slot 16 * (l / 32)
//    of each 32-wide slice.  A fragment load touches a line per row, which a
//    throughput-bound layer could not afford (the tiled kernels keep those);
//  * tiles are 32 rows x 32 * kWO channels, so there are four to eight times as many
//    workgroups;
//  * the waves' sums meet in LDS, and every thread finishes four channels of
//    a row: the residual, the scales and the offset terms it will need are
//    requested before the reduction starts, so the end of the kernel waits
//    for none of them.
// Workgroups are numbered rows first, so that an XCD's workgroups share
// channel tiles: at few rows the weights are the traffic.
//
// Folded layouts (kMode 0: three digit planes; 1: one plane of fixed-point
// scales): the sums are integers, so the result is the tiled kernels' bit for
// bit.  Per-group layout (kMode 2, G = 64): each wave folds its groups into
// fp32 as the tiled kernel does and the waves' partial sums are added in wave
// order; no value passes through more roundings than there (at most two per
// step of its wave, then as many as there are other waves with a step).
#pragma once

#include "igemm.h"
#include "qcode.h"
#include "xexpand.h"

namespace fgq {

struct WavekArgs {
  ig::ActArgs x;
  const float* sx;
  const void* weights;    // int8 planes, or the per-group layout's codes
  const int32_t* bias;    // [planes][O] (folded layouts)
  const float* scale;     // [O] grid steps (kMode 0), or alpha [Kp/64][O32] (kMode 2)
  const int32_t* fl;      // fractional length (kMode 1)
  const float* res;       // residual, or null
  float* y;               // fp32 output, or null
  uint8_t* q;             // code output, or null
  const float* oscale;    // its scale
  int32_t code_bits;      // 0, 8 or 4
  int32_t vec;            // codes of four channels of a row are one aligned piece
  int32_t weights_bytes, alpha_bytes, nks, O32;
  uint32_t inv_c, inv_s;  // ceil(2^32 / C), ceil(2^32 / S) (S > 1)
};

fgq_status launch_wavek_group(const WavekArgs& a, int bits, hipStream_t st);

namespace {

using namespace ig;

// Where a kernel that finishes four channels of a row per thread writes them.
struct PieceOut {
  float* y;         // fp32 output, or null
  uint8_t* q;       // code output, or null
  int32_t code_bits;
  bool vec;         // code pieces are whole and aligned
};

// Channels e .. e+3 of the output (n elements), of which `left` are in the row.
// fp32 pieces are 16 bytes at any 4-byte boundary, which the memory pipeline
// takes whole: as single stores (and single loads of the bias and the scales)
// the channel counts off 4 took up to 1.4 times as long as the tiled kernel
// (fixed-point scales, 2037 rows, 256 -> 218: 4.6 us there, 6.3; 1568 rows,
// 176 -> 242: 4.8 there, 5.1 singly, 4.3 here).
template <bool kR>
__device__ inline void store_piece(const PieceOut& out, const QScale& qs, const float __attribute__((ext_vector_type(4))) v,
                                   int64_t e, int left, int64_t n) {
  typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));  // any row alignment
  const int nv = left < 4 ? left : 4;
  if (out.y) {
    if (nv == 4) {
      if (check_store(kSiteStoreY, e, 4, n)) __builtin_nontemporal_store(static_cast<v4fu>(v), reinterpret_cast<v4fu*>(out.y + e));
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (c < nv && check_store(kSiteStoreY, e + c, 1, n)) __builtin_nontemporal_store(v[c], out.y + e + c);
    }
  }
  if (out.code_bits == 8) {
    const uint32_t cw = qcode4<kR>(v[0], v[1], v[2], v[3], qs);
    if (out.vec) {
      if (check_store(kSiteStoreY, e, 4, n)) __builtin_nontemporal_store(cw, reinterpret_cast<uint32_t*>(out.q + e));
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (c < nv && check_store(kSiteStoreY, e + c, 1, n)) out.q[e + c] = static_cast<uint8_t>(cw >> (8 * c));
    }
  } else if (out.code_bits == 4) {  // O is even: pieces of two or four channels
    uint32_t cw = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) cw |= qcode<kR>(v[c], qs) << (4 * c);
    if (out.vec) {
      if (check_store(kSiteStoreY, e / 2, 2, (n + 1) / 2))
        __builtin_nontemporal_store(static_cast<uint16_t>(cw), reinterpret_cast<uint16_t*>(out.q + e / 2));
    } else {
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (2 * c < nv && check_store(kSiteStoreY, e / 2 + c, 1, (n + 1) / 2))
          out.q[e / 2 + c] = static_cast<uint8_t>(cw >> (8 * c));
    }
  }
}

template <int kBits, int kMode, int kWO, int kWK>
__global__ __launch_bounds__(64 * kWO * kWK, 2) void wavek_kernel(WavekArgs a) {
  constexpr int kWG = 64 * kWO * kWK;
  constexpr int kPlanes = kMode == 0 ? 3 : 1;
  constexpr int kPitch = 36;               // words of a tile row in LDS
  constexpr int kChunks = 32 * 8 * kWO;    // four-channel pieces of the tile
  constexpr int kCh = (kChunks + kWG - 1) / kWG;
  typedef typename std::conditional<kBits == 8, v4i, v2i>::type raw_t;
  typedef float v4f __attribute__((ext_vector_type(4)));
  typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));  // any row alignment
  typedef int v4iu __attribute__((ext_vector_type(4), aligned(4)));
  __shared__ __attribute__((aligned(16))) int red[kWO * kWK][32 * kPitch];

  const int tid = threadIdx.x;
  const int lane = tid % 64, half = lane / 32;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int wo = wave % kWO, wk = wave / kWO;
  const int tile = xcd_swizzle(blockIdx.x, a.x.n_otiles * a.x.n_mtiles);
  const int m0 = (tile % a.x.n_mtiles) * 32;
  const int ot0 = (tile / a.x.n_mtiles) * 32 * kWO, o0 = ot0 + 32 * wo;
  const int nk = (a.x.K + kKT - 1) / kKT;
  const int O = a.x.O, M = a.x.M;

  // ---- operands
  const Buf xrs = make_buf(a.x.q, a.x.q_bytes, kSiteActs, kBufFlags);
  const Buf wrs = make_buf(a.weights, a.weights_bytes, kMode == 2 ? kSiteCodes : kSitePlanes, kBufFlags);
  const int m = m0 + lane % 32;
  const bool rowok = m < M;
  int hi0, wi0, rowbase;
  {
    const int mm = rowok ? m : 0;
    const int wo_ = mm % a.x.Wo, t = mm / a.x.Wo;
    const int ho = t % a.x.Ho, b = t / a.x.Ho;
    hi0 = ho * a.x.sh - a.x.ph;
    wi0 = wo_ * a.x.sw - a.x.pw;
    rowbase = (b * a.x.H + hi0) * a.x.W + wi0;
  }
  auto load_x = [&](int ks, raw_t (&x)[4]) {
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int k = kKT * ks + 32 * h + 16 * half;
      // exact for k < 65536 (no prepared layout is longer): k * (inv * C - 2^32) < 2^32
      const int rs = static_cast<int>(__umulhi(static_cast<uint32_t>(k), a.inv_c));
      const int c = k - rs * a.x.C;
      const int r = a.x.S > 1 ? static_cast<int>(__umulhi(static_cast<uint32_t>(rs), a.inv_s)) : rs;
      const int s = rs - r * a.x.S;
      const int hi = hi0 + r, wi = wi0 + s;
      const bool ok = rowok & (k < a.x.K) & (static_cast<unsigned>(hi) < static_cast<unsigned>(a.x.H)) &
                      (static_cast<unsigned>(wi) < static_cast<unsigned>(a.x.W));
      const uint32_t e = static_cast<uint32_t>((rowbase + r * a.x.W + s) * a.x.C + c);
      if constexpr (kBits == 8)
        x[h] = buf_load_b128(xrs, ok ? e : kOutOfRange, 0);
      else
        x[h] = buf_load_b64(xrs, ok ? e >> 1 : kOutOfRange, 0);
    }
  };
  constexpr uint32_t kMask = kMode == 2 ? 0x7F7F7F7Fu : 0x80808080u;  // uint8: q - 128, or 127 - q
  auto frag = [&](const raw_t& x) -> v4i {
    if constexpr (kBits == 8) {
      const int k = static_cast<int>(kMask);
      return v4i{x.x ^ k, x.y ^ k, x.z ^ k, x.w ^ k};
    } else {
      return unpack_u4x16(static_cast<uint32_t>(x.x), static_cast<uint32_t>(x.y));
    }
  };

  // Weights of one step: planes (fragment order), or 16 code bytes and the
  // step's two group scales.  Channel tiles past the layout read zeros.
  struct Weights {
    v4i w[kMode == 2 ? 1 : kPlanes][kMode == 2 ? 1 : 4];
    float al[2];
  };
  constexpr int kTileB = kPlanes * 2 * 1024;
  const int wbase = kMode == 2 ? (o0 / 32) * nk * 1024 + 16 * lane : (o0 / 32) * a.nks * kTileB + 16 * lane;
  const Buf ars = make_buf(a.scale, a.alpha_bytes, kSiteAlpha, kBufFlags);
  const int abase = o0 + lane % 32 < a.O32 ? 4 * (o0 + lane % 32) : static_cast<int>(kOutOfRange);
  auto load_w = [&](int ks, Weights& w) {
    if constexpr (kMode == 2) {
      w.w[0][0] = buf_load_b128(wrs, wbase, ks * 1024);
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
        w.al[blk] = __builtin_bit_cast(float, buf_load_b32(ars, abase, (2 * ks + blk) * a.O32 * 4));
    } else {
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int j = 0; j < kPlanes; ++j)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            w.w[j][2 * blk + h] = buf_load_b128(wrs, wbase + (2 * j + h) * 1024, (2 * ks + blk) * kTileB);
    }
  };

  raw_t xr[2][4];
  Weights wr[2];
  auto load = [&](auto U, int i) {  // this wave's i-th step (past the last: the layer's last, never used)
    constexpr int u = decltype(U)::value;
    const int ks = wk + i * kWK < nk ? wk + i * kWK : nk - 1;
    load_w(ks, wr[u]);
    load_x(ks, xr[u]);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  load(I0{}, 0);
  load(I1{}, 1);

  // ---- what the end of the kernel needs of its pieces: chunk t is row t /
  // (8 kWO) of the tile, channels 4 * (t % (8 kWO)) + [0, 4)
  const bool vec = a.vec != 0;
  v4f resv[kCh], scv[kCh];
  v4i biasv[kCh][kPlanes];
  const float sx = *a.sx;
  const int fl = kMode == 1 ? *a.fl : 0;
  const float os = a.code_bits ? *a.oscale : 1.0f;
#pragma unroll
  for (int i = 0; i < kCh; ++i) {
    const int t = tid + kWG * i;
    const int mr = m0 + t / (8 * kWO), ch = ot0 + 4 * (t % (8 * kWO));
    const bool in = t < kChunks && mr < M;
    const int64_t e = static_cast<int64_t>(mr) * O + ch;
    resv[i] = v4f{0, 0, 0, 0};
    scv[i] = v4f{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < kPlanes; ++j) biasv[i][j] = v4i{0, 0, 0, 0};
    if (a.res && in) {
      if (ch + 4 <= O) {
        if (check_store(kSiteStoreY, e, 4, static_cast<int64_t>(M) * O))  // the output's extent
          resv[i] = __builtin_nontemporal_load(reinterpret_cast<const v4fu*>(a.res + e));
      } else {
#pragma unroll
        for (int c = 0; c < 3; ++c)
          if (ch + c < O && check_store(kSiteStoreY, e + c, 1, static_cast<int64_t>(M) * O)) resv[i][c] = a.res[e + c];
      }
    }
    if constexpr (kMode != 2) {  // (up to three values past the last channel: still inside the prepared buffer)
      if (t < kChunks && ch < O) {
        if constexpr (kMode == 0) scv[i] = *reinterpret_cast<const v4f*>(a.scale + ch);
        if constexpr (kBits == 8)
#pragma unroll
          for (int j = 0; j < kPlanes; ++j) biasv[i][j] = *reinterpret_cast<const v4iu*>(a.bias + j * O + ch);
      }
    }
  }

  // ---- this wave's part of the reduction
  v16i acc[kPlanes];
  v16f facc;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    facc[r] = 0.0f;
#pragma unroll
    for (int j = 0; j < kPlanes; ++j) acc[j][r] = 0;
  }
  auto compute = [&](const raw_t (&x)[4], const Weights& w) {
    if constexpr (kMode == 2) {
      const v4i kMinus127 = {static_cast<int>(0x81818181u), static_cast<int>(0x81818181u),
                             static_cast<int>(0x81818181u), static_cast<int>(0x81818181u)};
      const v16i kZero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) {
        const v4i w0 = expand_ternary16(static_cast<uint32_t>(w.w[0][0][2 * blk]));
        const v4i w1 = expand_ternary16(static_cast<uint32_t>(w.w[0][0][2 * blk + 1]));
        v16i p = kZero;
        if constexpr (kBits == 8) {
          p = __builtin_amdgcn_mfma_i32_32x32x32_i8(kMinus127, w0, p, 0, 0, 0);
          p = __builtin_amdgcn_mfma_i32_32x32x32_i8(kMinus127, w1, p, 0, 0, 0);
        }
        p = __builtin_amdgcn_mfma_i32_32x32x32_i8(frag(x[2 * blk]), w0, p, 0, 0, 0);
        p = __builtin_amdgcn_mfma_i32_32x32x32_i8(frag(x[2 * blk + 1]), w1, p, 0, 0, 0);
        const float s = kBits == 8 ? -w.al[blk] : w.al[blk];
#pragma unroll
        for (int r = 0; r < 16; ++r) facc[r] = fmaf(s, static_cast<float>(p[r]), facc[r]);
      }
    } else {
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const v4i xf = frag(x[h]);
#pragma unroll
        for (int j = 0; j < kPlanes; ++j)  // channels as rows: a lane gets four consecutive ones
          acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w.w[j][h], xf, acc[j], 0, 0, 0);
      }
    }
  };
  const int nw = wk < nk ? (nk - wk + kWK - 1) / kWK : 0;
  for (int i = 0; i < nw; i += 2) {
    compute(xr[0], wr[0]);
    if (i + 2 < nw) load(I0{}, i + 2);
    if (i + 1 < nw) {
      compute(xr[1], wr[1]);
      if (i + 3 < nw) load(I1{}, i + 3);
    }
  }

  // ---- the waves' sums, plane by plane
  v4i S[kCh][kPlanes];
  v4f F[kCh];
#pragma unroll
  for (int j = 0; j < kPlanes; ++j) {
    if (j > 0) __syncthreads();
    int* const mine = red[wave];
    if constexpr (kMode == 2) {  // lane: channel lane % 32 of rows 8 (r/4) + 4 half + r%4
#pragma unroll
      for (int r = 0; r < 16; ++r)
        mine[(8 * (r / 4) + 4 * half + r % 4) * kPitch + lane % 32] = __float_as_int(facc[r]);
    } else {  // lane: row lane % 32, channels 8 (r/4) + 4 half + r%4
#pragma unroll
      for (int qd = 0; qd < 4; ++qd)
        *reinterpret_cast<v4i*>(&mine[(lane % 32) * kPitch + 8 * qd + 4 * half]) =
            v4i{acc[j][4 * qd], acc[j][4 * qd + 1], acc[j][4 * qd + 2], acc[j][4 * qd + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kCh; ++i) {
      const int t = tid + kWG * i;
      if (t >= kChunks) break;
      const int at = (t / (8 * kWO)) * kPitch + 4 * (t % 8), w0 = (t / 8) % kWO;
      if constexpr (kMode == 2) {
        F[i] = v4f{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < kWK; ++k) F[i] += *reinterpret_cast<const v4f*>(&red[k * kWO + w0][at]);
      } else {
        S[i][j] = biasv[i][j];
#pragma unroll
        for (int k = 0; k < kWK; ++k) S[i][j] += *reinterpret_cast<const v4i*>(&red[k * kWO + w0][at]);
      }
    }
  }

  // ---- scales, residual, stores
  const double cd = kMode == 1 && fl > -2048 && fl < 2048 ? static_cast<double>(sx) * ldexp(1.0, -fl) : 0.0;
  const QScale qs = make_qscale(os, a.code_bits == 4 ? 4 : 8);
  const int64_t n = static_cast<int64_t>(M) * O;
  const PieceOut out{a.y, a.q, a.code_bits, vec};
  with_rcp(qs, [&](auto rcp) {
    constexpr bool kR = decltype(rcp)::value;
#pragma unroll
    for (int i = 0; i < kCh; ++i) {
      const int t = tid + kWG * i;
      const int mr = m0 + t / (8 * kWO), ch = ot0 + 4 * (t % (8 * kWO));
      if (t >= kChunks || mr >= M || ch >= O) continue;
      const int64_t e = static_cast<int64_t>(mr) * O + ch;
      v4f v;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if constexpr (kMode == 0) {
          const float c0 = sx * scv[i][c];
          const float c1 = c0 * 255.0f, c2 = c0 * 65025.0f;
          v[c] = fmaf(static_cast<float>(S[i][2 % kPlanes][c]), c2,
                      fmaf(static_cast<float>(S[i][1 % kPlanes][c]), c1, static_cast<float>(S[i][0][c]) * c0));
        } else if constexpr (kMode == 1) {
          v[c] = static_cast<float>(static_cast<double>(S[i][0][c]) * cd);
        } else {
          v[c] = F[i][c] * sx;
        }
        if (a.res) v[c] = add_relu(v[c], resv[i][c]);
      }
      store_piece<kR>(out, qs, v, e, O - ch, n);
    }
  });
}

// Eight waves per workgroup: eight share the K steps, or four where there are
// fewer than six, each with a second one for the next 32 channels.
inline int wavek_channel_waves(int nk) { return nk >= 6 ? 1 : 2; }

template <int kMode, int kBits>
fgq_status launch_wavek_bits(WavekArgs a, hipStream_t st) {
  const int nk = (a.x.K + kKT - 1) / kKT;
  const int wos = wavek_channel_waves(nk);
  a.x.n_mtiles = (a.x.M + 31) / 32;
  a.x.n_otiles = (a.x.O + 32 * wos - 1) / (32 * wos);
  const dim3 grid(static_cast<uint32_t>(a.x.n_mtiles * a.x.n_otiles));
  if (wos == 1)
    hipLaunchKernelGGL((wavek_kernel<kBits, kMode, 1, 8>), grid, dim3(512), 0, st, a);
  else
    hipLaunchKernelGGL((wavek_kernel<kBits, kMode, 2, 4>), grid, dim3(512), 0, st, a);
  return last_launch();
}

template <int kMode>
fgq_status launch_wavek_mode(const WavekArgs& a, int bits, hipStream_t st) {
  return bits == 8 ? launch_wavek_bits<kMode, 8>(a, st) : launch_wavek_bits<kMode, 4>(a, st);
}

}  // namespace
}  // namespace fgq
