// exact.hip -- direct per-group FGQ layer kernels.
//
// exact_conv: y = s_x * sum_g alpha_g * P_g with every group sum P_g formed
//   exactly in int32 (v_dot4 on four codes and four activations at a time)
//   and the alpha-weighted sum accumulated in fp64 in group order, then
//   rounded once to fp32.  Every fp64 product alpha*P is exact (24 + 15
//   bits), so the result equals the plain definition's fp64 evaluation bit
//   for bit.  This is the general path (any G, C, stride, padding, bits)
//   and the "v_dot4 VALU" variant of the G=4 layer.
// group_sums: the int32 P_g themselves for a range of output rows.
//
// uint8 activations are signed-offset (q ^ 0x80 = q - 128) so that the
// signed v_dot4_i32_i8 applies; P_g = P'_g + 128*T_g with T_g the sum of the
// group's codes, accumulated alongside.  Out-of-image taps read q = 0, i.e.
// q' = -128, so the identity also holds there.
#include "fgq_internal.h"
#include "qcode.h"

// Every floating-point expression here is evaluated exactly as written.
#pragma clang fp contract(off)

namespace fgq {
namespace {

constexpr int kTM = 64, kTO = 64, kKC = 64;
constexpr int kStride = kKC + 4;  // LDS row stride in bytes (bank spread)

__device__ inline uint32_t unpack_code_byte(uint32_t b) {
  // 4 two-bit codes -> 4 int8 in {-1,0,1}: spread to bytes, sign-extend.
  uint32_t x = (b & 3u) | ((b & 0xCu) << 6) | ((b & 0x30u) << 12) | ((b & 0xC0u) << 18);
  uint32_t hi = x & 0x02020202u;
  return x | (hi * 0x7Eu);
}

__device__ inline unsigned act_elem(const uint8_t* __restrict__ q, int bits, int64_t e) {
  if (bits == 8) return q[e];
  return (q[e >> 1] >> (4 * (e & 1))) & 15u;
}

// Element index of A[m][k] in the NHWC activation tensor, or -1 outside.
__device__ inline int64_t a_index(const ConvGeom& g, int64_t m, int64_t k) {
  const int64_t wo = m % g.Wo;
  const int64_t t = m / g.Wo;
  const int64_t ho = t % g.Ho;
  const int64_t b = t / g.Ho;
  const int64_t c = k % g.C;
  const int64_t rs = k / g.C;
  const int64_t s = rs % g.S;
  const int64_t r = rs / g.S;
  const int64_t hi = ho * g.sh - g.ph + r;
  const int64_t wi = wo * g.sw - g.pw + s;
  if (hi < 0 || hi >= g.H || wi < 0 || wi >= g.W) return -1;
  return ((b * g.H + hi) * g.W + wi) * g.C + c;
}

// A workgroup owns 64 rows x 64 channels and walks K in chunks of 64: the
// chunk's activations, codes (expanded to int8) and the scales of the groups
// that end in it are staged in LDS, the next chunk's loads are in flight
// while the current one is computed, and a thread owns 4 x 4 outputs.
//
// Bound: the vector ALU (per group and output a conversion to fp64 and a
// multiply-add, per four products one dot4).  The rows' (b, ho, wo) are
// decoded once, the taps once per chunk, group ends are counted, and all
// index arithmetic is in I (32 bits unless a size needs 64); with 64-bit
// divisions for every loaded word and every four products, and the scales
// fetched from memory at each group's end, they were what the kernel spent
// its time on: 86.0 -> 35.1 us a call on a 3x3 layer of 40 -> 100 channels,
// 8 x 29 x 31, G = 4.  That layer has 226 workgroups, at most one wave a SIMD,
// which issues vector instructions in 52% of its cycles and waits in 28%; with
// three (128 -> 128 channels, 28 x 28, 32 images) it is 83% of the issue rate.
//
// kVec: C % 4 == 0, so four consecutive k share one tap and are contiguous.
// kDot4: G % 4 == 0, so groups end on words of four k.
template <int kBits, bool kVec, bool kDot4, int kOut, class I>
__global__ __launch_bounds__(256) void exact_conv_kernel(
    const uint8_t* __restrict__ q, const float* __restrict__ sxp,
    const uint8_t* __restrict__ codes, const float* __restrict__ alpha,
    ConvGeom g, LayerOut out) {
  constexpr int kMaxGr = kDot4 ? kKC / 4 : kKC;  // groups that end in a chunk, at most
  constexpr int kAPitch = kMaxGr + 1;
  __shared__ __attribute__((aligned(16))) int8_t As[kTM * kStride];
  __shared__ __attribute__((aligned(16))) int8_t Ts[kTO * kStride];
  __shared__ float Al[kTO * kAPitch];
  const int tid = threadIdx.x;
  const int tx = tid % 16, ty = tid / 16;
  const int64_t m0 = static_cast<int64_t>(blockIdx.x) * kTM;
  const int64_t o0 = static_cast<int64_t>(blockIdx.y) * kTO;
  const I K = static_cast<I>(g.K), C = static_cast<I>(g.C), H = static_cast<I>(g.H), W = static_cast<I>(g.W);
  const int32_t G = g.G;
  const int64_t ng = g.K / g.G;
  const int64_t rb = ceil_div(g.K, 4);
  const uint32_t xor_mask = kBits == 8 ? 0x80808080u : 0u;
  const bool codes4 = rb % 4 == 0 && reinterpret_cast<uintptr_t>(codes) % 4 == 0;

  // This thread's four activation rows (ty + 16*it) and its word of the chunk.
  I hi0[4], wi0[4], rowb[4];
  bool rowok[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int64_t m = m0 + ty + 16 * it;
    rowok[it] = m < g.M;
    const I mm = rowok[it] ? static_cast<I>(m) : 0;
    const I wo = mm % static_cast<I>(g.Wo);
    const I t = mm / static_cast<I>(g.Wo);
    const I ho = t % static_cast<I>(g.Ho);
    hi0[it] = ho * g.sh - g.ph;
    wi0[it] = wo * g.sw - g.pw;
    rowb[it] = (t / static_cast<I>(g.Ho)) * H;
  }
  // Its code column and scale column (64 columns, four threads each).
  const int col = tid / 4, part = tid % 4;
  const bool colok = o0 + col < g.O;
  const uint8_t* crow = codes + (o0 + (colok ? col : 0)) * rb;
  const float* arow = alpha + (o0 + (colok ? col : 0)) * ng;

  uint32_t aw[4], cw;
  float al[kMaxGr / 4];
  auto load = [&](I kc) {
    const I k = kc + 4 * tx;
#pragma unroll
    for (int it = 0; it < 4; ++it) aw[it] = 0;
    if constexpr (kVec) {
      const I rs = k / C, c = k - rs * C;
      const I r = rs / g.S, s = rs - r * g.S;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const I hi = hi0[it] + r, wi = wi0[it] + s;
        if (rowok[it] && k < K && hi >= 0 && hi < H && wi >= 0 && wi < W) {
          const I e = ((rowb[it] + hi) * W + wi) * C + c;
          if (kBits == 8) {
            aw[it] = *reinterpret_cast<const uint32_t*>(q + e);
          } else {
            const uint32_t h = *reinterpret_cast<const uint16_t*>(q + e / 2);
            aw[it] = (h & 0xFu) | ((h & 0xF0u) << 4) | ((h & 0xF00u) << 8) | ((h & 0xF000u) << 12);
          }
        }
      }
    } else {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const I rs = (k + b) / C, c = (k + b) - rs * C;
        const I r = rs / g.S, s = rs - r * g.S;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const I hi = hi0[it] + r, wi = wi0[it] + s;
          if (rowok[it] && k + b < K && hi >= 0 && hi < H && wi >= 0 && wi < W)
            aw[it] |= act_elem(q, kBits, ((rowb[it] + hi) * W + wi) * C + c) << (8 * b);
        }
      }
    }
    cw = 0;
    const int64_t byte = kc / 4 + 4 * part;
    if (colok) {
      if (codes4) {
        if (byte < rb) cw = *reinterpret_cast<const uint32_t*>(crow + byte);
      } else {
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (byte + b < rb) cw |= static_cast<uint32_t>(crow[byte + b]) << (8 * b);
      }
    }
    // scales of the groups that end in the chunk
    const int64_t g0 = kc / G;
    const int ngc = static_cast<int>((kc + kKC < K ? kc + kKC : K) / G - g0);
#pragma unroll
    for (int i = 0; i < kMaxGr / 4; ++i) {
      const int gi = part + 4 * i;
      al[i] = colok && gi < ngc ? arow[g0 + gi] : 0.0f;
    }
  };

  double acc[4][4];
  int32_t P[4][4];
  int32_t T[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    T[i] = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[i][j] = 0.0;
      P[i][j] = 0;
    }
  }
  int32_t left = G;  // weights left in the current group

  // The current group's scaled sums into the fp64 accumulators, `gi` its
  // index among those that end in this chunk.
  auto fold = [&](int gi) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const double a = static_cast<double>(Al[(tx + 16 * j) * kAPitch + gi]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int32_t pt = P[i][j] + 128 * T[j];
        acc[i][j] = fma(a, static_cast<double>(pt), acc[i][j]);
        P[i][j] = 0;
      }
      T[j] = 0;
    }
  };

  load(0);
  for (I kc = 0; kc < K; kc += kKC) {
#pragma unroll
    for (int it = 0; it < 4; ++it)
      *reinterpret_cast<uint32_t*>(&As[(ty + 16 * it) * kStride + 4 * tx]) = aw[it] ^ xor_mask;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      *reinterpret_cast<uint32_t*>(&Ts[col * kStride + 4 * (part * 4 + b)]) = unpack_code_byte((cw >> (8 * b)) & 0xFFu);
#pragma unroll
    for (int i = 0; i < kMaxGr / 4; ++i) Al[col * kAPitch + part + 4 * i] = al[i];
    __syncthreads();
    if (kc + kKC < K) load(kc + kKC);

    const int kend = static_cast<int>(K - kc < kKC ? K - kc : kKC);
    int gi = 0;
    if constexpr (kDot4) {
      for (int wd = 0; 4 * wd < kend; ++wd) {
        int32_t a[4], t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const int32_t*>(&As[(ty + 16 * i) * kStride + 4 * wd]);
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = *reinterpret_cast<const int32_t*>(&Ts[(tx + 16 * j) * kStride + 4 * wd]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) P[i][j] = __builtin_amdgcn_sdot4(a[i], t[j], P[i][j], false);
        if (kBits == 8) {
#pragma unroll
          for (int j = 0; j < 4; ++j) T[j] = __builtin_amdgcn_sdot4(t[j], 0x01010101, T[j], false);
        }
        left -= 4;
        if (left == 0) {
          fold(gi++);
          left = G;
        }
      }
    } else {
      for (int kk = 0; kk < kend; ++kk) {
        int32_t a[4], t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = As[(ty + 16 * i) * kStride + kk];
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = Ts[(tx + 16 * j) * kStride + kk];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) P[i][j] += a[i] * t[j];
        if (kBits == 8) {
#pragma unroll
          for (int j = 0; j < 4; ++j) T[j] += t[j];
        }
        if (--left == 0) {
          fold(gi++);
          left = G;
        }
      }
    }
    __syncthreads();
  }

  const double sx = static_cast<double>(*sxp);
  with_out_scale<kOut>(out.scale, [&](const QScale& qs, auto rcp) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t m = m0 + ty + 16 * i;
      if (m >= g.M) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t o = o0 + tx + 16 * j;  // lanes tx and tx^1 hold channels o and o^1
        if (o < g.O)
          emit_out<kOut, decltype(rcp)::value>(out.y, out.q, qs, m * g.O + o, g.M * g.O, static_cast<int>(o),
                                               static_cast<float>(sx * acc[i][j]), out.res);
      }
    }
  });
}

// One thread per (row, o, g): P = sum over the group of t * q, exact.
template <int kBits>
__global__ __launch_bounds__(256) void group_sums_kernel(
    const uint8_t* __restrict__ q, const uint8_t* __restrict__ codes, ConvGeom g,
    int64_t row0, int64_t nrows, int32_t* __restrict__ P) {
  const int64_t ng = g.K / g.G;
  const int64_t total = nrows * g.O * ng;
  const int64_t rb = ceil_div(g.K, 4);
  for (int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; idx < total;
       idx += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t gi = idx % ng;
    const int64_t o = (idx / ng) % g.O;
    const int64_t m = row0 + idx / (ng * g.O);
    int32_t acc = 0;
    for (int64_t k = gi * g.G; k < (gi + 1) * g.G; ++k) {
      const uint32_t c = (codes[o * rb + k / 4] >> (2 * (k % 4))) & 3u;
      if (c == 0) continue;
      const int64_t e = a_index(g, m, k);
      const int32_t a = e >= 0 ? static_cast<int32_t>(act_elem(q, kBits, e)) : 0;
      acc += c == 1 ? a : -a;
    }
    P[idx] = acc;
  }
}

template <int kBits, int kOut>
fgq_status launch_exact_out(const uint8_t* q, const float* sx, const uint8_t* codes,
                            const float* alpha, const ConvGeom& g, const LayerOut& y, hipStream_t st) {
  const int64_t gx = ceil_div(g.M, kTM), gy = ceil_div(g.O, kTO);
  if (gx > 0x7fffffffLL || gy > 65535) return FGQ_ERR_SHAPE;
  const dim3 grid(static_cast<uint32_t>(gx), static_cast<uint32_t>(gy));
  const bool vec = (g.C % 4 == 0) && (reinterpret_cast<uintptr_t>(q) % 4 == 0);
  const bool dot4 = g.G % 4 == 0;
  // 32-bit indices while every row, element offset and reduction index
  // (with a chunk's overhang) fits
  const int64_t lim = (1LL << 31) - 4096;
  const bool small = g.M < lim && g.K < lim && g.B * (g.H + 2 * g.ph) * (g.W + 2 * g.pw) < lim &&
                     g.B * g.H * g.W * g.C < lim && g.H + 2LL * g.ph < lim && g.W + 2LL * g.pw < lim;
  auto go = [&](auto v, auto d) {
    constexpr bool kV = decltype(v)::value, kD = decltype(d)::value;
    if (small)
      hipLaunchKernelGGL((exact_conv_kernel<kBits, kV, kD, kOut, int32_t>), grid, dim3(256), 0, st, q, sx, codes, alpha, g, y);
    else
      hipLaunchKernelGGL((exact_conv_kernel<kBits, kV, kD, kOut, int64_t>), grid, dim3(256), 0, st, q, sx, codes, alpha, g, y);
  };
  using T = std::true_type;
  using F = std::false_type;
  if (vec && dot4) go(T{}, T{});
  else if (dot4) go(F{}, T{});
  else if (vec) go(T{}, F{});
  else go(F{}, F{});
  return last_launch();
}

template <int kBits>
fgq_status launch_exact_bits(const uint8_t* q, const float* sx, const uint8_t* codes,
                             const float* alpha, const ConvGeom& g, const LayerOut& y, hipStream_t st) {
  switch (y.bits) {
    case 0: return launch_exact_out<kBits, 0>(q, sx, codes, alpha, g, y, st);
    case 2: return launch_exact_out<kBits, 2>(q, sx, codes, alpha, g, y, st);
    case 2 | 8: return launch_exact_out<kBits, 2 | 8>(q, sx, codes, alpha, g, y, st);
    case 2 | 4: return launch_exact_out<kBits, 2 | 4>(q, sx, codes, alpha, g, y, st);
    case 8: return launch_exact_out<kBits, 8>(q, sx, codes, alpha, g, y, st);
    default: return launch_exact_out<kBits, 4>(q, sx, codes, alpha, g, y, st);
  }
}

}  // namespace

fgq_status launch_exact_conv(const uint8_t* q, const float* sx, const uint8_t* codes,
                             const float* alpha, const ConvGeom& g, const LayerOut& y, hipStream_t st) {
  return g.bits == 8 ? launch_exact_bits<8>(q, sx, codes, alpha, g, y, st)
                     : launch_exact_bits<4>(q, sx, codes, alpha, g, y, st);
}

fgq_status launch_group_sums(const uint8_t* q, const uint8_t* codes, const ConvGeom& g,
                             int64_t row0, int64_t nrows, int32_t* P, hipStream_t st) {
  const int64_t total = nrows * g.O * (g.K / g.G);
  if (total == 0) return FGQ_OK;
  int64_t blocks = ceil_div(total, 256);
  if (blocks > 65536) blocks = 65536;
  if (g.bits == 8)
    hipLaunchKernelGGL(group_sums_kernel<8>, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, st, q, codes, g, row0, nrows, P);
  else
    hipLaunchKernelGGL(group_sums_kernel<4>, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, st, q, codes, g, row0, nrows, P);
  return last_launch();
}

}  // namespace fgq
