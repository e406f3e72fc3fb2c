// fcx.hip -- the GEMM at few rows (fully-connected layers at small batch) in
// one launch: codes and scale bytes expanded in registers as in dfpx.hip, the
// K steps of a 16-channel tile divided among the waves of a workgroup.
//
// The split-K form (dfpx.hip) gives K to several workgroups, so its sums go
// through memory and a second kernel adds them.  Here a wave takes every
// kWaves-th pair of K steps, loads both operands straight into
// matrix-instruction fragments (all of a lane's 64 k of a step at once), two
// pairs ahead, and the waves' sums meet in LDS.  With the 16x16x64 form a tile
// is 16 channels, so 4096 channels occupy all 256 compute units.  Lane l is
// channel (or row) l % 16; its quarter g = l / 16 of a fragment's 64 k is half
// g % 2 of the pair's step g / 2, in the order the prepared layout stores
// (xlayout.h); the order of k inside a sum is free as long as both operands
// agree.  Weights are read once per 32 rows (more rows: by two workgroups,
// neighbours, so the second time from L2); the rows are read once per
// workgroup, from L2.
//
// The sums are integers, so the results are the split form's bit for bit.
#include "wavek.h"

namespace fgq {
namespace {

constexpr int kWaves = 8;

struct FcxArgs {
  const uint8_t* q;       // activations [M][K] (uint8) or [M][K/2] (uint4)
  const uint8_t* xcodes;  // codes, expanding-GEMM order
  const int8_t* xacodes;  // per plane: scale codes (or scale digits), same order
  const int32_t* bias;    // [planes][O]  128 * sum_k (weight of the plane) (uint8 offset term)
  const float* scale;     // [O] grid steps (three planes)
  const int32_t* fl;      // fractional length (one plane)
  const float* sx;
  const float* oscale;
  float* y;
  uint8_t* qo;
  int32_t code_bits, vec;
  int32_t M, K, O, nk, n_mtiles;
  int32_t q_bytes, xcodes_bytes, xacodes_bytes, xplane;  // xplane: bytes between planes
};

template <int kBits, int kG, int kMB, int kPlanes>
__global__ __launch_bounds__(64 * kWaves, 2) void fcx_kernel(FcxArgs a) {
  typedef typename std::conditional<kBits == 8, v4i, v2i>::type raw_t;
  typedef float v4f __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) v4i red[kWaves][64 * kMB];

  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int g = lane / 16, hf = g % 2;
  // Row tiles of one channel tile are neighbours: they read the same weights.
  const int tile = xcd_swizzle(blockIdx.x, gridDim.x);
  const int o0 = tile / a.n_mtiles * 16, m0 = tile % a.n_mtiles * 16 * kMB;
  const int np = (a.nk + 1) / 2;  // pairs of K steps
  const Buf qrs = make_buf(a.q, a.q_bytes, kSiteActs, kBufFlags);
  const Buf crs = make_buf(a.xcodes, a.xcodes_bytes, kSiteCodes, kBufFlags);
  const Buf ars = make_buf(a.xacodes, a.xacodes_bytes, kSiteScales, kBufFlags);

  constexpr int kAB = ACodes<kG>::kBytes;
  const int lane0 = ((o0 / 128) * a.nk * 4 + (o0 % 128) / 32) * 64 + o0 % 32 + lane % 16 + 32 * hf;
  raw_t xr[2][kMB][4];
  v4i cr[2];
  ACodes<kG> ar[2][kPlanes];
  auto load = [&](auto U, int i) {  // this wave's i-th pair
    constexpr int u = decltype(U)::value;
    const int ks = 2 * (wave + kWaves * i) + g / 2;
    const bool ok = ks < a.nk;
    const int ln = lane0 + 256 * ks;
    cr[u] = buf_load_b128(crs, ok ? 16 * ln : static_cast<int>(kOutOfRange), 0);
#pragma unroll
    for (int j = 0; j < kPlanes; ++j) ar[u][j].load(ars, ok ? j * a.xplane + kAB * ln : static_cast<int>(kOutOfRange));
#pragma unroll
    for (int b = 0; b < kMB; ++b) {
      const int m = m0 + 16 * b + lane % 16;
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const int k = kKT * ks + 64 * hf + 16 * h;
        const uint32_t e = static_cast<uint32_t>(m * a.K + k);
        const bool in = (m < a.M) & (k < a.K);
        if constexpr (kBits == 8)
          xr[u][b][h] = buf_load_b128(qrs, in ? e : kOutOfRange, 0);
        else
          xr[u][b][h] = buf_load_b64(qrs, in ? e >> 1 : kOutOfRange, 0);
      }
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  const int nw = wave < np ? (np - wave + kWaves - 1) / kWaves : 0;
  if (nw > 0) load(I0{}, 0);
  if (nw > 1) load(I1{}, 1);

  // ---- what the end of the kernel needs: thread t < 64 kMB finishes row
  // 16 (t / 64) + t % 16 of the tile, channels 4 ((t % 64) / 16) + [0, 4) of the tile
  const bool vec = a.vec != 0;
  const int mr = m0 + 16 * (tid / 64) + lane % 16, ch = o0 + 4 * g;
  const bool mine = wave < kMB && mr < a.M && ch < a.O;
  const float sx = *a.sx;
  const int fl = kPlanes == 1 ? *a.fl : 0;
  const float os = a.code_bits ? *a.oscale : 1.0f;
  v4f scv = {0, 0, 0, 0};
  v4i S[kPlanes];
#pragma unroll
  for (int j = 0; j < kPlanes; ++j) S[j] = v4i{0, 0, 0, 0};
  if (mine) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (ch + c < a.O) {
        if constexpr (kPlanes == 3) scv[c] = a.scale[ch + c];
        if constexpr (kBits == 8)
#pragma unroll
          for (int j = 0; j < kPlanes; ++j) S[j][c] = a.bias[j * a.O + ch + c];
      }
  }

  // ---- this wave's part of the reduction
  v4i acc[kPlanes][kMB];
#pragma unroll
  for (int j = 0; j < kPlanes; ++j)
#pragma unroll
    for (int b = 0; b < kMB; ++b) acc[j][b] = v4i{0, 0, 0, 0};
  auto compute = [&](auto U) {
    constexpr int u = decltype(U)::value;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      uint32_t sel[4];
      selectors<kG>(static_cast<uint32_t>(cr[u][h]), sel);
      v4i xf[kMB];
#pragma unroll
      for (int b = 0; b < kMB; ++b) {
        const raw_t& x = xr[u][b][h];
        if constexpr (kBits == 8) {
          const int k = static_cast<int>(0x80808080u);  // q - 128
          xf[b] = v4i{x.x ^ k, x.y ^ k, x.z ^ k, x.w ^ k};
        } else {
          xf[b] = unpack_u4x16(static_cast<uint32_t>(x.x), static_cast<uint32_t>(x.y));
        }
      }
#pragma unroll
      for (int j = 0; j < kPlanes; ++j) {
        const v4i wf = expand16(sel, ar[u][j].quarter(h));
#pragma unroll
        for (int b = 0; b < kMB; ++b) acc[j][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf, xf[b], acc[j][b], 0, 0, 0);
      }
    }
  };
  for (int i = 0; i < nw; i += 2) {
    compute(I0{});
    if (i + 2 < nw) load(I0{}, i + 2);
    if (i + 1 < nw) {
      compute(I1{});
      if (i + 3 < nw) load(I1{}, i + 3);
    }
  }

  // ---- the waves' sums, plane by plane (lane: row l % 16, channels 4 (l / 16) + [0, 4))
#pragma unroll
  for (int j = 0; j < kPlanes; ++j) {
    if (j > 0) __syncthreads();
#pragma unroll
    for (int b = 0; b < kMB; ++b) red[wave][64 * b + lane] = acc[j][b];
    __syncthreads();
    if (wave < kMB) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) S[j] += red[w][tid];
    }
  }
  if (!mine) return;

  const double cd = kPlanes == 1 && fl > -2048 && fl < 2048 ? static_cast<double>(sx) * ldexp(1.0, -fl) : 0.0;
  v4f v;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if constexpr (kPlanes == 3) {
      const float c0 = sx * scv[c];
      const float c1 = c0 * 255.0f, c2 = c0 * 65025.0f;
      v[c] = fmaf(static_cast<float>(S[2][c]), c2,
                  fmaf(static_cast<float>(S[1][c]), c1, static_cast<float>(S[0][c]) * c0));
    } else {
      v[c] = static_cast<float>(static_cast<double>(S[0][c]) * cd);
    }
  }
  const QScale qs = make_qscale(os, a.code_bits == 4 ? 4 : 8);
  const PieceOut out{a.y, a.qo, a.code_bits, vec};
  with_rcp(qs, [&](auto rcp) {
    store_piece<decltype(rcp)::value>(out, qs, v, static_cast<int64_t>(mr) * a.O + ch, a.O - ch,
                                      static_cast<int64_t>(a.M) * a.O);
  });
}

template <int kBits, int kMB, int kPlanes>
fgq_status launch_g(FcxArgs a, int G, hipStream_t st) {
  a.n_mtiles = static_cast<int32_t>(ceil_div(a.M, 16 * kMB));
  const dim3 grid(static_cast<uint32_t>(ceil_div(a.O, 16) * a.n_mtiles)), wg(64 * kWaves);
  switch (G) {
    case 4: hipLaunchKernelGGL((fcx_kernel<kBits, 4, kMB, kPlanes>), grid, wg, 0, st, a); break;
    case 8: hipLaunchKernelGGL((fcx_kernel<kBits, 8, kMB, kPlanes>), grid, wg, 0, st, a); break;
    case 16: hipLaunchKernelGGL((fcx_kernel<kBits, 16, kMB, kPlanes>), grid, wg, 0, st, a); break;
    case 32: hipLaunchKernelGGL((fcx_kernel<kBits, 32, kMB, kPlanes>), grid, wg, 0, st, a); break;
    // one scale byte a lane and step, of its 64 (or both halves' 128) weights
    default: hipLaunchKernelGGL((fcx_kernel<kBits, 64, kMB, kPlanes>), grid, wg, 0, st, a); break;
  }
  return last_launch();
}

template <int kBits, int kPlanes>
fgq_status launch_rows(const FcxArgs& a, int G, hipStream_t st) {
  if (a.M <= 16) return launch_g<kBits, 1, kPlanes>(a, G, st);
  return launch_g<kBits, 2, kPlanes>(a, G, st);
}

}  // namespace

// Measured in a graph (us a call, split form with its reduction -> here; G = 4,
// 1150 shapes: 1 to 64 rows, K 256 to 16384, 64 to 24000 channels):
//   three planes  M 1:  K 4096, O 4096 10.1 -> 4.6;  K 9216 18.9 -> 7.9
//                 M 16: K 12288, O 128 11.8 -> 9.7;  K 16384, O 64 12.3 -> 11.9
//                 M 32: K 4096, O 4096 13.0 -> 7.5, O 4112 13.1 -> 13.1, O 8000 16.8 -> 14.0
//                       K 6144, O 5000 16.0 -> 17.3, O 6000 22.5 -> 17.8
//                       K 8192, O 128 11.4 -> 11.3, O 4112 22.2 -> 21.4, O 8000 28.4 -> 23.3
//                       K 9216, O 256 11.5 -> 12.1; K 16384, O 512 13.6 -> 19.3
//                 M 64: K 4096, O 2080 15.1 -> 13.2, O 4096 18.7 -> 13.5, O 8000 21.0 -> 25.6
//                       K 8192, O 1000 15.8 -> 12.0, O 4096 20.9 -> 22.1
//                 M 48: K 6144, O 2080 15.8 -> 16.5, O 4096 18.6 -> 16.8
//                 M 33: K 5120, O 2080 14.0 -> 15.2; K 8192, O 2080 15.7 -> 20.8
//   one plane     M 1:  K 4096, O 4096 6.6 -> 3.6;   K 9216, O 1000 7.0 -> 4.5
//                 M 16: K 8192, O 128 6.9 -> 6.4;    K 11264, O 64 7.6 -> 7.9
//                       K 12288, O 64 7.3 -> 8.3, O 1024 7.7 -> 8.5, O 2048 8.2 -> 8.5, O 4096 10.6 -> 8.6
//                 M 11: K 12288, O 64 to 4096 at or below the split form; M 12: O 64 7.1 -> 7.3
//                 M 32: K 4096, O 128 6.8 -> 6.3, O 4096 8.0 -> 6.6, O 8000 9.0 -> 10.7
//                       K 9216, O 1000 7.9 -> 11.3
//                 M 64: K 4096, O 2048 8.5 -> 6.7, O 4096 9.8 -> 10.5
// and eagerly one launch costs the host 3 us less than two.  A wave's rounds
// of loads are a serial chain, longer the more rows a round has, so K is
// bounded by the rows; every workgroup reads all its rows, so past 16 rows
// the workgroups are bounded too.  With three planes a second workgroup on a
// unit is worth it up to 32 K steps; beyond, where the split form's own
// workgroups need a second round, or (past 32 rows, to 48 steps) where it
// writes the sums of many rows and channels.  (Four row blocks a workgroup instead of two
// workgroups: 11.5 -> 19.5 us at M 64, K 9216, O 1000, one plane; whole
// 64-byte runs a load, transposed between lanes: 2 to 10% slower.)
bool fcx_pick(const ConvGeom& g, bool dfp) {
  const int64_t nk = ceil_div(g.K, 128), cus = device_cus();
  if (g.M <= 16) return nk <= (dfp ? (g.M <= 11 || g.O > 2048 ? 96 : 80) : 128);
  const int64_t wgs = ceil_div(g.O, 16) * ceil_div(g.M, 32);
  if (dfp) return nk <= 32 && wgs <= cus;
  if (nk > 64 || wgs > 2 * cus) return false;
  if (wgs <= cus || nk <= 32) return true;
  int32_t sps = 0;
  const int64_t split_wgs = ceil_div(g.O, 128) * dfpx_splits(g.M, g.K, g.O, g.G, &sps);
  return split_wgs > cus || (g.M > 32 && nk <= 48 && g.M * g.O >= 1 << 17);
}

fgq_status launch_fcx(const uint8_t* q, const float* sx, const void* prepared, bool dfp, const ConvGeom& g,
                      const LayerOut& out, hipStream_t st) {
  const PreparedLayout L = dfp ? prepared_layout_dfp(g.O, g.K, g.G) : prepared_layout(g.O, g.K, g.G);
  const char* base = static_cast<const char*>(prepared);
  const auto al = [](const void* p, uintptr_t n) { return reinterpret_cast<uintptr_t>(p) % n == 0; };
  FcxArgs a;
  a.q = q;
  a.xcodes = reinterpret_cast<const uint8_t*>(base + L.xcodes_off);
  a.xacodes = reinterpret_cast<const int8_t*>(base + L.xacodes_off);
  a.bias = reinterpret_cast<const int32_t*>(base + L.bias_off);
  a.scale = dfp ? nullptr : reinterpret_cast<const float*>(base + L.scale_off);
  a.fl = reinterpret_cast<const int32_t*>(base);
  a.sx = sx;
  a.oscale = out.scale;
  a.y = out.bits == 0 ? out.y : nullptr;
  a.code_bits = out.bits;
  a.qo = out.bits ? out.q : nullptr;
  a.vec = g.O % 4 == 0 && al(a.qo, out.bits == 4 ? 2 : 4);
  a.M = static_cast<int32_t>(g.M);
  a.K = static_cast<int32_t>(g.K);
  a.O = static_cast<int32_t>(g.O);
  a.nk = static_cast<int32_t>(ceil_div(g.K, 128));
  a.q_bytes = static_cast<int32_t>(g.bits == 8 ? g.M * g.K : g.M * g.K / 2);
  a.xcodes_bytes = static_cast<int32_t>(L.xacodes_off - L.xcodes_off);
  a.xacodes_bytes = static_cast<int32_t>(L.total - L.xacodes_off);
  a.xplane = dfp ? 0 : static_cast<int32_t>(round_up(g.O, 128) * (L.Kp / 64) * dfpx_acode_bytes(g.G));
  if (g.bits == 8) return dfp ? launch_rows<8, 1>(a, g.G, st) : launch_rows<8, 3>(a, g.G, st);
  return dfp ? launch_rows<4, 1>(a, g.G, st) : launch_rows<4, 3>(a, g.G, st);
}

}  // namespace fgq
