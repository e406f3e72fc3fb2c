// tinyc.hip -- the one-plane layer (8-bit weights, or fixed-point scales) on
// images of four channels, a network's first layer: the rows of an image are
// staged once and the matrix instruction's fragments are read from them.
//
// The tiled kernel gathers such a layer tap by tap, four 4-byte loads with a
// bounds test each per 16-deep piece of the reduction, for every output row
// that uses the tap.  Here a workgroup keeps its channels' weights in
// registers and walks output rows: per unit (128 output pixels in 4, 2 or 1
// rows) it copies the input rows they use to LDS as they lie in memory, 4
// bytes a pixel, out-of-image pixels as zeros, and a wave reads the 16 bytes
// of four neighbouring taps of a pixel as one fragment piece.  For that the
// reduction is taken row by row with the row padded to kPR pieces of four taps
// (zero weights): slice n of 32 holds pieces 2n and 2n + 1.  The weights are
// gathered from the prepared plane once per workgroup, so its layout is the
// other kernels'.  The next unit's rows are requested before the current
// unit's matrix work.
//
// Channels are the instruction's rows, so a lane holds four consecutive
// channels of its pixel; a wave's 32 pixels x 64 channels pass through its own
// LDS tile (no barrier) and leave as 16-byte pieces of whole pixels.
//
// Scales: y = fp32(double(S) * cd), cd = s_x 2^-fl in fp64.  |S| <= 255 * 128 *
// 224 < 2^24 here, so while cd is itself an fp32 value, that is the fp32
// product of two fp32 values, rounded once either way, at a third of the
// instructions.
//
// Bound: a unit's phases one after another, three workgroups a unit covering
// part of it.  On a 7x7 layer of 64 channels, 64 images of 224 x 224 (56.9 us
// gathered tap by tap, 33.0 here): vector work 21.6 us of the SIMDs (14.5
// instructions an output wave), matrix work 6.0, the bytes 13.6 at the copy
// rate, bank conflicts of the tile 8.
#include "fold_kernel.h"

namespace fgq {
namespace {

using namespace ig;

struct TinyArgs {
  ActArgs x;
  const int8_t* planes;
  const int32_t* bias;
  const int32_t* fl;
  const float* sx;
  const float* oscale;
  float* y;
  uint8_t* q;
  int32_t planes_bytes, nks;
  int32_t pxw, rows, nseg, nhg, nunits;  // pixel blocks of 32 per row, rows per unit, units per row and image, all
  int32_t width, prows, words;           // patch: pixels per row, rows, pixels in all
};

// The largest patch, in rows and in 64-pixel pieces of a row (the registers
// that carry one): 7x7 at stride 2 over a 224-wide image takes 7 x 262 pixels.
constexpr int kRows = 8, kCols = 5;

template <int kPR, int kNS, int kOut>
__global__ __launch_bounds__(kThreads, 3) void tinyc_kernel(TinyArgs a) {
  constexpr int kCB = 2;                                         // 32-channel blocks per wave
  constexpr int kEsz = kOut == 0 ? 32 : kOut;                    // bits per output value
  constexpr int kRowB = 64 * kEsz / 8;                           // tile bytes per pixel
  constexpr int kPitch = kRowB + 16;
  constexpr int kPieces = 32 * kRowB / 16;                       // 16-byte pieces of a wave's tile
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  struct __attribute__((packed, aligned(4))) Piece { int v[4]; };
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ __attribute__((aligned(16))) int sbias[64];
  unsigned char* const tile = smem + (threadIdx.x / 64) * 32 * kPitch;
  int* const patch = reinterpret_cast<int*>(smem + 4 * 32 * kPitch);  // two stages of a.words

  const int tid = threadIdx.x, lane = tid % 64, half = lane / 32;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int og = blockIdx.y * 64;
  const int u0 = static_cast<int>(static_cast<int64_t>(blockIdx.x) * a.nunits / gridDim.x);
  const int u1 = static_cast<int>(static_cast<int64_t>(blockIdx.x + 1) * a.nunits / gridDim.x);
  if (u0 >= u1) return;

  const Buf xrs = make_buf(a.x.q, a.x.q_bytes, kSiteActs, kBufFlags);
  struct Unit { int b, ho, wo; };
  auto unit = [&](int u) {
    const int seg = u % a.nseg, t = u / a.nseg;
    return Unit{t / a.nhg, (t % a.nhg) * a.rows, seg * a.pxw * 32};
  };
  // Rows of one unit: wave w takes patch rows w, w + 4, ..., a lane the pixels
  // lane, lane + 64, ... of a row, so a row's bounds are scalar and a pixel's
  // column is tested once for all rows.
  constexpr int kLR = (kRows + 3) / 4;  // rows per wave
  uint32_t ld[kLR][kCols];
  auto request = [&](int u) {
    const Unit n = unit(u);
    const int hi0 = n.ho * a.x.sh - a.x.ph, wi0 = n.wo * a.x.sw - a.x.pw;
    uint32_t voff[kCols];
#pragma unroll
    for (int j = 0; j < kCols; ++j) {
      const int c = lane + 64 * j, wi = wi0 + c;
      const bool ok = (c < a.width) & (static_cast<unsigned>(wi) < static_cast<unsigned>(a.x.W));
      voff[j] = ok ? static_cast<uint32_t>(4 * wi) : kOutOfRange;
    }
#pragma unroll
    for (int i = 0; i < kLR; ++i) {
      const int r = wave + 4 * i, hi = hi0 + r;
      const bool ok = r < a.prows && static_cast<unsigned>(hi) < static_cast<unsigned>(a.x.H);
      const int soff = ok ? (n.b * a.x.H + hi) * a.x.W * 4 : 0;
#pragma unroll
      for (int j = 0; j < kCols; ++j) ld[i][j] = ok ? buf_load_b32(xrs, voff[j], soff) : 0u;
    }
  };
  auto publish = [&](int stage) {
#pragma unroll
    for (int i = 0; i < kLR; ++i) {
      const int r = wave + 4 * i;
      if (r < a.prows) {
#pragma unroll
        for (int j = 0; j < kCols; ++j) {
          const int c = lane + 64 * j;
          if (c < a.width) patch[stage * a.words + r * a.width + c] = static_cast<int>(ld[i][j] ^ 0x80808080u);  // q - 128
        }
      }
    }
  };
  request(u0);

  const float sx = *a.sx;
  const float os = out_scale_of<kOut>(a.oscale);
  const int32_t fl = *a.fl;

  // ---- weights: the channels' part of the plane through LDS as it lies in
  // memory (two channel tiles of Kp x 32 bytes), then this lane's pieces of
  // it: slice n, piece p = 2n + half is taps s = 4 (p % kPR) + [0, 4) of
  // filter row p / kPR.  (Gathered from memory tap by tap, 56 loads a lane
  // with their addresses took 12 us of the launch.)
  const Buf wrs = make_buf(a.planes, a.planes_bytes, kSitePlanes, kBufFlags);
  const int tileb = a.nks * 2048;  // bytes of one channel tile
  for (int t = 16 * tid; t < kCB * tileb; t += 16 * kThreads)
    *reinterpret_cast<v4i*>(smem + t) = buf_load_b128(wrs, (og / 32) * tileb + t, 0);
  __syncthreads();
  v4i w[kCB][kNS];
#pragma unroll
  for (int n = 0; n < kNS; ++n) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      // the tap's place in a channel tile, for either half of the wave
      int at[2];
      bool in[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = (2 * n + h) / kPR, s = 4 * ((2 * n + h) % kPR) + t;
        const int k = (r * a.x.S + s) * 4;
        in[h] = r < a.x.R && s < a.x.S;
        at[h] = in[h] ? (k / 32) * 1024 + ((k % 32) / 16) * 512 + k % 16 : 0;
      }
      const int off = (half ? at[1] : at[0]) + (lane % 32) * 16;
      const bool ok = half ? in[1] : in[0];
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) {
        const int v = *reinterpret_cast<const int*>(smem + cb * tileb + off);
        w[cb][n][t] = ok ? v : 0;
      }
    }
  }
  if (tid < 64) sbias[tid] = og + tid < a.x.O ? a.bias[og + tid] : 0;

  // ---- the wave's pixels: row wave / pxw of the unit, block wave % pxw
  const int prow = wave / a.pxw, pblk = wave % a.pxw;
  int foff[kNS];  // word of this lane's piece of slice n (rows past the filter: the last, on zero weights)
#pragma unroll
  for (int n = 0; n < kNS; ++n) {
    const int r = half ? (2 * n + 1) / kPR : 2 * n / kPR;
    const int s0 = 4 * (half ? (2 * n + 1) % kPR : 2 * n % kPR);
    foff[n] = (prow * a.x.sh + (r < a.x.R ? r : a.x.R - 1)) * a.width + (32 * pblk + lane % 32) * a.x.sw + s0;
  }

  const double cd = fl > -2048 && fl < 2048 ? static_cast<double>(sx) * ldexp(1.0, -fl) : 0.0;
  const float cf = static_cast<float>(cd);
  // (the code's v * y stays finite too, whatever the sign of s_x: |v| < 2^24 |cf|, y = 1 / os)
  const bool fast =
      static_cast<double>(cf) == cd && (kOut == 0 || fabsf(cf) * 16777216.0f / os < __builtin_huge_valf());
  __syncthreads();  // the weights are read; the patches take their place
  publish(0);
  __syncthreads();

  for (int u = u0; u < u1; ++u) {
    const int stage = (u - u0) & 1;
    if (u + 1 < u1) request(u + 1);
    const Unit n = unit(u);
    const int* const src = patch + stage * a.words;

    v16i acc[kCB];
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const v4i b = *reinterpret_cast<const v4i*>(&sbias[32 * cb + 8 * qd + 4 * half]);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[cb][4 * qd + i] = b[i];
      }
#pragma unroll
    for (int s = 0; s < kNS; ++s) {
      const Piece p = *reinterpret_cast<const Piece*>(src + foff[s]);
      const v4i xf = {p.v[0], p.v[1], p.v[2], p.v[3]};
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) acc[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[cb][s], xf, acc[cb], 0, 0, 0);
    }

    // ---- lane: pixel lane % 32, channels 32 cb + 8 qd + 4 half + [0, 4)
    const int ho = n.ho + prow, wo0 = n.wo + 32 * pblk;
    with_out_scale<kOut>(os, [&](const QScale& qs, auto rcp) {
      constexpr bool kR = decltype(rcp)::value;
      auto fill = [&](auto F) {
#pragma unroll
        for (int cb = 0; cb < kCB; ++cb)
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int S = acc[cb][4 * qd + i];
              v[i] = decltype(F)::value ? static_cast<float>(S) * cf : static_cast<float>(static_cast<double>(S) * cd);
            }
            unsigned char* const dst = tile + (lane % 32) * kPitch + (32 * cb + 8 * qd + 4 * half) * kEsz / 8;
            if constexpr (kOut == 0) {
              *reinterpret_cast<u32x4*>(dst) = u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]),
                                                     __float_as_uint(v[3])};
            } else {
              if constexpr (kOut == 8) {
                *reinterpret_cast<uint32_t*>(dst) = qcode4<kR, decltype(F)::value>(v[0], v[1], v[2], v[3], qs);
              } else {
                uint32_t c = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) c |= qcode<kR>(v[i], qs) << (4 * i);
                *reinterpret_cast<uint16_t*>(dst) = static_cast<uint16_t>(c);
              }
            }
          }
      };
      if (fast)
        fill(std::true_type{});
      else
        fill(std::false_type{});
    });
    // Lanes read pieces that other lanes of the wave wrote: LDS serves a wave
    // in order, and the fence keeps the compiler from moving the reads up.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (ho < a.x.Ho) {
      const int64_t e0 = (static_cast<int64_t>(n.b * a.x.Ho + ho) * a.x.Wo + wo0) * a.x.O + og;
      const int64_t nbytes = static_cast<int64_t>(a.x.M) * a.x.O * kEsz / 8;
      unsigned char* const out = kOut == 0 ? reinterpret_cast<unsigned char*>(a.y) : a.q;
#pragma unroll
      for (int t0 = 0; t0 < kPieces; t0 += 64) {
        const int t = t0 + lane;
        const int px = t / (kRowB / 16), piece = t % (kRowB / 16);
        if (wo0 + px < a.x.Wo && og + piece * (128 / kEsz) < a.x.O) {
          const u32x4 v = *reinterpret_cast<const u32x4*>(tile + px * kPitch + 16 * piece);
          const int64_t byte = (e0 + static_cast<int64_t>(px) * a.x.O) * kEsz / 8 + 16 * piece;
          if (check_store(kSiteStoreY, byte, 16, nbytes))
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(out + byte));
        }
      }
    }
    if (u + 1 < u1) publish(1 - stage);
    __syncthreads();
  }
}

template <int kPR, int kNS, int kOut>
fgq_status launch(const TinyArgs& a, hipStream_t st) {
  constexpr int kTiles = 4 * 32 * (64 * (kOut == 0 ? 32 : kOut) / 8 + 16);
  const int64_t ogs = ceil_div(a.x.O, 64);
  // as many workgroups as fit at once, each walking a run of units (their
  // rows overlap), the same number for every 64 channels
  const int64_t fit = 3LL * device_cus();
  const int64_t gx = std::max<int64_t>(1, std::min<int64_t>(a.nunits, fit / ogs));
  hipLaunchKernelGGL((tinyc_kernel<kPR, kNS, kOut>), dim3(static_cast<uint32_t>(gx), static_cast<uint32_t>(ogs)),
                     dim3(kThreads), std::max(kTiles + 8 * a.words, 2 * a.nks * 2048), st, a);
  return last_launch();
}

// Filter rows of up to 4 or 8 taps (1 or 2 pieces), as many of them as the
// form's slices hold; 0: neither.  11x11 filters (three pieces, 17 slices)
// stay with the tiled kernel: their weights fill the registers, 35 us there
// against 48 on 64 images of 224 x 224.
int tinyc_form(const ConvGeom& g) {
  if (g.S <= 4 && g.R <= 4) return 1;
  if (g.S <= 8 && g.R <= 7) return 2;
  return 0;
}

template <int kOut>
fgq_status launch_form(int form, const TinyArgs& a, hipStream_t st) {
  return form == 1 ? launch<1, 2, kOut>(a, st) : launch<2, 7, kOut>(a, st);
}

void tinyc_patch(const ConvGeom& g, int form, TinyArgs* a) {
  a->pxw = g.Wo <= 32 ? 1 : (g.Wo <= 64 ? 2 : 4);
  a->rows = 4 / a->pxw;
  a->width = static_cast<int32_t>((a->pxw * 32 - 1) * g.sw + 4 * form);
  a->prows = static_cast<int32_t>((a->rows - 1) * g.sh + g.R);
  a->words = a->width * a->prows;
}

// Whether the form pays on a layer it fits.  Measured on some 3500 layers (3x3
// to 7x7 filters, strides 1 to 4, 16 to 512 channels, 8 to 300 pixels a row, 1
// to 64 images, every output kind; time here over the tiled kernel's):
//  * Up to 64 channels.  Filters of form 1 gain (0.5 to 0.9) except where a
//    second round of units is half empty (33 pixels in 64, 1088 units, 4x4:
//    1.03 to 1.08) and on large fp32 outputs, bound by their stores (64
//    channels, 5120 units 1.02 to 1.04, 7168 1.06 to 1.10).  7x7 filters gain
//    where rows fill their units (112 pixels: 1 image 0.96, 8 0.94, 64 0.59) or
//    there are several units a workgroup (80 pixels: 1280 units 1.00, 5120
//    0.79); 64 fp32 channels on few units do not (28 units 1.02, 448 0.99).
//    A reduction of one K step (5x5) is short for the tiled kernel too: up to
//    32 channels 0.84 to 0.88 on few full units, but 1.0 to 1.17 on 448 to 896;
//    from 1536 units on 0.7 to 0.9, with half-empty units (65 pixels) 1.05 to
//    1.09; 64 channels of fp32 0.97 to 1.16.
//  * More channels: the tiled kernel's tile has 128 of them, so it stages the
//    image once for two workgroups here.  Codes of form 1: 0.5 to 0.97 where
//    rows fill three quarters of their units (half: 1.04 to 1.22; five eighths
//    0.7 to 0.97 from 5120 units on, 1280 up to 1.09), at stride 4 only past a
//    round of units (28 units 1.03).  fp32 outputs: 0.85 to 0.99 up to two
//    rounds, then up to 1.36.  7x7 codes: 112 units of 96 channels 1.14, 448
//    1.20, 896 0.99, 448 of 192 0.88, 1792 of 128 0.86; fp32 up to 1.24.  5x5
//    codes: 448 units of 256 channels 1.07, 896 0.93, 1792 of 128 0.92.  8-bit
//    codes of 96 channels (rows that are not whole 64-byte pieces) 1.00 to 1.11
//    at 7168 units.
bool tinyc_pays(const ConvGeom& g, int form, int out_bits, const TinyArgs& a) {
  const int64_t cus = device_cus();
  const int64_t full = 32LL * a.pxw * ceil_div(g.Wo, 32 * a.pxw);  // pixels of a row's units
  const int64_t units = g.B * ceil_div(g.Ho, a.rows) * (full / (32 * a.pxw));
  const int64_t tiles = units * ceil_div(g.O, 64);
  const auto filled = [&](int eighths) { return 8 * g.Wo >= eighths * full; };
  const bool f32 = out_bits == 0, two_steps = g.K > 128;
  if (g.O <= 64) {
    if (form == 1) {
      if (f32 && g.O > 32 && units > 16 * cus) return false;
      return (g.O <= 32 && g.sh <= 3) || 16 * g.Wo >= 9 * full || units <= 3 * cus || units > 6 * cus;
    }
    if (two_steps) return (filled(7) && (!f32 || g.O <= 32 || units > cus)) || units > 5 * cus;
    if (g.O <= 32 && units <= cus / 2) return filled(7);
    return (g.O <= 32 || !f32) && units > 5 * cus && filled(5);
  }
  if (out_bits == 8 && g.O % 64 != 0 && units > 16 * cus) return false;
  if (form == 1) {
    if (g.sh > 3 && tiles <= cus) return false;
    if (f32) return filled(6) && tiles <= 6 * cus;
    return filled(6) || (filled(5) && units > 5 * cus);
  }
  if (f32) return false;
  if (two_steps) return filled(units > 5 * cus ? 5 : 7) && tiles > 5 * cus;
  return filled(7) && tiles > 12 * cus;
}

}  // namespace

// Taken where its form fits (four 8-bit channels, outputs in whole aligned
// 16-byte pieces, a patch within the registers that carry it) and pays.  Other
// first layers (eight channels, 4-bit, three planes, residuals) stay with the
// tiled kernel.
bool tinyc_supported(const ConvGeom& g, const uint8_t* q, const LayerOut& out) {
  if (g.C != 4 || g.bits != 8 || (out.bits != 0 && out.bits != 8 && out.bits != 4)) return false;
  const int form = tinyc_form(g);
  if (form == 0 || g.sh > 64 || g.sw > 64 || reinterpret_cast<uintptr_t>(q) % 4 != 0) return false;
  TinyArgs a;
  tinyc_patch(g, form, &a);
  if (a.prows > kRows || a.width > 64 * kCols) return false;
  const int per = out.bits == 0 ? 4 : 128 / out.bits;
  const void* p = out.bits == 0 ? static_cast<const void*>(out.y) : out.q;
  if (g.O % per != 0 || reinterpret_cast<uintptr_t>(p) % 16 != 0) return false;
  const int64_t segs = ceil_div(g.Wo, 32 * a.pxw), units = g.B * ceil_div(g.Ho, a.rows) * segs;
  if (units >= (1LL << 31) || ceil_div(g.O, 64) > device_cus()) return false;
  return tinyc_pays(g, form, out.bits, a);
}

fgq_status launch_tinyc(const uint8_t* q, const float* sx, const void* prepared, const ConvGeom& g,
                        const LayerOut& out, hipStream_t st) {
  const PreparedLayout L = prepared_layout_dfp(g.O, g.K, g.G);
  const char* base = static_cast<const char*>(prepared);
  const int form = tinyc_form(g);
  TinyArgs a;
  fill_act_args(g, q, &a.x);
  a.planes = reinterpret_cast<const int8_t*>(base + L.planes_off);
  a.bias = reinterpret_cast<const int32_t*>(base + L.bias_off);
  a.fl = reinterpret_cast<const int32_t*>(base);
  a.sx = sx;
  a.oscale = out.scale;
  a.y = out.y;
  a.q = out.q;
  a.planes_bytes = static_cast<int32_t>(L.O32 * L.Kp);
  a.nks = static_cast<int32_t>(L.nks);
  tinyc_patch(g, form, &a);
  a.nseg = static_cast<int32_t>(ceil_div(g.Wo, 32 * a.pxw));
  a.nhg = static_cast<int32_t>(ceil_div(g.Ho, a.rows));
  a.nunits = static_cast<int32_t>(g.B * a.nhg * a.nseg);
  switch (out.bits) {
    case 0: return launch_form<0>(form, a, st);
    case 8: return launch_form<8>(form, a, st);
    default: return launch_form<4>(form, a, st);
  }
}

}  // namespace fgq
