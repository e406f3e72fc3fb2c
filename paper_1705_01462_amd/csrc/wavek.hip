// wavek.hip -- host entry of the kernels that divide K among a workgroup's
// waves (wavek.h): the rule that picks them and the argument set-up from the
// prepared buffers; instantiates the folded layouts.
#include "wavek.h"

namespace fgq {

// Measured on the layers of ResNet-50's four stages at batch 1 to 16 (us a
// call, tiled kernel -> this one; W workgroups, n K steps):
//   fixed-point scales   W 208, n 36: 17.8 -> 7.4;  W 200, n 18: 10.9 -> 5.4;
//                        W 100, n 4: 5.6 -> 4.8;    W 400, n 16: 10.1 -> 7.2;
//                        W 392, n 9: 7.6 -> 7.5;    W 784, n 18: 11.1 -> 13.0
//   three digit planes   W 208, n 36: 28.2 -> 10.6; W 196, n 5: 8.7 -> 5.9;
//                        W 100, n 4: 6.6 -> 6.4;    W 392, n 18: 16.3 -> 12.9;
//                        W 200, n 2: 5.5 -> 6.1;    W 392, n 9: 10.3 -> 11.5
//   groups of 64         W 208, n 36: 29.0 -> 7.5;  W 100, n 4: 6.2 -> 4.6;
//                        W 392, n 8: 9.2 -> 7.7;    W 392, n 4: 6.6 -> 8.1
// With at most a workgroup per compute unit the layer takes one workgroup's
// time, 4 to 5 us and little more per step; a second one on a unit costs as
// much again (the fragment loads of one already take most of its L1), which
// only a long reduction repays.  One K step leaves nothing to share, and
// three planes take longer to fetch than two to four steps of the tiled
// kernel.  Two whole steps of one plane into a larger fp32 output leave the
// tiled kernel little to lose (M 1528, O 158: 4.5 -> 5.0; M 34, O 68: 3.8 ->
// 4.3; M 3904, O 114: 4.6 -> 5.2; up to 32 rows or 64 channels 0.52 to 0.97).
bool wavek_pick(const ConvGeom& g, int kind, int out_bits) {
  if (g.C % 16 != 0) return false;  // other C: a fragment's 16 k are not one run of channels
  const int64_t nk = ceil_div(g.K, 128);
  const int64_t wgs = ceil_div(g.M, 32) * ceil_div(g.O, 32 * wavek_channel_waves(static_cast<int>(nk)));
  const int64_t cus = ig::device_cus();
  if (kind == kPrepDfp && out_bits == 0 && g.K == 256 && g.M > 32 && g.O > 64) return false;
  if (wgs <= cus) return nk >= (kind == kPrepFold ? 5 : 2);
  return wgs <= 2 * cus && nk >= (kind == kPrepGroup ? 8 : 16);
}

namespace {

WavekArgs make_args(const uint8_t* q, const float* sx, const ConvGeom& g, const LayerOut& out) {
  WavekArgs a;
  ig::fill_act_args(g, q, &a.x);
  a.sx = sx;
  a.weights = nullptr;
  a.bias = nullptr;
  a.scale = nullptr;
  a.fl = nullptr;
  a.res = out.res;
  a.y = (out.bits == 0 || (out.bits & 2)) ? out.y : nullptr;
  a.code_bits = out.bits & 12;
  a.q = a.code_bits ? out.q : nullptr;
  a.oscale = out.scale;
  const auto al = [](const void* p, uintptr_t n) { return reinterpret_cast<uintptr_t>(p) % n == 0; };
  a.vec = g.O % 4 == 0 && al(a.q, a.code_bits == 4 ? 2 : 4);
  a.weights_bytes = a.alpha_bytes = a.nks = a.O32 = 0;
  a.inv_c = static_cast<uint32_t>(((1ULL << 32) + g.C - 1) / g.C);
  a.inv_s = g.S > 1 ? static_cast<uint32_t>(((1ULL << 32) + g.S - 1) / g.S) : 0;
  return a;
}

}  // namespace

fgq_status launch_wavek(const uint8_t* q, const float* sx, const void* prepared, int kind, const ConvGeom& g,
                        const LayerOut& out, hipStream_t st) {
  WavekArgs a = make_args(q, sx, g, out);
  const char* base = static_cast<const char*>(prepared);
  const PreparedLayout L = kind == kPrepDfp ? prepared_layout_dfp(g.O, g.K, g.G) : prepared_layout(g.O, g.K, g.G);
  a.nks = static_cast<int32_t>(L.nks);
  a.O32 = static_cast<int32_t>(L.O32);
  a.weights = base + L.planes_off;
  if (kind == kPrepGroup) {
    a.scale = reinterpret_cast<const float*>(base + L.alpha_off);
    a.weights_bytes = static_cast<int32_t>(L.O32 * L.Kp / 4);
    a.alpha_bytes = static_cast<int32_t>(4 * L.nks * L.O32);
    return launch_wavek_group(a, g.bits, st);
  }
  a.bias = reinterpret_cast<const int32_t*>(base + L.bias_off);
  if (kind == kPrepDfp) {
    a.fl = reinterpret_cast<const int32_t*>(base);
    a.weights_bytes = static_cast<int32_t>(L.O32 * L.Kp);
    return launch_wavek_mode<1>(a, g.bits, st);
  }
  a.scale = reinterpret_cast<const float*>(base + L.scale_off);
  a.weights_bytes = static_cast<int32_t>(3 * L.O32 * L.Kp);
  return launch_wavek_mode<0>(a, g.bits, st);
}

}  // namespace fgq
