// The autograd wrappers' backward (gfx950): the gradient formed in the forward call times the
// upstream gradient of the loss, one pass each.
//   scale_rows     dlogits [T, V] times g, in dlogits' type. A row whose token is masked, clipped
//                  or outside the band is zero in dlogits: its flags say so and it is written
//                  without being read.
//   scale_to_bf16  a float32 gradient times g, rounded once to bf16.
// Both are HBM-bound streams with one 16-byte store per thread over many small workgroups, the
// shape in which a read-write stream moves the most bytes per second on MI355X.
#include <algorithm>

#include "dppo.h"
#include "dppo_device.h"
#include "grad_scale.h"

namespace dppo {

constexpr int kScaleNT = 512;

// Whether row `row` of dlogits holds anything but zeros, by the loss call's flags.
__device__ __forceinline__ bool row_live(const ScaleRowsArgs& a, int64_t row) {
  const uint32_t fl = a.flags[row];
  const float lt = a.loss_tok[row];
  const bool active = (fl & DPPO_FLAG_PPO) && ((fl & DPPO_FLAG_BAND) || !a.uses_band);
  return active || lt != lt;                     // a NaN row's gradient is NaN, not zero
}

template <bool BF16>
__device__ __forceinline__ u32x4 scaled(const u32x4& v, float g) {
  u32x4 o;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (BF16) o[k] = pack_bf16(bf16_lo(v[k]) * g, bf16_hi(v[k]) * g);
    else o[k] = __float_as_uint(__uint_as_float(v[k]) * g);
  }
  return o;
}

// dlogits as one run of 16-byte chunks, whatever rows they lie in (both buffers start on a 16-byte
// boundary), one chunk per thread over the n entries from row 0 on; a chunk is read if any row it
// touches is live. Against whole workgroups for each row, which leave threads idle at every row's
// end, and against torch's product (us, every row live): T = 1M, V = 1 bf16 3.9, 561, 10.4;
// T = 262144, V = 100 20, 207, 21; T = 65536, V = 1000 43, 56, 43; V = 4001 164, 213, 182; T = 32768,
// V = 6000 124, 161, 136; V = 8192 168, 169, 184; T = 16384, V = 32000, 40 % masked 284, 294, 355.
template <bool BF16>
__global__ __launch_bounds__(kScaleNT) void scale_rows(ScaleRowsArgs a, int64_t n) {
  constexpr int E = BF16 ? 8 : 4;
  const int64_t e0 = (int64_t)blockIdx.x * (kScaleNT * E);
  const int64_t at = e0 + (int)threadIdx.x * E;
  if (at >= n) return;
  float g = uload(a.g);
  if (BF16) g = bf16_to_f32(to_bf16(g));
  bool live = a.flags == nullptr;
  if (!live) {
    const uint32_t V = (uint32_t)a.V;
    const int64_t row0 = e0 / a.V;               // uniform over the workgroup
    // entries from row0's start: less than V + kScaleNT E
    const uint32_t first = (uint32_t)(e0 - row0 * a.V) + threadIdx.x * E;
    const uint32_t last = first + (uint32_t)(n - at < E ? n - at : E) - 1;
    const uint32_t r1 = last / V;
    for (uint32_t r = first / V; r <= r1; ++r) live = live || row_live(a, row0 + r);
  }
  if (at + E <= n) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (live) v = __builtin_nontemporal_load((const u32x4*)a.d + at / E);
    __builtin_nontemporal_store(scaled<BF16>(v, g), (u32x4*)a.out + at / E);
    return;
  }
  for (int64_t e = at; e < n; ++e) {
    if (BF16) ((uint16_t*)a.out)[e] = to_bf16(live ? bf16_to_f32(((const uint16_t*)a.d)[e]) * g : 0.0f * g);
    else ((float*)a.out)[e] = live ? ((const float*)a.d)[e] * g : 0.0f * g;
  }
}

__global__ __launch_bounds__(256) void scale_to_bf16(const float* src, uint16_t* dst, int64_t n,
                                                     const float* gp) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= n) return;
  const float g = uload(gp);
  if (i + 8 <= n) {
    const f32x4 x = __builtin_nontemporal_load((const f32x4*)(src + i));
    const f32x4 y = __builtin_nontemporal_load((const f32x4*)(src + i) + 1);
    const u32x4 o = {pack_bf16(x[0] * g, x[1] * g), pack_bf16(x[2] * g, x[3] * g),
                     pack_bf16(y[0] * g, y[1] * g), pack_bf16(y[2] * g, y[3] * g)};
    __builtin_nontemporal_store(o, (u32x4*)(dst + i));
    return;
  }
  for (int64_t e = i; e < n; ++e) dst[e] = to_bf16(src[e] * g);
}

hipError_t launch_scale_rows(const ScaleRowsArgs& a0, bool bf16, hipStream_t st) {
  ScaleRowsArgs a = a0;
  const int64_t E = bf16 ? 8 : 4;
  // rows of a launch, a multiple of E so that the next starts on a chunk (V < 2^31: not zero)
  const int64_t most = kLaunchThreads * E / a.V / E * E;
  for (int64_t t0 = 0; t0 < a0.T; t0 += most) {
    const int64_t off = t0 * a.V * (16 / E);
    a.d = (const char*)a0.d + off;
    a.out = (char*)a0.out + off;
    if (a0.flags) {
      a.flags = a0.flags + t0;
      a.loss_tok = a0.loss_tok + t0;
    }
    a.T = (int32_t)std::min(most, a0.T - t0);
    const int64_t n = a.T * (int64_t)a.V;
    const unsigned grid = (unsigned)(((n + E - 1) / E + kScaleNT - 1) / kScaleNT);
    if (bf16) scale_rows<true><<<grid, kScaleNT, 0, st>>>(a, n);
    else scale_rows<false><<<grid, kScaleNT, 0, st>>>(a, n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_scale_to_bf16(const float* src, void* dst, int64_t n, const float* g, hipStream_t st) {
  constexpr int64_t most = kLaunchThreads * 8;
  for (int64_t i = 0; i < n; i += most) {
    const int64_t m = std::min(most, n - i);
    scale_to_bf16<<<(unsigned)((m + 2047) / 2048), 256, 0, st>>>(src + i, (uint16_t*)dst + i, m, g);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dppo
