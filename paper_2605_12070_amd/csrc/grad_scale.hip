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

// Workgroups [row * per_row, (row + 1) * per_row) cover row `row`. Rows may start anywhere (d
// and out are contiguous and at the same offset within 16 bytes, so they share every row's phase):
// chunks are the 16-byte blocks of memory the row touches, the first and last entry by entry.
template <bool BF16>
__global__ __launch_bounds__(kScaleNT) void scale_rows(ScaleRowsArgs a, int per_row) {
  constexpr int ES = BF16 ? 2 : 4;
  constexpr int E = 16 / ES;
  const int64_t row = blockIdx.x / per_row;
  const int c = (int)(blockIdx.x % per_row) * kScaleNT + threadIdx.x;
  const char* src = (const char*)a.d + row * a.V * ES;
  char* dst = (char*)a.out + row * a.V * ES;
  const int ph = (int)(((uintptr_t)src & 15) / ES);
  const int e0 = c * E - ph;                     // the chunk's first entry, within the row
  if (e0 >= a.V) return;
  // the upstream gradient in dlogits' type, as a product of two tensors of that type takes it
  float g = uload(a.g);
  if (BF16) g = bf16_to_f32(to_bf16(g));
  bool live = true;                              // uniform over the workgroup
  if (a.flags != nullptr) {
    const uint32_t fl = a.flags[row];
    const float lt = a.loss_tok[row];
    const bool active = (fl & DPPO_FLAG_PPO) && ((fl & DPPO_FLAG_BAND) || !a.uses_band);
    live = active || lt != lt;                   // a NaN row's gradient is NaN, not zero
  }
  if (e0 >= 0 && e0 + E <= a.V) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (live) v = __builtin_nontemporal_load((const u32x4*)(src + (int64_t)e0 * ES));
    u32x4 o;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (BF16) o[k] = pack_bf16(bf16_lo(v[k]) * g, bf16_hi(v[k]) * g);
      else o[k] = __float_as_uint(__uint_as_float(v[k]) * g);
    }
    __builtin_nontemporal_store(o, (u32x4*)(dst + (int64_t)e0 * ES));
    return;
  }
  for (int j = 0; j < E; ++j) {
    const int e = e0 + j;
    if (e < 0 || e >= a.V) continue;
    if (BF16) {
      const float x = live ? bf16_to_f32(((const uint16_t*)src)[e]) : 0.0f;
      ((uint16_t*)dst)[e] = to_bf16(x * g);
    } else {
      const float x = live ? ((const float*)src)[e] : 0.0f;
      ((float*)dst)[e] = x * g;
    }
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

// A dispatch holds fewer than 2^32 threads (a grid that passes them is cut to 32 bits, with no
// error): what exceeds them goes in several launches.
constexpr int64_t kMaxThreads = 0xffffffff;

hipError_t launch_scale_rows(const ScaleRowsArgs& a0, bool bf16, hipStream_t st) {
  ScaleRowsArgs a = a0;
  const int64_t E = bf16 ? 8 : 4;
  const int64_t chunks = (a.V + 2 * E - 2) / E;      // at any phase
  const int64_t per_row = (chunks + kScaleNT - 1) / kScaleNT;
  const int64_t most = kMaxThreads / kScaleNT / per_row;   // 8 rows or more: V < 2^31
  for (int64_t t0 = 0; t0 < a0.T; t0 += most) {
    const int64_t off = t0 * a.V * (16 / E);
    a.d = (const char*)a0.d + off;
    a.out = (char*)a0.out + off;
    if (a0.flags) {
      a.flags = a0.flags + t0;
      a.loss_tok = a0.loss_tok + t0;
    }
    a.T = (int32_t)std::min(most, a0.T - t0);
    const unsigned grid = (unsigned)(per_row * a.T);
    if (bf16) scale_rows<true><<<grid, kScaleNT, 0, st>>>(a, (int)per_row);
    else scale_rows<false><<<grid, kScaleNT, 0, st>>>(a, (int)per_row);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_scale_to_bf16(const float* src, void* dst, int64_t n, const float* g, hipStream_t st) {
  constexpr int64_t most = kMaxThreads / 256 * 256 * 8;
  for (int64_t i = 0; i < n; i += most) {
    const int64_t m = std::min(most, n - i);
    scale_to_bf16<<<(unsigned)((m + 2047) / 2048), 256, 0, st>>>(src + i, (uint16_t*)dst + i, m, g);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dppo
