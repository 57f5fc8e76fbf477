// Internal interface of the autograd wrappers' backward kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dppo {

struct ScaleRowsArgs {
  const void* d;           // [T, V] contiguous, 16-byte aligned
  void* out;               // the same
  int32_t T, V;
  const uint8_t* flags;    // the loss call's flags, or NULL: every row is read
  const float* loss_tok;   // with flags: the call's per-token losses (NaN rows)
  int32_t uses_band;       // the call's rd_mode masks by the band
  const float* g;          // device scalar
};

hipError_t launch_scale_rows(const ScaleRowsArgs& a, bool bf16, hipStream_t st);
hipError_t launch_scale_to_bf16(const float* src, void* dst, int64_t n, const float* g, hipStream_t st);

}  // namespace dppo
