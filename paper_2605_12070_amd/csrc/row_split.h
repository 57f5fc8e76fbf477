// Which entries of a logits row the row kernels read as 16-byte chunks and which one by one. Host
// and device: a CPU test walks every offset and length.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dppo {

// A row of V entries cut into its whole aligned 16-byte chunks and the entries before and after
// them (fewer than a chunk at each end): nfull chunks from entry `lead` on, nedge single
// entries, the i-th of them entry<E>(i).
struct RowSplit {
  int lead, nfull, nedge;
  template <int E>
  __host__ __device__ __forceinline__ int entry(int i) const { return i < lead ? i : nfull * E + i; }
};
template <typename Tin>
__host__ __device__ __forceinline__ RowSplit split_row(const Tin* row, int V) {
  constexpr int E = 16 / (int)sizeof(Tin);
  RowSplit sp;
  const int lead = (int)((0u - (uint32_t)(uintptr_t)row) & 15u) / (int)sizeof(Tin);
  sp.lead = V < lead ? V : lead;
  sp.nfull = (V - sp.lead) / E;
  sp.nedge = V - sp.nfull * E;
  return sp;
}

// The chunks a wave reads for a short row (wave_rows): `bytes` of them from entry `first` of the
// row on, of which the entries [lo, hi) (counted from the first chunk's start) are the row's; the
// other nedge entries of the row are read one by one (RowSplit). fp32 rows are read as their own
// entries and nothing else. A bf16 row is read as the aligned chunks that cover it, up to 7 entries
// on either side, which the ABI's read contract for bf16 allows.
struct WaveSpan {
  int first, bytes, lo, hi, nedge;
};
template <typename Tin>
__host__ __device__ __forceinline__ WaveSpan wave_span(const Tin* row, int V) {
  constexpr int E = 16 / (int)sizeof(Tin);
  if constexpr (sizeof(Tin) == 2) {
    const int ph = (int)(((uintptr_t)row / sizeof(Tin)) & (E - 1));
    return {-ph, (ph + V + E - 1) / E * 16, ph, ph + V, 0};
  } else {
    const RowSplit sp = split_row(row, V);
    return {sp.lead, sp.nfull * 16, 0, sp.nfull * E, sp.nedge};
  }
}

}  // namespace dppo
