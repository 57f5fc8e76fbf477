// Loss stage with the LM head folded in (gfx950). The logits z = hidden weight^T exist only
// as LMH_BM x LMH_BN tiles in registers and LDS:
//   lmh_fwd_tiles  one tile per workgroup on the matrix cores, reduced to per-token partial
//                  log-sum-exps of each 128-entry vocabulary group; optionally also stores
//                  the group-normalised exponentials 2^(z log2 e - m2) as fp16;
//   lmh_tokens     per token: merges the partials into lse_t, forms z[t, y_t] as a dot
//                  product and runs the token math of Eq. 1-4 (ratios, band, PPO clip, loss,
//                  MIS weight w_t);
//   lmh_grad_scale turns the stored exponentials into G = w_t (softmax - onehot) in bf16,
//                  the operand of the two gradient products (lm_head_grad.hip);
//   lmh_bwd_tiles  vocabulary-chunk mode: recomputes a tile and writes G for one chunk.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "dppo.h"
#include "dppo_device.h"
#include "lm_head.h"
#include "token_math.h"

namespace dppo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

// Tile engine: hidden[m0 : m0 + BM] . weight[r0 : r0 + BN]^T on the matrix cores, fed by
// buffer-to-LDS loads (gfx950 writes lane l's 16 bytes at the wave's LDS base + 16 l, and
// zeros for a lane whose offset lies outside the resource, which bounds every access to
// the tile's rows and turns a K tail past d into zeros). There is no register staging:
// LMH_STAGES LDS stages form a ring. A stage holds the A and B tiles as rows of LMH_BK bf16
// of K (128 bytes); the 16-byte chunk c of row r sits at position c ^ sw(r), sw(r) = (r / 2)
// % 8, so the fragment reads of 16 lanes (16 consecutive rows, one chunk) cover all 64 banks.
// Each stage is its own LDS object, which lets the compiler track the loads into each
// separately.
// Wave (wm, wn) owns TM x TN tiles of 32 x 32 (v_mfma_f32_32x32x16_bf16, fp32 accumulation;
// operand lane l holds row l % 32, K 8 (l / 32) .. +7). With 4 waves, one per SIMD, a wave
// holds 128 x 128 accumulators in its 256 accumulation registers, which halves the LDS
// fragment reads per matrix-core instruction against a 128 x 64 wave tile. The vocabulary
// tile is the A operand, so an accumulator holds vocabulary rows in its registers and
// tokens across its lanes: a lane reduces over the vocabulary of its own tokens without
// crossing lanes (LmhLane below).
// With a single wave per SIMD no other wave covers a stall, so the instruction order is
// fixed by hand (scheduling fences between steps):
//  * a K step of 16 is TM TN MFMAs; the fragments of the next K step are read during it,
//    one read after each of the first TM + TN MFMAs (two fragment register sets, by the
//    parity of the step);
//  * the stage barrier sits before the last K step of a stage: by then every wave has read
//    all of that stage's fragments, so its slot is refilled (with stage kb + LMH_STAGES)
//    by loads spread one per MFMA over that last step, whose MFMAs also overlap the reads of
//    the next stage's first fragments;
//  * K is padded to whole turns of the ring; stages past d load zeros (the out-of-range
//    offset) and add nothing, which keeps the loop free of branches.
// After the K loop, epi(acc, scratch) runs on the accumulators, with the ring as scratch.
template <int WM_, int WN_, int TM_, int TN_>
struct Tile {
  static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_;   // waves, 32 x 32 tiles per wave
  static constexpr int BM = 32 * WM * TM, BN = 32 * WN * TN;
  static constexpr int kWaves = WM * WN;
  static constexpr int kIA = BM / 8 / kWaves;     // 1 KB loads per wave and stage, A
  static constexpr int kIB = BN / 8 / kWaves;     // and B
  static constexpr int kAEl = BM * LMH_BK;        // bf16 elements of the A tile (B follows)
  static constexpr int kStageEl = (BM + BN) * LMH_BK;
  static_assert(BM % (8 * kWaves) == 0 && BN % (8 * kWaves) == 0, "tile shape");
  static_assert((LMH_STAGES - 2) * (kIA + kIB) <= 63, "ring depth");
  static_assert(kWaves * 64 == LMH_THREADS, "workgroup size");
  static_assert(TN * 32 == LMH_GROUP, "a wave's columns form one group");
};
using Large = Tile<LMH_WM, LMH_WN, LMH_TM, LMH_TN>;
// One wave's group of 128 vocabulary rows by 32 tokens. 64 KB of LDS and 64 accumulation
// registers a lane: two workgroups share a CU, and one computes while the other waits or runs
// its epilogue.
using Small = Tile<4, 1, 1, 4>;
static_assert(Large::BM == LMH_BM && Large::BN == LMH_BN && Small::BM == LMH_SMALL &&
              Small::BN == LMH_SMALL, "tiles");
constexpr int kChunks = LMH_BK / 8;             // 16-byte chunks per staged row
constexpr int kRL = 64 / kChunks;               // rows covered by one wave-wide load
static_assert(LMH_BK == 64 && LMH_STAGES >= 2, "stage");
static_assert((LMH_BK / 16) % 2 == 0, "an even number of K steps per stage");

// Swizzled position of 16-byte chunk c in staged row r.
__device__ __forceinline__ int lmh_sw(int r) { return (r >> 1) & 7; }

template <int N> using IC = std::integral_constant<int, N>;

template <typename S_, typename Epi>
__device__ __forceinline__ void lmh_engine(const LmhArgs& m, int m0, int r0,
                                           uint16_t* (&st)[LMH_STAGES], Epi&& epi) {
  constexpr int TM = S_::TM, TN = S_::TN, BK = LMH_BK, KS = BK / 16, S = LMH_STAGES;
  constexpr int kIA = S_::kIA, kIB = S_::kIB, kAEl = S_::kAEl;
  constexpr int L = kIA + kIB;                  // loads per wave and stage
  constexpr int NF = TM + TN;                   // fragment reads per K step
  constexpr int NM = TM * TN;                   // MFMAs per K step
  constexpr int LPM = (L + NM - 1) / NM;        // refill loads per MFMA
  constexpr int RPM = (NF + NM - 1) / NM;       // fragment reads per MFMA
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / S_::WN, wn = wave % S_::WN;
  const int d = m.d;
  const int rows_a = min(S_::BM, m.T - m0);
  // a small tile may lie past V (an empty resource); a scalar by hand, so that the resource stays
  // in scalar registers and its loads need no loop over its values
  const int rows_b = __builtin_amdgcn_readfirstlane(max(0, min(S_::BN, m.V - r0)));
  const __amdgpu_buffer_rsrc_t ra = row_rsrc(m.hidden + (int64_t)m0 * d, rows_a * d * 2);
  const __amdgpu_buffer_rsrc_t rb = row_rsrc(m.weight + (int64_t)r0 * d, rows_b * d * 2);

  // Load i of wave w covers tile rows kRL (w I + i) .. +kRL-1: lane l takes row
  // kRL (w I + i) + l / kChunks at position l % kChunks, i.e. K chunk (l % kChunks) ^ sw(row).
  int goa[kIA], gob[kIB];
#pragma unroll
  for (int i = 0; i < kIA; ++i) {
    const int row = kRL * (wave * kIA + i) + lane / kChunks;
    goa[i] = (row * d + ((lane % kChunks) ^ lmh_sw(row)) * 8) * 2;
  }
#pragma unroll
  for (int i = 0; i < kIB; ++i) {
    const int row = kRL * (wave * kIB + i) + lane / kChunks;
    gob[i] = (row * d + ((lane % kChunks) ^ lmh_sw(row)) * 8) * 2;
  }
  // refill load i of stage kb into slot s: i < kIA of the A tile, else of the B tile
  auto load_one = [&](uint16_t* s, int kb, auto I) {
    constexpr int i = decltype(I)::value;
    const int k0 = kb * BK;
    if constexpr (i < kIA) {
      const int row = kRL * (wave * kIA + i) + lane / kChunks;
      const int kc = (lane % kChunks) ^ lmh_sw(row);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          ra, (__attribute__((address_space(3))) void*)(s + (wave * kIA + i) * 512), 16,
          (k0 + kc * 8 < d) ? goa[i] + k0 * 2 : 0x7fffff00, 0, 0, 0);
    } else {
      constexpr int ib = i - kIA;
      const int row = kRL * (wave * kIB + ib) + lane / kChunks;
      const int kc = (lane % kChunks) ^ lmh_sw(row);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rb, (__attribute__((address_space(3))) void*)(s + kAEl + (wave * kIB + ib) * 512), 16,
          (k0 + kc * 8 < d) ? gob[ib] + k0 * 2 : 0x7fffff00, 0, 0, 0);
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.0f;

  // Fragment sets by K-step parity. A fragment row's swizzle depends only on lane % 32 (the
  // rows of a wave's tiles step by 32), so every read is a per-lane base plus a constant.
  bf16x8 fa[2][TM], fb[2][TN];
  const int swz = lmh_sw(lane & 31);
  const int rowa = (wm * 32 * TM + (lane & 31)) * BK;
  const int rowb = kAEl + (wn * 32 * TN + (lane & 31)) * BK;
  // fragment read i of K step ks of slot s into set f: i < TM the A fragment mi = i, else
  // the B fragment ni = i - TM
  auto read_one = [&](const uint16_t* s, int ks, auto F, auto I) {
    constexpr int f = decltype(F)::value, i = decltype(I)::value;
    const int col = ((2 * ks + (lane >> 5)) ^ swz) * 8;
    if constexpr (i < TM)
      fa[f][i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(s + rowa + col + i * 32 * BK));
    else
      fb[f][i - TM] = __builtin_bit_cast(bf16x8, *(const u32x4*)(s + rowb + col + (i - TM) * 32 * BK));
  };
  // MFMA i of a K step on set f: mi = i / TN, ni = i % TN
  auto mfma_one = [&](auto F, auto I) {
    constexpr int f = decltype(F)::value, i = decltype(I)::value;
    acc[i / TN][i % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
        fb[f][i % TN], fa[f][i / TN], acc[i / TN][i % TN], 0, 0, 0);
  };
  // One K step on set f, reading K step rks of slot rs into set f ^ 1; with LOADS, the
  // refill of slot dst with stage kb as well. Order per MFMA: read, loads, MFMA.
  auto kstep = [&](auto F, const uint16_t* rs, int rks, auto LOADS, uint16_t* dst, int kb) {
    constexpr int f = decltype(F)::value;
    constexpr bool loads = decltype(LOADS)::value;
    auto one = [&](auto I) {
      constexpr int i = decltype(I)::value;
      [&]<int... vs>(std::integer_sequence<int, vs...>) {
        ((i * RPM + vs < NF ? read_one(rs, rks, IC<f ^ 1>{}, IC<(i * RPM + vs < NF ? i * RPM + vs : 0)>{})
                            : void()), ...);
      }(std::make_integer_sequence<int, RPM>{});
      if constexpr (loads) {
        [&]<int... vs>(std::integer_sequence<int, vs...>) {
          ((i * LPM + vs < L ? load_one(dst, kb, IC<(i * LPM + vs < L ? i * LPM + vs : 0)>{})
                             : void()), ...);
        }(std::make_integer_sequence<int, LPM>{});
      }
      mfma_one(IC<f>{}, IC<i>{});
      __builtin_amdgcn_sched_barrier(0);
    };
    [&]<int... is>(std::integer_sequence<int, is...>) {
      (one(IC<is>{}), ...);
    }(std::make_integer_sequence<int, NM>{});
  };
  // Barrier without a memory fence (a fence would wait for the loads still in flight); the
  // empty asm statements keep the compiler from moving memory accesses across it.
  auto barrier = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  const int nk = (d + BK - 1) / BK;
#pragma unroll
  for (int s = 0; s < S; ++s)
    [&]<int... vs>(std::integer_sequence<int, vs...>) {
      (load_one(st[s], s, IC<vs>{}), ...);
    }(std::make_integer_sequence<int, L>{});
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((S - 1) * L) : "memory");
  barrier();
  [&]<int... is>(std::integer_sequence<int, is...>) {
    (read_one(st[0], 0, IC<0>{}, IC<is>{}), ...);
  }(std::make_integer_sequence<int, NF>{});
  // stage kb in slot J
  auto stage = [&](auto J, int kb) {
    constexpr int j = decltype(J)::value;
    [&]<int... ks>(std::integer_sequence<int, ks...>) {
      (kstep(IC<ks & 1>{}, st[j], ks + 1, std::false_type{}, st[j], kb), ...);
    }(std::make_integer_sequence<int, KS - 1>{});
    // This wave's reads of slot j are done, and its loads of stage kb + 1 are once at most
    // the loads of the S - 2 later stages are outstanding; after the barrier, every wave's.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((S - 2) * L) : "memory");
    barrier();
    __builtin_amdgcn_sched_barrier(0);
    kstep(IC<(KS - 1) & 1>{}, st[(j + 1) % S], 0, std::true_type{}, st[j], kb + S);
  };
  for (int kb0 = 0; kb0 < nk; kb0 += S) {
    [&]<int... js>(std::integer_sequence<int, js...>) {
      (stage(IC<js>{}, kb0 + js), ...);
    }(std::make_integer_sequence<int, S>{});
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  barrier();

  // The ring is free from here on; the epilogue works on the accumulators in registers and
  // may use the ring as scratch.
  epi(acc, (float*)st[0]);
}

// Accumulator layout (v_mfma_f32_32x32x16_bf16 with the vocabulary tile as the A operand):
// acc[mi][ni] register r of lane l holds z for token
//   m0 + wm 32 TM + mi 32 + l % 32
// and vocabulary row
//   r0 + wn 32 TN + ni 32 + 8 (r / 4) + 4 (l / 32) + r % 4,
// so a lane sees one token per mi and, for each (ni, r / 4), four consecutive vocabulary rows.
template <typename S_>
struct LmhLane {
  int wm, wn, lane;
  __device__ LmhLane() : wm((threadIdx.x >> 6) / S_::WN), wn((threadIdx.x >> 6) % S_::WN), lane(threadIdx.x & 63) {}
  __device__ int token(int m0, int mi) const { return m0 + wm * 32 * S_::TM + mi * 32 + (lane & 31); }
  // tile-relative vocabulary row of register r of tile ni
  __device__ int vrow(int ni, int r) const {
    return wn * 32 * S_::TN + ni * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
  }
};

}  // namespace

#define LMH_RUN_ENGINE(S_, m, m0, r0, epi)                                                \
  do {                                                                                    \
    __shared__ __align__(16) uint16_t lmh_st[LMH_STAGES][S_::kStageEl];                   \
    uint16_t* ring[LMH_STAGES];                                                           \
    _Pragma("unroll") for (int i = 0; i < LMH_STAGES; ++i) ring[i] = lmh_st[i];            \
    lmh_engine<S_>(m, m0, r0, ring, epi);                                                   \
  } while (0)

// Forward: per-token partial log-sum-exp (log2 domain) of each 128-entry vocabulary group of
// the tile (one wave's columns): m2 = log2 e * the group's maximum, sum 2^(z log2 e - m2).
// With store_p the exponentials 2^(z log2 e - m2) in (0, 1] are also stored as fp16 into
// g [T, ldg], four consecutive vocabulary entries (8 bytes) per store: the row pass later
// scales them by w 2^(m2 - lse2) into the gradient, so the backward needs no second product.
// ldg is then a multiple of the tile width, so every tile's columns lie inside the row
// (entries past V are overwritten by the row pass); a buffer resource over the tile's token
// rows drops the stores of rows past T.
// An entry of z that is NaN or +inf makes the partial sum NaN; a group of only -inf logits
// contributes nothing.
template <typename S_>
__global__ __launch_bounds__(LMH_THREADS) void lmh_fwd_tiles(LmhArgs m) {
  const int m0 = blockIdx.x * S_::BM;
  const int nt = blockIdx.y;
  const int r0 = m.n0 + nt * S_::BN;
  const int ncols = min(S_::BN, m.n1 - r0);   // not positive in a small tile past V (no group there)
  auto epi = [&](f32x16 (&acc)[S_::TM][S_::TN], float*) {
    const LmhLane<S_> L;
    const bool ragged = ncols < S_::BN;       // only the last vocabulary tile
    const int grp = (r0 / LMH_GROUP) + L.wn;  // this wave's 128 columns
    const int prows = m.store_p ? min(S_::BM, m.T - m0) : 0;
    const __amdgpu_buffer_rsrc_t rp = row_rsrc(m.g + (int64_t)m0 * m.ldg, (int)(prows * m.ldg * 2));
#pragma unroll
    for (int mi = 0; mi < S_::TM; ++mi) {
      float mx = -INFINITY;
#pragma unroll
      for (int ni = 0; ni < S_::TN; ++ni)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float x = acc[mi][ni][r];
          mx = fmaxf(mx, (ragged && L.vrow(ni, r) >= ncols) ? -INFINITY : x);
        }
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));  // the two lanes that hold the token's group
      const float m2 = mx * kLog2e;
      const float sh = (mx == -INFINITY) ? 0.0f : m2;
      const int t = L.token(m0, mi);
      const int poff = (int)(((int64_t)(t - m0) * m.ldg + r0) * 2);
      float sum = 0.0f;
#pragma unroll
      for (int ni = 0; ni < S_::TN; ++ni)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int v0 = L.vrow(ni, 4 * q);
          float e[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            e[j] = exp2_hw(__builtin_fmaf(acc[mi][ni][4 * q + j], kLog2e, -sh));
            sum += (ragged && v0 + j >= ncols) ? 0.0f : e[j];
          }
          if (m.store_p) {
            u32x2 v;
            v.x = pack_f16(e[0], e[1]);
            v.y = pack_f16(e[2], e[3]);
            __builtin_amdgcn_raw_buffer_store_b64(v, rp, poff + v0 * 2, 0, 0);
          }
        }
      sum += __shfl_xor(sum, 32, 64);
      if (L.lane < 32 && t < m.T) {
        float* p = m.part + ((int64_t)t * lmh_groups(m.V) + grp) * 2;
        p[0] = (mx == -INFINITY) ? -INFINITY : m2;
        p[1] = sum;
      }
    }
  };
  LMH_RUN_ENGINE(S_, m, m0, r0, epi);
}

// One wave per token: merges the token's group partials into lse2, forms z[t, y_t] as a dot
// product of hidden[t] and weight[y_t] (fp32 accumulation), runs the token math (per-token
// outputs) and leaves the backward constants w, lse2, dy = w (p_y - 1) and ev.
//
// Latency-bound (8 bytes per token and group, 4 d bytes per token): a wave's partial and operand
// loads are issued before anything waits on them, and every token has a wave at once. It
// replaces a dot-product kernel, a merge with one workgroup per token whose five counter atomics
// per workgroup serialised (36 us at T = 1024, V = 32000, 103 us at T = 8192, V = 151936) and,
// in the chunked mode, a merge with one thread per token (515 us at T = 2048, V = 151936). When
// the call writes flags the loss sum takes the counters from them and no atomics run.
constexpr int kTokWaves = 4;                     // tokens (waves) per workgroup

__global__ __launch_bounds__(64 * kTokWaves) void lmh_tokens(RowArgs a, LmhArgs m, int count) {
  const int lane = threadIdx.x & 63;
  const int ngroups = lmh_groups(m.V);
  StatCount sc;
  for (int64_t t0 = (int64_t)blockIdx.x * kTokWaves; t0 < m.T; t0 += (int64_t)gridDim.x * kTokWaves) {
    const int64_t t = t0 + (threadIdx.x >> 6);
    if (t >= m.T) break;                         // the whole wave
    const bool valid = a.mask == nullptr || a.mask[t] != 0;
    const int64_t y = m.ids[t];
    const bool ev = valid && y >= 0 && y < m.V;  // uniform over the wave
    if (!ev) {
      if (lane == 0) {
        a.lp_out[t] = valid ? __builtin_nanf("") : 0.0f;
        a.loss_tok[t] = 0.0f;
        if (a.flags) a.flags[t] = valid ? (uint8_t)(DPPO_FLAG_VALID | DPPO_FLAG_BAD_ID) : (uint8_t)0;
        if (valid) sc.bad += 1;
        m.w[t] = 0.0f;
        m.lse2[t] = 0.0f;
        m.dy[t] = 0.0f;
        m.ev[t] = 0;
      }
      continue;
    }
    const TokenIn tin = token_inputs_lane(a, t);
    constexpr int U = 8;                         // partials per lane in flight
    const f32x2* p = (const f32x2*)m.part + t * ngroups;
    float n = -INFINITY, s = 0.0f;
    for (int q0 = lane; q0 < ngroups; q0 += 64 * U) {
      f32x2 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + 64 * u;
        v[u] = p[q < ngroups ? q : lane];        // in bounds: q0 < ngroups, so lane is
        if (q >= ngroups) v[u] = f32x2{-INFINITY, 0.0f};
      }
#pragma unroll
      for (int u = 0; u < U; ++u) merge_ns(n, s, v[u].x, v[u].y);
    }
    float zy = 0.0f;
    const uint16_t* h = m.hidden + t * m.d;
    const uint16_t* wr = m.weight + y * m.d;
#pragma unroll 4
    for (int k = lane * 8; k < m.d; k += 512) {
      const u32x4 hv = *(const u32x4*)(h + k);
      const u32x4 wv = *(const u32x4*)(wr + k);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        zy = __builtin_fmaf(bf16_lo(hv[i]), bf16_lo(wv[i]), zy);
        zy = __builtin_fmaf(bf16_hi(hv[i]), bf16_hi(wv[i]), zy);
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      zy += __shfl_xor(zy, off, 64);
      const float n2 = __shfl_xor(n, off, 64);
      const float s2 = __shfl_xor(s, off, 64);
      merge_ns(n, s, n2, s2);
    }
    const float l2 = (n == -INFINITY) ? __builtin_nanf("") : n + log2f(s);
    if (lane == 0) {
      const TokenOut o = token_math(a, tin, zy, l2);
      a.lp_out[t] = o.lp;
      a.loss_tok[t] = o.loss;
      if (a.flags) a.flags[t] = o.flags;
      count_stats(a, o.flags, sc);
      m.w[t] = o.w;
      m.lse2[t] = l2;
      m.dy[t] = o.dy;
      m.ev[t] = 1;
    }
  }
  if (count && lane == 0) flush_stats(a, sc);
}

// Full-vocabulary backward without a second product: lmh_grad_scale turns the stored
// exponentials into G = w (softmax - onehot) in place, one 16-byte chunk (8 entries) per
// thread: entry v of group q becomes w 2^(m2_q - lse2) e_v in bf16, the sampled entry dy, and
// the entries from V up to ldg zeros; a row that is not evaluated (masked, or a bad id) becomes
// zeros without being read. One chunk per thread and a grid of (chunks per row / 256) x T
// workgroups is the shape in which a read-write stream moves the most bytes per second on
// MI355X (as a per-row loop over four chunks per thread it took 1.0 ms at T = 8192,
// V = 151936).
__global__ __launch_bounds__(256) void lmh_grad_scale(LmhArgs m, int per_row, int64_t row0) {
  // per_row workgroups cover a row's chunks; consecutive workgroups walk along a row
  const int64_t row = row0 + blockIdx.x / per_row;
  const int c = (int)(blockIdx.x % per_row) * 256 + threadIdx.x;
  if (c >= (int)(m.ldg / 8)) return;
  const int v0 = 8 * c;
  uint16_t* grow = m.g + row * m.ldg;
  const bool ev = uload_u8(m.ev + row) != 0;              // uniform over the workgroup
  u32x4 out = {0u, 0u, 0u, 0u};
  if (ev && v0 < m.V) {
    const u32x4 e = __builtin_nontemporal_load((const u32x4*)(grow + v0));
    const float w = uload(m.w + row), l2 = uload(m.lse2 + row), dy = uload(m.dy + row);
    const int64_t y = uload(m.ids + row);
    const float m2 = m.part[(row * lmh_groups(m.V) + v0 / LMH_GROUP) * 2];
    const float f = w * exp2_hw(m2 - l2);
    float x[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[2 * j] = f16_lo_mul(e[j], f);
      x[2 * j + 1] = f16_hi_mul(e[j], f);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if ((int64_t)(v0 + j) == y) x[j] = dy;
      if (v0 + j >= m.V) x[j] = 0.0f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) out[j] = pack_bf16(x[2 * j], x[2 * j + 1]);
  }
  __builtin_nontemporal_store(out, (u32x4*)(grow + v0));
}

// Backward (vocabulary chunks): g[t, v - n0] = w_t (softmax(z_t)[v] - 1{v = y_t}) in bf16
// for the tile's rows of the chunk [n0, n1); tokens that were not evaluated get zeros. The
// last tile also zeroes the entries past the chunk up to the next multiple of 8, which the
// gradient products read as whole 16-byte chunks.
template <typename S_>
__global__ __launch_bounds__(LMH_THREADS) void lmh_bwd_tiles(LmhArgs m) {
  const int m0 = blockIdx.x * S_::BM;
  const int r0 = m.n0 + blockIdx.y * S_::BN;
  const int ncols = min(S_::BN, m.n1 - r0);
  auto epi = [&](f32x16 (&acc)[S_::TM][S_::TN], float*) {
    const LmhLane<S_> L;
#pragma unroll
    for (int mi = 0; mi < S_::TM; ++mi) {
      const int t = L.token(m0, mi);
      if (t >= m.T) continue;
      const bool ev = m.ev[t] != 0;
      const float wt = ev ? m.w[t] : 0.0f;
      const float l2 = m.lse2[t];
      const int64_t yr = m.ids[t] - r0;        // the token's id relative to the tile
      uint16_t* grow = m.g + (int64_t)t * m.ldg + (r0 - m.n0);
#pragma unroll
      for (int ni = 0; ni < S_::TN; ++ni)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // four consecutive vocabulary rows v0 .. v0 + 3 of this token
          const int v0 = L.vrow(ni, 4 * q);
          float o[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float p = exp2_hw(__builtin_fmaf(acc[mi][ni][4 * q + j], kLog2e, -l2));
            o[j] = ev ? wt * (p - ((int64_t)(v0 + j) == yr ? 1.0f : 0.0f)) : 0.0f;
          }
          if (v0 + 4 <= ncols) {
            u32x2 v;
            v.x = pack_bf16(o[0], o[1]);
            v.y = pack_bf16(o[2], o[3]);
            *(u32x2*)(grow + v0) = v;
          } else {
            const int end8 = (ncols + 7) & ~7;
            for (int j = 0; j < 4 && v0 + j < end8; ++j)
              grow[v0 + j] = v0 + j < ncols ? to_bf16(o[j]) : (uint16_t)0;
          }
        }
    }
  };
  LMH_RUN_ENGINE(S_, m, m0, r0, epi);
}

hipError_t launch_lmh_fwd_tiles(const LmhArgs& m, hipStream_t st) {
  const int n = m.n1 - m.n0;
  if (lmh_small_tiles(m.T, n, m.d)) {
    // every group has its tile, the one past V too (it stores the empty partial)
    const dim3 grid((m.T + Small::BM - 1) / Small::BM, lmh_groups(n));
    lmh_fwd_tiles<Small><<<grid, LMH_THREADS, 0, st>>>(m);
  } else {
    const dim3 grid((m.T + LMH_BM - 1) / LMH_BM, lmh_tiles(n));
    lmh_fwd_tiles<Large><<<grid, LMH_THREADS, 0, st>>>(m);
  }
  return hipGetLastError();
}

hipError_t launch_lmh_tokens(const RowArgs& a, const LmhArgs& m, bool count, hipStream_t st) {
  if (m.T <= 0) return hipSuccess;
  const int64_t groups = ((int64_t)m.T + kTokWaves - 1) / kTokWaves;
  // with counter atomics, few workgroups: five atomics each on the same addresses
  const int64_t most = count ? 256 : 0x7fffffff;
  lmh_tokens<<<(unsigned)(groups < most ? groups : most), 64 * kTokWaves, 0, st>>>(a, m, count ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_lmh_grad_scale(const LmhArgs& m, hipStream_t st) {
  if (m.ldg % 8 != 0 || m.ldg > (1 << 21)) return hipErrorInvalidValue;
  if (m.T <= 0) return hipSuccess;
  const int64_t per_row = (m.ldg / 8 + 255) / 256;
  const int64_t most = kLaunchThreads / 256 / per_row;      // per_row <= 1024
  for (int64_t r = 0; r < m.T; r += most) {
    lmh_grad_scale<<<(unsigned)(per_row * std::min(most, m.T - r)), 256, 0, st>>>(m, (int)per_row, r);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_lmh_bwd_tiles(const LmhArgs& m, hipStream_t st) {
  const int n = m.n1 - m.n0;
  if (lmh_small_tiles(m.T, n, m.d)) {
    const dim3 grid((m.T + Small::BM - 1) / Small::BM, (n + Small::BN - 1) / Small::BN);
    lmh_bwd_tiles<Small><<<grid, LMH_THREADS, 0, st>>>(m);
  } else {
    const dim3 grid((m.T + LMH_BM - 1) / LMH_BM, lmh_tiles(n));
    lmh_bwd_tiles<Large><<<grid, LMH_THREADS, 0, st>>>(m);
  }
  return hipGetLastError();
}

}  // namespace dppo

namespace dppo {

__global__ __launch_bounds__(256) void lmh_fill_zero(float* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0.0f;
}

hipError_t launch_lmh_zero(float* p, int64_t n, hipStream_t st) {
  for (int64_t i = 0; i < n; i += kLaunchThreads) {
    const int64_t k = std::min(kLaunchThreads, n - i);
    lmh_fill_zero<<<(unsigned)((k + 255) / 256), 256, 0, st>>>(p + i, k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dppo
