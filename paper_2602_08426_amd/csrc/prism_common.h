// Internal helpers shared by the libprism translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "prism.h"

namespace prism {

constexpr int kHeadDim = 128;           // the head dim of the 64-queries-per-wave attention kernel
constexpr int kMaxHeadDim = 256;        // head_dim is 64, 128 or 256
constexpr int kMaxBlocks = 2048;       // N <= 2048  (128K tokens at B = 64)
constexpr int kWave = 64;
constexpr int kMaxDevices = 64;         // GPUs of one process for which per-device host state is kept

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Validation shared by every entry point.  Returns PRISM_OK or an error code.
inline int check_params(const prism_params* p) {
  if (p == nullptr) return PRISM_ERR_INVALID_ARG;
  if (p->n_q_heads <= 0 || p->n_kv_heads <= 0 || p->seq_len <= 0) return PRISM_ERR_INVALID_ARG;
  if (p->n_q_heads % p->n_kv_heads != 0) return PRISM_ERR_INVALID_ARG;
  if (p->head_dim != 64 && p->head_dim != 128 && p->head_dim != 256) return PRISM_ERR_UNSUPPORTED;
  if (p->block != 64 && p->block != 128) return PRISM_ERR_UNSUPPORTED;
  const int64_t n = ((int64_t)p->seq_len + p->block - 1) / p->block;   // a ragged last block is allowed
  if (n > kMaxBlocks) return PRISM_ERR_UNSUPPORTED;
  // CSR offsets are int32
  const int64_t pairs = (p->flags & PRISM_FLAG_BIDIRECTIONAL) ? (int64_t)p->n_q_heads * n * n
                                                               : (int64_t)p->n_q_heads * n * (n + 1) / 2;
  if (pairs >= (int64_t)1 << 31) return PRISM_ERR_UNSUPPORTED;
  if ((int64_t)p->n_q_heads * n + 1 >= (int64_t)1 << 31) return PRISM_ERR_UNSUPPORTED;
  return PRISM_OK;
}

// N = ceil(L / B) (Sec. 3.1, Eq. "mean-pooling": the last block holds the remaining tokens)
inline int n_blocks(const prism_params* p) { return (p->seq_len + p->block - 1) / p->block; }

inline int check_bands(const prism_params* p) {
  if (p->d_high < 0 || p->d_low < 0 || p->d_high > p->head_dim || p->d_low > p->head_dim)
    return PRISM_ERR_INVALID_ARG;
  if (p->d_high == 0 && p->d_low == 0) return PRISM_ERR_INVALID_ARG;
  if (!(p->top_p > 0.0f) || !(p->top_p <= 1.0f)) return PRISM_ERR_INVALID_ARG;   // also rejects NaN
  return PRISM_OK;
}

// Element strides between consecutive heads of the caller's tensors.  One sequence per call has
// contiguous heads (L * d); a sequence of a packed variable-length batch [heads, T, d] is addressed
// through pointers moved to its first token and the strides of the whole batch (T * d, T).
struct HeadStrides {
  size_t q;      // Q and O
  size_t kv;     // K and V
  size_t lse;    // the log-sum-exp output
};
inline HeadStrides contiguous_heads(const prism_params* p) {
  const size_t s = (size_t)p->seq_len * p->head_dim;
  return HeadStrides{s, s, (size_t)p->seq_len};
}

// The sequences of one launch.  A call on one sequence has one entry; a packed variable-length batch is taken in
// groups of up to kMaxGroupSeqs sequences that share every launch.
constexpr int kMaxGroupSeqs = 16;
struct SeqInfo {
  int32_t tok0;      // first token inside the packed tensors
  int32_t L, N;      // tokens, blocks
  int32_t v_shift;   // from tok0 to its first token in what the attention reads as V
  int32_t blk0;      // blocks of the sequences in front of it in the group ...
  int32_t tile0;     // ... and their tiles (strips) of 16 blocks
  int32_t cap;       // entries of its col_idx part
  int32_t index;     // its number in the batch
  int64_t mask0;     // its part of the mask words, of row_ptr and of col_idx starts here
  int64_t row0;
  int64_t col0;
};
// kSeqs = 1: a kernel for calls on one sequence.  The table of 16 costs 1 KB of arguments and a search per workgroup,
// 1 - 2 % of the calls whose kernels take a few microseconds (2K tokens, one head: 38.9 -> 39.7 us).
template <int kSeqs>
struct SeqTableOf {
  int32_t n;         // sequences
  int32_t nsum;      // blocks of all of them
  int32_t tiles;     // tiles of 16 blocks of all of them
  int32_t nmax;      // blocks of the longest
  SeqInfo s[kSeqs];
};
using SeqTable = SeqTableOf<kMaxGroupSeqs>;
using OneSeq = SeqTableOf<1>;
inline OneSeq only_sequence(const SeqTable& t) { return OneSeq{t.n, t.nsum, t.tiles, t.nmax, {t.s[0]}}; }
inline int clamp_capacity(int64_t n) { return n > 0x7fffffff ? 0x7fffffff : (int)n; }   // CSR offsets are int32
inline void add_sequence(SeqTable* t, const prism_params* p, SeqInfo s) {
  s.N = n_blocks(p);
  s.L = p->seq_len;
  s.blk0 = t->nsum;
  s.tile0 = t->tiles;
  t->nsum += s.N;
  t->tiles += (s.N + 15) / 16;
  t->nmax = s.N > t->nmax ? s.N : t->nmax;
  t->s[t->n++] = s;
}
inline SeqTable one_sequence(const prism_params* p, int64_t col_capacity) {
  SeqTable t = {};
  SeqInfo s = {};
  s.cap = clamp_capacity(col_capacity);
  add_sequence(&t, p, s);
  return t;
}

// Calls run(table, params of its first sequence) for groups that cover the batch; fits(table) says whether the
// sequences of a table can share their launches (a table of one always can).  Windows of kVarlenWindow
// sequences are packed longest first, each group filled with what still fits.  Stops at the first error.
constexpr int kVarlenWindow = 64;
template <typename Fits, typename Run>
inline int for_each_group(const prism_params* params, const int32_t* cu_seqlens, int n_seqs, Fits fits, Run run) {
  int64_t mo = 0, ro = 0, co = 0;
  for (int w0 = 0; w0 < n_seqs; w0 += kVarlenWindow) {
    const int n = n_seqs - w0 < kVarlenWindow ? n_seqs - w0 : kVarlenWindow;
    prism_params ps[kVarlenWindow];
    SeqInfo info[kVarlenWindow];
    int order[kVarlenWindow];
    bool done[kVarlenWindow];
    for (int i = 0; i < n; ++i) {
      ps[i] = *params;
      ps[i].seq_len = cu_seqlens[w0 + i + 1] - cu_seqlens[w0 + i];
      const int64_t N = n_blocks(&ps[i]), h = params->n_q_heads;
      const int64_t cap = (params->flags & PRISM_FLAG_BIDIRECTIONAL) ? h * N * N : h * N * (N + 1) / 2;
      info[i] = SeqInfo{};
      info[i].tok0 = cu_seqlens[w0 + i];
      info[i].cap = clamp_capacity(cap);
      info[i].index = w0 + i;
      info[i].mask0 = mo;
      info[i].row0 = ro;
      info[i].col0 = co;
      mo += h * N * ((N + 63) / 64);
      ro += h * N + 1;
      co += cap;
      done[i] = false;
      int at = i;                                    // insertion sort: longest first, equal ones in batch order
      for (; at > 0 && ps[order[at - 1]].seq_len < ps[i].seq_len; --at) order[at] = order[at - 1];
      order[at] = i;
    }
    for (int i = 0; i < n; ++i) {
      if (done[i]) continue;
      SeqTable t = {};
      add_sequence(&t, &ps[order[i]], info[order[i]]);
      for (int j = i + 1; j < n && t.n < kMaxGroupSeqs; ++j) {
        if (done[j]) continue;
        SeqTable more = t;
        add_sequence(&more, &ps[order[j]], info[order[j]]);
        if (!fits(more)) continue;
        t = more;
        done[j] = true;
      }
      const int rc = run(t, ps[order[i]]);
      if (rc != PRISM_OK) return rc;
    }
  }
  return PRISM_OK;
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

inline int launch_status() {
  return hipGetLastError() == hipSuccess ? PRISM_OK : PRISM_ERR_HIP;
}

// ---- device helpers -------------------------------------------------------------
// Wave-wide reductions on the DPP cross-lane paths (no LDS round trips): two quad
// permutes, half-row and row mirrors, then the row broadcasts; lane 63 ends up with the
// result, which is returned to every lane through a scalar register.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp_f32(float old, float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                               __builtin_bit_cast(int, x), CTRL,
                                                               ROW_MASK, 0xF, false));
}
constexpr int kDppQuadSwap1 = 0xB1;      // quad_perm [1,0,3,2]
constexpr int kDppQuadSwap2 = 0x4E;      // quad_perm [2,3,0,1]
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;
constexpr int kDppRowBcast15 = 0x142;
constexpr int kDppRowBcast31 = 0x143;

__device__ __forceinline__ float wave_sum(float x) {
  x += dpp_f32<kDppQuadSwap1>(0.f, x);
  x += dpp_f32<kDppQuadSwap2>(0.f, x);
  x += dpp_f32<kDppRowHalfMirror>(0.f, x);
  x += dpp_f32<kDppRowMirror>(0.f, x);
  x += dpp_f32<kDppRowBcast15, 0xA>(0.f, x);
  x += dpp_f32<kDppRowBcast31, 0xC>(0.f, x);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
__device__ __forceinline__ float wave_max(float x) {
  x = fmaxf(x, dpp_f32<kDppQuadSwap1>(x, x));
  x = fmaxf(x, dpp_f32<kDppQuadSwap2>(x, x));
  x = fmaxf(x, dpp_f32<kDppRowHalfMirror>(x, x));
  x = fmaxf(x, dpp_f32<kDppRowMirror>(x, x));
  x = fmaxf(x, dpp_f32<kDppRowBcast15, 0xA>(x, x));
  x = fmaxf(x, dpp_f32<kDppRowBcast31, 0xC>(x, x));
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
// The sum over the butterfly of lane ^ 32, 16, 8, 4, 2, 1, without a trip through LDS for each (us of select_small_kernel at 2K tokens and
// one head 8.9 -> 8.2, 32/8 heads, 8192 13.7 -> 12.8, 20011 36.0 -> 33.7).  Rotated by 4 in its row a lane meets lane ^ 4 or the lane 8
// from that, which holds the same sum by then.
typedef unsigned int lane_swap_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double double_of(uint32_t lo, uint32_t hi) {
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  return double_of(__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, false),
                   __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ double wave_sum(double x) {
  uint64_t b = __builtin_bit_cast(uint64_t, x);
  lane_swap_t lo = __builtin_amdgcn_permlane32_swap((uint32_t)b, (uint32_t)b, false, false);
  lane_swap_t hi = __builtin_amdgcn_permlane32_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
  b = __builtin_bit_cast(uint64_t, double_of(lo[0], hi[0]) + double_of(lo[1], hi[1]));
  lo = __builtin_amdgcn_permlane16_swap((uint32_t)b, (uint32_t)b, false, false);
  hi = __builtin_amdgcn_permlane16_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
  x = double_of(lo[0], hi[0]) + double_of(lo[1], hi[1]);
  x += dpp_f64<0x128>(x);                            // row_ror:8
  x += dpp_f64<0x124>(x);                            // row_ror:4
  x += dpp_f64<kDppQuadSwap2>(x);
  x += dpp_f64<kDppQuadSwap1>(x);
  return x;
}
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ int dpp_i32(int old, int x) {
  return __builtin_amdgcn_update_dpp(old, x, CTRL, ROW_MASK, 0xF, false);
}
// inclusive prefix sum over the 64 lanes on the DPP paths: shifts by 1, 2, 3 inside a row of 16 lanes
// (a window of four), then by 4 and 8 for the banks they reach, then the row broadcasts
__device__ __forceinline__ int wave_scan_inclusive(int x) {
  int s = x;
  s += dpp_i32<0x111>(0, x);                         // row_shr:1
  s += dpp_i32<0x112>(0, x);                         // row_shr:2
  s += dpp_i32<0x113>(0, x);                         // row_shr:3
  s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xF, 0xE, false);   // row_shr:4, banks 1-3
  s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xF, 0xC, false);   // row_shr:8, banks 2-3
  s += dpp_i32<kDppRowBcast15, 0xA>(0, s);
  s += dpp_i32<kDppRowBcast31, 0xC>(0, s);
  return s;
}
// the same over each 16 lanes
__device__ __forceinline__ int row16_scan_inclusive(int x) {
  x += dpp_i32<0x111>(0, x);
  x += dpp_i32<0x112>(0, x);
  x += dpp_i32<0x114>(0, x);
  x += dpp_i32<0x118>(0, x);
  return x;
}
__device__ __forceinline__ int wave_sum(int x) {
  x += dpp_i32<kDppQuadSwap1>(0, x);
  x += dpp_i32<kDppQuadSwap2>(0, x);
  x += dpp_i32<kDppRowHalfMirror>(0, x);
  x += dpp_i32<kDppRowMirror>(0, x);
  x += dpp_i32<kDppRowBcast15, 0xA>(0, x);
  x += dpp_i32<kDppRowBcast31, 0xC>(0, x);
  return __builtin_amdgcn_readlane(x, 63);
}

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

// fp32 -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

// The sequence that holds index i of a numbering in which sequence s starts at mult * blk0[s].
template <int kSeqs>
__device__ __forceinline__ int seq_of(const SeqTableOf<kSeqs>& seqs, int i, int mult) {
  int s = 0;
  if (kSeqs == 1) return s;
  while (s + 1 < seqs.n && i >= mult * seqs.s[s + 1].blk0) ++s;
  return s;
}

}  // namespace prism
