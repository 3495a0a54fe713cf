// Block-sparse causal flash attention of libprism (gfx950, bf16 MFMA, fp32 online softmax).
//
// Sec. 2 "Block-Sparse Attention": dense QK^T / softmax / PV with online accumulation,
// restricted to the (q-block, kv-block) pairs listed in a CSR index list.
//
// Formulation.  Each wave owns 32 query rows and works on the TRANSPOSED problem so that
// every per-query quantity (running max, running sum, output scale) lives in one lane:
//     S^T = K Q^T      (v_mfma_f32_32x32x16_bf16: A = K tile rows, B = Q rows)
//     O^T += V^T P^T   (A = V^T rows, B = P^T, which is exactly the accumulator layout of S^T
//                       after bf16 conversion, so P never leaves registers)
// In the 32x32 accumulator layout lane l holds query column l%32 and, per 32-key tile,
// keys 8*(r/4) + 4*(l/32) + r%4 for r = 0..15.  One MFMA K-step of PV therefore consumes
// keys {16s + 8g + 4*(l/32) + i}; the V^T operand must present the same keys in the same
// slots.  The general kernel reads V, or a plain copy of it, and transposes on the way from LDS to the registers
// (ds_read_b64_tr_b16 hands a lane four keys of its dim).  The 64-queries-per-wave kernel reads an fp16 image of V^T: per kv
// block [d][B], whose key positions inside every group of 16 are permuted to
// pos = 8*hf + 4*g + i  for key = 8*g + 4*hf + i.  A 16-byte LDS read then yields one
// A operand.
#include "prism_common.h"

#include <mutex>
#include <type_traits>

namespace prism {

// =====================================================================================
// V re-layout: V [h_kv, L, 128], whole blocks  ->  fp16 image [h_kv, N, 128, 128] of V^T with permuted key positions (the
// 64-queries-per-wave kernel forms its P V product in fp16: 11 significant bits for P instead of 8).
// Every bf16 value of magnitude in [2^-17, 65504] (and zero) is an fp16 value, so the conversion is
// exact there; smaller magnitudes lose at most 2^-25 absolute.  A block holding a finite value beyond
// the fp16 range sets range_flags[kv head * N + block] = 1 (else 0): such inputs go through the
// general kernel, which reads V or its copy.  Bound by the bytes: where both are written, the copy is stored from the registers that V
// passes through (us, two kernels / one: 32/8 heads, 8192 tokens 16.1 / 13.0, 32768 50.6 / 38.1, 131072 194.6 / 145.1).
// =====================================================================================
constexpr int kImageRows = 128;                      // tokens of a block of the image
typedef uint16_t ImageTile[kImageRows][kHeadDim + 2];
template <int kThreads>
__device__ __forceinline__ void vt_image_tile(ImageTile& tile, int& s_over, const uint16_t* __restrict__ src,
                                              uint16_t* __restrict__ copy, uint16_t* __restrict__ dst16,
                                              int32_t* __restrict__ range_flag, int flag_value) {
  const int t = threadIdx.x;
  if (t == 0) s_over = 0;
  constexpr int RCH = kHeadDim / 8;                  // 16-byte chunks per token row
  for (int idx = t; idx < kImageRows * RCH; idx += kThreads) {
    const int row = idx / RCH, c = idx % RCH;        // V is read once: streaming (non-temporal) loads
    const u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + (size_t)row * kHeadDim + c * 8));
    if (copy != nullptr) *reinterpret_cast<u32x4*>(copy + (size_t)row * kHeadDim + c * 8) = x;
    uint32_t* dst = reinterpret_cast<uint32_t*>(&tile[row][c * 8]);   // 4-byte aligned: row stride 2*d + 4 B
    dst[0] = x[0]; dst[1] = x[1]; dst[2] = x[2]; dst[3] = x[3];
  }
  __syncthreads();
  constexpr int CPR = kImageRows / 8;                // 16-byte chunks per image row
  bool over = false;
  for (int idx = t; idx < kHeadDim * CPR; idx += kThreads) {
    const int d = idx / CPR, c = idx % CPR;
    uint32_t w16[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      // position p = c*8 + e inside the row; group a = p/16, hf = (p/8)&1, g = (p/4)&1, i = p&3
      const int p0 = c * 8 + e, p1 = p0 + 1;
      const int k0 = (p0 & ~15) + 8 * ((p0 >> 2) & 1) + 4 * ((p0 >> 3) & 1) + (p0 & 3);
      const int k1 = (p1 & ~15) + 8 * ((p1 >> 2) & 1) + 4 * ((p1 >> 3) & 1) + (p1 & 3);
      const float fa = bf16_bits_to_float(tile[k0][d]), fb = bf16_bits_to_float(tile[k1][d]);
      over |= (fabsf(fa) > 65504.f && fabsf(fa) < INFINITY) || (fabsf(fb) > 65504.f && fabsf(fb) < INFINITY);
      const _Float16 ha = (_Float16)fa, hb = (_Float16)fb;
      w16[e >> 1] = (uint32_t)__builtin_bit_cast(uint16_t, ha) | ((uint32_t)__builtin_bit_cast(uint16_t, hb) << 16);
    }
    *reinterpret_cast<uint4*>(dst16 + (size_t)d * kImageRows + c * 8) = make_uint4(w16[0], w16[1], w16[2], w16[3]);
  }
  if (over) s_over = 1;                              // benign race: every writer stores 1
  __syncthreads();
  if (t == 0) *range_flag = s_over != 0 ? flag_value : 0;
}

__global__ __launch_bounds__(256) void vt_image_kernel(const uint16_t* __restrict__ v, int N, size_t kv_head_stride,
                                                       uint16_t* __restrict__ copy, uint16_t* __restrict__ vt16, int32_t* __restrict__ range_flags) {
  __shared__ ImageTile tile;
  __shared__ int s_over;
  const int blk = blockIdx.x, kvh = blockIdx.y;
  const size_t at = ((size_t)kvh * N + blk) * kHeadDim * kImageRows;
  vt_image_tile<256>(tile, s_over, v + (size_t)kvh * kv_head_stride + (size_t)blk * kImageRows * kHeadDim,
                     copy != nullptr ? copy + at : nullptr, vt16 + at, range_flags + kvh * N + blk, 1);
}

// The copy of V alone: [h_kv, N * B, d], of which the L tokens are written.
__global__ __launch_bounds__(256) void v_copy_kernel(const uint16_t* __restrict__ v, size_t chunks, size_t from_stride,
                                                     size_t to_stride, uint16_t* __restrict__ copy) {
  const u32x4* from = reinterpret_cast<const u32x4*>(v + (size_t)blockIdx.y * from_stride);
  u32x4* to = reinterpret_cast<u32x4*>(copy + (size_t)blockIdx.y * to_stride);
  const size_t at = (size_t)blockIdx.x * 1024 + threadIdx.x;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (at + i * 256 < chunks) to[at + i * 256] = __builtin_nontemporal_load(from + at + i * 256);
}

// A queue entry names its sequence in the high bits of the head number (only where a group holds several).
constexpr int kSeqShift = 20;

// What decides, on the device, whether the lists and values of a sequence suit the specialised attention kernels: sequence
// s of the call is "dirty" when bit s of any word of the two arrays is set.
struct DirtyFlags {
  const int32_t* a;
  const int32_t* b;
  int32_t na, nb;
};
// The dirty sequences, one bit each.  The answer has a word of its own: every wave reads it behind the last barrier here,
// so a word that the caller goes on to write (the queue position, say) could change under a wave that reads late.
template <int kThreads>
__device__ __forceinline__ int dirty_sequences(const DirtyFlags& f) {
  __shared__ int verdict;
  if (threadIdx.x == 0) verdict = 0;
  int bad = 0;
  for (int i = threadIdx.x; i < f.na; i += kThreads) bad |= f.a[i];
  for (int i = threadIdx.x; i < f.nb; i += kThreads) bad |= f.b[i];
  __syncthreads();
  if (bad != 0) atomicOr(&verdict, bad);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(verdict);
}

// =====================================================================================
// Sparse attention kernel.  One workgroup works on one (q-head, q-block) row at a time;
// BLK/32 waves of 32 queries.
// LDS: K tile and V tile [BLK][d] bf16 (d = 64, 128, 256), 16-byte chunks XOR-swizzled by
// row so that the 16-lane column reads of K and the transposing reads of V are conflict-free.  Tiles are copied global -> LDS
// asynchronously, without passing through registers.
// Step per listed kv block (each tile buffer is refilled as soon as its last reader is done):
//     K(j) in LDS | S^T = K Q^T, requests of V(j) between the MFMAs | barrier
//     online softmax, requests of K(j+1) at its start or in it | wait V(j) | barrier | O^T += V^T P^T | wait K(j+1) | barrier
// Pairs of 64 x 256 have two buffers per tile (AttnCfg).  In the plain forms, where two workgroups share a CU, they
// fit at 64 x 64, 128 x 64 and 64 x 256 and are no gain over the range: us of attention, one buffer -> two, 32/8 heads: 128 x 64
// at 8192 tokens 127 -> 123, at 20000 331 -> 345, at 32768 755 -> 790; 64 x 256 at 16320 1374 -> 1432, at 32768 3159 -> 3257;
// 64 x 64 at 16384 298 -> 303, at 40000 1060 -> 1007.
// The workgroups are persistent: a workgroup pulls its next row from its XCD's queue at the top
// of the last step of the current row and reads that row's queue entry during the last PV, so
// a row switch exposes only the load of the Q rows and of the first K tile.
// =====================================================================================
// PAIR: a workgroup serves two neighbouring q-blocks of one q-head (twice the waves) and walks the
// union of their two lists, so a tile that both list is copied once.
template <int BLK, int D, bool PAIR = false>
struct AttnCfg {
  static constexpr int kRowWaves = BLK / 32;                // waves of one q-block
  static constexpr int kWaves = kRowWaves * (PAIR ? 2 : 1);
  static constexpr int kThreads = kWaves * 64;
  static constexpr int kTileBytes = BLK * D * 2;
  static constexpr int kChunks = kTileBytes / 16;          // 16-byte pieces per tile
  static constexpr int kPerThread = kChunks / kThreads;    // = D / 16 (D / 32 with PAIR)
  static constexpr int kKCpr = D / 8;                      // chunks per K row
  static constexpr int kDTiles = D / 32;                   // 32-dim tiles of the output
  static constexpr int kKSteps = D / 16;                   // MFMA k-steps of S^T = K Q^T
  static constexpr int kWavesPerSimd = D > 128 ? 1 : 2;    // register budget: 512 or 256 per lane
  // Where the requests of the next K tile go.  A wave that issues all its pieces of a tile in a row stands still until the
  // texture path has taken them, 500 - 1000 cycles of a step (S phase 2770 cycles, PV phase with as many MFMAs 1640).  The
  // V pieces are spread over the S MFMAs in every form; the K pieces over the maximum at B = 128, over the exponentials
  // at d = 256, where no second wave of the SIMD fills the gap; at B = 64 the softmax is too short to hide a later request.
  // us of attention, all in a row / V spread / K over the maximum too / K over the exponentials instead:
  // 128 x 128, 32/8 heads, 12345 tokens 281 / 274 / 271 / 270, 40001 1822 / 1752 / 1755 / 1754; 128 x 64, 12345
  // 195 / 189 / 186 / 183, 28001 591 / 592 / 590 / 605; 128 x 256, 4/4 heads, 16384 216 / 201 / 192 / 187; pair 64 x 256, 16/4,
  // 16384 714 / 701 / 697 / 682; pair 64 x 128, 8/2, 60000 605 / 584 / 591 / 592; 64 x 64, 32/8, 16384 305 / 298 / 298 / 316.
  static constexpr int kPiecesInMax = BLK == 128 && D <= 128 ? kPerThread : 0;
  static constexpr int kPiecesInExp = D > 128 ? kPerThread : 0;
  // Two buffers per tile.  A pair of 256-dim rows has the CU to itself, so nothing fills the gaps where its waves wait for a tile, and
  // the 160 KB hold both: the copies have a whole step to land, and a step has one barrier instead of three.  us of attention,
  // one buffer -> two: 16/4 heads, 16384 tokens 515 -> 486, 32/8, 8192 312 -> 304, 8/2, 32768 598 -> 555.  The requests lie over the
  // MFMAs of S, K and V by turns, one for two MFMAs (one for each MFMA of the first half 518, V's over the exponentials 504).  The
  // scores of the next block between the instructions of this one's softmax as well: 544; a lone wave is bound by issue there.
  static constexpr bool kTwo = PAIR && D > 128;
};

// Asynchronous global -> LDS tile copies (buffer_load_dwordx4 ... lds: every lane fetches 16
// bytes at rsrc.base + voffset + soffset and the wave's 64 pieces land contiguously in LDS
// at M0-base + 16*lane).  LDS slot p (16-byte units) of a tile belongs to (row, c') with c'
// the swizzled chunk position; the lane that fills it reads global chunk
// c = c' ^ swizzle(row), i.e. the swizzle is applied on the global side.
// Buffer (not flat/global) addressing is used on purpose: LDS reads issued while such
// copies are in flight then keep exact lgkmcnt tracking in the compiler.
typedef __attribute__((address_space(3))) void* lptr_t;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  // raw buffer, 32-bit data format, no swizzle, no TID addition
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// XOR applied to the chunk index of K-tile row `row` so that 16 consecutive rows put the same
// chunk on 16 different LDS bank groups: rows of 128 bytes (d = 64) come two to a 256-byte line,
// rows of 512 bytes (d = 256) wrap the banks twice.
template <int D>
__device__ __forceinline__ int k_row_swizzle(int row) {
  return D == 64 ? ((row >> 1) & 7) : (row & 15);
}

// byte offset inside a tile of the 16-byte piece that LDS slot p holds
template <int BLK, int D>
__device__ __forceinline__ int k_piece_offset(int p) {
  using C = AttnCfg<BLK, D>;
  const int row = p / C::kKCpr;
  return row * (D * 2) + (((p % C::kKCpr) ^ k_row_swizzle<D>(row)) << 4);
}
// XOR applied to the 64-byte groups of V-tile row `row`, so that the four keys of a transposing read lie in four bank groups: rows
// of 128 bytes (d = 64) come two to a 256-byte line.
template <int D>
__device__ __forceinline__ int v_row_swizzle(int row) {
  return D == 64 ? ((row >> 1) & 1) : (row & 3);
}
template <int BLK, int D>
__device__ __forceinline__ int v_piece_offset(int p) {
  using C = AttnCfg<BLK, D>;
  const int row = p / C::kKCpr;
  return row * (D * 2) + (((p % C::kKCpr) ^ (v_row_swizzle<D>(row) << 2)) << 4);
}

// this wave's first LDS slot of a tile's piece 0, wave-uniform and re-materialised per step so that the per-piece M0
// values are formed with scalar adds instead of being kept live (and spilled) across the whole loop
__device__ __forceinline__ int first_slot(int t) {
  int wave_base = __builtin_amdgcn_readfirstlane(t & ~63);
  asm volatile("" : "+s"(wave_base));
  return wave_base;
}

// the pieces [i0, i1) of the kPerThread 16-byte pieces that a thread copies of a tile
template <int BLK, int D, bool PAIR>
__device__ __forceinline__ void async_load_k_pieces(__amdgpu_buffer_rsrc_t rs, int tile_off, char* lds, int t,
                                                    int wave_base, int i0, int i1) {
  using C = AttnCfg<BLK, D, PAIR>;
#pragma unroll
  for (int i = i0; i < i1; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lptr_t)(lds + (i * C::kThreads + wave_base) * 16), 16,
                                             k_piece_offset<BLK, D>(i * C::kThreads + t), tile_off, 0, 0);
}

template <int BLK, int D, bool PAIR>
__device__ __forceinline__ void async_load_v_pieces(__amdgpu_buffer_rsrc_t rs, int tile_off, char* lds, int t,
                                                     int wave_base, int i0, int i1) {
  using C = AttnCfg<BLK, D, PAIR>;
#pragma unroll
  for (int i = i0; i < i1; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lptr_t)(lds + (i * C::kThreads + wave_base) * 16), 16,
                                             v_piece_offset<BLK, D>(i * C::kThreads + t), tile_off, 0, 0);
}

// One piece of such a copy, written as asm: the compiler, seeing the builtin, would wait for a copy into one of two buffers before
// it reads the other.  Waited for with wait_async_loads.
struct TileRsrc {
  u32x4 w;
};
__device__ __forceinline__ TileRsrc make_tile_rsrc(const void* base, uint32_t bytes) {
  const uint64_t b = (uint64_t)base;
  TileRsrc r;
  r.w[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  r.w[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(b >> 32) & 0xffffu));
  r.w[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r.w[3] = 0x00020000u;
  return r;
}
__device__ __forceinline__ void async_piece(const TileRsrc& rs, int lane_off, int tile_off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(lane_off), "s"(rs.w),
               "s"(tile_off)
               : "m0", "memory");
}

// Waits on the vector-memory counter, written with the builtin (immediate: vmcnt in bits 3:0,
// expcnt = 7 and lgkmcnt = 15 meaning "no wait") rather than inline asm, so that the compiler's
// own wait-count bookkeeping sees them: it then knows which tile copies have landed and adds no
// conservative vmcnt(0) of its own in front of the LDS reads of a finished tile.
__device__ __forceinline__ void wait_async_loads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
  asm volatile("" ::: "memory");
}
// all but the youngest tile copy (kPerThread = d/16 vector-memory operations per thread) are complete
template <int kPerThread>
__device__ __forceinline__ void wait_async_loads_but_last_tile() {
  static_assert(kPerThread <= 16, "vmcnt immediate");
  asm volatile("" ::: "memory");
  // vmcnt(kPerThread): low four bits in 3:0, the two high bits in 15:14
  __builtin_amdgcn_s_waitcnt(0x0F70 | (kPerThread & 15) | ((kPerThread >> 4) << 14));
  asm volatile("" ::: "memory");
}

// max / sum of a value with the lane 32 away (the two lanes that share a query), on the
// v_permlane32_swap cross-lane path: an LDS shuffle here would queue behind the tile traffic
// on the critical path of every step.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float other_half_max(float x) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float other_half_sum(float x) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Workgroup barrier of the tile loop: this wave's LDS accesses are complete, then s_barrier.
// Unlike __syncthreads() it carries no memory fence, so the compiler adds no wait for the global
// loads, stores and atomics in flight (the next tile copies, the previous row's output, the
// queue pull); the tile copies are waited for explicitly with vmcnt where their data is needed.
__device__ __forceinline__ void tile_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Queue entry of one row, written by queue_fill_kernel:
//   x = q-head, y = q-block u | (first valid key block << 16), z = index of that entry in
//   col_idx, w = end of the row's list (z == w: the row has no valid entry).
// Every queue (one per XCD) owns a contiguous segment of the table: `plan` = { start[8], len[8], len + 1 of the queues
// that were seen exhausted[8], flags[8], rows with a CU to themselves[8] }; a workgroup's pulls p = 0, 1, 2, ... from
// queue x are the entries start[x] + p while p < len[x].
enum { kItemEnd = 0, kItemRow = 2 };
// MI355X: 8 accelerator dies (XCDs), each with its own L2; workgroups are dealt to them round-robin,
// so the attention kernels keep one work queue per XCD (the plan below has room for exactly kXcds).
constexpr int kXcds = 8;
constexpr int kPlanStart = 0, kPlanLen = 8, kPlanCounter = 16, kPlanFlags = 24, kPlanAlone = 32, kPlanInts = 40;
// plan[kPlanFlags]: bit 0 = some list holds an entry that must be skipped (negative, beyond the
// row's last admissible block): such lists go through the general kernel, clean lists through the
// 64-queries-per-wave kernel, each sequence of a packed batch for itself; each of the two kernels returns at once when
// it is not its turn.
constexpr int kFlagDirtyLists = 1;

// Pull counters of the queues, on cache lines of their own: all pulls on one line are served one after the other, 16 ns
// each, which made 40 us of the 64 us that 2048 rows without any listed block took, and held the short rows at the end of
// a longer call back (us of attention, 8512 rows of 32/8 heads, 17024 tokens, B = 64 521 -> 449; 10016 of d = 64, 20001
// tokens 478 -> 377; 14336 of 28/4, 64K, B = 128 2514 -> 2483).  They start behind the workgroups' first rows, which are
// dealt out by workgroup number.  The counters of the plan are left to record that a queue was exhausted.
struct PullCounters {
  int32_t* at;
  int32_t stride;        // ints between two queues' counters
};
// the rows of queue x that are dealt to the first pulls of the workgroups x, x + n_queues, ...
__device__ __forceinline__ int dealt_rows(int x, int n_queues, int grid) {
  return x < n_queues ? (grid - x + n_queues - 1) / n_queues : 0;
}

// The longest rows of a short call have a CU to themselves.  With two workgroups on every CU a row among them advances a
// block in 2.25 us and alone in 1.3 (128 x 128, four waves): at 8K tokens its 62 blocks ended at 142 us, the other
// workgroups, out of rows, at 105 - 115.  plan[kPlanAlone + x] has bit p for the p-th row of queue x if it is such a
// row; it is dealt to workgroup x + 8 p, which shares its CU with workgroup x + 8 p + gridDim.x / 2 (in the order that
// the hardware places a grid of two workgroups per CU; otherwise only the gain is lost).  That one ends at once, and the
// workgroups behind it move up to its row.  Returns the workgroup's first row in its queue, or -1: it ends.  Of a packed batch a
// launch may leave the long rows to another kernel: the general kernel behind the 64-queries-per-wave kernel then heeds no
// mark (its counters start accordingly), and there the workgroup beside a row that is left goes on.
__device__ __forceinline__ int first_row(unsigned alone, int n_queues, bool heed) {
  const unsigned shift = n_queues == 1 ? 0 : 3;             // kXcds or one; divisions are 40 instructions each
  const int p = blockIdx.x >> shift, half = gridDim.x >> 1 >> shift;
  if (!heed || alone == 0 || p < half) return p;            // bits are set only where half <= 32
  const int mate = p - half;
  return (alone >> mate) & 1u ? -1 : p - __popc(alone & ((1u << mate) - 1u));
}

__device__ __forceinline__ int item_kind(int pulled, int seg_start, int seg_len, int* entry) {
  if (pulled >= seg_len) return kItemEnd;
  *entry = seg_start + pulled;
  return kItemRow;
}

// 64 entries of one of a pair's lists, one a lane.  Loaded one by one, two steps ahead, the entries came through the scalar
// cache, whose answers arrive in no order: the first LDS read of a step then waited for them, 300 - 1000 cycles of a
// step.  us of attention, entry by entry -> from here: 64 x 128, 8/2 heads, 60000 tokens 583 -> 550, 32/8, 12288 304 -> 292,
// 20480 557 -> 546, 32768 1329 -> 1314; 64 x 256, 16/4, 16384 680 -> 662.  The other forms, one list and one entry a step, gain
// nothing (128 x 128, 32/8, 20011 516 -> 524; 128 x 64, 32768 825 -> 839).
struct ListWindow {
  const int32_t* cols;
  int first, end, lane, held;
  __device__ __forceinline__ void fetch(int i) {
    first = i;
    held = cols[min(i + lane, end - 1)];
  }
  __device__ __forceinline__ void start(const int32_t* c, int i, int e, int l) {
    cols = c;
    end = e;
    lane = l;
    if (i < e) fetch(i);
  }
  // entry i, first <= i < end; i never goes back
  __device__ __forceinline__ int at(int i) {
    if (i - first >= 64) fetch(i);
    return __builtin_amdgcn_readlane(held, i - first);
  }
};

// kStreamOnly (PRISM_FLAG_STREAM_ONLY): the same tile copies, waits, barriers and queue traffic
// with the arithmetic left out; it measures how long the memory side of a call takes alone.
// kPair (B = 64, an even number of blocks, every list ascending and clean): items and plan describe PAIR
// rows (q-blocks 2u' and 2u' + 1 of a head, whose two lists lie one behind the other in col_idx); the
// workgroup walks the union of the two lists in ascending order, copies every tile of the union once,
// and the waves of a q-block compute only in the steps whose block their own list names.  `flags` is what
// the list check found.  A kernel launched behind another one takes what that one left (only_dirty): behind the pair
// kernel, which returns at once if any sequence is dirty, the whole call then (kDirtyCall; both give the same bits); behind
// the 64-queries-per-wave kernel the one sequence of the call (kDirtyCall) or the dirty ones of a packed batch
// (kDirtySequences), so that no sequence's bits follow from the others'.
enum { kEverything, kDirtyCall, kDirtySequences };
template <int BLK, bool kStreamOnly, int D, bool kPair, bool kKeepMask>
__global__ __launch_bounds__((AttnCfg<BLK, D, kPair>::kThreads), (AttnCfg<BLK, D, kPair>::kWavesPerSimd)) void sparse_attn_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ vals, size_t v_head_stride,
    const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, const int4* __restrict__ items,
    int32_t* __restrict__ plan, PullCounters pulls, DirtyFlags flags,
    uint16_t* __restrict__ out, float* __restrict__ lse, int h, int h_kv, SeqTable seqs,
    HeadStrides hs, int causal, int only_dirty) {
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the kernel's signature
  using C = AttnCfg<BLK, D, kPair>;
  constexpr int KS = C::kKSteps, DT = C::kDTiles;
  constexpr int KT = BLK / 32;                       // 32-key tiles per kv block
  constexpr bool kTwo = C::kTwo && !kStreamOnly;
  __shared__ __attribute__((aligned(16))) char lds_k[C::kTileBytes * (kTwo ? 2 : 1)];
  __shared__ __attribute__((aligned(16))) char lds_v[C::kTileBytes * (kTwo ? 2 : 1)];
  __shared__ int next_item, next_queue;
  int take = ~0;                                            // the sequences that are this launch's to do
  if (kPair) {
    if (dirty_sequences<C::kThreads>(flags) != 0) return;   // the plain kernel takes this call
  } else if (only_dirty != kEverything) {
    const int dirty = dirty_sequences<C::kThreads>(flags);
    if (blockIdx.x == 0 && threadIdx.x == 0) plan[kPlanFlags] = dirty != 0 ? kFlagDirtyLists : 0;
    if (dirty == 0) return;                                 // the kernel launched in front of this one took it
    if (only_dirty == kDirtySequences) take = dirty;
  }

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int l32 = lane & 31, hf = lane >> 5;
  const int g = h / h_kv;
  // which of the two q-blocks of a pair row this wave belongs to (wave-uniform)
  const int sub = kPair ? __builtin_amdgcn_readfirstlane(wave / C::kRowWaves) : 0;
  // log2(e) / sqrt(d)
  const float sm_scale = 1.4426950408889634f * (D == 64 ? 0.125f : (D == 128 ? 0.08838834764831845f : 0.0625f));

  // LDS read offsets of this lane inside a 32-row slab: row l32, swizzled chunk
  // (2*step + hf) ^ swizzle(row).
  constexpr int kDepth = 8;                                // LDS reads kept in flight
  constexpr int kGroups = D > 128 ? 4 : DT;                // 64-byte groups of a V row that the swizzle mixes
  int koff[KS], voff[kGroups];
#pragma unroll
  for (int st = 0; st < KS; ++st) koff[st] = l32 * (D * 2) + (((2 * st + hf) ^ k_row_swizzle<D>(l32)) << 4);
  // V: lane l supplies the address of 4 dims of key 4*hf + (l%16)/4 of a 16-key step, and receives 4 keys of dim l%32.  Two such
  // reads make an operand that one 16-byte read of a transposed image would be, at no more than 1 % (us of attention on an image that
  // is there, transposed / as given: 128 x 128, 32/8 heads, 20011 tokens 612.8 / 614.2, 16 heads, 19290, bidirectional 514.7 / 516.1,
  // 128 x 64, 8192 119.2 / 119.7, 12345 192.5 / 193.8, 32768 981.3 / 980.8, 8/2, 40000 289.1 / 292.3, 64 x 64, 16384 310.5 / 312.3, 32000
  // 932 / 929, pair 64 x 128, 32768 1478 / 1469, 16 heads, 30000 986 / 982).  Packed batches then need no image, and the others a plain copy:
  // preparation and attention, image / copy: 128 x 128, 20011 627 / 629, bidirectional 19290 535 / 530, 64 x 128, 32768 1545 / 1525.
#pragma unroll
  for (int i = 0; i < kGroups; ++i) {
    const int key = 4 * hf + ((lane >> 2) & 3);
    voff[i] = key * (D * 2) + ((i ^ v_row_swizzle<D>(key)) << 6) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
  }
  // one A operand of O^T += V^T P^T: dims 32*dt ..+31, keys 16*st + {8*g + 4*hf + i}
  auto v_frag = [&](int dt, int st) __attribute__((always_inline)) {
    typedef __attribute__((address_space(3))) bf16x4* lv4_t;
    const char* at = lds_v + voff[dt % kGroups] + (dt / kGroups) * (kGroups * 64) + st * (16 * D * 2);
    const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lv4_t)at), b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lv4_t)(at + 8 * D * 2));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  // Persistent workgroups pull rows from per-XCD queues (workgroups are dealt round-robin to the
  // 8 XCDs, and each XCD has its own L2).  A queue runs through neighbouring q-blocks of one
  // q-head at a time, so the 64 workgroups of an XCD work on neighbouring rows of one head: such
  // rows list many of the same key blocks (stripes, sinks, local windows; all of them for dense
  // lists) at about the same position of their lists, and the tile one of them fetches is still
  // in the XCD's L2 when the others ask for it.
  // A workgroup whose queue is exhausted goes on with rows of another XCD's queue, so the XCDs
  // finish together although the lists of one may take longer per block than those of another;
  // it leaves the loop once it has seen every queue exhausted.
  const int n_queues = gridDim.x < kXcds ? 1 : kXcds;
  int my_queue = blockIdx.x % n_queues;
  int seg_start = plan[kPlanStart + my_queue];
  int seg_len = plan[kPlanLen + my_queue];
  const unsigned alone = plan[kPlanAlone + my_queue];
  asm volatile("" ::"s"(seg_start), "s"(seg_len), "s"(alone));   // three requests, one wait (8/2 heads, 4096 tokens 37.2 -> 36.4 us)
  int32_t* __restrict__ counter = pulls.at;

  // The queue is pulled when a workgroup is about to become free (at the top of the last
  // step of its row), so neighbouring rows of the queue start close together; the pull and the
  // read of the next row's queue entry are hidden behind that last step.
  int lane_zero;                                     // 0, but opaque to the compiler
  asm volatile("v_mov_b32 %0, 0" : "=v"(lane_zero));
  constexpr bool kBehind = BLK == 128 && D == kHeadDim;      // this form stands behind the 64-queries-per-wave kernel
  const int first = first_row(alone, n_queues, !kBehind || only_dirty != kDirtySequences);
  if (first < 0) return;
  if (t == 0) next_item = first;
  __syncthreads();
  int cur_x = 0, cur_y = 0, cur_z = 0, cur_w = 0;     // the current row's queue entry, wave-uniform
  int kind_cur;
  {
    int e = 0;
    kind_cur = item_kind(__builtin_amdgcn_readfirstlane(next_item), seg_start, seg_len, &e);
    if (kind_cur == kItemRow) {
      const int4 it0 = items[e];
      cur_x = it0.x; cur_y = it0.y; cur_z = it0.z; cur_w = it0.w;
    }
  }
  __syncthreads();
  // requests of the last step of a row (not re-initialised per row: overwriting a register that a
  // load in flight will write would force a wait for every older memory operation)
  int4 item_nxt = make_int4(0, 0, 0, 0);
  int pulled_reg = 0;
  // two buffers per tile: where the current ones start, and this lane's places in pieces 0 and 1 of a K tile and in a piece of V
  int buf = 0;
  const int k_lane0 = kTwo ? k_piece_offset<BLK, D>(t) : 0, k_lane1 = kTwo ? k_piece_offset<BLK, D>(C::kThreads + t) : 0;
  const int v_lane = kTwo ? v_piece_offset<BLK, D>(t) : 0;

  for (;;) {
    if (kind_cur == kItemEnd) {
      // Own queue exhausted: look (one coherent read of the 8 pull counters, no atomic) for a
      // queue that still has rows, nearest first round the ring, and pull from it.  A counter
      // only grows, so a queue seen exhausted stays so; the atomic pull decides who gets a row.
      if (wave == 0) {
        if (lane == 0) plan[kPlanCounter + my_queue] = seg_len + 1;
        int taken = 0x7fffffff, len = 0;
        if (lane < n_queues) {
          taken = __hip_atomic_load(counter + lane * pulls.stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          len = plan[kPlanLen + lane];
        }
        const unsigned long long open = __ballot(taken < len);
        int pick = -1;
        for (int s = 1; s < n_queues && pick < 0; ++s) {
          const int x = my_queue + s < n_queues ? my_queue + s : my_queue + s - n_queues;
          if ((open >> x) & 1ull) pick = x;
        }
        if (lane == 0) {
          next_queue = pick;
          if (pick >= 0) next_item = atomicAdd(counter + pick * pulls.stride, 1);
        }
      }
      __syncthreads();
      const int pick = __builtin_amdgcn_readfirstlane(next_queue);
      if (pick < 0) break;
      my_queue = pick;
      seg_start = plan[kPlanStart + my_queue];
      seg_len = plan[kPlanLen + my_queue];
      int e = 0;
      kind_cur = item_kind(__builtin_amdgcn_readfirstlane(next_item), seg_start, seg_len, &e);
      if (kind_cur == kItemRow) {
        const int4 it0 = items[e];
        cur_x = it0.x; cur_y = it0.y; cur_z = it0.z; cur_w = it0.w;
      }
      __syncthreads();
      continue;
    }
    cur_x = __builtin_amdgcn_readfirstlane(cur_x);
    cur_y = __builtin_amdgcn_readfirstlane(cur_y);
    cur_z = __builtin_amdgcn_readfirstlane(cur_z);
    cur_w = __builtin_amdgcn_readfirstlane(cur_w);
    const int sq = seqs.n > 1 ? cur_x >> kSeqShift : 0;
    const int hq = seqs.n > 1 ? cur_x & ((1 << kSeqShift) - 1) : cur_x;
    const int L = seqs.s[sq].L, N = seqs.s[sq].N, tok0 = seqs.s[sq].tok0;
    const int vmax_nc = N - 1;
    const int tail = L - (N - 1) * BLK;              // tokens in the last block (BLK unless ragged)
    const uint32_t head_bytes = (uint32_t)L * D * 2;
    const int32_t* __restrict__ cols = col_idx + seqs.s[sq].col0;
    const int u = cur_y & 0xffff;
    int v = (cur_y >> 16) & 0xffff;
    int it = cur_z;
    const int end = cur_w;
    const bool mine = ((take >> sq) & 1) != 0;
    const bool has_work = kind_cur == kItemRow && it < end && mine;
    const int kvh = hq / g;
    // `u` is the index of the row among the head's rows: a q-block, or a pair of them
    const int qrow = u * (C::kWaves * 32) + wave * 32 + l32;   // >= L for the padding rows of a ragged last block
    const int u_own = kPair ? 2 * u + sub : u;                 // the q-block this wave's queries belong to
    int kind_nxt = kItemEnd;

    if (!has_work) {
      // a row without a valid entry (o = 0, lse = -inf), or another kernel's: no tile work; pull the next row right away
      if (kind_cur == kItemRow && mine && qrow < L) {
        uint16_t* op = out + (size_t)hq * hs.q + (size_t)(tok0 + qrow) * D + hf * (D / 2);
#pragma unroll
        for (int c = 0; c < D / 16; ++c) *reinterpret_cast<uint4*>(op + c * 8) = make_uint4(0u, 0u, 0u, 0u);
        if (lse != nullptr && hf == 0) lse[(size_t)hq * hs.lse + tok0 + qrow] = -INFINITY;
      }
      if (t == 0) next_item = atomicAdd(counter + my_queue * pulls.stride, 1);
      __syncthreads();
      int e = 0;
      kind_cur = item_kind(__builtin_amdgcn_readfirstlane(next_item), seg_start, seg_len, &e);
      if (kind_cur == kItemRow) {
        const int4 it0 = items[e];
        cur_x = it0.x; cur_y = it0.y; cur_z = it0.z; cur_w = it0.w;
      }
      __syncthreads();
      continue;
    }

    // K and V of this kv head as buffer resources (tile v starts at byte v * kTileBytes).
    // K is the caller's tensor: rows past L in a ragged last block are outside the resource and
    // read as zeros, as are those of V.
    const __amdgpu_buffer_rsrc_t krs = make_rsrc(k + (size_t)kvh * hs.kv + (size_t)tok0 * D, head_bytes);
    const __amdgpu_buffer_rsrc_t vrs = make_rsrc(vals + (size_t)kvh * v_head_stride + (size_t)(tok0 + seqs.s[sq].v_shift) * D, head_bytes);
    const int vmax = causal ? u_own : vmax_nc;
    // With two buffers per tile, step j reads the buffers j & 1, and both tiles of the next block are copied into the others; `buf` is
    // where they start, and what the lanes' read offsets hold already.
    TileRsrc krs2 = {}, vrs2 = {};
    if constexpr (kTwo) {
      krs2 = make_tile_rsrc(k + (size_t)kvh * hs.kv + (size_t)tok0 * D, head_bytes);
      vrs2 = make_tile_rsrc(vals + (size_t)kvh * v_head_stride + (size_t)(tok0 + seqs.s[sq].v_shift) * D, head_bytes);
    }
    auto other_buffer = [&]() __attribute__((always_inline)) {
      const int by = buf == 0 ? C::kTileBytes : -C::kTileBytes;
      buf += by;
#pragma unroll
      for (int st = 0; st < KS; ++st) koff[st] += by;
#pragma unroll
      for (int i = 0; i < kGroups; ++i) voff[i] += by;
    };
    auto copy_k = [&](int blk, int at, int wave_base, int i) __attribute__((always_inline)) {
      // (16 rows from one piece to the next but one: the same swizzle)
      async_piece(krs2, (i & 1) ? k_lane1 : k_lane0, blk * C::kTileBytes + (i & ~1) * (C::kThreads * 16),
                  (uint32_t)(size_t)lds_k + at + (i * C::kThreads + wave_base) * 16);
    };
    auto copy_v = [&](int blk, int at, int wave_base, int i) __attribute__((always_inline)) {
      async_piece(vrs2, v_lane, blk * C::kTileBytes + i * (C::kThreads * 16),
                  (uint32_t)(size_t)lds_v + at + (i * C::kThreads + wave_base) * 16);
    };

    // Pair rows: the two lists [it, mid) and [mid, end) are walked together, smallest block first;
    // `act` says whose list names the block (bit 0: q-block 2u, bit 1: q-block 2u + 1).
    constexpr int kNoEntry = 0x7fffffff;
    int mid = 0, ia = 0, ib = 0, act = 0, act_next = 0;
    ListWindow list_a, list_b;
    bool active = true;                               // this wave computes in the current step
    auto pair_advance = [&](int* vout, int* actout) __attribute__((always_inline)) {
      // precondition: ia < mid or ib < end
      const int ca = ia < mid ? list_a.at(ia) : kNoEntry;
      const int cb = ib < end ? list_b.at(ib) : kNoEntry;
      const int vv = ca < cb ? ca : cb;
      const int aa = (ca == vv ? 1 : 0) | (cb == vv ? 2 : 0);
      ia += aa & 1;
      ib += aa >> 1;
      *vout = vv;
      *actout = aa;
    };
    if (kPair) {
      mid = __builtin_amdgcn_readfirstlane(row_ptr[seqs.s[sq].row0 + (size_t)hq * N + 2 * u + 1]);
      mid = mid < it ? it : (mid > end ? end : mid);
      ia = it;
      ib = mid;
      list_a.start(cols, ia, mid, lane);
      list_b.start(cols, ib, end, lane);
      pair_advance(&v, &act);                          // has_work: at least one entry
      active = ((act >> sub) & 1) != 0;
    }

    // Q fragments (B operand of S^T = K Q^T): query row 32*wave + l32, dims 16*ks + 8*hf ..+7
    bf16x8 qf[KS];
    {
      const uint16_t* qp = q + (size_t)hq * hs.q + (size_t)(tok0 + min(qrow, L - 1)) * D + hf * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
    }
    if constexpr (kTwo) {
      const int wave_base = first_slot(t);
#pragma unroll
      for (int i = 0; i < C::kPerThread; ++i) copy_k(v, buf, wave_base, i);
#pragma unroll
      for (int i = 0; i < C::kPerThread; ++i) copy_v(v, buf, wave_base, i);
    } else {
      async_load_k_pieces<BLK, D, kPair>(krs, v * C::kTileBytes, lds_k, t, first_slot(t), 0, C::kPerThread);
    }
    wait_async_loads();
    // At d = 256 a lane holds 128 accumulators, 64 registers of Q and 32 scores beside the operands.  What the maximum moves
    // in nearly every step, the accumulators, has to be in VGPRs (build.py), and the Q fragments, which only the MFMAs read,
    // in AGPRs, from where they are read in place.  A 64 x 256 step of the pair form then is 417 vector instructions instead of
    // 746.  us of attention, accumulators in AGPRs / in VGPRs / and Q pinned here: pair 64 x 256, 16/4 heads, 16384 tokens
    // 665 / 535 / 522, 28/4, 32768 2297 / 1917 / 1889; plain 64 x 256, 16/4, 16330 659 / 533 / 519; 128 x 256, 16384 529 / 450 / 438.
    if (D > 128) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qf[ks]));
    }
    tile_barrier();

    f32x16 oacc[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
    float m_run = -INFINITY;          // running max, in units of log2: s * sm_scale
    float l_run = 0.f;                // this lane's share of the running sum
    int v_next = 0;

    // One step = one listed kv block.  kLast distinguishes the last step of the row: an ordinary
    // step starts the copy of the next K tile after its S^T phase, the last one pulls the queue.
    auto step = [&](auto last_tag) __attribute__((always_inline)) {
      constexpr bool kLast = decltype(last_tag)::value;
      if (kLast && t == 0) pulled_reg = atomicAdd(counter + my_queue * pulls.stride, 1);

      // ---- V(j) -> LDS, requested piece by piece between the MFMAs of S^T, in flight during the softmax ----
      const int wave_base = first_slot(t);
      const bool computes = !kStreamOnly && active;
      if (!computes && !kTwo) async_load_v_pieces<BLK, D, kPair>(vrs, v * C::kTileBytes, lds_v, t, wave_base, 0, C::kPerThread);
      const int other = C::kTileBytes - buf;
      if (!computes && kTwo && !kLast) {
#pragma unroll
        for (int i = 0; i < C::kPerThread; ++i) copy_k(v_next, other, wave_base, i);
#pragma unroll
        for (int i = 0; i < C::kPerThread; ++i) copy_v(v_next, other, wave_base, i);
      }

      f32x16 sacc[KT];
      if (kPair) {
        // whatever the registers hold: without this the compiler writes zeros for the steps a wave sits out, and does
        // so in every step (48 moves; 4 % of a 64 x 64 step)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) asm volatile("" : "=v"(sacc[kt]));
      }
      if (computes) {
      // ---- S^T = K Q^T ----
      // Flat software pipeline over the KT*KS (tile, k-step) pairs: the LDS read of step
      // i + kDepth is issued right after the MFMA of step i, in source order.
      const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      {
        constexpr int kSteps = KT * KS;
        constexpr int kSlab = 32 * D * 2;              // bytes of 32 key rows
        static_assert(kSteps >= kDepth, "pipeline deeper than the phase");
        bf16x8 fr[kDepth];
#pragma unroll
        for (int i = 0; i < kDepth; ++i)
          fr[i] = *reinterpret_cast<const bf16x8*>(lds_k + (i % KT) * kSlab + koff[i / KT]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
          const int kt = i % KT, ks = i / KT;          // consecutive MFMAs: independent accumulators
          sacc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % kDepth], qf[ks], ks == 0 ? zero16 : sacc[kt], 0, 0, 0);
          if (i + kDepth < kSteps) {
            const int j = i + kDepth;
            fr[i % kDepth] = *reinterpret_cast<const bf16x8*>(lds_k + (j % KT) * kSlab + koff[j / KT]);
          }
          constexpr int kEvery = kSteps / C::kPerThread;
          static_assert(kSteps % C::kPerThread == 0, "a piece per kEvery MFMAs");
          if (!kTwo && i % kEvery == 0)
            async_load_v_pieces<BLK, D, kPair>(vrs, v * C::kTileBytes, lds_v, t, wave_base, i / kEvery, i / kEvery + 1);
          if (kTwo && !kLast && i % kEvery == 0) copy_k(v_next, other, wave_base, i / kEvery);
          if (kTwo && !kLast && i % kEvery == kEvery / 2) copy_v(v_next, other, wave_base, i / kEvery);
          __builtin_amdgcn_sched_barrier(0);
        }
      }

      }

      // every wave is done reading K(j): K(j+1) can start now and land during softmax + PV
      if (!kTwo) tile_barrier();
      constexpr int kNow = C::kPerThread - C::kPiecesInMax - C::kPiecesInExp;
      if (!kLast && !kTwo)
        async_load_k_pieces<BLK, D, kPair>(krs, v_next * C::kTileBytes, lds_k, t, wave_base, 0, computes ? kNow : C::kPerThread);

      bf16x8 pf[KT][2];
      if (kPair) {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int s = 0; s < 2; ++s) asm volatile("" : "=v"(pf[kt][s]));
      }
      if (computes) {
      // ---- causal mask inside the diagonal block ----
      if (causal && v == u_own) {
        int last = (wave % C::kRowWaves) * 32 + l32 - 4 * hf;    // key kloc is kc behind 4 * hf
        // kKeepMask leaves the compares to the compiler, which forms them once in front of the row loop and keeps the
        // results in spilled scalar registers; otherwise they are formed here (the dispatch has both sides)
        if (!kKeepMask) asm volatile("" : "+v"(last));
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int kc = kt * 32 + 8 * (r >> 2) + (r & 3);
            if (kc > last) sacc[kt][r] = -INFINITY;
          }
      }

      // ---- keys past the end of the sequence (ragged last block) ----
      if (v == N - 1 && tail < BLK) {
        int left = tail - 4 * hf;
        if (!kKeepMask) asm volatile("" : "+v"(left));
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int kc = kt * 32 + 8 * (r >> 2) + (r & 3);
            if (kc >= left) sacc[kt][r] = -INFINITY;
          }
      }

      // ---- online softmax (per query = per lane pair l, l^32) ----
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        if (!kLast && !kTwo && C::kPiecesInMax > 0) {
          constexpr int kEach = C::kPiecesInMax / KT;
          static_assert(kEach * KT == C::kPiecesInMax, "pieces per 32 keys");
          async_load_k_pieces<BLK, D, kPair>(krs, v_next * C::kTileBytes, lds_k, t, wave_base, kNow + kt * kEach, kNow + (kt + 1) * kEach);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[kt][r]);
      }
      mx = other_half_max(mx);
      const float m_new = fmaxf(m_run, mx * sm_scale);       // finite: every query sees a key
      if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) { // some query's max moved: rescale
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < DT; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
        m_run = m_new;
      }
      // p = 2^(s*scale - m) as bf16 pairs (the PV operand); the row sum adds the fp32 values with
      // plain adds: the dot-product instructions that would add the rounded pairs run on the
      // matrix pipe and stall behind the other workgroup's MFMAs (measured: 2.2x slower there).
      float psum0 = 0.f, psum1 = 0.f;
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          if (!kLast && !kTwo && C::kPiecesInExp > 0) {
            constexpr int kEach = C::kPiecesInExp / (2 * KT), kFirst = kNow + C::kPiecesInMax;
            static_assert(kEach * 2 * KT == C::kPiecesInExp, "pieces per 16 keys");
            async_load_k_pieces<BLK, D, kPair>(krs, v_next * C::kTileBytes, lds_k, t, wave_base,
                                               kFirst + (2 * kt + s) * kEach, kFirst + (2 * kt + s + 1) * kEach);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int j = 0; j < 8; j += 2) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(sacc[kt][8 * s + j], sm_scale, -m_new));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(sacc[kt][8 * s + j + 1], sm_scale, -m_new));
            const f32x2 pp = {p0, p1};
            const bf16x2 pb = __builtin_convertvector(pp, bf16x2);
            pf[kt][s][j] = pb[0];
            pf[kt][s][j + 1] = pb[1];
            psum0 += p0;
            psum1 += p1;
          }
        }
      }
      l_run += psum0 + psum1;

      }

      if (kLast) {
        if (t == 0) next_item = pulled_reg;         // the queue position pulled at the top of the step
        wait_async_loads();                          // this wave's share of V(j) has landed
      } else if (!kTwo) {
        wait_async_loads_but_last_tile<C::kPerThread>();   // ... while the younger loads of K(j+1) may still be in flight
      }
      if (!kTwo || kLast) tile_barrier();            // V(j) complete

      if (kLast) {
        // the next row's queue entry, read through a per-lane (vector) address so that it arrives
        // on the vector-memory counter and is waited for after the PV phase; a scalar load would be
        // waited for by the very next LDS read
        int e_nxt = 0;
        kind_nxt = item_kind(__builtin_amdgcn_readfirstlane(next_item), seg_start, seg_len, &e_nxt);
        if (kind_nxt == kItemRow) item_nxt = items[e_nxt + lane_zero];
      }

      if (computes) {
      // ---- O^T += V^T P^T ----  (same flat pipeline over the DT*KT*2 (d-tile, k-step) pairs)
      {
        constexpr int kPer = KT * 2;                   // k-steps per d-tile
        constexpr int kSteps = DT * kPer;
        static_assert(kSteps >= kDepth, "pipeline deeper than the phase");
        bf16x8 fr[kDepth];
#pragma unroll
        for (int i = 0; i < kDepth; ++i)
          fr[i] = v_frag(i % DT, i / DT);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
          const int dt = i % DT, st = i / DT;          // consecutive MFMAs: independent accumulators
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % kDepth], pf[st >> 1][st & 1], oacc[dt], 0, 0, 0);
          if (i + kDepth < kSteps) {
            const int j = i + kDepth;
            fr[i % kDepth] = v_frag(j % DT, j / DT);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }

      }

      wait_async_loads();              // this wave's share of K(j+1) (or the next row's entry) has landed
      tile_barrier();                  // K(j+1) complete; everyone is done reading V(j)
      if (kTwo) other_buffer();
    };

    // The list is walked one entry ahead of its use: col_idx[it + 1] is requested here and
    // before the MFMA phases of every block, and read only after the waits that end the block,
    // so the latency of the index load is never on the critical path of a block.
    if (kPair) {
      for (;;) {
        if (ia >= mid && ib >= end) break;
        pair_advance(&v_next, &act_next);
        step(std::false_type{});
        v = v_next;
        act = act_next;
        active = ((act >> sub) & 1) != 0;
      }
      step(std::true_type{});
    } else {
    int ahead = it + 1 < end ? cols[it + 1] : -1;
    for (;;) {
      // next valid entry (v_next <= vmax): normally the entry fetched one block ago; entries
      // that must be skipped (negative or beyond vmax) take the slow path
      int nx = it + 1;
      v_next = __builtin_amdgcn_readfirstlane(ahead);
      if (nx < end && !(v_next >= 0 && v_next <= vmax)) {
        ++nx;
        while (nx < end) {
          v_next = __builtin_amdgcn_readfirstlane(cols[nx]);
          if (v_next >= 0 && v_next <= vmax) break;
          ++nx;
        }
      }
      if (nx >= end) break;
      ahead = nx + 1 < end ? cols[nx + 1] : -1;
      step(std::false_type{});
      it = nx;
      v = v_next;
    }
    step(std::true_type{});
    }

    // ---- epilogue: O = O^T / l, bf16, [q][d] ----
    const float l_tot = other_half_sum(l_run);
    const float inv_l = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    uint16_t* op = out + (size_t)hq * hs.q + (size_t)(tok0 + qrow) * D;
    if (qrow < L) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const int d0 = dt * 32 + gq * 8 + hf * 4;
          const f32x2 a = {oacc[dt][gq * 4 + 0] * inv_l, oacc[dt][gq * 4 + 1] * inv_l};
          const f32x2 b = {oacc[dt][gq * 4 + 2] * inv_l, oacc[dt][gq * 4 + 3] * inv_l};
          const bf16x2 ab = __builtin_convertvector(a, bf16x2);
          const bf16x2 bb = __builtin_convertvector(b, bf16x2);
          uint2 w;
          w.x = *reinterpret_cast<const uint32_t*>(&ab);
          w.y = *reinterpret_cast<const uint32_t*>(&bb);
          *reinterpret_cast<uint2*>(op + d0) = w;
        }
    }
    if (lse != nullptr && hf == 0 && qrow < L)
      lse[(size_t)hq * hs.lse + tok0 + qrow] =
          l_tot > 0.f ? (m_run + log2f(l_tot)) * 0.6931471805599453f : -INFINITY;

    // ---- the row pulled in the last step becomes the current one ----
    kind_cur = kind_nxt;
    cur_x = __builtin_amdgcn_readfirstlane(item_nxt.x);
    cur_y = __builtin_amdgcn_readfirstlane(item_nxt.y);
    cur_z = __builtin_amdgcn_readfirstlane(item_nxt.z);
    cur_w = __builtin_amdgcn_readfirstlane(item_nxt.w);
  }
#endif
}

// =====================================================================================
// The same computation with kQ = 64 queries per wave (B = 128, d = 128, whole blocks, clean lists): workgroup =
// 2 waves = one (q-head, q-block) row, one wave per SIMD, two workgroups per CU; or with kQ = 32: 4 waves of
// 256 registers a lane, still two workgroups per CU, which take a listed block in 1.3 instead of 2.2 us when a row is
// alone on its CU (the dispatch says which calls want that).  With kQ = 64 every K / V^T
// fragment read from LDS feeds two MFMAs, K and V^T travel as 64-key half tiles through two LDS
// buffers each, and the row loop (software-pipelined over half-steps, softmax in the shadow of the
// neighbouring half-steps' MFMAs, accumulators and Q fragments in AGPRs) is a generated,
// hand-scheduled instruction sequence: prism_attn_w64_body.inc (and _w32_), written by gen_attn_w64.py, which
// also documents the register map and the pipeline.  This function supplies the persistent-workgroup
// loop around it: the same per-XCD queues as the general kernel.
// =====================================================================================
template <int kQ>
__global__ __launch_bounds__(128 / kQ * 64, kQ == 64 ? 1 : 2) void sparse_attn_w64_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ vt,
    const int32_t* __restrict__ col_idx, const int4* __restrict__ items, int32_t* __restrict__ plan,
    PullCounters pulls, DirtyFlags flags, uint16_t* __restrict__ out, float* __restrict__ lse, int h, int h_kv,
    SeqTable seqs, HeadStrides hs, int causal) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(1024))) char lds_tiles[65536];
  __shared__ int s_pulled, s_queue;
  const int dirty = dirty_sequences<128 / kQ * 64>(flags);  // the general kernel takes these
  if (dirty == (1 << seqs.n) - 1) return;

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int g = h / h_kv;
  const int n_queues = gridDim.x < kXcds ? 1 : kXcds;
  int my_queue = blockIdx.x % n_queues;
  int seg_start = plan[kPlanStart + my_queue];
  int seg_len = plan[kPlanLen + my_queue];
  const unsigned alone = plan[kPlanAlone + my_queue];
  asm volatile("" ::"s"(seg_start), "s"(seg_len), "s"(alone));   // three requests, one wait (8/2 heads, 4096 tokens 37.2 -> 36.4 us)
  int32_t* __restrict__ counter = pulls.at;
  const uint32_t lds_base = (uint32_t)(size_t)lds_tiles;
  int pulled = 0;
  const int first = first_row(alone, n_queues, true);
  if (first < 0) {
    // the row on this CU may be one of those that the general kernel takes
    const int mate = (int)(blockIdx.x - gridDim.x / 2) / kXcds;
    if (seqs.n == 1 || ((dirty >> (items[seg_start + mate].x >> kSeqShift)) & 1) == 0) return;
  }
  if (t == 0) pulled = first < 0 ? atomicAdd(counter + my_queue * pulls.stride, 1) : first;
  for (;;) {
    // hand the pulled queue position to both waves
    __syncthreads();
    if (t == 0) s_pulled = pulled;
    __syncthreads();
    int pos = __builtin_amdgcn_readfirstlane(s_pulled);
    if (pos >= seg_len) {
      // Own queue exhausted: go on with rows of the nearest queue that still has some.  A pull
      // counter only grows, so a queue seen exhausted stays so; the atomic decides who gets a row.
      __syncthreads();
      if (wave == 0) {
        int ln = lane;
        asm volatile("" : "+v"(ln));                        // addresses formed here, not kept across the row loop
        if (ln == 0) plan[kPlanCounter + my_queue] = seg_len + 1;
        int found_pos = -1, found_queue = -1;
        for (;;) {
          int taken = 0x7fffffff, len = 0;
          if (ln < n_queues) {
            taken = __hip_atomic_load(counter + ln * pulls.stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            len = plan[kPlanLen + ln];
          }
          const unsigned long long open = __ballot(taken < len);
          if (open == 0ull) break;
          int pick = -1;
          for (int s = 1; s <= n_queues && pick < 0; ++s) {
            const int x = (my_queue + s) % n_queues;
            if ((open >> x) & 1ull) pick = x;
          }
          int got = 0;
          if (ln == 0) got = atomicAdd(counter + pick * pulls.stride, 1);
          got = __builtin_amdgcn_readfirstlane(got);
          if (got < plan[kPlanLen + pick]) {
            found_pos = got;
            found_queue = pick;
            break;
          }
        }
        if (lane == 0) {
          s_pulled = found_pos;
          s_queue = found_queue;
        }
      }
      __syncthreads();
      pos = __builtin_amdgcn_readfirstlane(s_pulled);
      const int nq = __builtin_amdgcn_readfirstlane(s_queue);
      if (nq < 0) break;                                    // every queue is exhausted
      my_queue = nq;
      seg_start = plan[kPlanStart + my_queue];
      seg_len = plan[kPlanLen + my_queue];
    }
    const int4 it0 = items[seg_start + pos];
    const int head_word = __builtin_amdgcn_readfirstlane(it0.x);
    const int sq = seqs.n > 1 ? head_word >> kSeqShift : 0;
    const int hq = seqs.n > 1 ? head_word & ((1 << kSeqShift) - 1) : head_word;
    const int L = seqs.s[sq].L, N = seqs.s[sq].N;
    const uint32_t k_bytes = (uint32_t)L * kHeadDim * 2;
    const uint32_t vt_bytes = (uint32_t)N * 128u * kHeadDim * 2;
    const int u = __builtin_amdgcn_readfirstlane(it0.y) & 0xffff;
    const int c_first = (__builtin_amdgcn_readfirstlane(it0.y) >> 16) & 0xffff;   // first listed block
    const int it = __builtin_amdgcn_readfirstlane(it0.z);
    const int end = __builtin_amdgcn_readfirstlane(it0.w);
    // The next row's queue position is pulled when this row is almost done (inside the row loop, at
    // the start of its last PV phase) and looked at after it: pulling at the start of a row would
    // reserve a row that its neighbours in the queue have long passed by the time it is started.

    const int q0 = u * 128 + wave * kQ;                                          // this wave's first query
    const size_t tok0 = (size_t)seqs.s[sq].tok0 + q0;                            // its token in the tensors
    const size_t row0 = (size_t)hq * hs.q + tok0 * kHeadDim;                     // its element offset in Q / O
    const bool mine = ((dirty >> sq) & 1) == 0;
    if (it >= end || !mine) {
      // a row without entries (o = 0, lse = -inf), or the general kernel's
      const int r = lane;                                   // one row per lane
      if (mine && r < kQ) {
        uint16_t* op = out + row0 + (size_t)r * kHeadDim;
#pragma unroll
        for (int c = 0; c < 16; ++c) *reinterpret_cast<uint4*>(op + c * 8) = make_uint4(0u, 0u, 0u, 0u);
        if (lse != nullptr) lse[(size_t)hq * hs.lse + tok0 + r] = -INFINITY;
      }
      if (t == 0) pulled = atomicAdd(counter + my_queue * pulls.stride, 1);
      continue;
    }
    const uint16_t* q_row = q + row0;
    uint16_t* o_row = out + row0;
    float* lse_row = lse != nullptr ? lse + (size_t)hq * hs.lse + tok0 : nullptr;
    const int kvh = hq / g;
    const uint16_t* k_head = k + (size_t)kvh * hs.kv + (size_t)seqs.s[sq].tok0 * kHeadDim;
    const uint16_t* vt_head = vt + ((size_t)seqs.s[sq].blk0 * h_kv + (size_t)kvh * N) * 128 * kHeadDim;
    const int32_t* col_row = col_idx + seqs.s[sq].col0 + it;
    const int n_entries = end - it;
    int32_t* pull_counter = counter + __builtin_amdgcn_readfirstlane(my_queue * pulls.stride);
    int pulled_next;
    if constexpr (kQ == 64) {
#include "prism_attn_w64_body.inc"
    } else {
#include "prism_attn_w32_body.inc"
    }
    if (t == 0) pulled = pulled_next;
  }
#endif
}

// One wave per row: does the row's list hold an entry the attention kernels must skip?
// With need_sorted (the pair kernel merges two lists) a list that is not strictly ascending counts too.
__global__ __launch_bounds__(256) void queue_validate_kernel(const int32_t* __restrict__ row_ptr,
                                                             const int32_t* __restrict__ col_idx, int h,
                                                             int N, int cap, int causal, int need_sorted,
                                                             const int32_t* __restrict__ range_flags,
                                                             int n_range_flags, int32_t* __restrict__ plan) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  // values of V beyond the fp16 range (flagged per block by vt_image_kernel) also need the general kernel
  const int fi = blockIdx.x * 256 + threadIdx.x;
  if (fi < n_range_flags && range_flags[fi] != 0) atomicOr(plan + kPlanFlags, kFlagDirtyLists);
  if (r >= h * N) return;
  int b = row_ptr[r], e = row_ptr[r + 1];
  const bool clamped = b < 0 || b > cap || e < b || e > cap;
  b = b < 0 ? 0 : (b > cap ? cap : b);
  e = e < b ? b : (e > cap ? cap : e);
  const int vmax = causal ? r % N : N - 1;
  bool bad = clamped;
  for (int i = b + lane; i < e; i += 64) {
    const int v = col_idx[i];
    bad |= v < 0 || v > vmax;
    if (need_sorted && i + 1 < e) bad |= col_idx[i + 1] <= v;
  }
  if (__ballot(bad) != 0ull && lane == 0) atomicOr(plan + kPlanFlags, kFlagDirtyLists);
}

// =====================================================================================
// Work queues.  The rows (q-head, q-block) are put in the order
//     (phase, length class, q-head, q-block descending)
// and every (phase, class) group of that order is cut into one contiguous part per queue, the
// parts of a group holding equal work (listed blocks + one per row).  A queue is the sequence of
// its parts.  So each XCD walks neighbouring q-blocks of one q-head at a time, all XCDs go
// through the long rows of a phase first and its short rows last (no long row is started at the
// end of the call), and the queues hold equal work.
//   phase = kv head / heads_per_phase: the kv heads are taken a few at a time so that the K and
//       V of the heads in flight fit the 256 MB memory-side cache (at 128K tokens a kv head is
//       67 MB of K + V and all eight do not fit).
//   class: list length in (512, ..], (256, 512], (128, 256], ... (1, 2], [0, 1].
//   queue_count_kernel  (one workgroup per q-head): rows and work of the head per class.
//   queue_rank_kernel   (one workgroup per q-head): every row's rank in its group and its part,
//       and the number of rows of every (group, part).
//   queue_fill_kernel   (one thread per row): the row's position in its queue and its entry.
// =====================================================================================
// N = rows per head: q-blocks, or pairs of q-blocks (stride = 2: row r of the plan covers the two
// consecutive lists of q-blocks 2r and 2r + 1 of the index lists).
struct PlanCfg {
  int h, g, N, heads_per_phase, n_phases, n_queues, cap, causal, stride;
};
// Two sets of kXcds pull counters, `stride` ints apart, in row_part (stride 0: not in this launch), and the queues and
// workgroups of the kernels that pull from them.
struct CounterInit {
  int stride;
  int n_queues[2], grid[2];
};
constexpr int kCounterStride = 32;        // ints: a 128-byte line
constexpr int kClasses = 11;
constexpr int kMaxGroups = 512;           // (phase, class) groups held in LDS by queue_fill_kernel

// class 0: more than 512 listed blocks, class c = 1 .. 9: (2^(9-c), 2^(10-c)], class 10: 0 or 1
__device__ __forceinline__ int length_class(int len) {
  if (len <= 1) return kClasses - 1;
  const int k = 31 - __builtin_clz(len - 1);           // len in (2^k, 2^(k+1)]
  return k > 9 ? 0 : 9 - k;
}

// list bounds of row r clamped to [0, cap] (and end >= begin)
__device__ __forceinline__ void row_bounds(const int32_t* __restrict__ row_ptr, int r, int cap, int stride,
                                           int* beg, int* end) {
  int b = row_ptr[(size_t)r * stride], e = row_ptr[(size_t)r * stride + stride];
  b = b < 0 ? 0 : (b > cap ? cap : b);
  e = e < b ? b : (e > cap ? cap : e);
  *beg = b;
  *end = e;
}

// bins = { rows[h][kClasses], work[h][kClasses] }; parts[n_phases][kClasses][8] is cleared here.
__global__ __launch_bounds__(256) void queue_count_kernel(const int32_t* __restrict__ row_ptr, PlanCfg c,
                                                          int32_t* __restrict__ bins,
                                                          int32_t* __restrict__ parts,
                                                          int32_t* __restrict__ plan) {
  __shared__ int s_rows[kClasses], s_work[kClasses];
  const int t = threadIdx.x, hq = blockIdx.x;
  if (t < kClasses) {
    s_rows[t] = 0;
    s_work[t] = 0;
  }
  for (int i = hq * 256 + t; i < c.n_phases * kClasses * 8; i += c.h * 256) parts[i] = 0;
  if (hq == 0 && t < kPlanInts - kPlanFlags) plan[kPlanFlags + t] = 0;
  __syncthreads();
  for (int u = t; u < c.N; u += 256) {
    int beg, end;
    row_bounds(row_ptr, hq * c.N + u, c.cap, c.stride, &beg, &end);
    const int cls = length_class(end - beg);
    atomicAdd(&s_rows[cls], 1);
    atomicAdd(&s_work[cls], end - beg + 1);
  }
  __syncthreads();
  if (t < kClasses) {
    bins[hq * kClasses + t] = s_rows[t];
    bins[(c.h + hq) * kClasses + t] = s_work[t];
  }
}

// row_rank[r] = rank of row r inside its (phase, class) group; row_part[r] = group * 8 + part.
__global__ __launch_bounds__(256) void queue_rank_kernel(const int32_t* __restrict__ row_ptr, PlanCfg c,
                                                         const int32_t* __restrict__ bins,
                                                         int32_t* __restrict__ parts,
                                                         int32_t* __restrict__ row_rank,
                                                         int32_t* __restrict__ row_part) {
  __shared__ int s_rows_before[kClasses];            // rows of the group in earlier heads
  __shared__ long long s_work_before[kClasses], s_work_total[kClasses];
  __shared__ int s_parts[kClasses * 8];
  __shared__ long long s_wave_total[kClasses][4];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, hq = blockIdx.x;
  const int phase = (hq / c.g) / c.heads_per_phase;
  if (t < kClasses) {
    s_rows_before[t] = 0;
    s_work_before[t] = 0;
    s_work_total[t] = 0;
  }
  __syncthreads();
  {
    const int h0 = phase * c.heads_per_phase * c.g;
    const int h1 = min(c.h, h0 + c.heads_per_phase * c.g);
    for (int i = t; i < (h1 - h0) * kClasses; i += 256) {
      const int hh = h0 + i / kClasses, k = i % kClasses;
      const int w = bins[(c.h + hh) * kClasses + k];
      if (hh < hq) {
        atomicAdd(&s_rows_before[k], bins[hh * kClasses + k]);
        atomicAdd(reinterpret_cast<unsigned long long*>(&s_work_before[k]), (unsigned long long)w);
      }
      atomicAdd(reinterpret_cast<unsigned long long*>(&s_work_total[k]), (unsigned long long)w);
    }
  }
  for (int i = t; i < kClasses * 8; i += 256) s_parts[i] = 0;

  // Thread t owns the rows i = t*per .. t*per + per - 1 of the head's order (q-block N-1-i).
  // Per class, rows and work of a thread travel through the scan as one number: work * 2^16 + rows
  // (a head has at most 2048 rows).
  const int per = (c.N + 255) / 256;
  long long mine[kClasses];
#pragma unroll
  for (int k = 0; k < kClasses; ++k) mine[k] = 0;
  for (int j = 0; j < per; ++j) {
    const int i = t * per + j;
    if (i >= c.N) break;
    int beg, end;
    row_bounds(row_ptr, hq * c.N + (c.N - 1 - i), c.cap, c.stride, &beg, &end);
    const int cls = length_class(end - beg);
    const long long add = ((long long)(end - beg + 1) << 16) + 1;
#pragma unroll
    for (int k = 0; k < kClasses; ++k) mine[k] += k == cls ? add : 0;
  }
  long long before[kClasses];                        // exclusive prefix over the threads
#pragma unroll
  for (int k = 0; k < kClasses; ++k) {
    long long incl = mine[k];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const long long y = __shfl_up(incl, off, 64);
      if (lane >= off) incl += y;
    }
    if (lane == 63) s_wave_total[k][wave] = incl;
    before[k] = incl - mine[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kClasses; ++k)
    for (int w = 0; w < wave; ++w) before[k] += s_wave_total[k][w];

  for (int j = 0; j < per; ++j) {
    const int i = t * per + j;
    if (i >= c.N) break;
    const int r = hq * c.N + (c.N - 1 - i);
    int beg, end;
    row_bounds(row_ptr, r, c.cap, c.stride, &beg, &end);
    const int cls = length_class(end - beg);
    const long long add = ((long long)(end - beg + 1) << 16) + 1;
    long long upto = 0;                              // this row included
#pragma unroll
    for (int k = 0; k < kClasses; ++k)
      if (k == cls) {
        before[k] += add;
        upto = before[k];
      }
    const int rank = (int)(upto & 0xffff) - 1;
    const long long w_incl = (upto >> 16) + s_work_before[cls];
    int x = 0;
    if (c.n_queues > 1) {
      x = (int)(((w_incl - 1) * c.n_queues) / s_work_total[cls]);
      x = x < 0 ? 0 : (x > c.n_queues - 1 ? c.n_queues - 1 : x);
    }
    row_rank[r] = s_rows_before[cls] + rank;
    row_part[r] = (phase * kClasses + cls) * 8 + x;
    atomicAdd(&s_parts[cls * 8 + x], 1);
  }
  __syncthreads();
  for (int i = t; i < kClasses * 8; i += 256)
    if (s_parts[i] > 0) atomicAdd(&parts[phase * kClasses * 8 + i], s_parts[i]);
}

// The thread of a row writes the row's queue entry: list bounds clamped to [0, cap], and the
// first entry that names a valid key block (0 <= v <= u for causal attention, 0 <= v < N
// otherwise).  Queue x holds, group after group, the rows of its part of the group; workgroup 0
// also writes the plan (segment starts and lengths, no queue exhausted).  The call's last launch
// of it turns the first entries of row_part into the pull counters of the two attention kernels: the
// thread that has read an entry, the last to do so, writes the counter that takes its place.
__global__ __launch_bounds__(256) void queue_fill_kernel(const int32_t* __restrict__ row_ptr,
                                                         const int32_t* __restrict__ col_idx, PlanCfg c,
                                                         const int32_t* __restrict__ parts,
                                                         const int32_t* __restrict__ row_rank,
                                                         int32_t* __restrict__ row_part,
                                                         int32_t* __restrict__ plan,
                                                         int4* __restrict__ items, CounterInit ci) {
  __shared__ int s_parts[kMaxGroups * 8];            // rows of (group, part)
  __shared__ int s_before[kMaxGroups * 8];           // rows of the same part in earlier groups
  __shared__ int s_start[8];
  const int t = threadIdx.x;
  const int n_groups = c.n_phases * kClasses;
  for (int i = t; i < n_groups * 8; i += 256) s_parts[i] = parts[i];
  __syncthreads();
  if (t < 8) {
    int run = 0;
    for (int gq = 0; gq < n_groups; ++gq) {
      s_before[gq * 8 + t] = run;
      run += s_parts[gq * 8 + t];
    }
    s_start[t] = run;                                // length of queue t, turned into its start below
  }
  __syncthreads();
  if (t == 0) {
    int start = 0;
    for (int x = 0; x < 8; ++x) {
      const int len = s_start[x];
      s_start[x] = start;
      if (blockIdx.x == 0) {
        plan[kPlanStart + x] = start;
        plan[kPlanLen + x] = len;
        plan[kPlanCounter + x] = 0;
      }
      start += len;
    }
  }
  __syncthreads();

  const int r = blockIdx.x * 256 + t;
  if (r >= c.h * c.N) return;
  const int hq = r / c.N, u = r - hq * c.N;
  const int gp = row_part[r], x = gp & 7;
  if (ci.stride > 0 && r % ci.stride == 0 && r < 2 * kXcds * ci.stride) {
    const int k = r / ci.stride, set = k / kXcds;
    row_part[r] = dealt_rows(k % kXcds, ci.n_queues[set], ci.grid[set]);
  }
  int in_earlier_parts = 0;
  for (int y = 0; y < x; ++y) in_earlier_parts += s_parts[(gp & ~7) + y];
  const int entry = s_start[x] + s_before[gp] + row_rank[r] - in_earlier_parts;
  int beg, end;
  row_bounds(row_ptr, r, c.cap, c.stride, &beg, &end);
  const int vmax = c.causal ? u : c.N - 1;
  int it = beg, v = 0;
  if (c.stride == 1) {
    while (it < end) {
      v = col_idx[it];
      if (v >= 0 && v <= vmax) break;
      ++it;
    }
    if (it >= end) v = 0;
  }                                                  // pair rows: clean lists, the kernel finds its first block
  if (entry >= 0 && entry < c.h * c.N) items[entry] = make_int4(hq, u | (v << 16), it, end);
}

// =====================================================================================
// Everything in front of the attention kernels in one launch, for calls of up to kPrepMaxRows rows whose kv heads
// form one phase: workgroup 0 (and 1, where the pair kernel may take the call) builds a queue plan, the next
// `n_check` workgroups look the lists over, the rest write the V image: the fp16 image and the copy, or the copy alone where the
// 64-queries-per-wave kernel cannot take the call.  The parts do not depend on each other;
// the attention kernels read what the list check and the image found through DirtyFlags.
// Such calls are bound by launches: a kernel with next to no work takes 4.5 us, and as four to nine kernels the same
// work took 34 of 266 us per layer at 8K tokens and 14 of 47 us at 2K tokens and one head (the attention dispatch has
// the figures of both sides).
// =====================================================================================
constexpr int kPrepThreads = 1024;
constexpr int kPrepMaxRows = 8 * kPrepThreads;
constexpr int kCheckRows = 64;             // rows per list-check workgroup
struct PrepArgs {
  const int32_t *row_ptr, *col_idx;
  const uint16_t* v;                       // read for the image of the launch, if it writes one
  uint16_t *vt16, *copy;                   // null: not written
  int32_t *range_flags, *check;
  int4 *items, *pair_items;
  int32_t *plan, *pair_plan;
  int32_t *counters, *pair_counters;       // without a second plan: counters of the first one for a second kernel
  int32_t counter_stride;
  int32_t grid, pair_grid;                 // workgroups of the attention kernels
  float alone;                             // a row this many times the work of an average workgroup has a CU to itself (0: none)
  float halve;                             // every row has, where the longest is a CU's average work over this or more (0: no)
  int32_t h, h_kv, n_queues, pair_queues, n_check;
  int32_t block, head_dim;
  uint8_t n_plans, causal, need_sorted;
  size_t kv_head_stride;
};

// One workgroup writes the plan of all rows: the order, parts and entries of queue_count / rank / fill_kernel for one
// phase.  Wave w owns the rows 64*CH*w .. of the order (q-head, sequence, q-block descending), 64 at a time; rank and
// work of a row inside its length class come from ballots and prefix sums over the wave, then over the 16 waves.
struct PlanLds {
  int rows[16][kClasses], work[16][kClasses];       // per wave: totals, then what lies in front of the wave
  float scale[kClasses];                            // parts per unit of work
  int start[kClasses][9];                           // first rank of the class that belongs to part x
  int before[kClasses][8], qlen[8], qstart[8];
  int total;                                        // entries + 3 per row (a row costs about three blocks beside its own)
  int above[8];                                     // rows of queue x with that much work
  unsigned alone[8];
  int longest;
};
__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)x), hi = __builtin_amdgcn_readfirstlane((int)(x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
// stride = 2: rows are pairs of q-blocks (every sequence has an even number of them).
template <int CH, bool kOne>
__device__ __forceinline__ void plan_rows(PlanLds& m, const PrepArgs& a, const SeqTable& seqs, int stride,
                                          int n_queues, int grid, int32_t* __restrict__ counters,
                                          int32_t* __restrict__ more_counters, int4* __restrict__ items, int32_t* __restrict__ plan) {
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int per_head = seqs.nsum >> (stride - 1);
  const int R = a.h * per_head;
  // What the rows need to know of their sequence: a call of one sequence (kOne) holds it in scalar registers.  Looked up in
  // LDS for every row and use it was 40 % of the instructions, which bind this workgroup: 32.0 -> 29.0 us at 5024 rows,
  // 16.1 -> 14.4 at 3104 (d = 64), 20.4 -> 19.0 at 4096, 41.1 -> 40.4 at 8192.
  const int n0 = __builtin_amdgcn_readfirstlane(seqs.s[0].N), cap0 = __builtin_amdgcn_readfirstlane(seqs.s[0].cap);
  const int64_t row_at0 = uniform64(seqs.s[0].row0), col_at0 = uniform64(seqs.s[0].col0);
  auto n_of = [&](int s) { return kOne ? n0 : seqs.s[s].N; };
  auto cap_of = [&](int s) { return kOne ? cap0 : seqs.s[s].cap; };
  auto row0_of = [&](int s) { return kOne ? row_at0 : (int64_t)seqs.s[s].row0; };
  auto col0_of = [&](int s) { return kOne ? col_at0 : (int64_t)seqs.s[s].col0; };
  // Row i of the order: its sequence, q-head and number inside the head.
  struct Row {
    int s, hq, u;
  };
  // (a fp32 product instead of an integer division: i < 2^13, so (i + 1/2) / per_head is at least 2^-14 of itself
  // away from a whole number and the rounding errors of the product, below 2^-22, cannot cross one)
  const float per_head_inv = 1.0f / (float)per_head;
  auto row = [&](int i) {
    Row r;
    r.hq = (int)(((float)i + 0.5f) * per_head_inv);
    const int rem = i - r.hq * per_head;
    r.s = kOne ? 0 : seq_of(seqs, rem * stride, 1);
    r.u = (n_of(r.s) >> (stride - 1)) - 1 - (kOne ? rem : rem - (seqs.s[r.s].blk0 >> (stride - 1)));
    return r;
  };
  auto index = [&](int c) { return (wave * CH + c) * 64 + lane; };
  // The bounds of all rows are requested at once, and at the end the first entries of all lists: two memory round trips
  // for the workgroup.  What remains is a few hundred instructions per 64 rows of a wave on one CU, 9.5 us at 2048 rows
  // (an integer division per row and part and a prefix sum over every class, there or not, took 11.1 us).
  int beg[CH], len[CH];                               // len = -1 past the last row
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int i = index(c);
    beg[c] = 0;
    len[c] = -1;
    if (i < R) {
      const Row r = row(i);
      const int32_t* rp = a.row_ptr + row0_of(r.s) + ((size_t)r.hq * (n_of(r.s) >> (stride - 1)) + r.u) * stride;
      beg[c] = rp[0];
      len[c] = rp[stride];
    }
  }
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int i = index(c);
    if (i < R) {
      const int cap = cap_of(kOne ? 0 : row(i).s);
      const int b = beg[c] < 0 ? 0 : (beg[c] > cap ? cap : beg[c]), e = len[c];
      beg[c] = b;
      len[c] = (e < b ? b : (e > cap ? cap : e)) - b;
    }
  }
  int rank[CH], cum[CH];
  // Lane k counts the rows and the work of class k that the wave has met.  64 neighbouring rows fall into two or three
  // classes: one round per class that is there.
  int crow = 0, cwork = 0;
  // work of a row: its entries + 1; a list with repeated entries weighs no more than 2 * kMaxBlocks
  auto weight = [&](int c) { return min(len[c], 2 * kMaxBlocks) + 1; };
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int cls = len[c] < 0 ? -1 : length_class(len[c]);
    rank[c] = cum[c] = 0;
    unsigned long long todo = __ballot(cls >= 0);
    while (todo != 0ull) {                              // uniform
      const int k = __builtin_amdgcn_readlane(cls, __builtin_ctzll(todo));
      const unsigned long long mine = __ballot(cls == k);
      const int incl = wave_scan_inclusive(cls == k ? weight(c) : 0);
      const int r0 = __builtin_amdgcn_readlane(crow, k), w0 = __builtin_amdgcn_readlane(cwork, k);
      if (cls == k) {
        rank[c] = r0 + __popcll(mine & ((1ull << lane) - 1ull));
        cum[c] = w0 + incl;
      }
      const int r1 = r0 + __popcll(mine), w1 = w0 + __builtin_amdgcn_readlane(incl, 63);
      crow = lane == k ? r1 : crow;
      cwork = lane == k ? w1 : cwork;
      todo &= ~mine;
    }
  }
  if (lane < kClasses) {
    m.rows[wave][lane] = crow;
    m.work[wave][lane] = cwork;
  }
  if (t < 8) m.alone[t] = m.above[t] = 0;
  if (t == 8) m.total = m.longest = 0;
  __syncthreads();
  if (t < 16 * kClasses) {                            // 16 lanes a class, one for each wave
    const int k = t >> 4, w = t & 15;
    const int nr = m.rows[w][k], nw = m.work[w][k];
    const int r = row16_scan_inclusive(nr), work = row16_scan_inclusive(nw);
    m.rows[w][k] = r - nr;
    m.work[w][k] = work - nw;
    if (w == 15) {
      atomicAdd(&m.total, work + 2 * r);
      m.scale[k] = work > 0 ? (float)n_queues / (float)work : 0.f;
      for (int x = 0; x < 9; ++x) m.start[k][x] = r;
    }
  }
  if (a.halve > 0.f) {
    int longest = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) longest = max(longest, len[c]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) longest = max(longest, __shfl_xor(longest, off, 64));
    if (lane == 0) atomicMax(&m.longest, longest);
  }
  __syncthreads();
  // part of the row that ends at work `w` of its class: grows with w, 0 .. n_queues - 1
  auto part = [&](int w, int k) { return min((int)((float)(w - 1) * m.scale[k]), n_queues - 1); };
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    if (len[c] >= 0) {
      const int k = length_class(len[c]);
      rank[c] += m.rows[wave][k];
      cum[c] += m.work[wave][k];
      const int x1 = part(cum[c], k);
      const int prev = rank[c] == 0 ? -1 : part(cum[c] - weight(c), k);
      for (int x = prev + 1; x <= x1; ++x) m.start[k][x] = rank[c];
    }
  }
  __syncthreads();
  if (t < 16 * 8) {                                   // 16 lanes a queue, one for each class
    const int x = t >> 4, k = t & 15;
    const int n = k < kClasses ? m.start[k][x + 1] - m.start[k][x] : 0;
    const int upto = row16_scan_inclusive(n);
    if (k < kClasses) m.before[k][x] = upto - n;
    if (k == 15) m.qlen[x] = upto;
  }
  __syncthreads();
  // lane x < 8: where queue x starts
  const int qlen = lane < 8 ? m.qlen[lane] : 0;
  const int qstart = row16_scan_inclusive(qlen) - qlen;
  if (lane < 8) m.qstart[lane] = qstart;              // every wave the same
  const bool marks = stride == 1 && (a.alone > 0.f || a.halve > 0.f);     // some row may have a CU to itself
  auto count = [&](unsigned alone) __attribute__((always_inline)) {
    plan[kPlanAlone + t] = (int)alone;
    // the first pulls of queue t belong to the workgroups t, t + n_queues, ... that first_row leaves
    const int all = dealt_rows(t, n_queues, grid), dealt = all - __popc(alone);
    counters[t * a.counter_stride] = dealt;
    if (more_counters != nullptr) more_counters[t * a.counter_stride] = kOne ? dealt : all;
  };
  if (t < 8) {
    plan[kPlanStart + t] = qstart;
    plan[kPlanLen + t] = qlen;
    plan[kPlanCounter + t] = 0;
    plan[kPlanFlags + t] = 0;
    if (!marks) count(0);
  }
  const float alone_from = stride == 1 && a.alone > 0.f ? a.alone * (float)m.total / (float)grid : INFINITY;
  const int half = grid / 2 / n_queues;
  // rank becomes the row's entry, cum its list's first element
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    if (len[c] < 0) continue;
    const int k = length_class(len[c]), x = part(cum[c], k);
    const int entry = m.before[k][x] + rank[c] - m.start[k][x];
    if ((float)len[c] > alone_from) {
      atomicAdd(&m.above[x], 1);
      if (entry < half) atomicOr(&m.alone[x], 1u << entry);
    }
    rank[c] = m.qstart[x] + entry;
    cum[c] = 0;
    if (stride == 1 && len[c] > 0)
      cum[c] = a.col_idx[col0_of(kOne ? 0 : row(index(c)).s) + beg[c]];
  }
  if (marks) {
    // (in front of the entries, whose stores the workgroup would wait for at a barrier behind them: 42.8 -> 39.8 us in a
    // packed batch of 4640 rows)
    __syncthreads();
    if (t < 8) {
      const bool halve = (float)m.total < a.halve * (float)m.longest * (float)(grid / 2);
      count(halve ? ~0u >> (32 - half) : m.above[t] <= half * 5 / 8 ? m.alone[t] : 0);
    }
  }
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    if (len[c] < 0) continue;
    const Row r = row(index(c));
    const int end = beg[c] + len[c];
    int it = beg[c], v = cum[c];
    if (stride == 1) {
      const int vmax = a.causal ? r.u : n_of(r.s) - 1;
      if (len[c] == 0 || v < 0 || v > vmax) {          // rare: look for the first entry that names a valid block
        const int32_t* cols = a.col_idx + col0_of(r.s);
        for (v = 0; it < end; ++it) {
          const int w = cols[it];
          if (w >= 0 && w <= vmax) {
            v = w;
            break;
          }
        }
      }
    }                                                  // pair rows: clean lists, the kernel finds its first block
    items[rank[c]] = make_int4(kOne ? r.hq : r.hq | (r.s << kSeqShift), r.u | (v << 16), it, end);
  }
}

// Which sequences have, among the 64 rows of this workgroup, a list with an entry to skip (queue_validate_kernel's
// question)?
__device__ __forceinline__ void check_rows(const PrepArgs& a, const SeqTable& seqs, int wg, int& s_bad) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int R = a.h * seqs.nsum;
  int bad_seqs = 0;
  for (int j = 0; j < kCheckRows / 16; ++j) {
    const int r = wg * kCheckRows + j * 16 + wave;
    if (r >= R) break;
    const int s = seq_of(seqs, r, a.h);
    const int rr = r - a.h * seqs.s[s].blk0, N = seqs.s[s].N, cap = seqs.s[s].cap;
    int b = a.row_ptr[seqs.s[s].row0 + rr], e = a.row_ptr[seqs.s[s].row0 + rr + 1];
    bool bad = b < 0 || b > cap || e < b || e > cap;
    b = b < 0 ? 0 : (b > cap ? cap : b);
    e = e < b ? b : (e > cap ? cap : e);
    const int vmax = a.causal ? rr % N : N - 1;
    const int32_t* cols = a.col_idx + seqs.s[s].col0;
    for (int i = b + lane; i < e; i += 64) {
      const int v = cols[i];
      bad |= v < 0 || v > vmax;
      if (a.need_sorted && i + 1 < e) bad |= cols[i + 1] <= v;
    }
    if (bad) bad_seqs |= 1 << s;
  }
  if (threadIdx.x == 0) s_bad = 0;
  __syncthreads();
  if (bad_seqs != 0) atomicOr(&s_bad, bad_seqs);
  __syncthreads();
  if (threadIdx.x == 0) a.check[wg] = s_bad;
}

union PrepLds {
  PlanLds plan;
  ImageTile tile;
};
// Where block `blk` of a sequence lies in a kv head of the copy.
__device__ __forceinline__ uint16_t* copy_block(const PrepArgs& a, const SeqTable& seqs, int kvh, int s, int blk) {
  return a.copy + ((size_t)kvh * seqs.nsum + seqs.s[s].blk0 + blk) * ((size_t)a.block * a.head_dim);
}
// The part of the V image that belongs to workgroup `wg` of the launch's image workgroups: with the fp16 image ...
__device__ __forceinline__ void prep_image(PrepLds& lds, int& s_over, const PrepArgs& a, const SeqTable& seqs, int wg) {
  const int s = seq_of(seqs, wg, a.h_kv);
  const int rr = wg - a.h_kv * seqs.s[s].blk0, N = seqs.s[s].N;
  const int kvh = rr / N, blk = rr - kvh * N;
  vt_image_tile<kPrepThreads>(lds.tile, s_over,
                              a.v + (size_t)kvh * a.kv_head_stride + ((size_t)seqs.s[s].tok0 + (size_t)blk * kImageRows) * kHeadDim,
                              a.copy != nullptr ? copy_block(a, seqs, kvh, s, blk) : nullptr,
                              a.vt16 + (size_t)wg * kHeadDim * kImageRows, a.range_flags + wg, 1 << s);
}
// ... and the copy alone.
__device__ __forceinline__ void prep_copy(const PrepArgs& a, const SeqTable& seqs, int wg) {
  const int s = seq_of(seqs, wg, a.h_kv);
  const int rr = wg - a.h_kv * seqs.s[s].blk0, N = seqs.s[s].N;
  const int kvh = rr / N, blk = rr - kvh * N;
  const int chunks = min(a.block, seqs.s[s].L - blk * a.block) * a.head_dim / 8;       // of 16 bytes
  const u32x4* from = reinterpret_cast<const u32x4*>(
      a.v + (size_t)kvh * a.kv_head_stride + ((size_t)seqs.s[s].tok0 + (size_t)blk * a.block) * a.head_dim);
  u32x4* to = reinterpret_cast<u32x4*>(copy_block(a, seqs, kvh, s, blk));
  for (int i = threadIdx.x; i < chunks; i += kPrepThreads) to[i] = __builtin_nontemporal_load(from + i);
}
// The smallest calls feel what lies in front of their work: with the shortest plans first, and without a look
// at each of sixteen sequences where there is one, 32 rows of one head take 4.3 us instead of 4.9.
__global__ __launch_bounds__(kPrepThreads, 8) void prep_kernel(PrepArgs a, SeqTable table) {
  __shared__ PrepLds lds;
  // The table in LDS: indexed by a lane's own sequence the kernel argument would be copied to scratch memory.
  __shared__ SeqTable seqs;
  if (threadIdx.x == 0) {
    seqs.n = table.n;
    seqs.nsum = table.nsum;
    seqs.s[0] = table.s[0];
  }
  if (table.n > 1) {
#pragma unroll
    for (int i = 1; i < kMaxGroupSeqs; ++i)
      if (i < table.n && threadIdx.x == i) seqs.s[i] = table.s[i];
  }
  __syncthreads();
  __shared__ int s_over;
  int wg = blockIdx.x;
  if (wg >= a.n_plans) {
    wg -= a.n_plans;
    if (wg < a.n_check) {
      check_rows(a, seqs, wg, s_over);
      return;
    }
    wg -= a.n_check;
    if (a.vt16 != nullptr) prep_image(lds, s_over, a, seqs, wg);
    else prep_copy(a, seqs, wg);
    return;
  }
  const int stride = 1 + wg;
  const int R = a.h * seqs.nsum / stride;
  const int n_queues = wg == 0 ? a.n_queues : a.pair_queues;
  int4* items = wg == 0 ? a.items : a.pair_items;
  int32_t* plan = wg == 0 ? a.plan : a.pair_plan;
  int32_t* counters = wg == 0 ? a.counters : a.pair_counters;
  int32_t* more = a.n_plans == 1 ? a.pair_counters : nullptr;
  const int grid = wg == 0 ? a.grid : a.pair_grid;
  // The waves take 64 * CH rows each in turn, so a CH too large leaves the last waves idle (5024 rows at 8 instead of 5 are
  // ten waves' work): an instance for every 1024 rows.  us of the launch, with 1, 2, 4 and 8 only -> now: 20011 tokens 30.6 -> 24.4,
  // 32/8 heads, 28000 (7008 rows) 37.0 -> 33.6; packed batches of 2900 rows 20.6 -> 17.5, 4640 37.8 -> 29.1, 7000 43.1 -> 38.3.
  // At 64 registers a lane, for two workgroups to a CU, the largest instances spill 11 or 12 of them.
  auto run = [&](auto one) __attribute__((always_inline)) {
    constexpr bool kOne = decltype(one)::value;
    if (R <= kPrepThreads) plan_rows<1, kOne>(lds.plan, a, seqs, stride, n_queues, grid, counters, more, items, plan);
    else if (R <= 2 * kPrepThreads) plan_rows<2, kOne>(lds.plan, a, seqs, stride, n_queues, grid, counters, more, items, plan);
    else if (R <= 3 * kPrepThreads) plan_rows<3, kOne>(lds.plan, a, seqs, stride, n_queues, grid, counters, more, items, plan);
    else if (R <= 4 * kPrepThreads) plan_rows<4, kOne>(lds.plan, a, seqs, stride, n_queues, grid, counters, more, items, plan);
    else if (R <= 5 * kPrepThreads) plan_rows<5, kOne>(lds.plan, a, seqs, stride, n_queues, grid, counters, more, items, plan);
    else if (R <= 6 * kPrepThreads) plan_rows<6, kOne>(lds.plan, a, seqs, stride, n_queues, grid, counters, more, items, plan);
    else if (R <= 7 * kPrepThreads) plan_rows<7, kOne>(lds.plan, a, seqs, stride, n_queues, grid, counters, more, items, plan);
    else plan_rows<8, kOne>(lds.plan, a, seqs, stride, n_queues, grid, counters, more, items, plan);
  };
  if (seqs.n == 1) run(std::true_type{});
  else run(std::false_type{});
}

}  // namespace prism

using namespace prism;

// ---- workspace layout: [ copy of V        (packed batches: where they read one, or have room)
//                            items[h*N] (queue entries) | row_rank[h*N] | row_part[h*N] |
//                            bins[2*h*kClasses] | parts[h_kv*kClasses*8] | plan[kPlanInts] |
//                            fp16 V image | range_flags[h_kv*N]        where the fp16 image is read |
//                            pair_items[h*N/2] | pair_plan[kPlanInts]  where the pair kernel may run ] ----
struct AttnWs {
  size_t copy, items, row_rank, row_part, bins, parts, plan, image16, range_flags, pair_items, pair_plan, total;
};
// The fp16 image exists where the 64-queries-per-wave kernel can take the call: whole blocks only.  Ragged lengths stay
// with the general kernel, which reads V as it is given: fp16 loses bits of values below 2^-17 and has nothing left of
// them at 2^-25.  (Attention alone, us, general kernel against this one with fp16: 8 heads, 8100 tokens 91 and 77;
// 32 heads, 8100 183 and 165; 20011 539 and 541; 32001 1052 and 1025.  With bf16 P and V in this kernel the error
// of a lagging maximum, 0.0020 instead of the general kernel's 0.0017, or the rescaling without the lag, 570 at 20011.)
static bool w64_shape(const prism_params* p) {
  return p->block == 128 && p->head_dim == kHeadDim && p->seq_len % 128 == 0;
}

// B = 64 with an even number of blocks: a second plan over pairs of q-blocks for the pair kernel
static bool pair_shape(const prism_params* p) { return p->block == 64 && n_blocks(p) % 2 == 0; }

// The layout for `N` blocks (those of one sequence, or of a group of a packed batch).
static AttnWs attn_layout(const prism_params* p, size_t N, bool with_copy, bool with16, bool pairs) {
  const size_t rows = (size_t)p->n_q_heads * N;
  const size_t image_bytes = (size_t)p->n_kv_heads * N * p->block * p->head_dim * 2;
  AttnWs w;
  size_t off = 0;
  w.copy = off;     off = align_up(off + (with_copy ? image_bytes : 0), 256);
  w.items = off;    off = align_up(off + rows * sizeof(int4), 256);
  w.row_rank = off; off = align_up(off + rows * sizeof(int32_t), 256);
  w.row_part = off; off = align_up(off + rows * sizeof(int32_t), 256);
  w.bins = off;     off = align_up(off + (size_t)2 * p->n_q_heads * kClasses * sizeof(int32_t), 256);
  w.parts = off;    off = align_up(off + (size_t)p->n_kv_heads * kClasses * 8 * sizeof(int32_t), 256);
  w.plan = off;     off = align_up(off + kPlanInts * sizeof(int32_t), 256);
  w.image16 = off;
  w.range_flags = off;
  if (with16) {
    off = align_up(off + image_bytes, 256);
    w.range_flags = off;
    off = align_up(off + (size_t)p->n_kv_heads * N * sizeof(int32_t), 256);
  }
  w.pair_items = off;
  w.pair_plan = off;
  if (pairs) {
    off = align_up(off + rows / 2 * sizeof(int4), 256);
    w.pair_plan = off;
    off = align_up(off + kPlanInts * sizeof(int32_t), 256);
  }
  w.total = off;
  return w;
}
// elements between the kv heads of the copy of V, whose sequences start with a block each
static size_t copy_head_stride(const prism_params* p, size_t N) { return N * p->block * p->head_dim; }
static AttnWs attn_ws(const prism_params* p) { return attn_layout(p, n_blocks(p), true, w64_shape(p), pair_shape(p)); }

static int check_image(const prism_params* params, const void* img, size_t bytes) {
  if (img == nullptr || (reinterpret_cast<uintptr_t>(img) & 255u) != 0 ||
      bytes < attn_ws(params).total)
    return PRISM_ERR_WORKSPACE;
  return PRISM_OK;
}

// Facts about the device the calls run on, asked from the runtime once per device.
struct DeviceFacts {
  int cus;          // compute units
};
static int device_facts(DeviceFacts* out) {
  static std::mutex mu;
  static DeviceFacts facts[kMaxDevices];
  static bool known[kMaxDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PRISM_ERR_HIP;
  std::lock_guard<std::mutex> lock(mu);
  if (!known[dev]) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return PRISM_ERR_HIP;
    facts[dev].cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    known[dev] = true;
  }
  *out = facts[dev];
  return PRISM_OK;
}

// The memory-side cache holds 256 MB; the K and V of the kv heads that are in flight together are
// kept to kCacheBudgetBytes of it.
constexpr size_t kCacheBudgetBytes = (size_t)160 << 20;

// kv heads whose K and V fit that budget together, at least one
static int heads_in_cache(const prism_params* p, const SeqTable& seqs) {
  size_t tokens = 0;
  for (int i = 0; i < seqs.n; ++i) tokens += seqs.s[i].L;
  const size_t fit = kCacheBudgetBytes / (tokens * p->head_dim * 2 * 2);
  return fit < 1 ? 1 : (fit > 0x7fffffff ? 0x7fffffff : (int)fit);
}

static int persistent_grid(int rows, int wgs_per_cu) {
  DeviceFacts f;
  if (device_facts(&f) != PRISM_OK) return -1;
  const int resident = f.cus * wgs_per_cu;
  return rows < resident ? rows : resident;
}

extern "C" int prism_sparse_attn_workspace_bytes(const prism_params* params, size_t* bytes) {
  if (bytes == nullptr) return PRISM_ERR_INVALID_ARG;
  int rc = check_params(params);
  if (rc != PRISM_OK) return rc;
  *bytes = attn_ws(params).total;
  return PRISM_OK;
}

// The parts of the V image by kernels of their own.
static int v_image_core(const prism_params* params, const HeadStrides& hs, const void* v_bf16, const AttnWs& W, char* ws,
                        bool copy, bool image16, hipStream_t st) {
  const uint16_t* v = (const uint16_t*)v_bf16;
  const size_t chunks = (size_t)params->seq_len * params->head_dim / 8;     // 16 bytes each
  uint16_t* to = copy ? reinterpret_cast<uint16_t*>(ws + W.copy) : nullptr;
  if (copy && !image16)
    hipLaunchKernelGGL(v_copy_kernel, dim3((unsigned)((chunks + 1023) / 1024), params->n_kv_heads), dim3(256), 0, st, v, chunks, hs.kv,
                       copy_head_stride(params, n_blocks(params)), to);
  if (image16)
    hipLaunchKernelGGL(vt_image_kernel, dim3(n_blocks(params), params->n_kv_heads), dim3(256), 0, st, v, n_blocks(params), hs.kv, to,
                       reinterpret_cast<uint16_t*>(ws + W.image16), reinterpret_cast<int32_t*>(ws + W.range_flags));
  return launch_status();
}

extern "C" int prism_v_image(const prism_params* params, const void* v_bf16, void* v_image,
                             size_t v_image_bytes, void* stream) {
  int rc = check_params(params);
  if (rc != PRISM_OK) return rc;
  if (!v_bf16) return PRISM_ERR_INVALID_ARG;
  rc = check_image(params, v_image, v_image_bytes);
  if (rc != PRISM_OK) return rc;
  return v_image_core(params, contiguous_heads(params), v_bf16, attn_ws(params), static_cast<char*>(v_image),
                      true, w64_shape(params), static_cast<hipStream_t>(stream));
}

template <int BLK, bool kStreamOnly, int D, bool kPair = false, bool kKeepMask = false>
static void launch_attn(int grid, hipStream_t st, const PullCounters& pulls, const uint16_t* q, const uint16_t* k, const uint16_t* v, size_t v_head_stride,
                        const int32_t* row_ptr, const int32_t* col_idx, const int4* items, int32_t* plan,
                        const DirtyFlags& flags, uint16_t* out, float* lse, int h, int h_kv, const SeqTable& seqs,
                        const HeadStrides& hs, int causal, int only_dirty) {
  hipLaunchKernelGGL((sparse_attn_kernel<BLK, kStreamOnly, D, kPair, kKeepMask>), dim3(grid),
                     dim3(AttnCfg<BLK, D, kPair>::kThreads), 0, st, q, k, v, v_head_stride, row_ptr, col_idx, items, plan,
                     pulls, flags, out, lse, h, h_kv, seqs, hs, causal, only_dirty);
}

// the three kernels that turn index lists into the queue plan of `pc`
static void build_plan(const PlanCfg& pc, const int32_t* row_ptr, const int32_t* col_idx, int32_t* bins,
                       int32_t* parts, int32_t* row_rank, int32_t* row_part, int32_t* plan, int4* items,
                       const CounterInit& ci, hipStream_t st) {
  const int R = pc.h * pc.N;
  hipLaunchKernelGGL(queue_count_kernel, dim3(pc.h), dim3(256), 0, st, row_ptr, pc, bins, parts, plan);
  hipLaunchKernelGGL(queue_rank_kernel, dim3(pc.h), dim3(256), 0, st, row_ptr, pc, bins, parts, row_rank,
                     row_part);
  hipLaunchKernelGGL(queue_fill_kernel, dim3((R + 255) / 256), dim3(256), 0, st, row_ptr, col_idx, pc,
                     parts, row_rank, row_part, plan, items, ci);
}

// The whole attention of the sequences in `seqs` (arguments already validated; several sequences only where
// R <= kPrepMaxRows and one phase, and where w64_shape says the same of all).  With `v_bf16` null the V image in `ws` takes
// its place; with `writes_copy` the call writes that image, whole, whatever it reads of it.
static int attn_core(const prism_params* params, const HeadStrides& hs, const SeqTable& sequences, const AttnWs& W,
                     const void* q_bf16, const void* k_bf16, const void* v_bf16, char* ws, bool writes_copy,
                     const int32_t* row_ptr, const int32_t* col_idx, void* out_bf16, float* lse, hipStream_t st) {
  const int h = params->n_q_heads, h_kv = params->n_kv_heads, d = params->head_dim;
  // The general kernel reads the copy where there is one: V itself may lie where the outputs go, and its tile copies ask for
  // 16-byte alignment.
  const bool reads_copy = v_bf16 == nullptr || writes_copy;
  SeqTable seqs = sequences;
  for (int i = 0; i < seqs.n; ++i) seqs.s[i].v_shift = reads_copy ? seqs.s[i].blk0 * params->block - seqs.s[i].tok0 : 0;
  const int N = seqs.nsum;
  const int R = h * N;
  int4* items = reinterpret_cast<int4*>(ws + W.items);
  int32_t* row_rank = reinterpret_cast<int32_t*>(ws + W.row_rank);
  int32_t* row_part = reinterpret_cast<int32_t*>(ws + W.row_part);
  int32_t* bins = reinterpret_cast<int32_t*>(ws + W.bins);
  int32_t* parts = reinterpret_cast<int32_t*>(ws + W.parts);
  int32_t* plan = reinterpret_cast<int32_t*>(ws + W.plan);
  // resident workgroups per CU, by the LDS the two tiles of a workgroup take (2 * B * d * 2 bytes of the
  // CU's 160 KB) and its waves: 2 at B = 128, d = 128 (64 KB, 4 waves).  At d = 256 a wave has a SIMD to itself: one
  // workgroup of four waves, or two of two at B = 64.  Two of these share the LDS and the copies of the CU, which a call
  // bound by its longest rows feels and another one does not: from four rows per CU on, where the preparation looks for the
  // longest row, the lists decide (halve, below); elsewhere it is two beyond 11 rows per CU.  us of estimate and attention, one / two
  // / by the lists: 16/4 heads, 8100 tokens (2032 rows) 274 / 296 / 275, 10001 (2512) 336 / 359 / 336, 12065 (3024) 420 / 424 / 422,
  // 30016 (7504) 1968 / 1334 / 1335; 32/8, 2063 (1056) 100 / 108 / 101, 4000 (2016) 183 / 176 / 176, 5050 (2528) 241 / 216 / 217, 8100
  // (4064) 453 / 340 / 344, 16300 (8160) 1156 / 824 / 825; 28/4, 4001 (1764) 159 / 176 / 159, 6050 (2660) 246 / 245 / 245; 7/1, 24065
  // (2639) 223 / 247 / 223.
  const int tile_pair = 2 * params->block * d * 2;
  int per_cu = (160 * 1024) / tile_pair;
  per_cu = per_cu > 4 ? 4 : per_cu;
  const bool looks = R <= kPrepMaxRows && heads_in_cache(params, seqs) >= h_kv;
  const int two_wide_rows = (looks ? 4 : 11) * persistent_grid(0x7fffffff, 1);
  if (d > 128) per_cu = params->block == 64 && R > two_wide_rows ? 2 : 1;
  else if (params->block == 128 && per_cu > 2) per_cu = 2;
  const int grid = persistent_grid(R, per_cu);
  if (grid <= 0) return PRISM_ERR_HIP;

  // queue plan: kv heads in phases that fit the memory-side cache
  PlanCfg pc;
  pc.h = h;
  pc.g = h / h_kv;
  pc.N = N;
  pc.n_queues = grid < kXcds ? 1 : kXcds;
  pc.heads_per_phase = heads_in_cache(params, seqs);
  pc.n_phases = (h_kv + pc.heads_per_phase - 1) / pc.heads_per_phase;
  if (pc.n_phases * kClasses > kMaxGroups) {                               // very many kv heads: larger phases
    pc.n_phases = kMaxGroups / kClasses;
    pc.heads_per_phase = (h_kv + pc.n_phases - 1) / pc.n_phases;
    pc.n_phases = (h_kv + pc.heads_per_phase - 1) / pc.heads_per_phase;
  }
  pc.cap = seqs.s[0].cap;
  pc.causal = (params->flags & PRISM_FLAG_BIDIRECTIONAL) ? 0 : 1;
  pc.stride = 1;
  const int causal = pc.causal;
  // Which rows have a CU to themselves (first_row), where the grid fills the chip with two workgroups per CU.  A row that
  // shares its CU advances a block in 2.25 us where the average workgroup, over all of a call, takes 3 (four waves of
  // 32 queries; the general kernel 3.3 and 4), so from 1.4 times the average work on it would be the last to end.  us of
  // preparation and attention, without / 1.0 / 1.1 / 1.25 / 1.4: 32/8 heads, 8192 tokens 155.2 / 141.4 / 140.8 / 140.5 / 140.8,
  // 8100 177.8 / 165.4 / 164.5 / 164.6 / 165.2, 8/2 heads, 8192 78.6 / 76.3 / 75.9 / 76.6 / 76.2; below 1.4 other calls lose:
  // 16 heads, 19290, bidirectional 459 / 480 / 462 / 461 / 461, 4 heads, 128K 1640 / 1691 / 1646 / 1640 / 1638, the eight packed
  // prompts of perf/cases.py 656 / 663 / 659 / 659 / 657.
  // A CU with one workgroup does less than one with two, and the workgroup that ended does not come back: a queue (an XCD)
  // with more such rows than 5/8 of its CUs has none alone.  us without / with / only up to 5/8, M rows of N blocks among h * N
  // with one block (h x N, M): four waves 32 x 124, 128 278 / 253 / 252, 8 x 100, 288 332 / 382 / 333; two waves (beyond kW32MaxRows
  // rows) 14 x 300, 128 737 / 705 / 703, 288 859 / 1425 / 862; general kernel 32 x 124, 128 305 / 281 / 281, 8 x 100, 288 329 / 452 / 329;
  // d = 64 32 x 124, 128 205 / 200 / 199, 8 x 100, 288 217 / 310 / 217.  Causal, one of 8 heads with full lists, N = 512, whose 73
  // longest rows lie in three queues: four waves 1276 / 1333 / 1276, general kernel 1361 / 1286 / 1362.
  constexpr float kAlone = 1.4f;
  const bool full = grid == persistent_grid(0x7fffffff, 2) && grid % (2 * kXcds) == 0 && grid / (2 * kXcds) <= 32;
  const float alone = params->block == 128 && per_cu == 2 && full ? kAlone : 0.f;
  // Wide rows (d = 256, two workgroups per CU): all have a CU to themselves, so half of the workgroups end, where the longest row
  // bounds the call, a CU's average work (entries + 3 a row) being less than 1.2 times the longest row.  us of estimate
  // and attention, one / two per CU, at that ratio: 16/2 heads, 11305 tokens (0.90) 355 / 393, 16/8, 11309 (0.94) 384 / 401, 8/1, 24071
  // (1.17) 229 / 245; 4/2, 45368 (1.21) 819 / 846, 16/4, 12066 (1.25) 455 / 434.  Calls of several phases or more than kPrepMaxRows
  // rows have two, whose preparation does not look for the longest row (16/16, 11298 (0.95) 617 / 546, 15288 (1.12) 746 / 703).
  const float halve = d > 128 && per_cu == 2 && full ? 1.2f : 0.f;
  const bool stream_only = (params->flags & PRISM_FLAG_STREAM_ONLY) != 0;
  const uint16_t* qp = (const uint16_t*)q_bf16;
  const uint16_t* kp = (const uint16_t*)k_bf16;
  const uint16_t* vp = reads_copy ? reinterpret_cast<const uint16_t*>(ws + W.copy) : (const uint16_t*)v_bf16;
  const size_t v_head_stride = reads_copy ? copy_head_stride(params, N) : hs.kv;
  const bool with16 = w64_shape(params);
  uint16_t* vp16 = with16 ? reinterpret_cast<uint16_t*>(ws + W.image16) : nullptr;
  int32_t* range_flags = with16 ? reinterpret_cast<int32_t*>(ws + W.range_flags) : nullptr;
  uint16_t* op = (uint16_t*)out_bf16;
  // Whole blocks of 128 tokens go through the 64-queries-per-wave kernel when every list of a sequence is clean
  // (decided on the device, so the general kernel is queued behind it, takes the sequences whose lists or values turn
  // out to need it and returns at once where none do).
  const bool w64 = with16 && !stream_only && !(params->flags & PRISM_FLAG_GENERAL_KERNEL);
  // B = 64 with an even number of blocks: the pair kernel (two q-blocks per workgroup sharing the tiles of
  // the union of their lists) takes the call when every list is ascending and clean; decided on the
  // device in the same way.
  // Below kPairMinRows rows the call is short and launch-bound, and the second plan and the list check
  // (four more launches) cost more than the shared tiles save (measured: 25 -> 42 us at 32 rows).
  // At d = 64 a tile is 8 KB and the plain kernel is not bound by its copies: the pair form is 5 % slower
  // even on all-ones lists, where the two lists of a pair coincide (750 -> 712 TFLOP/s at 16K tokens;
  // d = 128: 948 -> 993, d = 256: 438 -> 753).
  // At d = 256, where a workgroup of the plain form has two waves for the four SIMDs of its CU, pairs win from 11 rows per CU on: us
  // of estimate and attention, plain / pairs: 16/4 heads, 8192 tokens (2048 rows) 278 / 294, 8/2, 16384 (2048) 292 / 300, 16/2, 11264
  // (2816) 374 / 381, 16/4, 11264 (2816) 414 / 392, 28/4, 6656 (2912) 277 / 261, 12/4, 16384 (3072) 321 / 318, 8/2, 24576 (3072) 609 /
  // 523, 32/8, 6144 (3072) 262 / 253, 28/4, 8192 (3584) 334 / 308, 4/2, 57344 (3584) 924 / 786.
  const int pair_rows = d > 128 ? 11 * persistent_grid(0x7fffffff, 1) : 4096;
  const bool pair = W.pair_plan != W.pair_items && !stream_only && !(params->flags & PRISM_FLAG_GENERAL_KERNEL) &&
                    ((R >= pair_rows && d >= 128) || (params->flags & PRISM_FLAG_PAIR_KERNEL));
  const int only_dirty = w64 && seqs.n > 1 ? kDirtySequences : (w64 || pair ? kDirtyCall : kEverything);
  int4* pair_items = reinterpret_cast<int4*>(ws + W.pair_items);
  int32_t* pair_plan = reinterpret_cast<int32_t*>(ws + W.pair_plan);
  const int pair_grid = pair ? persistent_grid(R / 2, d > 128 ? 1 : 2) : 0;   // 4 waves and 2 * 64 * d * 2 bytes of LDS each
  if (pair && pair_grid <= 0) return PRISM_ERR_HIP;
  const int pair_queues = pair_grid < kXcds ? 1 : kXcds;
  const int n_range_flags = w64 ? h_kv * N : 0;
  const bool writes_image16 = v_bf16 != nullptr && with16 && (w64 || writes_copy);

  // One launch prepares the call up to kPrepMaxRows rows in one phase: the V image is written beside the plan of a single workgroup.  us,
  // one launch / separate kernels, B = 128, 32/8 heads, copy and fp16 image: 2048 rows 14.0 / 35.9, 4096 27.1 / 45.1, 8192 47.2 / 61.7; the copy
  // alone (ragged): 2048 10.3 / 28.4, 4096 21.4 / 32.9, 5024 28.4 / 33.7, 8192 39.3 / 42.3; with a plan of pairs: B = 64, 8192 31.6 / 52.6, d = 256,
  // 4096 22.1 / 50.8; 32 rows 4.2.  Beyond, the plan takes longer than the image.  Calls that write none (prism_sparse_attn_pre, most packed
  // batches) would have their line lower: 2048 rows 10 / 18, 4096 17.0 / 18.6, 5024 21.9 / 18.6, 8192 32.4 / 18.8, of calls of 700 - 1300 us
  // (attention and all, 5024 677 / 673, 8192 1275 / 1280, where the separate kernels plan no row with a CU to itself).
  DirtyFlags flags = {plan + kPlanFlags, nullptr, 1, 0};
  // Two sets of pull counters in row_part, which the preparation is done with: of the pair kernel and the one behind it, or
  // of the 64-queries-per-wave kernel and the one behind it.  A short table holds them closer together.
  const bool one_launch = R <= kPrepMaxRows && pc.n_phases == 1;
  const int last_fill_rows = pair ? R / 2 : R;             // of queue_fill_kernel, whose threads write the counters
  int counter_stride = kCounterStride;
  while ((size_t)counter_stride * 2 * kXcds * sizeof(int32_t) > W.bins - W.row_part ||
         (!one_launch && counter_stride * 2 * kXcds > last_fill_rows))
    counter_stride >>= 1;
  const PullCounters pulls = {row_part, counter_stride}, second_pulls = {row_part + counter_stride * kXcds, counter_stride};
  if (one_launch) {
    PrepArgs pa = {};
    pa.row_ptr = row_ptr;
    pa.col_idx = col_idx;
    pa.v = (const uint16_t*)v_bf16;
    pa.vt16 = writes_image16 ? vp16 : nullptr;
    pa.copy = writes_copy ? reinterpret_cast<uint16_t*>(ws + W.copy) : nullptr;
    pa.block = params->block;
    pa.head_dim = d;
    pa.range_flags = range_flags;
    pa.check = row_rank;
    pa.items = items;
    pa.pair_items = pair_items;
    pa.plan = plan;
    pa.pair_plan = pair_plan;
    pa.h = h;
    pa.h_kv = h_kv;
    pa.causal = (uint8_t)pc.causal;
    pa.n_queues = pc.n_queues;
    pa.pair_queues = pair_queues;
    pa.n_plans = pair ? 2 : 1;
    pa.n_check = only_dirty != kEverything ? (R + kCheckRows - 1) / kCheckRows : 0;
    pa.need_sorted = pair ? 1 : 0;
    pa.counters = pulls.at;
    pa.pair_counters = second_pulls.at;
    pa.counter_stride = pulls.stride;
    pa.grid = grid;
    pa.alone = alone;
    pa.halve = halve;
    pa.pair_grid = pair_grid;
    pa.kv_head_stride = hs.kv;
    const int prep_grid = pa.n_plans + pa.n_check + (writes_copy || writes_image16 ? h_kv * N : 0);
    hipLaunchKernelGGL(prep_kernel, dim3(prep_grid), dim3(kPrepThreads), 0, st, pa, seqs);
    flags = DirtyFlags{row_rank, range_flags, pa.n_check, n_range_flags};
  } else {
    if (writes_copy || writes_image16) {
      const int rc = v_image_core(params, hs, v_bf16, W, ws, writes_copy, writes_image16, st);
      if (rc != PRISM_OK) return rc;
    }
    // (over a thousand rows here: more than kPrepMaxRows, or kv heads that do not fit the memory-side cache together)
    const CounterInit later = {};
    const CounterInit ci = {counter_stride, {pc.n_queues, pair ? pair_queues : pc.n_queues}, {grid, pair ? pair_grid : grid}};
    build_plan(pc, row_ptr, col_idx, bins, parts, row_rank, row_part, plan, items, pair ? later : ci, st);
    if (pair) {
      PlanCfg pp = pc;
      pp.N = N / 2;
      pp.stride = 2;
      pp.n_queues = pair_queues;
      build_plan(pp, row_ptr, col_idx, bins, parts, row_rank, row_part, pair_plan, pair_items, ci, st);
    }
    if (only_dirty != kEverything) {
      const int by_flags = (n_range_flags + 255) / 256;
      hipLaunchKernelGGL(queue_validate_kernel, dim3((R + 3) / 4 > by_flags ? (R + 3) / 4 : by_flags), dim3(256), 0, st,
                         row_ptr, col_idx, h, N, pc.cap, causal, pair ? 1 : 0, range_flags, n_range_flags, plan);
    }
  }
  if (pair) {
#define PRISM_PAIR(D)                                                                                        \
  launch_attn<64, false, D, true>(pair_grid, st, second_pulls, qp, kp, vp, v_head_stride, row_ptr, col_idx, pair_items, pair_plan, flags, \
                                  op, lse, h, h_kv, seqs, hs, causal, 0)
    if (d == 64) PRISM_PAIR(64);
    else if (d == 128) PRISM_PAIR(128);
    else PRISM_PAIR(256);
#undef PRISM_PAIR
  }
  if (w64) {
    // The same bits from two waves of 64 queries or from four of 32.  Four take 1.3 instead of 2.2 us per block of a
    // row that has a CU to itself, two need half the LDS reads per block and are 3 % faster where every CU is busy
    // to the end (2048 rows of 64 blocks: 543 against 558 us).  Up to kW32MaxRows rows, 8 per resident workgroup, the
    // longest rows decide how long a call takes (us, two waves -> four): 8 heads, 8K tokens (512 rows) 93 -> 71;
    // 32 heads, 8K (2048) 184 -> 152; 4 heads, 128K (4096) 1010 -> 836; 32 heads, 16K (4096) 396 -> 392; beyond it, with
    // as many heads, two waves win: 17K (4352 rows) 457 and 460, 20096 tokens (5024) 515 and 530, 32K (8192) 1056 and 1068.
    // (Few heads with long rows would still want four: 5 heads, 128K, 5120 rows 888 -> 703.)
    constexpr int kW32MaxRows = 4096;
    if (R <= kW32MaxRows)
      hipLaunchKernelGGL(sparse_attn_w64_kernel<32>, dim3(grid), dim3(256), 0, st, qp, kp, vp16, col_idx, items, plan,
                         pulls, flags, op, lse, h, h_kv, seqs, hs, causal);
    else
      hipLaunchKernelGGL(sparse_attn_w64_kernel<64>, dim3(grid), dim3(128), 0, st, qp, kp, vp16, col_idx, items, plan,
                         pulls, flags, op, lse, h, h_kv, seqs, hs, causal);
  }
  // Plain 64 x 128 beyond kPrepMaxRows rows keeps its mask compares across the row loop.  us of attention before they were
  // formed in place / formed / kept: 32/8 heads, 16448 tokens (8224 rows) 546 / 558 / 549, 30016 1086 / 1115 / 1091, 28/4 heads,
  // 33328 1121 / 1148 / 1130.  Forming them once costs a workgroup about 1 us, which short calls notice (32 rows 15 -> 16,
  // 7968 rows 433 -> 436), and the other shapes are faster without: 64 x 64 at 16448 tokens 413 -> 401, 64 x 256 at 16320
  // 1406 -> 1375, 128 x 64 at 32768 804 -> 795, 128 x 128 at 40001 1669 -> 1662.
#define PRISM_ATTN(BLK, SO, D, KEEP)                                                                          \
  launch_attn<BLK, SO, D, false, KEEP>(grid, st, w64 ? second_pulls : pulls, qp, kp, vp, v_head_stride, row_ptr, col_idx, items, plan, flags, op, lse, h, h_kv, seqs, \
                          hs, causal, only_dirty)
  if (stream_only) {
    // measurement aid of the d = 128 kernels only
    if (d != 128) return PRISM_ERR_UNSUPPORTED;
    if (params->block == 128) PRISM_ATTN(128, true, 128, false);
    else PRISM_ATTN(64, true, 128, false);
  } else if (params->block == 128) {
    if (d == 64) PRISM_ATTN(128, false, 64, false);
    else if (d == 128) PRISM_ATTN(128, false, 128, false);
    else PRISM_ATTN(128, false, 256, false);
  } else {
    if (d == 64) PRISM_ATTN(64, false, 64, false);
    else if (d == 128 && R > kPrepMaxRows) PRISM_ATTN(64, false, 128, true);
    else if (d == 128) PRISM_ATTN(64, false, 128, false);
    else PRISM_ATTN(64, false, 256, false);
  }
#undef PRISM_ATTN
  return launch_status();
}

extern "C" int prism_sparse_attn_pre(const prism_params* params, const void* q_bf16,
                                     const void* k_bf16, void* v_image, size_t v_image_bytes,
                                     const int32_t* row_ptr, const int32_t* col_idx,
                                     int64_t col_count, void* out_bf16, float* lse, void* stream) {
  int rc = check_params(params);
  if (rc != PRISM_OK) return rc;
  if (!q_bf16 || !k_bf16 || !row_ptr || !col_idx || !out_bf16 || col_count < 0)
    return PRISM_ERR_INVALID_ARG;
  rc = check_image(params, v_image, v_image_bytes);
  if (rc != PRISM_OK) return rc;
  return attn_core(params, contiguous_heads(params), one_sequence(params, col_count),
                   attn_ws(params), q_bf16, k_bf16, nullptr, static_cast<char*>(v_image), false,
                   row_ptr, col_idx, out_bf16, lse, static_cast<hipStream_t>(stream));
}

extern "C" int prism_sparse_attn(const prism_params* params, const void* q_bf16, const void* k_bf16,
                                 const void* v_bf16, const int32_t* row_ptr, const int32_t* col_idx,
                                 int64_t col_count, void* out_bf16, float* lse, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  int rc = check_params(params);
  if (rc != PRISM_OK) return rc;
  if (!q_bf16 || !k_bf16 || !v_bf16 || !row_ptr || !col_idx || !out_bf16 || col_count < 0)
    return PRISM_ERR_INVALID_ARG;
  rc = check_image(params, workspace, workspace_bytes);
  if (rc != PRISM_OK) return rc;
  return attn_core(params, contiguous_heads(params), one_sequence(params, col_count),
                   attn_ws(params), q_bf16, k_bf16, v_bf16, static_cast<char*>(workspace), true, row_ptr,
                   col_idx, out_bf16, lse, static_cast<hipStream_t>(stream));
}

// ---- packed variable-length batches: groups of sequences, one after the other on the stream ---------
extern "C" int prism_sparse_attn_varlen_workspace_bytes(const prism_params* params, const int32_t* cu_seqlens,
                                                        int n_seqs, size_t* bytes) {
  if (bytes == nullptr) return PRISM_ERR_INVALID_ARG;
  int rc = prism_varlen_layout(params, cu_seqlens, n_seqs, nullptr, nullptr, nullptr);
  if (rc != PRISM_OK) return rc;
  size_t need = 0;
  for (int s = 0; s < n_seqs; ++s) {
    prism_params ps = *params;
    ps.seq_len = cu_seqlens[s + 1] - cu_seqlens[s];
    const size_t b = attn_ws(&ps).total;
    need = b > need ? b : need;
  }
  *bytes = need;
  return PRISM_OK;
}

extern "C" int prism_sparse_attn_varlen(const prism_params* params, const int32_t* cu_seqlens, int n_seqs,
                                        const void* q_bf16, const void* k_bf16, const void* v_bf16,
                                        const int32_t* row_ptr, const int32_t* col_idx, void* out_bf16,
                                        float* lse, void* workspace, size_t workspace_bytes, void* stream) {
  size_t need = 0;
  int rc = prism_sparse_attn_varlen_workspace_bytes(params, cu_seqlens, n_seqs, &need);
  if (rc != PRISM_OK) return rc;
  if (!q_bf16 || !k_bf16 || !v_bf16 || !row_ptr || !col_idx || !out_bf16) return PRISM_ERR_INVALID_ARG;
  if (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 || workspace_bytes < need)
    return PRISM_ERR_WORKSPACE;
  const size_t d = params->head_dim, T = params->seq_len;
  const HeadStrides hs{T * d, T * d, T};
  hipStream_t st = static_cast<hipStream_t>(stream);
  // B = 64 in pairs of q-blocks: every sequence of the group has an even number of blocks
  auto pairs = [&](const SeqTable& t) {
    bool even = params->block == 64;
    for (int i = 0; i < t.n; ++i) even = even && t.s[i].N % 2 == 0;
    return even;
  };
  // Whole blocks of 128 and ragged lengths have kernels of their own (w64_shape), here as in calls on one sequence:
  // a group is of one kind.
  auto kind = [&](const SeqInfo& q) {
    prism_params ps = *params;
    ps.seq_len = q.L;
    return w64_shape(&ps);
  };
  // These calls leave no image and read V itself, where it is aligned for the tile copies and apart from the outputs: a group
  // that needs the room of a copy has it then.
  const uintptr_t v0 = reinterpret_cast<uintptr_t>(v_bf16), v1 = v0 + params->n_kv_heads * T * d * 2;
  auto overlaps = [&](const void* p, size_t bytes) {
    const uintptr_t p0 = reinterpret_cast<uintptr_t>(p);
    return p != nullptr && p0 < v1 && v0 < p0 + bytes;
  };
  const bool copy = (v0 & 15u) != 0 || overlaps(out_bf16, params->n_q_heads * T * d * 2) || overlaps(lse, params->n_q_heads * T * 4);
  auto layout = [&](const SeqTable& t) {
    const AttnWs w = attn_layout(params, t.nsum, true, kind(t.s[0]), pairs(t));
    return copy || w.total <= workspace_bytes ? w : attn_layout(params, t.nsum, false, kind(t.s[0]), pairs(t));
  };
  // Sequences share their launches while the one-launch preparation can take them all, their heads form one phase
  // and the workspace holds them.
  auto fits = [&](const SeqTable& t) {
    return (int64_t)params->n_q_heads * t.nsum <= kPrepMaxRows && params->n_q_heads < (1 << kSeqShift) &&
           kind(t.s[t.n - 1]) == kind(t.s[0]) && heads_in_cache(params, t) >= params->n_kv_heads &&
           layout(t).total <= workspace_bytes;
  };
  auto run = [&](const SeqTable& t, const prism_params& ps) {
    const size_t tok = t.n > 1 ? 0 : t.s[0].tok0;
    SeqTable at = t;
    if (t.n == 1) at.s[0].tok0 = 0, at.s[0].row0 = 0, at.s[0].col0 = 0;   // one sequence: through the pointers
    const int64_t ro = t.n > 1 ? 0 : t.s[0].row0, co = t.n > 1 ? 0 : t.s[0].col0;
    return attn_core(&ps, hs, at, layout(t), (const uint16_t*)q_bf16 + tok * d, (const uint16_t*)k_bf16 + tok * d,
                     (const uint16_t*)v_bf16 + tok * d, static_cast<char*>(workspace), copy, row_ptr + ro, col_idx + co,
                     (uint16_t*)out_bf16 + tok * d, lse != nullptr ? lse + tok : nullptr, st);
  };
  return for_each_group(params, cu_seqlens, n_seqs, fits, run);
}
