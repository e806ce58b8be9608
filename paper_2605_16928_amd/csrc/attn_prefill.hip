// Prefill-time attention on bf16 MFMA: rtp_local_attn / rtp_dense_attn with q_start != NULL, and the
// p >= 1 case of rtp_sparse_attn_prefill (the paper's prefill rule: retrieval heads dense, local heads
// sink + window; Sec. 3.2 and Sec. 4.2).
//
// Flash-style tiling written for the CDNA MFMA register layout.  A wave owns 32 queries and computes
// the TRANSPOSED score tile  S^T = K Q^T  with v_mfma_f32_32x32x16_bf16: the K tile is the A operand
// (read from LDS, row-major, 16-byte reads), Q^T the B operand (held in registers for the whole
// kernel).  In the accumulator layout a lane then holds 16 keys of ONE query (column = lane % 32), so
// the online-softmax state (running max, running sum, rescale factor) is a per-lane scalar and the
// only cross-lane traffic is one exchange with lane ^ 32 per tile.  The probabilities stay in place:
// the accumulator registers, rounded to bf16, ARE the B operand of  O^T = V^T P^T  (the key order
// inside the contraction is permuted identically for both operands), so P never touches LDS.  Only V
// has to be transposed, by the LDS reads that fetch the operands.
//
// Workgroup = 4 waves = 128 queries of one (sequence, head); key tiles of 64; heads of one KV group
// are adjacent in the grid so that they meet in L2; late (long) query tiles are scheduled first.
#include "common.h"
#include "index_project.h"
#include "prefill_scan.h"

#include <algorithm>
#include <type_traits>
#include <vector>

namespace rtp {

constexpr int kPfThreads = 256;
constexpr int kPfQ = 128;          // queries per workgroup
constexpr int kPwQ = 256;          // of the wide kernel
constexpr int kPfK = 64;           // keys per tile
constexpr int kPfPart = kHeadDim + 4;   // floats per partial row: max, sum, 2 pad, unnormalised output[128]

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct PrefillArgs {
  const uint16_t* q;
  const uint16_t* K;
  const uint16_t* V;
  int64_t row_stride, head_stride;
  const int64_t* seq_start;     // NULL: one sequence starting at token 0
  const int32_t* q_start;       // NULL: q_start_host
  int64_t q_start_host;
  int32_t n_q, n_q_heads, n_kv_heads, sink, window;
  float scale, scale_log2;
  uint16_t* out;
  float* lse;
  int32_t n_heads;
  bool by_die;                  // local band: a KV head to a die
  uint8_t heads[128];           // query heads this launch computes, ascending
  int32_t n_splits;             // wide kernel: key range of every query tile cut into this many parts
  int32_t n_sub;                // ... and every part into this many sub-ranges that share the part's reference maxima
  float* part;                  // n_splits * n_sub > 1: partial results [range, head slot, query, kPfPart]
  // sparse mode only (per-query top-p over the indexer scores):
  const uint16_t* qI;           // bf16 [n_ret, n_q, 16]
  const uint16_t* kI;           // bf16 [n_ret, >= pos0 + n_q, 16]
  int64_t kI_head_stride;
  float p, index_scale;
  float* tau;                   // optional [n_ret, n_q] (the three also in dense mode, where they are known without a search)
  int32_t* count;
  float* mass;
  float* sel_thr;               // [n_ret, n_q]: a candidate is kept iff its raw index product is >= this
  int32_t f16;                  // q, K, V and out are fp16 (else bf16)
  // selecting mode: which key tiles can hold a kept pair at all
  float* tile_max;              // [n_ret * ceil(n_q / 32), n_t64]: largest raw index product of a 32-query group in a 64-key tile
  int32_t n_t64;                // row length of tile_max
  int32_t* act_list;            // [n_ret, ceil(n_q / 256), n_t64]: the 64-key tiles a 256-query tile has to visit, ascending
  int32_t* act_count;           // [n_ret, ceil(n_q / 256)]
  int32_t* act_range;           // {longest list, shortest list} of the launch (the search resets, the list kernel updates)
  int32_t n_splits_even;        // key ranges per query tile when the lists are about equally long
  // a threshold search cut into launches, n_slice workgroups per 32-query group (short chunks; see prefill_select_kernel)
  int32_t n_slice;
  float* sl_max;                // [groups, n_slice, 32]: the slices' row maxima
  double* sl_hist;              // [2, groups, n_slice, 128, 32]: the slices' histograms (running sums), of the current sweep and the one before
  struct SelState* sl_state;    // [2, n_ret, n_q]: what a scan found, read by the next launch
  int32_t* sl_again;            // [groups]: 1 = some query's threshold lies in the open-ended bin, the last launch searches the group;
                                // 2 = the group's search is complete
  // queries regrouped by how much they keep (prefill_order_kernel); NULL: every launch takes them by position, and units is NULL too
  int32_t* order;               // [n_ret, n_q]: the query of every place
  int32_t* order_on;            // [n_ret, blocks]: how the block's queries stand, kOrder...
  int32_t order_block;          // queries per block, a multiple of kPwQ
  int32_t one_round;            // workgroups of a search launch that run at the same time
  int32_t order_whole;          // the first digits came from whole rows: kOrderOwnAlike asks for whole groups too
  // the attention launch's work, cut by the lists' lengths (prefill_plan_kernel); NULL: n_splits ranges of every list.  A query tile has two
  // lists then: list i of its first waves (the ordinary act_list), and of the others, where they keep little, list n_lists + i, which is
  // in more_list: queries in the order of what they keep have one such tile to a block at the most
  int32_t* n_units;             // how many there are; 0: nothing is regrouped, n_splits ranges of every list all the same
  int2* units;                  // [n_units]: {list, range | ranges << 8 | first wave << 16 | past the last << 20 | kUnitExact}
  int2* list_info;              // [2 * n_lists]: {tiles, the same waves << 16 | kUnitExact}, n_lists = n_ret * ceil(n_q / 256)
  int2* list_ranges;            // [2 * n_lists]: {ranges | past the last wave << 16, where the first one's partials are}, in 256-row pieces of `part`
  int32_t* more_list;           // [n_ret, blocks, n_t64]
  int32_t part_cap;             // pieces there is room for
};

enum { kOrderOwnAlike = 0, kOrderOwn = 1, kOrderByKept = 2 };  // by position, their last sweeps about equally long; by position; regrouped
constexpr int kUnitExact = 1 << 30, kFewKept = 64;
enum { kSelRebased = 1, kSelOpen = 2, kSelClassShift = 8 };   // SelState::flags; the class of prefill_order_kernel above them
struct SelState {               // one query between two launches of a search
  double Z, above;
  float selM, x_max;
  int32_t prefix, flags;
};

// Key ranges a selecting launch behind a threshold search really uses: the grid is sized for lists that differ
// wildly in length (many short ranges); when the shortest list is at least half the longest there is nothing to
// even out and the few long ranges of the dense rule are cheaper (fewer partials to write and merge).
__device__ __forceinline__ int listed_splits(const PrefillArgs& a) {
  const int longest = a.act_range[0], shortest = a.act_range[1];
  return (2 * shortest >= longest) ? min(a.n_splits_even, a.n_splits) : a.n_splits;
}

__device__ __forceinline__ int32_t* more_list_of(const PrefillArgs& a, int j, int q_tile) {
  const int blocks = (a.n_q + a.order_block - 1) / a.order_block;
  return a.more_list + ((int64_t)j * blocks + q_tile * kPwQ / a.order_block) * a.n_t64;
}

enum { kModeDense = 0, kModeSparse = 1 };
// Per-query threshold search of the sparse mode: a score s is mapped to the integer
// q = floor((M - s) * 2^17) (M = row maximum; q clamps at 2^21 - 1, i.e. 16 below the maximum) and
// the threshold is the smallest q whose cumulative mass from q = 0 reaches p * Z, found digit by
// digit in base 128 (bin widths 1/8, 1/1024, 1/131072 in score units).  Masses are summed in fp64.
constexpr int kSelBins = 128;
constexpr float kSelScale = 131072.0f;
constexpr int kSelQMax = (1 << 21) - 1;
constexpr int kPfTileBytes = kPfK * kHeadDim * 2 * 2;                 // one staged K + V tile
constexpr int kSelListCap = 24;      // entries per lane of the member lists: with the histogram 80 KB, two workgroups per compute unit
constexpr int kSelMfma = 2;          // index-score MFMAs of a wave in flight (the SIMD's other waves cover their latency)
constexpr int kSelRing = 4, kSelRingWide = 8;   // index-key tiles in flight per wave during the threshold search; where only some of its sweeps run

__device__ __forceinline__ int sel_q_of_t(float tt) {       // tt = M - s >= 0
  return (int)fminf(tt * kSelScale, (float)kSelQMax);
}

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const f32x2 f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}
// The attention tensors' element type is a template flag of the kernels (F16 = IEEE binary16, else bf16): two
// floats rounded (nearest even) and packed, and the 32 x 32 x 16 MFMA on 16-bit operands with fp32 accumulation.
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
template <bool F16> __device__ __forceinline__ uint32_t pack16(float a, float b) {
  if constexpr (F16) {
    const f32x2 f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, f16x2));
  } else {
    return pack_bf16(a, b);
  }
}
template <bool F16> __device__ __forceinline__ f32x16 mfma32(const u32x4 a, const u32x4 b, const f32x16 c) {
  if constexpr (F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// Largest of 16 matrix-core results, none NaN: medians for the first of each half (they make the compiler wait for the
// matrix core, which it does not do for operands of an assembly statement), then three-operand maxima -- the compiler
// has no way to one that does not first canonicalise every operand.
__device__ __forceinline__ float max16_nn(const float (&v)[16]) {
  float a = max_nn(v[0], v[1]), b = max_nn(v[2], v[3]);
#pragma unroll
  for (int i = 4; i < 16; i += 4) {
    asm("v_max3_f32 %0, %0, %1, %2" : "+v"(a) : "v"(v[i]), "v"(v[i + 1]));
    asm("v_max3_f32 %0, %0, %1, %2" : "+v"(b) : "v"(v[i + 2]), "v"(v[i + 3]));
  }
  return max_nn(a, b);
}

// The local heads' band.  What bounds it is each wave's chain through a tile (scores, maximum, probabilities, PV: about 2.3 us
// with one wave per SIMD, where 16 + 16 MFMAs take 0.4), overlapped only with the other workgroup of the compute unit.
// Staging by direct loads and transposing reads instead of through registers, the first PV operands read under the softmax
// and maxima in two short chains: 4096 queries at 128K, 28 heads: 241 -> 175 to 205 us (590 to 690 TFLOP/s); 333 queries: 89 -> 82 us; a
// prompt of 2037 with 6 heads: 31.5 -> 29 us.  Measured without gain: four buffers, three tiles ahead (92 and 32 us: memory
// latency is not the limit); the band on the wide kernel (twice as long: its masked blocks leave the pipelined path).
// GROUPS = 2, for launches of at most one workgroup per compute unit whose bands may have four tiles: a second group of four waves
// takes every other tile of the same queries, with buffers and a running maximum of its own, and the first one merges the two at the
// end.  Launch, us (GPU time alone), one group / two: 28 heads, 333 queries behind 131072 tokens, window 2048: 70.3 / 49.3; 200
// behind 5000, window 512: 28.4 / 22.2; 256 of a prompt (four tiles) 12.4 / 12.2, but 128 to 192 (two, three) 9.3 / 10.2, 64 (one) 6.0 / 7.9.
template <bool F16, int GROUPS>
__global__ __launch_bounds__(kPfThreads * GROUPS, 2) void flash_prefill_local_kernel(const PrefillArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem_all[GROUPS * 2 * kPfTileBytes];

  const int grp = GROUPS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kPfThreads);
  unsigned char* const smem = smem_all + grp * 2 * kPfTileBytes;
  const int tid = (int)threadIdx.x - grp * kPfThreads, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 5, r = lane & 31;
  int h, b, t0, split = 0;
  const int group = a.n_q_heads / a.n_kv_heads;
  if (GROUPS == 2 || !a.by_die) {
    h = a.heads[blockIdx.x];
    b = a.n_splits > 1 ? 0 : (int)blockIdx.z;
    split = a.n_splits > 1 ? (int)blockIdx.z : 0;
    t0 = ((int)gridDim.y - 1 - (int)blockIdx.y) * kPfQ;
  } else {
    // Workgroups go to the eight dies in turn, each with an L2 of its own, and every die takes an eighth of the work in one piece: KV head by
    // KV head, within one the query tiles (late ones first), within a tile the query heads, so that the workgroups a die runs at a
    // time read one KV head's rows of a few thousand tokens.  With the heads side by side in the grid a die read all KV heads' windows
    // at once: 4096 queries at 128K tokens 180 -> 171 us, the last 8192 of 1M (window 4096) 625 -> 595.  (Launches of few workgroups lose the
    // microsecond that finding the place takes.)
    const int per_head = (a.n_q + kPfQ - 1) / kPfQ, n_unit = a.n_heads * per_head;
    const int die = (int)blockIdx.x & 7, chunk = (n_unit + 7) >> 3;
    const int unit = die * chunk + ((int)blockIdx.x >> 3);
    if (unit >= n_unit) return;
    const int any = unit / per_head, kv = a.heads[any] / group;
    int first = any, last = any;                              // the KV head's slots
    while (first > 0 && a.heads[first - 1] / group == kv) --first;
    while (last + 1 < a.n_heads && a.heads[last + 1] / group == kv) ++last;
    const int in_group = unit - first * per_head, n_in = last - first + 1;
    h = a.heads[first + in_group % n_in];
    b = 0;
    t0 = (per_head - 1 - in_group / n_in) * kPfQ;
  }
  const int kvh = h / group;
  const int pos0 = a.q_start ? a.q_start[b] : (int)a.q_start_host;
  const int64_t tok0 = a.seq_start ? a.seq_start[b] : 0;
  const float ninf = -__builtin_huge_valf();

  // ---- this lane's query (column r of the wave's 32) ----
  const int t = t0 + wave * 32 + r;
  const bool qok = t < a.n_q;
  const int m = pos0 + t;
  const int64_t qrow = (((int64_t)b * a.n_q + t) * a.n_q_heads + h) * kHeadDim;
  u32x4 qreg[8];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    qreg[kk] = qok ? *reinterpret_cast<const u32x4*>(a.q + qrow + kk * 16 + g * 8) : (u32x4){0u, 0u, 0u, 0u};
  }

  // ---- key tiles this workgroup needs ----
  const int m_lo = pos0 + t0;
  const int m_hi = pos0 + min(t0 + kPfQ, a.n_q) - 1;
  const int kt_end = m_hi / kPfK;                       // inclusive
  const int kt_w0 = max(a.sink, m_lo - a.window + 1) / kPfK;
  const int ks_end = min((a.sink + kPfK - 1) / kPfK, kt_w0);    // sink tiles not already inside the band
  const int n_band = ks_end + (kt_end - kt_w0 + 1);
  const int it_lo = GROUPS == 2 ? n_band * split / a.n_splits : 0;    // this workgroup's range of them
  const int n_tiles = (GROUPS == 2 ? n_band * (split + 1) / a.n_splits : n_band) - it_lo;

  const uint16_t* Kg = a.K + (int64_t)kvh * a.head_stride + tok0 * a.row_stride;
  const uint16_t* Vg = a.V + (int64_t)kvh * a.head_stride + tok0 * a.row_stride;

  f32x16 O[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) O[db][i] = 0.f;
  float mrow = ninf, lrow = 0.f;
  const float c = a.scale_log2;
  const int m_wave_lo = pos0 + t0 + wave * 32;
  const int m_wave_hi = pos0 + min(t0 + wave * 32 + 32, a.n_q) - 1;

  // ---- tile movers: direct global->LDS loads into a layout that the transposing reads like (see the wide kernel).
  // Rows past the last needed key repeat that key; zero_past() then clears their V rows. ----
  constexpr int kRows = 16;                                   // tile rows one load of the whole workgroup covers
  const uint32_t lds_base = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int ld_row = 4 * wave + (lane >> 4), ld_pos = lane & 15;
  const int ld_ck = ld_pos ^ (ld_row & 15);
  const int ld_cv = ((((ld_pos >> 1) ^ (2 * (ld_row & 3))) << 1) | (ld_pos & 1));
  uint32_t off_k[4], off_v[4];                                // of a tile that lies wholly inside the keys
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    off_k[j] = (uint32_t)(((int64_t)(kRows * j + ld_row) * a.row_stride + ld_ck * 8) * 2);
    off_v[j] = (uint32_t)(((int64_t)(kRows * j + ld_row) * a.row_stride + ld_cv * 8) * 2);
  }
  auto load_tile = [&](int n0, int buf) __attribute__((always_inline)) {
    if (n0 + kPfK - 1 <= m_hi) {
      const unsigned char* const kb = reinterpret_cast<const unsigned char*>(Kg + (int64_t)n0 * a.row_stride);
      const unsigned char* const vb = reinterpret_cast<const unsigned char*>(Vg + (int64_t)n0 * a.row_stride);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t dst = lds_base + buf * kPfTileBytes + (j < 4 ? 0 : kPfTileBytes / 2) + ((j & 3) * 4 + wave_s) * 1024;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(j < 4 ? off_k[j & 3] : off_v[j & 3]),
                     "s"(j < 4 ? kb : vb) : "memory", "m0");
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int n = min(n0 + kRows * (j & 3) + ld_row, m_hi);
      const uint16_t* src = (j < 4 ? Kg + ld_ck * 8 : Vg + ld_cv * 8) + (int64_t)n * a.row_stride;
      const uint32_t dst = lds_base + buf * kPfTileBytes + (j < 4 ? 0 : kPfTileBytes / 2) + ((j & 3) * 4 + wave_s) * 1024;
      // (assembly: through the intrinsic every later LDS read would wait for all outstanding direct loads)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory", "m0");
    }
  };
  auto loads_landed = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
  auto zero_past = [&](int n0, int buf) __attribute__((always_inline)) {      // a masked probability is 0, and 0 * inf is not
    for (int i = tid; i < kPfK * 16; i += kPfThreads)
      if (n0 + (i >> 4) > m_hi) *reinterpret_cast<u32x4*>(smem + buf * kPfTileBytes + kPfTileBytes / 2 + i * 16) = (u32x4){0u, 0u, 0u, 0u};
  };
  const int rd_k = r * 256, rd_kx = (g ^ (r & 15)) << 4;
  const int rd_j = lane & 15;
  const int rd_v = kPfTileBytes / 2 + (4 * g + (rd_j >> 2)) * 256 + 8 * (rd_j & 3);
  const int rd_vx = (((lane >> 4) & 1) ^ (2 * (rd_j >> 2))) << 5;
  auto read_k = [&](const unsigned char* tile, int kb, int kk) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(tile + kb * 8192 + rd_k + ((kk << 5) ^ rd_kx));
  };
  auto read_v = [&](const unsigned char* tile, int kb, int tt, int db) __attribute__((always_inline)) {
    const unsigned char* p0 = tile + rd_v + (kb * 32 + 16 * tt) * 256 + ((db << 6) ^ rd_vx);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0 + 8 * 256));
    return __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  // ---- one key tile: S^T = K Q^T, online softmax, O^T += V^T P^T -----------------------------------
  auto compute_tile = [&](int buf, int n0) {
    const unsigned char* tile = smem + buf * kPfTileBytes;
    f32x16 S[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) S[kb][i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        S[kb] = mfma32<F16>(read_k(tile, kb, kk), qreg[kk], S[kb]);
      }
    }
    // interior tiles (every key visible to every query of the wave) skip the mask arithmetic
    const bool edge = (n0 + kPfK - 1 > m_wave_lo) || (n0 <= m_wave_hi - a.window);
    if (edge) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int n = n0 + kb * 32 + (i >> 2) * 8 + g * 4 + (i & 3);
          bool ok = qok && n <= m;
          ok = ok && (n < a.sink || n > m - a.window);
          S[kb][i] = ok ? S[kb][i] : ninf;
        }
      }
    }
    u32x4 va[4];                                             // the first PV operands arrive under the softmax
#pragma unroll
    for (int db = 0; db < 4; ++db) va[db] = read_v(tile, 0, 0, db);
    float s0[16], s1[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) { s0[i] = S[0][i]; s1[i] = S[1][i]; }
    float mx = max_nn(max16_nn(s0), max16_nn(s1));
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = max_nn(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    const float mnew = fmaxf(mrow, mx);
    uint32_t P[2][8];
    if (mnew == ninf) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 8; ++i) P[kb][i] = 0u;
    } else {
      const float mc = mnew * c;
      float lsum = 0.f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
          const float p0 = fast_exp2(fmaf(S[kb][i], c, -mc));
          const float p1 = fast_exp2(fmaf(S[kb][i + 1], c, -mc));
          lsum += p0 + p1;
          P[kb][i >> 1] = pack16<F16>(p0, p1);
        }
      }
      const float corr = fast_exp2((mrow - mnew) * c);     // 1 where the maximum did not move
      lrow = lrow * corr + lsum;
      if (__ballot(mnew > mrow) != 0ull) {                   // rescale only when some query's maximum grew
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) O[db][i] *= corr;
      }
      mrow = mnew;
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const u32x4 pb = (u32x4){P[kb][4 * tt], P[kb][4 * tt + 1], P[kb][4 * tt + 2], P[kb][4 * tt + 3]};
#pragma unroll
        for (int db = 0; db < 4; ++db) {
          const u32x4 v = va[db];
          if (kb * 2 + tt < 3) va[db] = read_v(tile, (kb * 2 + tt + 1) >> 1, (tt + 1) & 1, db);
          O[db] = mfma32<F16>(v, pb, O[db]);
        }
      }
    }
  };

  {
    // Software pipeline: the loads of the group's next tile are in flight while this one is computed from the other buffer.
    // (Steps are counted alike in both groups: the barriers are the workgroup's.)
    const int steps = (n_tiles + GROUPS - 1) / GROUPS;
    auto tile_of = [&](int i) { return i * GROUPS + grp; };
    auto tile_n0 = [&](int i) { const int it = it_lo + i; return (it < ks_end ? it : kt_w0 + (it - ks_end)) * kPfK; };
    auto landed = [&](int i) __attribute__((always_inline)) {        // publishes the tiles of step i
      loads_landed();
      __syncthreads();
      const int n0 = tile_n0(tile_of(i));
      // (the last tile alone, in the last step)
      if (GROUPS == 1 ? n0 + kPfK - 1 > m_hi : i == steps - 1) {
        if (tile_of(i) < n_tiles) zero_past(n0, i & 1);
        __syncthreads();
      }
    };
    if (tile_of(0) < n_tiles) load_tile(tile_n0(tile_of(0)), 0);
    if (n_tiles > 0) landed(0);
    for (int i = 0; i < steps; ++i) {
      if (tile_of(i + 1) < n_tiles) load_tile(tile_n0(tile_of(i + 1)), (i + 1) & 1);
      if (GROUPS == 1 || tile_of(i) < n_tiles) compute_tile(i & 1, tile_n0(tile_of(i)));
      if (i + 1 < steps) landed(i + 1);
    }
  }
  if constexpr (GROUPS == 2) {
    // group 1 leaves its state, register by register, in the tile buffers; group 0 goes on with both
    __syncthreads();
    float* const sh = reinterpret_cast<float*>(smem_all) + tid;
    if (grp == 1) {
      sh[0] = mrow;
      sh[kPfThreads] = lrow;
#pragma unroll
      for (int i = 0; i < 64; ++i) sh[(2 + i) * kPfThreads] = O[i >> 4][i & 15];
    }
    __syncthreads();
    if (grp == 1) return;
    const float m1 = sh[0], l1 = sh[kPfThreads], mnew = fmaxf(mrow, m1);
    if (mnew != ninf) {
      const float c0 = fast_exp2((mrow - mnew) * c), c1 = fast_exp2((m1 - mnew) * c);
      lrow = lrow * c0 + l1 * c1;
#pragma unroll
      for (int i = 0; i < 64; ++i) O[i >> 4][i & 15] = O[i >> 4][i & 15] * c0 + sh[(2 + i) * kPfThreads] * c1;
      mrow = mnew;
    }
  }

  // ---- normalise and store ----
  const float ltot = lrow + __shfl_xor(lrow, 32);
  if (!qok) return;
  if (GROUPS == 2 && a.n_splits > 1) {
    float* prow = a.part + (((int64_t)split * a.n_heads + blockIdx.x) * a.n_q + t) * kPfPart;
    if (g == 0) { prow[0] = mrow; prow[1] = ltot; prow[2] = 0.f; }
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        *reinterpret_cast<float4*>(prow + 4 + db * 32 + i4 * 8 + g * 4) =
            make_float4(O[db][i4 * 4], O[db][i4 * 4 + 1], O[db][i4 * 4 + 2], O[db][i4 * 4 + 3]);
    return;
  }
  const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
  uint16_t* orow = a.out + qrow;
#pragma unroll
  for (int db = 0; db < 4; ++db) {
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const u32x2 w = (u32x2){pack16<F16>(O[db][i4 * 4] * inv, O[db][i4 * 4 + 1] * inv),
                              pack16<F16>(O[db][i4 * 4 + 2] * inv, O[db][i4 * 4 + 3] * inv)};
      *reinterpret_cast<u32x2*>(orow + db * 32 + i4 * 8 + g * 4) = w;
    }
  }
  if (a.lse && g == 0) {
    a.lse[((int64_t)b * a.n_q + t) * a.n_q_heads + h] = ltot > 0.f ? mrow * a.scale + logf(ltot) : ninf;
  }
}

// ---- per-query top-p threshold search (selecting mode of rtp_sparse_attn_prefill) ---------------------
// Sec. 3.2, S = Top-P(s(m, .), p), applied to every prefill query over its causal candidates n <= m.
//
// 32 queries of one retrieval head form a group, whose waves sweep the index keys 0..m up to four times:
// sweep 0 finds the row maximum M; sweeps 1-3 histogram the softmax mass over the integer
// q = floor(min((M - s) * 2^17, 2^21 - 1)) one base-128 digit at a time (all candidates in sweep 1, only
// the members of the digit prefix found so far in sweeps 2 and 3) and scan the histogram from the top of
// the score range for the bin where the cumulative mass reaches p * Z.  The index-score tile of 32 keys
// x 32 queries is ONE MFMA (K = 16) in the transposed layout, so a lane holds 16 keys of its own query.
//
// What makes the sweeps cheap:
//  - index keys are fetched kSelRing tiles ahead into registers, through a scalar base address;
//  - interior tiles (every key a candidate of every query of the wave) carry no mask arithmetic;
//  - the histogram of a group is laid out [bin][query]: the 32 queries of a wave sit in 32 different
//    LDS bank pairs whatever their bins, so an fp64 LDS atomic of the wave sees only the two-way
//    conflict between the two lanes of one query;
//  - q is a monotone function of the raw MFMA product x (s = x * index_scale), so "q lies in the digit
//    prefix" is an interval of x.  Its two end points are found once per query and sweep by bisection
//    over the float bit patterns, evaluating the very expression that defines q -- the comparisons of
//    sweeps 2, 3 and of the attention kernel are then exact restatements of that definition, and only members
//    do any further arithmetic;
//  - sweep 0 records the largest product of the group in every pair of key tiles, and sweeps 2 and 3 -- whose
//    members all lie at or above a known bound -- pass over the pairs that cannot hold one.
// t = M - x * index_scale as ONE fused operation (one rounding): the definition every sweep, the end points
// of the digit intervals and the final threshold share
__device__ __forceinline__ float sel_t(float M, float x, float index_scale) { return __builtin_fmaf(-x, index_scale, M); }

// Smallest float x (as a raw product) with sel_t(M, x) < bound; -inf if every finite x qualifies.
// sel_t is non-increasing in x, so the predicate flips once from false to true.  The exact-arithmetic solution is an
// ulp or two of the larger operand away from the flip: a probe on either side of it usually leaves three or four
// bisection steps of the 32 (a probe only ever narrows the bracket, so a poor guess costs time and nothing else).
__device__ __forceinline__ float sel_first_below(float M, float index_scale, float bound) {
  if (bound == __builtin_huge_valf()) return -__builtin_huge_valf();
  uint32_t lo = float_key(-__builtin_huge_valf()), hi = float_key(__builtin_huge_valf());
  auto probe = [&](uint32_t k) {
    if (sel_t(M, key_float(k), index_scale) < bound) hi = k; else lo = k + 1;
  };
  const float guess = (M - bound) / index_scale, off = fmaxf(fabsf(M), bound) * 0x1p-21f / index_scale;
  if (fabsf(guess) < 1e30f) {
    const uint32_t below = float_key(guess - off), above = float_key(guess + off);
    if (below > lo && below < hi) probe(below);
    if (above > lo && above < hi) probe(above);
  }
  while (lo < hi) probe(lo + ((hi - lo) >> 1));
  return key_float(lo);
}

// A workgroup is the eight waves of one group, which split its key range between them; 128 vector registers and 80 KB of
// LDS let two workgroups share a compute unit (of a launch that leaves it one, some have sixteen waves): four waves per SIMD (3.5 on average, by the counters) issue under each other's latencies (with two, 221 registers and loads two rounds of eight tiles ahead, the search
// took 23.7 ms on the last 8192-query chunk of a 1,048,576-token context, 18.4 to 19.5 now; the same code held to 128
// registers 19.4).  The waves add into ONE histogram (LDS atomics; 32 KB); the per-lane member
// lists of sweeps 2 and 3 are emptied when a half tile might overrun one.  All waves meet at
// barriers around every scan, so the phases are uniform over the workgroup.
// What bounds the sweeps there: sweep 0 (1.9 ms, was 2.4) and sweep 3 their vector instructions per tile; sweep 1
// (7.4, was 9.3) the LDS atomics -- an fp64 one holds the compute unit's LDS for 8.6 cycles, i.e. 34 per SIMD and wave of
// 64 pairs, as many as its seven vector instructions take --; sweep 2 the LDS stores (4.6 cycles
// each whatever the number of lanes) and draining the lists.  Over every tile sweeps 2 and 3 take 6.3 and 2.0 ms, over the tiles that the regrouped
// queries of that chunk leave them (see below) 3.4 and 1.9 as launches of their own.  Skipping the stores of the pairs without a member by a
// branch measured slower (7.5 ms over every tile); one store of a table entry per round of sweeps 2 and 3 gave 0.4 %, which the runs of one side differ by.
// One group per workgroup: when a few queries of a chunk have their threshold deep in the
// background while the others' sweeps 2 and 3 visit a handful of tiles, short workgroups let the dispatcher even
// the load out.
// A chunk of few groups leaves most of the chip idle that way (333 queries of 4 heads: 44 workgroups, 0.88 ms at 128K
// tokens).  Then the search runs as five launches with n_slice workgroups per group, each sweeping a slice of the
// group's keys: STEP = 0 .. 3 are the sweeps -- a launch first scans what the slices of the launch before left
// (maxima, histograms as running sums: plain stores and sums in slice order, no atomics), the same in every slice -- and
// kSelFinish scans the last histogram; the kernel boundaries are the only synchronisation.  Every sum has the same
// terms as in one workgroup, in fp64.  0.88 -> 0.19 ms there (0.20 with whole histograms added up by every slice: 32 KB times
// the slices, twice; sweeps 2 and 3 with their scans 61.7 -> 57.5 and 47.1 -> 43.1 us).  (A group with a query whose threshold lies in the open-ended
// bin, see below, leaves that form: its sweeps 0 and 1 are thrown away and one workgroup of the last launch searches it as a whole.)
//
// A threshold inside the open-ended last coarse bin (candidates 15.875 or more below the row maximum) is not
// taken as "keep everything": the workgroup repeats sweep 1 with the reference lowered by 15.875 for the queries
// concerned -- the mass above that bin is already known, the bin's members are spread over 128 new coarse bins --
// until the threshold bin is an ordinary one (or 24 rounds, about 380 score units, are used up).
//
// At the limit of 128 registers the forms that run the whole search keep 68 to 84 bytes per lane in scratch, the slices of sweep 3
// eight: addresses and ends of ranges that are stored before a sweep and read back at the start of the next one or behind it, none of it inside
// the loops over tiles.
constexpr int kSelThreads = 512;
constexpr int kSelThreadsFew = 1024;               // alone on its compute unit, keys for more than kSelFewRounds rounds of
constexpr int kSelFewRounds = 90;                  // 32 * kSelRing: see rtp_sparse_attn_prefill
constexpr float kSelLumpT = 15.875f;               // (kSelBins - 1) / 8: where the open-ended bin starts
constexpr double kSelLumpScale = 7843180.797657975;   // exp(15.875)
constexpr int kSelMaxRounds = 24;
// STEP of prefill_select_kernel beside the sweeps 0 .. 3: the whole search; its end after sliced sweeps; the first digit of whole
// rows, and of sliced ones, left to prefill_order_kernel
constexpr int kSelAll = -1, kSelFinish = 4, kSelFirst = 5, kSelScan = 6;

// ---- queries regrouped by how much they keep ----
// A 32-query group of the search's last sweeps and a 256-query tile of the attention launch have to visit every key tile that one
// of their queries keeps a key in.  Where queries that keep a few tokens stand among queries that keep tenths of the context, that
// is nearly every tile for every group.  So, once the first digit of every threshold is known (and with it, from the histogram, about how many candidates
// a query keeps), the queries of a block are brought into the order of that number, in half octaves, those that keep most first, and by position within a class; the
// sweeps behind, the tile lists and the attention launch take them in this order.  Thresholds, kept sets, counts and masses do not depend on it;
// outputs do by the order of fp32 sums and the rounding of probabilities to 16 bits, against a reference from other keys or, where few are kept,
// in two parts.  Share of the key tiles that 256-query tiles visit, by position / regrouped: last 8192 queries of 1M tokens with Zipf
// clusters 0.996 / 0.46, 4096 queries at 128K with clusters of 32 at p = 0.9 and 0.8 0.985 / 0.66 and 0.985 / 0.37, with a few hard
// queries among easy ones 0.18 / 0.064; ten classes per decade or whole octaves instead change little (0.455, 0.48 on the first).
// A block's order is left alone unless, for queries that keep more than 1/64, 1/256 or 1/1024 of the context, a sixteenth of its tiles
// would be spared a query that does: sweep 2 then finds the tiles' maxima as sweep 0 left them, for these groups.  If then none
// or a quarter of them and more keep more than 1/2048, a group's last sweeps are not cut into slices (4096 queries at 128K tokens that all keep a
// sixth: sweeps 2 and 3 640 us in slices, 590 without; one that keeps 800 of 1M among 8191 that keep 20: 670 and 1550).
constexpr int kOrderThreads = 1024;
constexpr int kOrderMax = 8192;                    // queries of a block
constexpr int kOrderClasses = 64;
constexpr int kFewClass = 12;                      // below it: fewer than kFewKept kept
static_assert(kFewKept == 1 << (kFewClass / 2), "half octaves");
__global__ __launch_bounds__(kOrderThreads) void prefill_order_kernel(const PrefillArgs a) {
  constexpr int NW = kOrderThreads / 64, ROUNDS = kOrderMax / kOrderThreads, TILES = kOrderMax / kPwQ;
  __shared__ int at[kOrderClasses][ROUNDS * NW];   // places of a wave's round within a class, then before it
  __shared__ int class_at[kOrderClasses];
  __shared__ uint32_t tile_has[3];                 // which tiles hold a query of a class from here on
  __shared__ int n_hard[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = blockIdx.y, first = blockIdx.x * a.order_block, n = min(a.order_block, a.n_q - first);
  const SelState* const st = a.sl_state + (int64_t)j * a.n_q + first;
  int32_t* const order = a.order + (int64_t)j * a.n_q + first;
  for (int i = tid; i < kOrderClasses * ROUNDS * NW; i += kOrderThreads) (&at[0][0])[i] = 0;
  for (int i = tid; i < (n + kPwQ - 1) / kPwQ; i += kOrderThreads) a.act_count[(int64_t)j * ((a.n_q + kPwQ - 1) / kPwQ) + first / kPwQ + i] = 0;
  if (tid < 4) { if (tid < 3) tile_has[tid] = 0; n_hard[tid] = 0; }
  __syncthreads();
  const float keys = (float)(a.q_start_host + first + n);
  int cls[ROUNDS], rank[ROUNDS];
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k) {
    if (k * kOrderThreads >= n) break;                             // (the same for the whole workgroup)
    const int i = k * kOrderThreads + tid;
    const bool on = i < n;
    cls[k] = on ? kOrderClasses - 1 - (st[i].flags >> kSelClassShift) : kOrderClasses - 1;      // (the class that keeps most comes first)
    uint64_t same = __ballot(on);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
      const uint64_t bit = __ballot((cls[k] >> b) & 1);
      same &= (cls[k] >> b) & 1 ? bit : ~bit;
    }
    rank[k] = __popcll(same & ((1ull << lane) - 1ull));
    if (on && rank[k] == 0) at[cls[k]][k * NW + wave] = __popcll(same);
#pragma unroll
    for (int q = 0; q < 3; ++q) {                                  // 1/64, 1/256, 1/1024 of the context
      const float least = 2.f * (__builtin_amdgcn_logf(keys) - (6.f + 2.f * q));
      const uint64_t hard = __ballot(on && (float)(kOrderClasses - 1 - cls[k]) >= least);
      if (lane == 0 && hard != 0ull) {
        atomicOr(&tile_has[q], 1u << (i / kPwQ));
        atomicAdd(&n_hard[q], __popcll(hard));
      }
    }
    const uint64_t deep = __ballot(on && (float)(kOrderClasses - 1 - cls[k]) >= 2.f * (__builtin_amdgcn_logf(keys) - 11.f));
    if (lane == 0 && deep != 0ull) atomicAdd(&n_hard[3], __popcll(deep));
  }
  __syncthreads();
  const int n_tiles = (n + kPwQ - 1) / kPwQ;
  bool on = false;
#pragma unroll
  for (int q = 0; q < 3; ++q) on = on || 16 * (__popc(tile_has[q]) - (n_hard[q] + kPwQ - 1) / kPwQ) >= n_tiles;
  if (tid == 0) a.order_on[j * gridDim.x + blockIdx.x] = on ? kOrderByKept : n_hard[3] > 0 && 4 * n_hard[3] < n ? kOrderOwn : kOrderOwnAlike;
  if (!on) {                                                        // (the same for the whole workgroup)
    for (int i = tid; i < n; i += kOrderThreads) order[i] = first + i;
    return;
  }
  // sixteen threads go through a class, eight entries each
  constexpr int PER = ROUNDS * NW / 16;
  static_assert(kOrderThreads == 16 * kOrderClasses && PER * 16 == ROUNDS * NW && TILES <= 32, "one run of entries per thread, one bit per tile");
  {
    const int c = tid >> 4, e0 = (tid & 15) * PER;
    int sum = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) sum += at[c][e0 + e];
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int up = __shfl_up(incl, o, 16);
      if ((tid & 15) >= o) incl += up;
    }
    int run = incl - sum;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int v = at[c][e0 + e];
      at[c][e0 + e] = run;
      run += v;
    }
    if ((tid & 15) == 15) class_at[c] = incl;
  }
  __syncthreads();
  if (wave == 0) {
    const int v = class_at[lane];
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o);
      if (lane >= o) incl += up;
    }
    class_at[lane] = incl - v;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k) {
    const int i = k * kOrderThreads + tid;
    if (i < n) order[class_at[cls[k]] + at[cls[k]][k * NW + wave] + rank[k]] = first + i;
  }
}

// Least and greatest of 32 positions, lane and lane ^ 32 holding the same one.
__device__ __forceinline__ void position_range(int m, int& lo, int& hi) {
  lo = hi = m;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) {
    lo = min(lo, __shfl_xor(lo, o));
    hi = max(hi, __shfl_xor(hi, o));
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  hi = __builtin_amdgcn_readfirstlane(hi);
}

template <int STEP, int THREADS = kSelThreads, bool ORDERED = false>
__global__ __launch_bounds__(THREADS, 4) void prefill_select_kernel(const PrefillArgs a) {
  constexpr bool kSliced = STEP >= 0 && STEP < kSelFinish;             // this launch sweeps a slice of the group's keys
  constexpr bool kWhole = STEP == kSelAll || STEP == kSelFinish;       // ... or can run the whole search
  constexpr int NW = THREADS / 64;                             // waves of the workgroup
  // (the sweeps of a sliced search that stay with their slices' keys for a few rounds only are quicker with the short one: 333 queries
  // behind 131072 tokens, sweeps 1 and 2 60.2 and 55.2 us against 61.9 and 56.3)
  constexpr int RING = STEP == 0 || STEP == kSelFirst || (ORDERED && kSliced) ? kSelRingWide : kSelRing;
  __shared__ double hist[kSelBins][32];                            // 32 KB
  __shared__ float list_all[NW][kSelListCap][64];                  // per-lane member lists of sweeps 2 and 3 (48 KB)
  float (*max_all)[32] = reinterpret_cast<float (*)[32]>(&list_all[0][0][0]);   // sweep 0: the waves' row maxima
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (tile numbers are scalars)
  const int g = lane >> 5, r = lane & 31;
  // Workgroups go round-robin over the chip's 8 dies, each with its own L2.  The 1-D grid is decoded so
  // that a die works on ONE head (8 / n_heads dies per head): all its waves then stream the same index
  // keys and meet in that L2.
  int j, qtile;
  const int n_qtiles = (a.n_q + 31) / 32;
  const int n_slice = kSliced ? a.n_slice : 1;
  if (a.n_heads <= 8 && 8 % a.n_heads == 0) {
    const int per_head = 8 / a.n_heads;                            // dies per head
    const int die = blockIdx.x & 7, k = blockIdx.x >> 3;
    j = die / per_head;
    qtile = k * per_head + die % per_head;
  } else {
    j = blockIdx.x % a.n_heads;
    qtile = blockIdx.x / a.n_heads;
  }
  if (kWhole && blockIdx.x == 0 && tid == 0) {                     // for prefill_active_tiles_kernel, which runs next
    a.act_range[0] = 0;
    a.act_range[1] = 0x7fffffff;
  }
  if (qtile >= n_qtiles * n_slice) return;                         // (the whole workgroup)
  int slice = qtile / n_qtiles;
  if (ORDERED && (int)gridDim.x <= a.one_round) {
    // one round of two workgroups per compute unit: all slices of what keeps most first, and the second half in reverse, so that the second workgroup
    // of a compute unit has the less to do the more the first one has
    const int n_here = n_qtiles * n_slice, half = (n_here + 1) / 2;
    if (qtile >= half) qtile = n_here - 1 - (qtile - half);
    slice = qtile % n_slice;
    qtile /= n_slice;
  } else {
    qtile -= slice * n_qtiles;
  }
  // first query of the group; long rows first, or what keeps most
  const int t0 = (ORDERED ? qtile : n_qtiles - 1 - qtile) * 32;
  const int pos0 = (int)a.q_start_host;
  // The lanes past the last query of a partial group repeat that query (their results are not stored): every lane
  // then has a causal range that ends where its group's does, and the group's interior tiles need no mask.  (Masking
  // those lanes instead puts the whole range of a partial group on the masked path of one wave: the search takes 10.7 against 0.9 ms
  // for a chunk of 333 queries behind 131072 tokens.)
  const bool qok = t0 + r < a.n_q;
  int t = min(t0 + r, a.n_q - 1);
  if (ORDERED) t = a.order[(int64_t)j * a.n_q + t];
  const int m = pos0 + t;
  const float ninf = -__builtin_huge_valf(), pinf = __builtin_huge_valf();
  const float cs = a.index_scale;
  const uint16_t* kIg = a.kI + (int64_t)j * a.kI_head_stride;
  const u32x4 qIreg = *reinterpret_cast<const u32x4*>(a.qI + ((int64_t)j * a.n_q + t) * kIndexDim + g * 8);
  const int n_rows = pos0 + a.n_q;                                 // index-key rows that exist
  int m_lo = pos0 + t0;
  int m_hi = pos0 + min(t0 + 32, a.n_q) - 1;
  // whether the table holds the group's maxima; where its queries were brought together after sweep 0, sweep 2 makes its row
  bool own_table = true;
  int order_mode = kOrderOwn;
  if (ORDERED) {
    position_range(m, m_lo, m_hi);
    order_mode = a.order_on[j * ((a.n_q + a.order_block - 1) / a.order_block) + t0 / a.order_block];
    own_table = order_mode != kOrderByKept;
  }
  const int n_tiles = m_hi / 32 + 1;
  const int n_interior = (m_lo + 1) / 32;                          // tiles with nb + 31 <= m_lo
  float (*lst)[64] = list_all[wave];
  // this group's row of the tile-maximum table: written in sweep 0 (one entry per pair of key tiles, i.e. per 64
  // keys), read in sweeps 2 and 3, whose members all lie at or above x_lo -- a tile pair whose maximum is below
  // every query's x_lo holds none.  Sweep 3 replaces the entries of the pairs it visits by +inf (some query of
  // the group has a product at or above its own x_lo there, so it may keep a key) or -inf (none can); the pairs
  // it skips keep a maximum below every x_lo.  The attention launch's tile lists are built from the result.
  float* tmx = a.tile_max + ((int64_t)j * ((a.n_q + 31) / 32) + t0 / 32) * a.n_t64;
  float xlo_wave = ninf;            // smallest x_lo over the wave's queries
  float xlo_wave_top = ninf;        // and the largest
  bool reach_known = false;         // sweep 3: the tile in hand is certain to hold a product at or above its query's x_lo
  bool kept_much = false;           // regrouped queries that keep so much that few pairs will be without a kept key
  int n_looked = 0, n_needed = 0;   // sweep 3 (and 2, if it makes the table): tile pairs whose reach was worked out, and those found within reach
  int lcnt = 0;                     // entries in this lane's member list
  const uint32_t lst_base = (uint32_t)(size_t)(__attribute__((address_space(3))) float*)&lst[0][lane];

  auto load_k = [&](int tile) __attribute__((always_inline)) {
    const int nrow = min(tile * 32 + r, n_rows - 1);               // rows past the chunk are causally masked anyway
    return *reinterpret_cast<const u32x4*>(kIg + (int64_t)nrow * kIndexDim + g * 8);
  };
  // the same for a tile of the mask-free range, all of whose rows exist (what is fetched ahead past the last whole tile
  // is not used): a scalar base and one lane offset, no vector arithmetic
  const uint32_t k_lane = (uint32_t)(r * kIndexDim + g * 8) * 2u;
  const int last_whole = n_rows / 32 - 1;
  auto load_k_whole = [&](int tile) __attribute__((always_inline)) {
    const unsigned char* base = reinterpret_cast<const unsigned char*>(kIg) + (int64_t)min(tile, last_whole) * (32 * kIndexDim * 2);
    return *reinterpret_cast<const u32x4*>(base + k_lane);
  };
  // the group's waves clear their histogram together (followed by a barrier at the call sites)
  auto zero_hist = [&]() __attribute__((always_inline)) {
    double* h = &hist[0][0];
    for (int i = tid; i < kSelBins * 32; i += THREADS) h[i] = 0.0;
  };
  // One candidate's mass into bin `bin` of this lane's query.
  auto add_mass = [&](int bin, float tt) __attribute__((always_inline)) {
    const float wgt = fast_exp2(tt * -1.4426950408889634f);        // exp(s - M)
    atomicAdd(&hist[bin][r], (double)wgt);
  };

  float selM = ninf;                // the query's reference: its row maximum, lowered by 15.875 per repeat of sweep 1
  float selM8 = ninf;               // 8 * selM and 8 * index_scale for sweep 1
  const float cs8 = cs * 8.0f;
  float x_lo = ninf, x_top = pinf;  // sweeps 2, 3: members of the prefix have x_lo <= x <= x_top
  float x_max = ninf;               // the row's largest raw product
  float x_mid = 0.f, x_half = 0.f;  // sweep 3: middle of [x_lo, min(x_top, x_max)] and the larger distance of its ends from it
  int shift = 0;
  float mx_lane = ninf;             // sweep 0: the lane's largest product

  // Weighs the listed members of every lane: lane-private lists, so the only cross-lane step is the loop bound.
  // Four entries at a time: their reads, exponentials and atomics overlap (one by one, a drain is a chain of LDS round
  // trips that costs a wave more than the pairs between two drains).
  auto drain_list = [&]() __attribute__((always_inline)) {
#pragma unroll 1
    for (int k = 0; __ballot(k < lcnt) != 0ull; k += 4) {
      float x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = lst[k + u][lane];          // (the capacity is a multiple of 4; what lies past the end is not used)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (k + u < lcnt) {
          const float tt = sel_t(selM, x[u], cs);
          add_mass((sel_q_of_t(tt) >> shift) & (kSelBins - 1), tt);
        }
      }
    }
    lcnt = 0;
  };

  // Stores x at the LDS address `end` and advances it, in the lanes whose median equals x.
  auto append_if_member = [](uint32_t& end, float x, float median) __attribute__((always_inline)) {
    uint64_t lanes;
    asm volatile("s_mov_b64 %1, exec\n\tv_cmpx_eq_f32_e64 exec, %2, %3\n\tds_write_b32 %0, %2\n\tv_add_u32_e32 %0, 0x100, %0\n\t"
                 "s_mov_b64 exec, %1"
                 : "+v"(end), "=&s"(lanes) : "v"(x), "v"(median) : "memory");
  };

  // What one tile contributes in phase PH (0: maximum, 1: all candidates -- of a repeated sweep 1: those at or below
  // the lowered reference --, 2 / 3: members of the digit prefix): SI = its 32 x 32 index products, nb = its first
  // key.  MASKED: causality and the lowered reference are tested pair by pair.
  float t_least = ninf;             // masked sweep 1: candidates have 8 (M - s) >= t_least
  auto tile_work = [&](auto PH, auto MASKED, const f32x16& SI, int nb) __attribute__((always_inline)) -> float {
    constexpr int phase = decltype(PH)::value;
    constexpr bool masked = decltype(MASKED)::value;
    if (phase == 0) {
      // scaling by a positive constant is monotone, so the maximum is taken on the raw products
      float v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int n = nb + (i >> 2) * 8 + g * 4 + (i & 3);
        v[i] = (!masked || n <= m) ? SI[i] : ninf;
      }
      return max16_nn(v);
    } else if (phase == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int n = nb + (i >> 2) * 8 + g * 4 + (i & 3);
        // 8 * (M - x * scale) straight from 8 M and 8 * scale: scaling by a power of two commutes with both
        // roundings, so this IS 8 * sel_t(M, x, scale), one multiplication less per pair
        float tt8 = sel_t(selM8, SI[i], cs8);
        // a repeated sweep takes the candidates at or below the lowered reference only (the others were
        // counted above the open-ended bin); a query that does not repeat has reference -inf and takes none.  What is left
        // out adds a weight of zero to the last bin: no branch per pair
        if (masked) tt8 = n <= m && tt8 >= t_least ? tt8 : 1e9f;
        // first digit of q: floor(min(tt * 2^17, 2^21 - 1)) >> 14 == floor(min(tt * 8, (2^21 - 1) / 2^14))
        const int bin = (int)fminf(tt8, 127.99993896484375f);
        // exp(s - M) = exp2(tt * -log2(e)); the constant carries the 1/8, again exactly
        atomicAdd(&hist[bin][r], (double)fast_exp2(tt8 * -0.18033688011112042f));
      }
    } else {
      // Members of the digit prefix (about one pair in a hundred in sweep 2, one in ten thousand in
      // sweep 3) are only noted here -- their raw product goes to the lane's list -- and weighed
      // with all lanes busy (drain_list); weighing them where they turn up would run the exponential
      // and the atomic for one or two active lanes at a time.
      // Membership x_lo <= x <= x_top is one median and one comparison, which switches the other lanes off for the
      // store at the list's end and the step of the end: three vector instructions per pair.
      // MASKED: a key that the query does not see is taken as -inf, which no finite lower end lets in.
      float v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int n = nb + (i >> 2) * 8 + g * 4 + (i & 3);
        v[i] = (!masked || n <= m) ? SI[i] : ninf;
      }
      const float lo = masked ? fmaxf(x_lo, -3.4028234663852886e38f) : x_lo;
      bool go = true;
      float reach = 0.f;
      if (phase == 3) {
        // does any lane have a member in this tile?  Its products' smallest distance from the middle of the lane's
        // range says so, one and a half vector instructions per pair (rounding is monotone, so a member is
        // never further away than the range's ends as subtracted the same way; a tile let through for nothing is harmless)
        float d = pinf;
#pragma unroll
        for (int i = 0; i < 16; i += 2) d = fminf(fminf(fabsf(v[i] - x_mid), fabsf(v[i + 1] - x_mid)), d);
        go = __ballot(d <= x_half) != 0ull;
        // can some query of the wave keep a key of this tile?  Its final threshold is at or above x_lo, so a
        // tile whose largest visible product is below x_lo for every query holds no kept pair
        reach = 1.f;
        if (!reach_known) reach = __ballot(max16_nn(v) >= x_lo) != 0ull ? 1.f : 0.f;
      } else if (ORDERED && !reach_known) {
        go = __ballot(max16_nn(v) >= x_lo) != 0ull;
        reach = go ? 1.f : 0.f;
      }
      if (go) {
        // A half tile adds at most 8 entries, so the lists are emptied when some lane has no room for 8 more.  The list's
        // end travels as an LDS address.
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          if (__ballot(lcnt > kSelListCap - 8) != 0ull) drain_list();
          uint32_t end = lst_base + (uint32_t)lcnt * 256u;
#pragma unroll
          for (int i = hf * 8; i < hf * 8 + 8; ++i) append_if_member(end, v[i], __builtin_amdgcn_fmed3f(v[i], lo, x_top));
          lcnt = (int)((end - lst_base) >> 8);
        }
      }
      return reach;
    }
    return 0.f;
  };

  // Sweep 0: the maxima of a round's tile pairs over the wave's 32 queries x 64 keys, to the table.  The pairs share the steps across
  // lanes: the halves of two are swapped into one register, the rows of two such into one, then four steps inside the rows.
  auto swapped = [](float a, float b) __attribute__((always_inline)) {
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return max_nn(__uint_as_float(x[0]), __uint_as_float(x[1]));
  };
  auto pair_maxima = [&](const float (&top)[RING / 2], float* to) __attribute__((always_inline)) {
    float x = swapped(top[0], top[1]);                             // lanes 0 .. 31: of pair 0, the others: of pair 1
    int at = lane >> 5;
    if constexpr (RING == 8) {
      const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(swapped(top[2], top[3])), false, false);
      x = max_nn(__uint_as_float(y[0]), __uint_as_float(y[1]));    // rows of 16 lanes: pairs 0, 2, 1, 3
      at = (lane >> 5) | ((lane >> 3) & 2);
    }
#define RTP_STEP(CTRL) x = max_nn(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true)));
    RTP_STEP(0xB1) RTP_STEP(0x4E) RTP_STEP(0x141) RTP_STEP(0x140)  // quad_perm [1,0,3,2] and [2,3,0,1], row_half_mirror, row_mirror
#undef RTP_STEP
    if constexpr (RING == 4) {
      const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
      x = max_nn(__uint_as_float(y[0]), __uint_as_float(y[1]));
    }
    if ((lane & (RING == 8 ? 15 : 31)) == 0) to[at] = x;
  };

  // One sweep over the tiles [tile_begin, tile_end) in rounds of RING: a round's index-key registers are refilled
  // (for the next round) as soon as its MFMAs have read them, so a load has a round's arithmetic -- of this wave and
  // of the SIMD's three others -- to land in.  No tail test: the mask-free range is a whole number of rounds, and in
  // the masked range a tile past the last one holds only keys n > m, which the causal mask drops.
  // Sweeps 2 and 3 consult the maximum table pair by pair: skip what cannot hold a member, and in sweep 3 note which
  // pairs a query can keep a key in.  no_look: nearly every pair can hold a member and is needed (see sweep_picked);
  // the pairs keep their maxima in the table, which is the conservative answer.
  // Regrouped queries that keep much (kept_much): of 64 pairs the first 8 are looked at, and the others if one of these was not needed.
  auto sweep = [&](auto PH, auto MASKED, int tile_begin, int tile_end, bool no_look = false) __attribute__((always_inline)) {
    if (tile_begin >= tile_end) return;
    constexpr int phase_ = decltype(PH)::value;
    constexpr bool kSkip = phase_ == 2 || phase_ == 3;
    static_assert(kSelMfma == 2, "a batch of MFMAs is one 64-key tile of the maximum table");
    constexpr bool masked_ = decltype(MASKED)::value;
    auto fetch = [&](int tile) { return masked_ ? load_k(tile) : load_k_whole(tile); };
    u32x4 ring[RING];
    float top[RING / 2];                                           // sweep 0: the lanes' maxima of the round's pairs
    float tm[RING / 2];                                        // the table entries of the tile pairs in the ring
#pragma unroll
    for (int u = 0; u < RING; ++u) ring[u] = fetch(tile_begin + u);
    if (kSkip) {
#pragma unroll
      for (int u = 0; u < RING / 2; ++u) tm[u] = tmx[(tile_begin >> 1) + u];
    }
#pragma unroll 1
    for (int first = tile_begin; first < tile_end; first += RING) {
#pragma unroll
      for (int hb = 0; hb < RING; hb += kSelMfma) {            // kSelMfma MFMAs in flight at a time
        // no member possible in this pair of tiles: only the prefetches for the next round are issued
        bool skip = false;
        if (ORDERED && kSkip && kept_much && (((first + hb) >> 1) & 63) == 0) no_look = false;
        if (kSkip) {
          const float pair_max = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(tm[hb / 2])));
          const bool maxima = !ORDERED || own_table;               // (else +-inf, from sweep 2, and nothing before it)
          skip = !no_look && pair_max < xlo_wave && (maxima || phase_ == 3);
          // a maximum at or above EVERY query's x_lo is at or above its own query's: no need to look
          reach_known = no_look || (maxima && (phase_ == 2 || pair_max >= xlo_wave_top));
          tm[hb / 2] = tmx[((first + RING + hb) >> 1)];
        }
        if (skip) {
#pragma unroll
          for (int u = 0; u < kSelMfma; ++u) ring[hb + u] = fetch(first + RING + hb + u);
          continue;
        }
        f32x16 SI[kSelMfma];
#pragma unroll
        for (int u = 0; u < kSelMfma; ++u) {
#pragma unroll
          for (int i = 0; i < 16; ++i) SI[u][i] = 0.f;
          SI[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[hb + u]),
                                                          __builtin_bit_cast(bf16x8, qIreg), SI[u], 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kSelMfma; ++u) ring[hb + u] = fetch(first + RING + hb + u);
        float tmax = ninf;
#pragma unroll
        for (int u = 0; u < kSelMfma; ++u) {
          __builtin_amdgcn_sched_barrier(0);       // one tile at a time: hoisting four tiles' operands runs out of registers
          const float v = tile_work(PH, MASKED, SI[u], (first + hb + u) * 32);
          tmax = phase_ == 0 ? (u == 0 ? v : max_nn(tmax, v)) : fmaxf(tmax, v);
        }
        if (phase_ == 0) {
          mx_lane = max_nn(mx_lane, tmax);
          top[hb / 2] = tmax;
        }
        // the last sweep knows better than the maximum: can one of the wave's queries keep a key of the pair?
        // (a pair known to reach keeps its maximum, which says the same)
        // (and sweep 2 finds the first answer where sweep 0 saw the queries in other groups)
        if ((phase_ == 3 || (ORDERED && phase_ == 2)) && !reach_known) {
          n_looked += 1;
          n_needed += tmax > 0.f ? 1 : 0;
          if (lane == 0) tmx[(first + hb) >> 1] = tmax > 0.f ? pinf : ninf;
          if (ORDERED && kept_much) {
            if ((((first + hb) >> 1) & 63) == 7) no_look = n_needed >= 8;
            if (tmax <= 0.f) n_needed = 0;                         // (here: how many of the last pairs in a row were needed)
          }
        } else if (ORDERED && phase_ == 2 && !own_table) {
          if (lane == 0) tmx[(first + hb) >> 1] = pinf;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (phase_ == 0) pair_maxima(top, tmx + (first >> 1));
    }
  };
  const int n_plain = n_interior / RING * RING;            // whole rounds of interior tiles run without masks
  // this wave's share: an equal run of the rounds, the masked ones of the edge (one or two) at the end
  const int plain_rounds = n_plain / RING, rounds = (n_tiles + RING - 1) / RING;
  // (ORDERED: where the last sweeps will take about equally long everywhere, the rest of a group's search is left to its first workgroup)
  const bool rest_whole = STEP == 2 && ORDERED && order_mode == kOrderOwnAlike && a.order_whole != 0;
  if (rest_whole && slice != 0) return;
  const int share = (rest_whole ? 0 : slice * NW) + wave, shares = (rest_whole ? 1 : n_slice) * NW;
  const int round_lo = (int)((int64_t)rounds * share / shares), round_hi = (int)((int64_t)rounds * (share + 1) / shares);
  const int plain_lo = min(round_lo, plain_rounds) * RING, plain_hi = min(round_hi, plain_rounds) * RING;
  const int edge_lo = max(round_lo, plain_rounds) * RING, edge_hi = round_hi * RING;
  // Sweeps 2 and 3 over the mask-free range, 512 tiles (256 entries of the maximum table) at a time: where at most
  // a quarter of a stretch's tile pairs can hold a member, only those are fetched and looked at, one after the other -- with a
  // peaked score law that is a handful of pairs in a million keys --; otherwise the streaming sweep above runs over the stretch,
  // consulting the table per pair unless that can skip next to nothing and, in sweep 3, nine in ten of the pairs
  // the wave has looked at turned out to hold a product some query can keep (a group with one moderately hard query
  // among easy ones is not such a case: looking tells which pairs that query really keeps a key in).
  auto sweep_picked = [&](auto PH, int tile_begin, int tile_end) __attribute__((always_inline)) {
    constexpr int phase_ = decltype(PH)::value;
#pragma unroll 1
    for (int tb = tile_begin; tb < tile_end; tb += 512) {
      const int te = min(tb + 512, tile_end);
      if (ORDERED && phase_ == 2 && !own_table) {
        sweep(PH, std::false_type{}, tb, te);
        continue;
      }
      auto entry = [&](int k) {
        const int pair = (tb >> 1) + k * 64 + lane;
        return pair < (te >> 1) ? tmx[pair] : ninf;
      };
      int n_on = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) n_on += __popcll(__ballot(entry(k) >= xlo_wave));
      if (4 * n_on > (te - tb) >> 1) {
        // next to nothing to skip, and (sweep 3) the pairs looked at so far nearly all turned out to be needed: do not look
        const bool no_look = (!ORDERED || own_table) && 16 * n_on > 15 * ((te - tb) >> 1) && (phase_ == 2 || (n_looked >= 64 && 10 * n_needed >= 9 * n_looked));
        sweep(PH, std::false_type{}, tb, te, no_look);
        continue;
      }
#pragma unroll 1
      for (int k = 0; k < 4; ++k) {
        const float tmv = entry(k);
        uint64_t todo = __ballot(tmv >= xlo_wave);
        while (todo != 0ull) {
          const int pl = __builtin_ctzll(todo);
          todo &= todo - 1ull;
          const int tile = tb + 2 * (k * 64 + pl);
          reach_known = (!ORDERED || own_table) && (phase_ == 2 || __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tmv), pl)) >= xlo_wave_top);
          f32x16 SI[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int i = 0; i < 16; ++i) SI[u][i] = 0.f;
            SI[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, load_k_whole(tile + u)),
                                                            __builtin_bit_cast(bf16x8, qIreg), SI[u], 0, 0, 0);
          }
          float tmax = ninf;
#pragma unroll
          for (int u = 0; u < 2; ++u) tmax = fmaxf(tmax, tile_work(PH, std::false_type{}, SI[u], (tile + u) * 32));
          if (phase_ == 3 && !reach_known && lane == 0) tmx[tile >> 1] = tmax > 0.f ? pinf : ninf;
        }
      }
    }
  };
  auto sweep_all = [&](auto PH) __attribute__((always_inline)) {
    constexpr int phase_ = decltype(PH)::value;
    if constexpr (phase_ == 2 || phase_ == 3) sweep_picked(PH, plain_lo, plain_hi);
    else sweep(PH, std::false_type{}, plain_lo, plain_hi);
    sweep(PH, std::true_type{}, edge_lo, edge_hi);
    if (phase_ == 2 || phase_ == 3) drain_list();
  };

  double Z = 0.0, above = 0.0;
  int prefix = 0;                 // digits of the threshold found so far
  float sel_mass = 1.f;
  float cut = pinf;               // keep a candidate iff reference - s < cut
  double cum = 0.0, hsel = 0.0;
  int bsel = kSelBins - 1;
  // The threshold bin: this query's bins from the top of the score range (bin 0) down.  The two lanes of the query and
  // every wave of the group take one run of bins each and leave its sum; every one of them then goes through the
  // runs' sums and the bins of the run that crosses, on the same numbers in the same order.  (All of them going through
  // all 128 bins is a chain of LDS reads and additions of 32000 cycles, three times per workgroup.)  One barrier; the
  // sums live in the lists' memory, idle between sweeps.  `whole`: the histogram holds all candidates, take Z from it.
  constexpr int kRuns = kSelThreads / 32, kRunBins = kSelBins / kRuns;
  double (*run_sum)[32] = reinterpret_cast<double (*)[32]>(&list_all[0][0][0]);
  static_assert(kSelBins % kRuns == 0 && sizeof(double) * 32 * kRuns + sizeof(int) * NW <= sizeof(list_all), "runs of equal length");
  // About how many candidates the query keeps: the mass of every bin by the weight of its middle, run by run above the run that crosses.
  float kept_about = 0.f;
  auto count_kept = [&](const double (&rs)[kRuns], double target, auto&& bin_mass) __attribute__((always_inline)) {
    const int run = bsel / kRunBins;
    kept_about = 0.f;
#pragma unroll
    for (int i = 0; i < kRuns; ++i) kept_about += i < run ? (float)rs[i] * fast_exp2(((float)i + 0.5f) * 1.44269504f) : 0.f;
#pragma unroll
    for (int i = 0; i < kRunBins; ++i) {
      const int b = run * kRunBins + i;
      const float share = b < bsel ? 1.f : (b > bsel ? 0.f : fminf((float)((target - cum) / hsel), 1.f));
      kept_about += share * (float)bin_mass(i) * fast_exp2(((float)b + 0.5f) * 0.18033688f);
    }
  };
  auto scan = [&](bool whole, bool take) __attribute__((always_inline)) {
    if (THREADS == kSelThreads || tid < kSelThreads) {
      double h[kRunBins], sum = 0.0;
#pragma unroll
      for (int i = 0; i < kRunBins; ++i) h[i] = hist[(wave * 2 + g) * kRunBins + i][r];
#pragma unroll
      for (int i = 0; i < kRunBins; ++i) sum += h[i];
      run_sum[wave * 2 + g][r] = sum;
    }
    __syncthreads();
    if (!take) return;
    double rs[kRuns];
#pragma unroll
    for (int i = 0; i < kRuns; ++i) rs[i] = run_sum[i][r];
    if (whole) {
      Z = 0.0;
#pragma unroll
      for (int i = 0; i < kRuns; ++i) Z += rs[i];
    }
    const double target = (double)a.p * Z;
    const ThresholdBin t = threshold_bin<kRuns, kRunBins>(above, target, rs, [&](int i) __attribute__((always_inline)) { return hist[i][r]; });
    bsel = t.bin;
    cum = t.above;
    hsel = t.mass;
    if (STEP == kSelFirst) count_kept(rs, target, [&](int i) __attribute__((always_inline)) { return hist[bsel / kRunBins * kRunBins + i][r]; });
  };

  // ---- sweep 0: the row maxima ----
  // (of this workgroup's share of the keys, in every wave)
  auto row_maxima = [&]() __attribute__((always_inline)) {
    sweep_all(std::integral_constant<int, 0>{});
    float mx = fmaxf(mx_lane, __shfl_xor(mx_lane, 32));
    if (g == 0) max_all[wave][r] = mx;
    zero_hist();
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NW; ++k) mx = fmaxf(mx, max_all[k][r]);
    x_max = mx;
    selM = mx * cs;
    __syncthreads();                                                // the maxima are read: the lists' memory is free again
  };
  bool rebased = false;             // the reference is not the row maximum
  // after a scan of sweep 1: is this query's threshold in the open-ended bin?
  auto in_open_bin = [&]() __attribute__((always_inline)) { return bsel == kSelBins - 1 && hsel > 0.0; };
  // the same for any query of the workgroup (flags in the lists' memory, idle in this phase; the barrier also says
  // that every wave has read the histograms)
  auto any_of = [&](bool mine_) __attribute__((always_inline)) {
    int* flags = reinterpret_cast<int*>(reinterpret_cast<double (*)[32]>(&list_all[0][0][0]) + kRuns);
    const bool mine = __ballot(mine_) != 0ull;
    if (lane == 0) flags[wave] = mine ? 1 : 0;
    __syncthreads();
    int any = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) any |= flags[w];
    return any != 0;
  };

  // ---- sweep 1: the first digit; repeated with a lowered reference while some query's threshold lies in the
  // open-ended bin ----
  auto first_digit = [&]() __attribute__((always_inline)) {
    bool repeat_me = false;
    for (int round = 0; round < kSelMaxRounds; ++round) {
      selM8 = (round == 0 || repeat_me) ? selM * 8.0f : ninf;       // (exact unless it overflows)
      if (round == 0) {
        sweep_all(std::integral_constant<int, 1>{});
      } else {
        t_least = 0.f;                                              // (no mask-free form: repeats are rare)
        sweep(std::integral_constant<int, 1>{}, std::true_type{}, plain_lo, plain_hi);
        sweep(std::integral_constant<int, 1>{}, std::true_type{}, edge_lo, edge_hi);
      }
      __syncthreads();                                              // every wave of the group has added its masses
      scan(round == 0, round == 0 || repeat_me);
      // the threshold in the open-ended bin: everything above it is counted (cum), its members go round again
      repeat_me = (round == 0 || repeat_me) && in_open_bin() && round + 1 < kSelMaxRounds;
      if (!any_of(repeat_me)) break;
      if (repeat_me) {
        rebased = true;
        selM -= kSelLumpT;
        Z *= kSelLumpScale;
        above = cum * kSelLumpScale;
      }
      zero_hist();
      __syncthreads();
    }
    prefix = bsel;
    above = cum;
  };

  // ---- sweeps 2 and 3: the second and third digit among the members of the prefix ----
  auto member_range = [&](int phase) __attribute__((always_inline)) {
    // members of the prefix: prefix << shift <= q < (prefix + 1) << shift; for the non-negative
    // tt = M - s of a candidate that is qlo / 2^17 <= tt < qhi / 2^17 (the last bin is open-ended),
    // and in terms of the raw product x: first x with tt < hi bound <= x < first x with tt < lo bound
    shift = 7 * (4 - phase);                                        // of the prefix found so far: 14, then 7
    const int qlo = prefix << shift, qhi = (prefix + 1) << shift;
    const float lo_t = (float)qlo * (1.0f / kSelScale);
    const float hi_t = qhi > kSelQMax ? pinf : (float)qhi * (1.0f / kSelScale);
    x_lo = sel_first_below(selM, cs, hi_t);
    // the largest x that is still a member: the float just below the first x with tt < lo bound
    x_top = key_float(float_key(sel_first_below(selM, cs, lo_t)) - 1u);
    // the very first range of a reference that is the row maximum is open upwards: t of the maximum itself is the
    // rounding error of M = max * scale and may be a hair below zero (a lowered reference keeps its bound:
    // what lies above it has been counted)
    if (qlo == 0 && !rebased) x_top = pinf;
    {
      const float hi = fminf(x_top, x_max), lo = fmaxf(x_lo, -1e38f);
      x_mid = 0.5f * lo + 0.5f * hi;
      x_half = fmaxf(hi - x_mid, x_mid - lo);
    }
    xlo_wave = -wave_max_f32(-x_lo);
    xlo_wave_top = wave_max_f32(x_lo);
    shift -= 7;                                                     // of this sweep's digit: 7, then 0
  };

  // a sliced search: the histogram of the group from what its slices left in the launch before
  const int groups = a.n_heads * n_qtiles, grp = j * n_qtiles + qtile;
  constexpr int kHistN = kSelBins * 32;
  // A slice leaves every run of a histogram as its running sums, so that the run's sum is its last entry.  Each slice of the next
  // launch then fetches the runs' sums and, of each query, the one run that crosses, where adding up all 128 bins is 32 KB per
  // slice in every slice.  Sums of running sums are running sums again (rounding keeps their order).
  static_assert(STEP == kSelAll || THREADS == kRuns * 32, "one thread per run and query");
  static_assert((kSelScan & 1) == 0 && (kSelFinish & 1) == 0, "histograms alternate between launches");
  const int my_run = wave * 2 + g;
  auto leave_runs = [&](double* own) __attribute__((always_inline)) {
    double c = 0.0;
#pragma unroll
    for (int i = 0; i < kRunBins; ++i) {
      c += hist[my_run * kRunBins + i][r];
      own[(my_run * kRunBins + i) * 32 + r] = c;
    }
  };
  auto scan_slices = [&](int n, bool whole) __attribute__((always_inline)) {
    const double* const old = a.sl_hist + ((int64_t)(1 - (STEP & 1)) * groups + grp) * n * kHistN + r;   // (kSelScan and sweep 2: of sweep 1)
    double (*crossing)[32] = run_sum + kRuns;                       // running sums of each query's crossing run
    static_assert(sizeof(double) * 32 * (kRuns + kRunBins) <= sizeof(list_all), "both fit the lists' memory");
    auto over_slices = [&](int bin) __attribute__((always_inline)) {
      double sum = 0.0;
#pragma unroll 8
      for (int k = 0; k < n; ++k) sum += old[(int64_t)k * kHistN + bin * 32];
      return sum;
    };
    run_sum[my_run][r] = over_slices(my_run * kRunBins + kRunBins - 1);
    __syncthreads();
    double rs[kRuns];
#pragma unroll
    for (int i = 0; i < kRuns; ++i) rs[i] = run_sum[i][r];
    if (whole) {
      Z = 0.0;
#pragma unroll
      for (int i = 0; i < kRuns; ++i) Z += rs[i];
    }
    const double target = (double)a.p * Z;
    const ThresholdRun run = threshold_run<kRuns>(above, target, rs);
    if (my_run < kRunBins) crossing[my_run][r] = over_slices(run.run * kRunBins + my_run);
    __syncthreads();
    double c[kRunBins];
#pragma unroll
    for (int i = 0; i < kRunBins; ++i) c[i] = crossing[i][r];
    const ThresholdBin t = threshold_in_run<kRuns, kRunBins>(run, target, c);
    bsel = t.bin;
    cum = t.above;
    hsel = t.mass;
    if (STEP == kSelScan) count_kept(rs, target, [&](int i) __attribute__((always_inline)) { return i == 0 ? c[0] : c[i] - c[i > 0 ? i - 1 : 0]; });
    __syncthreads();                                                // the sums are read: the lists' memory is free again
  };
  // what a launch hands to the next one, per query
  SelState* const state0 = a.sl_state + (int64_t)j * a.n_q + t;
  SelState* const state1 = state0 + (int64_t)a.n_heads * a.n_q;
  auto take = [&](const SelState& st) __attribute__((always_inline)) {
    Z = st.Z; above = st.above; selM = st.selM; x_max = st.x_max; prefix = st.prefix;
    rebased = (st.flags & kSelRebased) != 0;
  };
  // (48 kept keys a pair on the average: 1/43 of the context per query, more than a run of tokens that a query keeps for itself)
  auto see_how_much = [&](int flags) __attribute__((always_inline)) {
    float kept = fast_exp2(0.5f * (float)(flags >> kSelClassShift));
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) kept += __shfl_xor(kept, o);
    kept_much = !own_table && __builtin_amdgcn_readfirstlane(kept * 64.f >= 48.f * (float)n_rows ? 1 : 0) != 0;
  };
  auto leave = [&](SelState* st, int flags) __attribute__((always_inline)) {
    *st = SelState{Z, above, selM, x_max, prefix, (rebased ? kSelRebased : 0) | flags};
  };
  // the class of prefill_order_kernel: half octaves of the kept count
  auto class_of_kept = [&]() __attribute__((always_inline)) {
    return (int)fminf(fmaxf(2.f * __builtin_amdgcn_logf(kept_about), 0.f), (float)(kOrderClasses - 2));
  };
  auto last_digits = [&]() __attribute__((always_inline)) {
#pragma unroll 1
    for (int phase = 2; phase < 4; ++phase) {
      member_range(phase);
      zero_hist();
      __syncthreads();
      if (phase == 2) sweep_all(std::integral_constant<int, 2>{});
      else sweep_all(std::integral_constant<int, 3>{});
      __syncthreads();
      scan(false, true);
      prefix = (prefix << 7) | bsel;
      above = cum;
      __syncthreads();                                              // every wave has read the histograms
    }
  };
  auto results = [&]() __attribute__((always_inline)) {
    // a threshold inside the open-ended last coarse bin (only after the last repeat) keeps every candidate
    const bool lump = (prefix >> 14) == kSelBins - 1;
    cut = lump ? pinf : (float)(prefix + 1) * (1.0f / kSelScale);
    sel_mass = (lump || !(Z > 0.0)) ? 1.f : (float)((cum + hsel) / Z);
    if (!qok || g != 0 || wave != 0) return;
    const int64_t o = (int64_t)j * a.n_q + t;
    a.sel_thr[o] = sel_first_below(selM, cs, cut);
    if (a.mass) a.mass[o] = sel_mass;
    // kept: candidates with floor((M - s) * 2^17) <= the threshold's digit string, i.e. s > M - cut
    if (a.tau) a.tau[o] = cut != pinf ? selM - cut : ninf;
  };
  auto row_max_of_slices = [&]() __attribute__((always_inline)) {
    x_max = ninf;
    for (int k = 0; k < a.n_slice; ++k) x_max = fmaxf(x_max, a.sl_max[((int64_t)grp * a.n_slice + k) * 32 + r]);
    selM = x_max * cs;
  };
  if constexpr (STEP == kSelFirst) {
    row_maxima();
    first_digit();
    if (qok && g == 0 && wave == 0) leave(state0, class_of_kept() << kSelClassShift);
    return;
  }
  if constexpr (STEP == kSelScan) {
    row_max_of_slices();
    scan_slices(a.n_slice, true);
    prefix = bsel;
    above = cum;
    const int open = in_open_bin() ? kSelOpen | ((kOrderClasses - 1) << kSelClassShift) : class_of_kept() << kSelClassShift;
    if (qok && g == 0 && wave == 0) leave(state0, open);
    return;
  }
  if constexpr (kSliced) {
    const int64_t mine_at = (int64_t)grp * n_slice + slice;
    double* const own = a.sl_hist + ((int64_t)(STEP & 1) * groups * n_slice + mine_at) * kHistN;          // written by this launch
    if constexpr (STEP == 0) {
      row_maxima();
      if (tid < 32) a.sl_max[mine_at * 32 + r] = x_max;
      return;
    }
    if constexpr (STEP == 1) {
      row_max_of_slices();
      selM8 = selM * 8.0f;
      zero_hist();
      __syncthreads();
      sweep_all(std::integral_constant<int, 1>{});
    } else if constexpr (STEP >= 2) {
      if (STEP == 3 && a.sl_again[grp] != 0) return;                  // (the same for the whole workgroup)
      int again = 0;
      if (STEP == 2 && ORDERED) {
        const SelState st = *state0;
        take(st);
        see_how_much(st.flags);
        again = any_of((st.flags & kSelOpen) != 0) ? 1 : 0;
        if (rest_whole) {
          if (tid == 0) a.sl_again[grp] = 2;
          __syncthreads();
          last_digits();
          results();
          return;
        }
      } else if (STEP == 2) {
        row_max_of_slices();
        scan_slices(n_slice, true);
        again = any_of(in_open_bin()) ? 1 : 0;
        prefix = bsel;
        above = cum;
      } else {
        const SelState st = *state0;
        take(st);
        if (ORDERED) see_how_much(st.flags);
        scan_slices(n_slice, false);
        prefix = (prefix << 7) | bsel;
        above = cum;
      }
      if (STEP == 2) {
        if (slice == 0 && tid == 0) a.sl_again[grp] = again;
        if (again) return;
      }
      if (slice == 0 && tid < 32 && !(STEP == 2 && ORDERED)) leave(STEP == 2 ? state0 : state1, 0);
      member_range(STEP);
      zero_hist();
      __syncthreads();
      sweep_all(std::integral_constant<int, STEP>{});
    }
    __syncthreads();
    leave_runs(own);
    return;
  }

  const int again = STEP == kSelFinish ? a.sl_again[grp] : 1;
  if (again == 2) return;
  if (again == 0) {
    take(*state1);
    scan_slices(a.n_slice, false);
    prefix = (prefix << 7) | bsel;
  } else {
    own_table = true;
    row_maxima();
    first_digit();
    last_digits();
  }
  results();
}

// ---- the wide kernel: dense and selecting modes ------------------------------------------------------
// Same data flow as above for a workgroup of 256 queries whose eight waves of 32, two per SIMD at at most 256 registers
// each, share every staged K/V tile.  (Built and measured as four waves of 64 queries, one per SIMD, too: every A operand
// read from LDS -- a K row block, a V^T row block -- then feeds two MFMAs, which halves the LDS operand traffic per flop, at the
// price of registers, 2 x 64 output accumulators and 64 for the two Q operand sets.  A lone wave on a SIMD issues an
// independent 32x32x16 MFMA every 38 cycles and a vector instruction every ~6, two waves reach the pipes' 32 and 4; in this
// kernel's own address patterns eight waves read K rows from LDS at ~250 bytes per clock and V^T (the transposing read) at
// ~96, four waves at ~160 and ~63 -- enough for either shape, so the second instruction stream wins: eight waves were 3 to
// 16 % faster at every depth of the 131072- and 1048576-token configurations.)
//
// Nothing hides latency by itself at two waves per SIMD, so the loop is software-pipelined over
// 32-key blocks: while the softmax of block i runs on the vector ALU, the matrix pipe executes the PV
// MFMAs of block i-1; the two are independent instruction streams inside one basic block and are
// interleaved with scheduling-group hints.  For that the accumulators must never be touched by the
// vector ALU inside the loop (the register allocator would otherwise shuttle them between the two
// register files), so there is no running maximum: every query takes a FIXED reference
// maximum from the scores of the first key tile and the probabilities are exp2(s - ref), which fp32 and
// bf16 represent over +-126 binades.  After the pass the row sums tell whether a reference was off by
// more than that leaves room for (sum outside [2^-60, 2^100], or not finite); the workgroup then
// repeats its keys with the classical running-maximum recurrence (exact_pass).  Real score rows
// have their maximum at the first tokens; the repeat exists for correctness, not for speed.
// K/V tiles rotate through three LDS buffers (the PV of a tile's last block reads its V^T while the
// next tile is current).  One workgroup barrier per 64-key tile, in its middle: it publishes tile it + 1, whose loads every
// wave has waited for, and behind it every wave is done with tile it - 1, whose buffer the loads of tile it + 2 fill.
//
// Tiles that every query of the workgroup sees in full -- all but the first and the four or five on the diagonal --
// run in a loop without a branch (steady, below), the others block by block with element masks and nothing
// interleaved.  Inside the branches that served both before, the register allocator moved accumulators at the joins,
// and every stream began by waiting for its first LDS operands, all eight waves at once; in the loop a stream reads
// the next one's first operands.  Attention launch of 4 heads x 4096 queries at 128K tokens: 1300 -> 1066 us selecting,
// 1250 -> 918 us dense (1.18 PFLOP/s); last 8192-query chunk of 1M tokens, selecting, over every tile: 20.3 -> 17.3 to 17.7 ms (operands three
// and two steps ahead instead of five and four: 17.7 and 1141 us).  Over the 0.46 of the tiles that its queries regrouped leave (ORDERED):
// 8.9 ms; the 4096 at 128K, 0.66 of the tiles: 825 us.  Per 32 x 32 block the two waves of a SIMD issue 16 MFMAs
// of 32 cycles, 24 LDS reads and, by the counters, 64 (dense) or 122 (selecting) other vector instructions each, with the matrix
// pipe busy 59 and 48 % of the cycles and the LDS, at the rates of these reads, about half of them.  Spreading a block's softmax
// over both streams (it used to run beside the PV MFMAs alone) took the dense call of this shape from 1132 to 1124 us, 333
// queries' launch from 132 to 129 and left the selecting last chunk of 1M as it was.  The dense launch runs at a die clock of 1.71 to
// 1.75 GHz, against 2.4 when idle: it has come to what the chip's power allows.  The selecting one (1.98 GHz, matrix pipe busy 51 %) has
// not; it issues twice the other vector instructions.
constexpr int kPwThreads = 512;
constexpr int kPwStages = 3;
// One staged tile: 64 K rows then 64 V rows, 256 bytes each, no padding -- the tiles are written by
// direct global->LDS loads (16 bytes per lane, a wave's 64 lanes fill 1 KiB contiguously), so bank
// spreading comes from the order of the 16-byte chunks inside a row instead: K row n keeps chunk c at
// position c ^ (n % 16) (the MFMA operand read takes one chunk of 16 consecutive rows), V row n keeps
// 32-byte unit u at position u ^ 2 (n % 4): a transposing operand read has each half-wave take, from four rows,
// the two units 2 db and 2 db + 1 (its two 16-lane groups), and with this order those eight (row, unit) pieces
// land on the eight different bank groups of a row (u ^ (n % 8), the first layout, put the two groups' pieces on
// the same four: a third of the kernel's LDS cycles were bank conflicts by the counters, none now; the kernel is
// bound by instruction issue and runs as long).
constexpr int kPwTileBytes = 2 * kPfK * kHeadDim * 2;
constexpr int kSmemWide = kPwTileBytes * kPwStages;


// ORDERED: a selecting launch over regrouped queries, in planned units (without any where nothing is regrouped, the order being by position).
template <int MODE, bool F16 = false, bool ORDERED = false>
__global__ __launch_bounds__(kPwThreads, 2) void flash_prefill_wide_kernel(const PrefillArgs a) {
  constexpr int NW = kPwThreads / 64;        // waves per workgroup; each owns 32 queries
  constexpr int RG = 4 * NW;                 // tile rows one load instruction of the whole workgroup covers
  constexpr int GH = 64 / RG;                // such loads per wave for the K rows of a tile (and as many for V)
  constexpr bool SPARSE = MODE == kModeSparse;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kSmemWide];
  unsigned char* const Ls = smem;       // stage s: K rows at Ls + s * kPwTileBytes, V rows 16 KiB further

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (the branches on a wave's queries are scalar)
  const int g = lane >> 5, r = lane & 31;
  // A selecting launch behind a threshold search (one sequence) is laid out (key range, query tile, head slot): the
  // query tiles' lists differ wildly in length, and with the key range as the fastest index the ranges of a long
  // list go round all eight dies (workgroups are dealt to the dies in turn) instead of piling up on one.
  // The grid of such a launch is sized for the finer cut; the ranges really used (listed_splits) take the
  // first workgroups of the grid in the same (key range, query tile, head slot) order, the others leave.
  constexpr bool listed = SPARSE;
  const int n_wide = (a.n_q + kPwQ - 1) / kPwQ;
  static_assert(!ORDERED || SPARSE, "only behind a search");
  const int n_units = ORDERED ? *a.n_units : 0;
  int n_parts = listed && n_units == 0 ? listed_splits(a) : a.n_splits;
  int n_sub = a.n_sub;
  int n_splits = n_parts * n_sub;
  int hslot = blockIdx.x, split, qt_rev = blockIdx.y, b = 0;
  bool exact_only = false, more = false;
  int list = 0, wave_lo = 0, wave_hi = NW;            // the unit's list and the waves whose queries it is for
  if (ORDERED && n_units > 0) {
    if ((int)blockIdx.x >= n_units) return;
    const int2 unit = a.units[blockIdx.x];
    const int what = __builtin_amdgcn_readfirstlane(unit.y);
    list = __builtin_amdgcn_readfirstlane(unit.x);
    const int n_lists = a.n_heads * n_wide;
    more = list >= n_lists;
    const int tile = more ? list - n_lists : list;
    hslot = tile / n_wide;
    qt_rev = tile - hslot * n_wide;
    split = what & 0xff;
    n_splits = n_parts = (what >> 8) & 0xff;
    n_sub = 1;
    wave_lo = (what >> 16) & 0xf;
    wave_hi = (what >> 20) & 0xf;
    exact_only = (what & kUnitExact) != 0;
  } else if (listed) {
    const int lin = (int)blockIdx.x + (int)gridDim.x * ((int)blockIdx.y + (int)gridDim.y * (int)blockIdx.z);
    split = lin % n_splits;
    qt_rev = (lin / n_splits) % n_wide;
    hslot = lin / (n_splits * n_wide);
    if (hslot >= a.n_heads) return;
  } else {
    b = blockIdx.z / n_splits;
    split = (int)blockIdx.z - b * n_splits;
  }
  const int h = a.heads[hslot];
  constexpr bool ordered = ORDERED;                     // (hard queries first, their tiles have the long lists)
  const int t0 = (ordered ? qt_rev : n_wide - 1 - qt_rev) * kPwQ;
  const int kvh = h / (a.n_q_heads / a.n_kv_heads);
  const int pos0 = a.q_start ? a.q_start[b] : (int)a.q_start_host;
  const int64_t tok0 = a.seq_start ? a.seq_start[b] : 0;
  const float ninf = -__builtin_huge_valf();

  // ---- this lane's query (column r of the wave's 32) ----
  const bool my_wave = !ORDERED || (wave >= wave_lo && wave < wave_hi);
  const bool qok = my_wave && t0 + wave * 32 + r < a.n_q;
  const int32_t* const order = ordered ? a.order + (int64_t)hslot * a.n_q : nullptr;
  int tq = t0 + wave * 32 + r;
  if (ordered) tq = order[min(tq, a.n_q - 1)];
  const int mq = pos0 + tq;
  const int64_t qrow = (((int64_t)b * a.n_q + tq) * a.n_q_heads + h) * kHeadDim;
  u32x4 qreg[8];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk)
    qreg[kk] = qok ? *reinterpret_cast<const u32x4*>(a.q + qrow + kk * 16 + g * 8) : (u32x4){0u, 0u, 0u, 0u};

  // ---- key tiles this workgroup needs ----
  int m_lo = pos0 + t0;
  int m_hi = pos0 + min(t0 + kPwQ, a.n_q) - 1;
  if (ordered) {
    int lo = 0x7fffffff, hi = 0;
#pragma unroll
    for (int k = 0; k < kPwQ / 64; ++k) {
      const int m = pos0 + order[min(t0 + k * 64 + lane, a.n_q - 1)];
      lo = min(lo, m);
      hi = max(hi, m);
    }
    lo = min(lo, __shfl_xor(lo, 32));
    hi = max(hi, __shfl_xor(hi, 32));
    int unused;
    position_range(lo, m_lo, unused);
    position_range(hi, unused, m_hi);
  }
  const int kt_end = m_hi / kPfK;                       // inclusive
  // selecting mode with a threshold search in front: only the tiles on this query tile's list (ascending
  // 64-key tile numbers, written by prefill_active_tiles_kernel) can hold a kept pair
  const int qt_list = t0 / kPwQ;
  const int32_t* const alist = !listed ? nullptr : more ? more_list_of(a, hslot, qt_list) : a.act_list + ((int64_t)hslot * n_wide + qt_list) * a.n_t64;
  const int n_tiles = !listed ? kt_end + 1 : n_units > 0 ? a.list_info[list].x : a.act_count[(int64_t)hslot * n_wide + qt_list];
  const uint16_t* Kg = a.K + (int64_t)kvh * a.head_stride + tok0 * a.row_stride;
  const uint16_t* Vg = a.V + (int64_t)kvh * a.head_stride + tok0 * a.row_stride;

  f32x16 O[4];
  float mrow = ninf, lrow = 0.f;
  const float c = a.scale_log2;
  const int q_last = pos0 + a.n_q - 1;
  // the wave's first query position and its last; -1 for a wave without queries
  int m_w_lo = -1, m_w_hi = -1;
  if (my_wave && t0 + wave * 32 < a.n_q) {
    m_w_lo = ordered ? m_lo : pos0 + t0 + wave * 32;
    m_w_hi = ordered ? m_hi : min(m_w_lo + 31, q_last);
  }

  // ---- selecting mode: a key is kept by a query iff the raw index product reaches the query's
  // threshold (found by prefill_select_kernel; -inf keeps every candidate).  The index-score block of
  // 32 keys x 32 queries is one MFMA (K = 16) in the layout of the attention scores. ----
  u32x4 qIreg = (u32x4){0u, 0u, 0u, 0u};
  float selThr = ninf;
  int sel_cnt = 0;
  const uint16_t* kIg = nullptr;
  const int n_rows = pos0 + a.n_q;                      // index-key rows that exist
  if (SPARSE) {
    const int j = hslot;
    kIg = a.kI + (int64_t)j * a.kI_head_stride;
    if (qok) {
      qIreg = *reinterpret_cast<const u32x4*>(a.qI + ((int64_t)j * a.n_q + tq) * kIndexDim + g * 8);
      selThr = a.sel_thr[(int64_t)j * a.n_q + tq];
    }
  }
  // index keys of the 32-key block at nb0 (rows past the chunk repeat the last one: causally masked anyway)
  auto load_ki = [&](int nb0) __attribute__((always_inline)) {
    const int nrow = min(nb0 + r, n_rows - 1);
    return *reinterpret_cast<const u32x4*>(kIg + (int64_t)nrow * kIndexDim + g * 8);
  };
  // drops the keys a query does not keep from its scores and counts the kept ones; run AFTER mask_block
  // (causality shows as -inf there)
  auto select_block = [&](f32x16& S, const u32x4 ki) __attribute__((always_inline)) {
    f32x16 SI;
#pragma unroll
    for (int i = 0; i < 16; ++i) SI[i] = 0.f;
    SI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ki), __builtin_bit_cast(bf16x8, qIreg), SI, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const bool keep = SI[i] >= selThr && S[i] != ninf;
      sel_cnt += keep ? 1 : 0;
      S[i] = keep ? S[i] : ninf;
    }
  };

  // ---- tile movers: direct global->LDS loads, no staging registers (rows past the last needed key
  // repeat that key: they are masked for every query, and real data keeps 0 * V finite) ----
  // Load j (0..GH-1: K, GH..2GH-1: V) of a wave covers rows RG * (j % GH) + 4 * wave + lane / 16 of the
  // tile, lane % 16 is the 16-byte position inside the row; the lane fetches the chunk that belongs there.
  const uint32_t lds_base = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)Ls;
  const int ld_row = 4 * wave + (lane >> 4);
  const int ld_pos = lane & 15;
  const int ld_ck = ld_pos ^ (ld_row & 15);                                          // K chunk of this lane
  const int ld_cv = ((((ld_pos >> 1) ^ (2 * (ld_row & 3))) << 1) | (ld_pos & 1));    // V chunk of this lane
  auto load_piece = [&](int n0, int slot, int j) __attribute__((always_inline)) {
    const int jj = j % GH;
    const int n = min(n0 + RG * jj + ld_row, m_hi);
    const uint16_t* src = (j < GH ? Kg + ld_ck * 8 : Vg + ld_cv * 8) + (int64_t)n * a.row_stride;
    const uint32_t dst = lds_base + slot * kPwTileBytes + (j < GH ? 0 : kPwTileBytes / 2) + (jj * NW + wave) * 1024;
    // Written as assembly on purpose: through the compiler's own intrinsic every later LDS read waits
    // for ALL outstanding direct loads (it cannot tell the buffers apart), which serialises the
    // pipeline; completion is awaited explicitly (loads_landed) before the barrier that publishes a tile.
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory", "m0");
  };
  // The same for a tile that lies wholly inside the key range (every tile but the last): the tile's first
  // K and V rows as scalar base addresses, the lane's place inside the tile as a 32-bit offset computed
  // once -- no vector arithmetic per load (the general form costs seven vector instructions per piece,
  // two of them quarter-rate multiplies, a tenth of the kernel's issue slots).
  uint32_t off_k[GH], off_v[GH];
#pragma unroll
  for (int jj = 0; jj < GH; ++jj) {
    off_k[jj] = (uint32_t)(((int64_t)(RG * jj + ld_row) * a.row_stride + ld_ck * 8) * 2);
    off_v[jj] = (uint32_t)(((int64_t)(RG * jj + ld_row) * a.row_stride + ld_cv * 8) * 2);
  }
  auto load_piece_full = [&](int n0_any, int slot, int j) __attribute__((always_inline)) {
    const int n0 = __builtin_amdgcn_readfirstlane(n0_any);   // (a listed tile's number was loaded from memory)
    const int jj = j % GH;
    const unsigned char* base = reinterpret_cast<const unsigned char*>((j < GH ? Kg : Vg) + (int64_t)n0 * a.row_stride);
    const uint32_t dst = lds_base + slot * kPwTileBytes + (j < GH ? 0 : kPwTileBytes / 2) + (jj * NW + wave) * 1024;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(j < GH ? off_k[jj] : off_v[jj]), "s"(base)
                 : "memory", "m0");
  };
  auto load_tile = [&](int n0, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2 * GH; ++j) load_piece(n0, slot, j);
  };
  auto loads_landed = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
  // operand read addresses (bytes inside a staged tile)
  const int rd_k = r * 256, rd_kx = (g ^ (r & 15)) << 4;                              // K: + kb * 8192, chunk (2 kk) ^ ...
  const int rd_j = lane & 15, rd_G = (lane >> 4) & 1;
  const int rd_v = kPwTileBytes / 2 + (4 * g + (rd_j >> 2)) * 256 + 8 * (rd_j & 3);   // V: + (kb * 32 + 16 tt + 8 h) * 256
  const int rd_vx = (rd_G ^ (2 * (rd_j >> 2))) << 5;                                  //    unit (2 db) ^ ...
  auto read_k = [&](const unsigned char* tile, int kb, int kk) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(tile + kb * 8192 + rd_k + ((kk << 5) ^ rd_kx));
  };
  // the 8 keys x 1 dim a lane needs of V^T for MFMA (tt, db): two transposing reads of 4 keys each
  auto read_v = [&](const unsigned char* tile, int kb, int tt, int db) __attribute__((always_inline)) {
    const unsigned char* p0 = tile + rd_v + (kb * 32 + 16 * tt) * 256 + ((db << 6) ^ rd_vx);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0 + 8 * 256));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  // ---- MFMA streams ----
  // scores of key block kb of the staged tile, for the wave's query blocks
  auto mfma_S = [&](const unsigned char* tile, int kb, f32x16& S) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) S[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const u32x4 ka = read_k(tile, kb, kk);
      S = mfma32<F16>(ka, qreg[kk], S);
    }
  };
  // In the steady loop K operands are read kAheadK steps ahead, V operands kAheadV, the first ones during the stream before
  // (ka_first, va_first): with every wave of the workgroup at the same place (the barrier in every tile) nothing else covers
  // their LDS latency.
  constexpr int kAheadK = 5, kAheadV = 4, kPairsPV = 4;
  u32x4 ka_first[kAheadK];
  s16x8 va_first[kAheadV];
  auto first_k = [&](const unsigned char* tile, int kb) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < kAheadK; ++kk) ka_first[kk] = read_k(tile, kb, kk);
  };
  auto first_v = [&](const unsigned char* tile, int kb) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < kAheadV; ++k) va_first[k] = read_v(tile, kb, k >> 2, k & 3);
  };
  // O^T += V^T P^T for key block kb of the staged tile
  auto mfma_PV = [&](const unsigned char* tile, int kb, const uint32_t (&P)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const u32x4 va = __builtin_bit_cast(u32x4, read_v(tile, kb, tt, db));
        const u32x4 pb = (u32x4){P[4 * tt], P[4 * tt + 1], P[4 * tt + 2], P[4 * tt + 3]};
        O[db] = mfma32<F16>(va, pb, O[db]);
      }
    }
  };
  // per-element visibility without control flow: key nb0 + off, off = (i / 4) * 8 + g * 4 + i % 4, is
  // visible iff off <= hi, a per-lane bound
  auto mask_block = [&](f32x16& S, int nb0) __attribute__((always_inline)) {
    const int base = nb0 + g * 4;
    const int hi = qok ? mq - base : -1;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int off = (i >> 2) * 8 + (i & 3);
      S[i] = off <= hi ? S[i] : ninf;
    }
  };
  // l += both halves of a packed pair of probabilities, i.e. the values as rounded to bf16 (what the PV
  // product multiplies): one instruction, and of a kind the compiler leaves where it is written (plain
  // additions get collected behind the last MFMA of the sequence, where nothing hides them)
  // (the compiler's own dot product intrinsic gets collected the same way).  The result of a dot
  // instruction must not be read by another kind of vector instruction for three wait states, and
  // the compiler does not look into assembly text: row_sum_settled() goes between the last
  // row_sum_add and the first use.
  auto row_sum_settled = [&](float& l) __attribute__((always_inline)) { asm volatile("s_nop 3" : "+v"(l)); };
  auto row_sum_add = [&](float& l, uint32_t pk) __attribute__((always_inline)) {
    if constexpr (F16) asm volatile("v_dot2c_f32_f16 %0, %1, %2" : "+v"(l) : "v"(pk), "v"(0x3c003c00u));
    else asm volatile("v_dot2c_f32_bf16 %0, %1, %2" : "+v"(l) : "v"(pk), "v"(0x3f803f80u));
  };
  // probabilities against the fixed reference; masked scores are -inf and give exactly 0.  Summed as rounded to 16 bits where
  // the steady loop could have run the block, unrounded where it could not: rows of few tokens live in such blocks, and their
  // log-sum would carry the rounding (chunk of 172 tokens at position 0: 2.2e-4 instead of 1.2e-4 off).  fp16: a probability above
  // 65504 is rounded to infinity, which the PV product takes and the unrounded sum does not show; the sum of such a block is the rounded one,
  // i.e. infinite, so that the range is repeated in the exact pass.
  auto softmax_fixed = [&](const f32x16& S, uint32_t (&P)[8], const bool rounded) __attribute__((always_inline)) {
    const float mc = mrow * c;
    float lsum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      const float p0 = fast_exp2(fmaf(S[i], c, -mc));
      const float p1 = fast_exp2(fmaf(S[i + 1], c, -mc));
      lsum += p0 + p1;
      P[i >> 1] = pack16<F16>(p0, p1);
    }
    if (F16 || rounded) {                                // (the same for the whole wave)
      float as_rounded = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) row_sum_add(as_rounded, P[i]);
      row_sum_settled(as_rounded);
      if (rounded || !(as_rounded < __builtin_huge_valf())) lsum = as_rounded;
    }
    lrow += lsum;
  };
  // The steady-state step, two hand-interleaved streams over which the block's 16 probabilities are spread, so that each MFMA
  // (32 cycles of the matrix pipe) has about one of them beside it (1 fma, 1 exp, half a convert and half a packed dot product on
  // the vector ALU): pv_beside_softmax runs the PV MFMAs of the previous block and the first pairs, scores_beside_softmax
  // the score MFMAs of the next block and the rest.  Scheduling fences keep the compiler from regrouping them; V^T operands are
  // read kAheadV steps ahead (the first ones are in va_first) and, at the first stream's end, the first K operands of
  // the second (block next_kb of next_tile).  SEL (the selecting mode): the block's index-score MFMA in front and every
  // probability gated by its query's keep test (one compare, one select, one add for the count per probability).
  f32x16 SI;
  float mc, l_blk;
  int cnt_blk;
  auto pair = [&](auto sel_tag, int k, const f32x16& S, uint32_t (&Pout)[8]) __attribute__((always_inline)) {
    constexpr bool SEL = decltype(sel_tag)::value;
    float p0 = fast_exp2(fmaf(S[2 * k], c, -mc));
    float p1 = fast_exp2(fmaf(S[2 * k + 1], c, -mc));
    if (SEL) {
      const bool k0 = SI[2 * k] >= selThr, k1 = SI[2 * k + 1] >= selThr;
      p0 = k0 ? p0 : 0.f;
      p1 = k1 ? p1 : 0.f;
      cnt_blk += (k0 ? 1 : 0) + (k1 ? 1 : 0);
    }
    Pout[k] = pack16<F16>(p0, p1);
    row_sum_add(l_blk, Pout[k]);
  };
  auto pv_beside_softmax = [&](auto sel_tag, const unsigned char* tile, int kb, const uint32_t (&Pin)[8], const f32x16& S,
                               uint32_t (&Pout)[8], const u32x4 ki, const unsigned char* next_tile, int next_kb) __attribute__((always_inline)) {
    constexpr bool SEL = decltype(sel_tag)::value;
    mc = mrow * c;
    l_blk = 0.f;
    cnt_blk = 0;
    if (SEL) {
#pragma unroll
      for (int i = 0; i < 16; ++i) SI[i] = 0.f;
      SI = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ki), __builtin_bit_cast(bf16x8, qIreg), SI, 0, 0, 0);
    }
    s16x8 va[8];
    auto read_va = [&](int k) __attribute__((always_inline)) { va[k] = read_v(tile, kb, k >> 2, k & 3); };   // k = tt * 4 + db
#pragma unroll
    for (int k = 0; k < kAheadV; ++k) va[k] = va_first[k];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int tt = k >> 2, db = k & 3;
      if (k + kAheadV < 8) read_va(k + kAheadV);
      if (k == 8 - kAheadV) first_k(next_tile, next_kb);
      const u32x4 pb = (u32x4){Pin[4 * tt], Pin[4 * tt + 1], Pin[4 * tt + 2], Pin[4 * tt + 3]};
      O[db] = mfma32<F16>(__builtin_bit_cast(u32x4, va[k]), pb, O[db]);
      if (k & 1) { if (k / 2 < kPairsPV) pair(sel_tag, k / 2, S, Pout); }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto scores_beside_softmax = [&](auto sel_tag, const unsigned char* tile, int kb, f32x16& Snext, const f32x16& S, uint32_t (&Pout)[8],
                                   auto&& work) __attribute__((always_inline)) {
    constexpr bool SEL = decltype(sel_tag)::value;
    u32x4 ka[8];
#pragma unroll
    for (int kk = 0; kk < kAheadK; ++kk) ka[kk] = ka_first[kk];
#pragma unroll
    for (int i = 0; i < 16; ++i) Snext[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      if (kk + kAheadK < 8) ka[kk + kAheadK] = read_k(tile, kb, kk + kAheadK);
      Snext = mfma32<F16>(ka[kk], qreg[kk], Snext);
      work(kk);
      if (kk & 1) { if (kPairsPV + kk / 2 < 8) pair(sel_tag, kPairsPV + kk / 2, S, Pout); }
      __builtin_amdgcn_sched_barrier(0);
    }
    row_sum_settled(l_blk);
    lrow += l_blk;
    if (SEL) sel_cnt += cnt_blk;
  };
  // does the 32-key block starting at nb0 need per-element masks for some query of this wave?
  auto needs_mask = [&](int nb0) __attribute__((always_inline)) {
    return nb0 + 31 > m_w_lo;
  };
  // can some query of this wave see a key of the block at all?
  auto is_active = [&](int nb0) __attribute__((always_inline)) {
    return nb0 <= m_w_hi;
  };

  auto tile_n0 = [&](int it) __attribute__((always_inline)) {
    return (listed ? alist[it] : it) * kPfK;
  };
  const int p_lo = (int)((int64_t)n_tiles * (split / n_sub) / n_parts), p_hi = (int)((int64_t)n_tiles * (split / n_sub + 1) / n_parts);
  const int sub = split % n_sub;
  const int it_lo = p_lo + (int)((int64_t)(p_hi - p_lo) * sub / n_sub);
  const int it_hi = p_lo + (int)((int64_t)(p_hi - p_lo) * (sub + 1) / n_sub);
  auto slot_of = [&](int it) __attribute__((always_inline)) { return (it - it_lo) % kPwStages; };
  auto tile_at = [&](int it) __attribute__((always_inline)) { return Ls + slot_of(it) * kPwTileBytes; };

  bool redo = exact_only;
  if (it_lo < it_hi && !exact_only) {
    f32x16 S;
    uint32_t P0[8], P1[8];
    lrow = 0.f;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) O[db][i] = 0.f;
    // first keys of tiles it, it + 1, it + 2 (clamped to the range's last tile) and, one iteration ahead of its
    // first use, it + 3: a listed tile's number comes from memory
    int n_t0 = tile_n0(it_lo), n_t1 = tile_n0(min(it_lo + 1, it_hi - 1)), n_t2 = tile_n0(min(it_lo + 2, it_hi - 1));
    int n_t3 = tile_n0(min(it_lo + 3, it_hi - 1));
    load_tile(n_t0, 0);
    load_tile(n_t1, 1);
    // reference maxima: the largest score of the part's first tile, masks ignored (always finite).  A sub-range further
    // on takes the same reference -- its probabilities are rounded to 16 bits exactly as if the part were
    // walked in one go -- from a copy of that tile in the buffer that is free until half 1 of its own first tile.
    const unsigned char* const t_ref = it_lo == p_lo ? Ls : Ls + 2 * kPwTileBytes;
    if (it_lo != p_lo) load_tile(tile_n0(p_lo), 2);
    loads_landed();
    __syncthreads();
    mrow = ninf;
#pragma unroll
    for (int kb = 1; kb >= 0; --kb) {
      mfma_S(t_ref, kb, S);
      float mx = S[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, S[i]);
      mrow = fmaxf(mrow, fmaxf(mx, __shfl_xor(mx, 32)));
    }
    if (it_lo != p_lo) mfma_S(Ls, 0, S);                 // S now holds block (it_lo, 0)

    // Invariant at the start of half hf of tile it: S holds the scores of that block if it is active
    // for this wave; if `pend`, the probabilities of the last active block wait in P1 (hf = 0, V in
    // the previous tile's buffer) or P0 (hf = 1); tiles it and it + 1 are in LDS.  The loads of tile
    // it + 2 go out during half 1 (their buffer held tile it - 1, last read in half 0) and every wave
    // waits for its own before the barrier that ends half 0 of tile it + 1.
    bool pend = false;
    u32x4 ki0 = (u32x4){0u, 0u, 0u, 0u}, ki1 = ki0;       // index keys of the current tile's two key blocks
    if (SPARSE) {
      ki0 = load_ki(n_t0);
      ki1 = load_ki(n_t0 + 32);
    }
    auto next_tiles = [&](int it) __attribute__((always_inline)) {
      n_t0 = n_t1;
      n_t1 = n_t2;
      n_t2 = n_t3;
      n_t3 = tile_n0(min(it + 4, it_hi - 1));
    };
    // one half of a tile that some query may not see in full (masks by element, nothing interleaved)
    auto half = [&](int it, auto hf_tag) __attribute__((always_inline)) {
      constexpr int hf = decltype(hf_tag)::value;
      const int nb0 = n_t0 + hf * 32;
      const unsigned char* t_pend = hf == 0 ? tile_at(it - 1) : tile_at(it);
      const uint32_t (&Pin)[8] = hf == 0 ? P1 : P0;
      uint32_t (&Pout)[8] = hf == 0 ? P0 : P1;
      if (pend) mfma_PV(t_pend, 1 - hf, Pin);
      bool rounded = pend || (hf == 0 && it == it_lo && it_lo != p_lo);    // some block of the part was before
      pend = false;
      if (is_active(nb0)) {
        if (needs_mask(nb0)) {
          mask_block(S, nb0);
          rounded = false;
        }
        if (SPARSE) select_block(S, hf == 0 ? ki0 : ki1);
        softmax_fixed(S, Pout, rounded);
        pend = true;
      }
      if (SPARSE && hf == 1) {                             // the next tile's index keys: a tile's time to arrive
        ki0 = load_ki(n_t1);
        ki1 = load_ki(n_t1 + 32);
      }
      if (hf == 0) {
        if (is_active(nb0 + 32)) mfma_S(tile_at(it), 1, S);
        loads_landed();
        __syncthreads();
      } else {
        // past the last tile the same loads re-fetch it into a buffer nobody reads: no branches
        load_tile(n_t2, slot_of(it + 2));
        if (it + 1 < it_hi && is_active(n_t1)) mfma_S(tile_at(it + 1), 0, S);
      }
    };
    int it = it_lo;
    auto edge_tile = [&]() __attribute__((always_inline)) {
      half(it, std::integral_constant<int, 0>{});
      half(it, std::integral_constant<int, 1>{});
      next_tiles(it);
      ++it;
    };
    edge_tile();
    // The steady loop: tiles every query of the workgroup sees in full, the tile to fetch a whole one.  The tile
    // before was visible as well, so every wave with queries has probabilities pending; a wave without queries only
    // fetches its share of the tiles.
    auto steady = [&]() __attribute__((always_inline)) { return it < it_hi && n_t0 + kPfK - 1 <= m_lo && n_t2 + kPfK - 1 <= m_hi; };
    if (steady()) {
      if (m_w_hi >= 0) {
        f32x16 S1;
        first_v(tile_at(it - 1), 1);
        do {
          constexpr std::integral_constant<bool, SPARSE> sel{};
          pv_beside_softmax(sel, tile_at(it - 1), 1, P1, S, P0, ki0, tile_at(it), 1);
          scores_beside_softmax(sel, tile_at(it), 1, S1, S, P0, [&](int) __attribute__((always_inline)) {});
          first_v(tile_at(it), 0);
          loads_landed();
          __syncthreads();
          pv_beside_softmax(sel, tile_at(it), 0, P0, S1, P1, ki1, tile_at(it + 1), 0);
          if (SPARSE) {                                    // the next tile's index keys: a tile's time to arrive
            ki0 = load_ki(n_t1);
            ki1 = load_ki(n_t1 + 32);
          }
          const int n2 = n_t2, s2 = slot_of(it + 2);
          scores_beside_softmax(sel, tile_at(it + 1), 0, S, S1, P1,
                                [&](int kk) __attribute__((always_inline)) { if (kk < 2 * GH) load_piece_full(n2, s2, kk); });
          first_v(tile_at(it), 1);
          next_tiles(it);
          ++it;
        } while (steady());
      } else {
        do {
          loads_landed();
          __syncthreads();
#pragma unroll
          for (int j = 0; j < 2 * GH; ++j) load_piece_full(n_t2, slot_of(it + 2), j);
          next_tiles(it);
          ++it;
        } while (steady());
      }
    }
    while (it < it_hi) edge_tile();
    if (pend) mfma_PV(tile_at(it_hi - 1), 1, P1);        // drain: PV of the last block
    loads_landed();

    // was every reference within reach?  A query that can see a key of this key range (always, with
    // the whole band of a local launch; from the range's first key on, in a dense one) must have a sum
    // in the comfortable middle of the fp32 range; everything else (0, tiny, huge, inf, NaN) repeats.
    bool bad = false;
    const float ltot = lrow + __shfl_xor(lrow, 32);
    // selecting mode: a query that kept no key of this range legitimately sums to zero
    const int n_kept = SPARSE ? sel_cnt + __shfl_xor(sel_cnt, 32) : 0;
    const bool sees_key = SPARSE ? n_kept > 0 : (qok && tile_n0(it_lo) <= mq);
    // (fp16 probabilities: nothing above 65504 -- a larger one is infinite and shows in the sum -- and a
    // row whose largest probability is below 2^-6 may have most of its mass in subnormals.  Few kept keys may have a smaller sum: a subnormal is
    // off by at most 2^-25, and n of those are within 2^-11 of a sum of n * 2^-14, as the rounding of n normal probabilities is.  A query
    // that keeps a few keys of a range, all far below its first tile's best, is one of 256 in hundreds of tiles nearly always, and the whole range was
    // repeated for it.  Attention launch at 128K tokens, 333, 2000 and 4096 queries (clusters): 365 -> 150, 1547 -> 606, 1472 -> 939 us.)
    float least = F16 ? 0x1p-6f : 0x1p-60f;
    if (SPARSE && F16) least = fminf(least, (float)n_kept * 0x1p-14f);
    bad = bad || (sees_key && !(ltot > least && ltot < 0x1p100f));
    redo = __syncthreads_or(bad ? 1 : 0) != 0;
  }

  if (redo) {
    // ---- exact pass: running maximum, accumulators rescaled in place; only the next tile's loads are in flight.  For queries that
    // keep few keys (their tiles' lists are short once they stand together) and references out of reach (rare).  In bf16 the probabilities are multiplied
    // in two parts, rounded and the rest: a sum of a few terms does not average a rounding to 8 bits. ----
    constexpr bool kParts = ORDERED && !F16;
    f32x16 S;
    uint32_t P[8], Q[kParts ? 8 : 1];
    mrow = ninf;
    lrow = 0.f;
    sel_cnt = 0;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) O[db][i] = 0.f;
    __syncthreads();
    if (it_lo < it_hi) load_tile(tile_n0(it_lo), 0);
    for (int it = it_lo; it < it_hi; ++it) {
      const int buf = (it - it_lo) & 1;
      const unsigned char* const tile = Ls + buf * kPwTileBytes;
      loads_landed();
      __syncthreads();
      if (it + 1 < it_hi) load_tile(tile_n0(it + 1), buf ^ 1);
      for (int kb = 0; kb < 2; ++kb) {
        const int nb0 = tile_n0(it) + kb * 32;
        if (!is_active(nb0)) continue;
        if (kb == 0) mfma_S(tile, 0, S); else mfma_S(tile, 1, S);
        mask_block(S, nb0);
        if (SPARSE) {
          const int before = sel_cnt;
          select_block(S, load_ki(nb0));
          if (__ballot(sel_cnt != before) == 0ull) continue;      // no query of the wave keeps a key of the block
        }
        float mx = S[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, S[i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mnew = fmaxf(mrow, mx);
        const float msafe = mnew == ninf ? 0.f : mnew;
        const float mc = msafe * c;
        float lsum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
          const float p0 = fast_exp2(fmaf(S[i], c, -mc));
          const float p1 = fast_exp2(fmaf(S[i + 1], c, -mc));
          lsum += p0 + p1;
          P[i >> 1] = pack16<F16>(p0, p1);
          if constexpr (kParts) Q[i >> 1] = pack16<F16>(p0 - bf16_lo(P[i >> 1]), p1 - bf16_hi(P[i >> 1]));
        }
        const float corr = fast_exp2((mrow - msafe) * c);
        lrow = lrow * corr + lsum;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) O[db][i] *= corr;
        mrow = mnew;
        if (kb == 0) mfma_PV(tile, 0, P); else mfma_PV(tile, 1, P);
        if constexpr (kParts) { if (kb == 0) mfma_PV(tile, 0, Q); else mfma_PV(tile, 1, Q); }
      }
    }
  }

  // ---- normalise and store ----
  const float ltot = (it_lo < it_hi) ? lrow + __shfl_xor(lrow, 32) : 0.f;
  if (!qok) return;
  const float mfin = (it_lo < it_hi && ltot > 0.f) ? mrow : ninf;
  const int kept = sel_cnt + __shfl_xor(sel_cnt, 32);
  if (MODE == kModeDense && g == 0 && split == 0) {       // the statistics of the rule that keeps every candidate
    const int64_t o = (int64_t)hslot * a.n_q + tq;
    if (a.mass) a.mass[o] = 1.f;
    if (a.tau) a.tau[o] = ninf;
    if (a.count) a.count[o] = mq + 1;
  }
  if (n_splits > 1) {
    const int64_t at = ORDERED && n_units > 0 ? (int64_t)(a.list_ranges[list].y + split) * kPwQ + wave * 32 + r
                                         : ((int64_t)split * a.n_heads + hslot) * a.n_q + tq;
    float* prow = a.part + at * kPfPart;
    // (a sum that is not a number comes with a maximum that the merge does not take for a range without keys)
    if (g == 0) { prow[0] = it_lo < it_hi && ltot != ltot ? 0.f : mfin; prow[1] = ltot; prow[2] = __int_as_float(kept); }
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        *reinterpret_cast<float4*>(prow + 4 + db * 32 + i4 * 8 + g * 4) =
            ltot > 0.f ? make_float4(O[db][i4 * 4], O[db][i4 * 4 + 1], O[db][i4 * 4 + 2], O[db][i4 * 4 + 3])
                       : make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
  uint16_t* orow = a.out + qrow;
#pragma unroll
  for (int db = 0; db < 4; ++db) {
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const u32x2 w = ltot > 0.f ? (u32x2){pack16<F16>(O[db][i4 * 4] * inv, O[db][i4 * 4 + 1] * inv),
                                           pack16<F16>(O[db][i4 * 4 + 2] * inv, O[db][i4 * 4 + 3] * inv)}
                                 : (u32x2){0u, 0u};
      *reinterpret_cast<u32x2*>(orow + db * 32 + i4 * 8 + g * 4) = w;
    }
  }
  if (a.lse && g == 0) {
    a.lse[((int64_t)b * a.n_q + tq) * a.n_q_heads + h] = ltot > 0.f ? mfin * a.scale + logf(ltot) : ninf;
  }
  if (SPARSE && a.count && g == 0) a.count[(int64_t)hslot * a.n_q + tq] = kept;
}

// The first digit of a sliced search, for prefill_order_kernel.
static constexpr auto prefill_first_digit = prefill_select_kernel<kSelScan>;

// The 64-key tiles a 256-query tile of the selecting attention launch has to visit: tile n is on the list iff, for
// one of the tile's eight 32-query groups, the group's largest index product in the tile (tile_max, written by the
// first sweep of prefill_select_kernel) reaches the group's smallest threshold.  Every other tile holds no kept
// pair -- the keep test is product >= threshold -- so leaving it out changes no output, count or sum.
// Grid (query tiles, retrieval heads); the list is ascending.  A thread takes one tile at a time and the eight groups' entries of it at
// once: a chain of dependent loads, and few workgroups, is all there is to this launch (with 256 threads, a group's entry loaded only if the
// groups before had none: 67 us where every tile is on the list, 245 where few are, for 8192 queries behind 1M tokens; 22 now).
// Regrouped queries, grid (.., .., 2): the groups whose queries all keep few keys get a list of their own, which the attention launch walks
// with more exact probabilities; they are all of the query tile's groups, or its last ones (the second list then) in one tile of a block.
constexpr int kListThreads = 1024, kListThreadsFew = 256;    // (up to 32768 keys: two rounds of 256 threads, 4.0 us for 2037 against 5.1)
template <int THREADS>
__global__ __launch_bounds__(THREADS) void prefill_active_tiles_kernel(const PrefillArgs a) {
  constexpr int G = kPwQ / 32;
  const int j = blockIdx.y, qt = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t0 = qt * kPwQ;
  const bool second = blockIdx.z != 0;
  __shared__ float thr[G];
  __shared__ int last[G];                               // the last position of every group (-1: a group past the chunk)
  __shared__ int many[G];                               // some query of the group keeps more than few keys
  __shared__ int wave_n[2][THREADS / 64];
  const int pos0 = (int)a.q_start_host;
  const bool by_kept = a.units && a.order_on[j * ((a.n_q + a.order_block - 1) / a.order_block) + t0 / a.order_block] == kOrderByKept;
  if (tid < kPwQ) {
    int t = t0 + tid;
    const bool qok = t < a.n_q;
    if (a.order && qok) t = a.order[(int64_t)j * a.n_q + t];
    float v = qok ? a.sel_thr[(int64_t)j * a.n_q + t] : __builtin_huge_valf();
    int m = qok ? pos0 + t : -1;
    int cls = by_kept && qok ? a.sl_state[(int64_t)j * a.n_q + t].flags >> kSelClassShift : 0;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) {
      v = fminf(v, __shfl_xor(v, o));
      m = max(m, __shfl_xor(m, o));
      cls = max(cls, __shfl_xor(cls, o));
    }
    if ((tid & 31) == 0) {
      thr[tid >> 5] = v;
      last[tid >> 5] = m;
      many[tid >> 5] = cls >= kFewClass ? 1 : 0;
    }
  }
  __syncthreads();
  // this list's groups
  int n_many = by_kept ? 0 : G;
#pragma unroll
  for (int i = 0; i < G; ++i) if (by_kept && many[i]) n_many = i + 1;
  const bool exact = n_many == 0 || second;
  const int lo = second ? n_many : 0, hi = second || n_many == 0 ? G : n_many;
  const int n_wide = gridDim.x, list_no = (second ? (int)gridDim.y * n_wide : 0) + j * n_wide + qt;
  if (second && (n_many == 0 || n_many == G)) {
    if (tid == 0) a.list_info[list_no] = make_int2(0, 0);
    return;
  }
  // the groups' rows of the table, each as far as the group's last query sees
  float least[G];
  int n_of[G], n_pairs = 0;
#pragma unroll
  for (int i = 0; i < G; ++i) {
    least[i] = thr[i];
    n_of[i] = last[i] < 0 || i < lo || i >= hi ? 0 : last[i] / kPfK + 1;
    n_pairs = max(n_pairs, n_of[i]);
  }
  const float* tm = a.tile_max + ((int64_t)j * ((a.n_q + 31) / 32) + t0 / 32) * a.n_t64;
  int32_t* list = second ? more_list_of(a, j, qt) : a.act_list + ((int64_t)j * n_wide + qt) * a.n_t64;
  auto entries = [&](int p, float (&v)[G]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < G; ++i) v[i] = p < n_of[i] ? tm[(int64_t)i * a.n_t64 + p] : -__builtin_huge_valf();
  };
  int base = 0;
  float v[G];
  entries(tid, v);
  for (int p0 = 0, odd = 0; p0 < n_pairs; p0 += THREADS, odd ^= 1) {
    const int p = p0 + tid;
    bool on = false;
#pragma unroll
    for (int i = 0; i < G; ++i) on = on || (p < n_of[i] && v[i] >= least[i]);
    entries(p + THREADS, v);
    const uint64_t bal = __ballot(on);
    if (lane == 0) wave_n[odd][wave] = __popcll(bal);
    __syncthreads();
    int before = base;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
      const int n = wave_n[odd][w];
      if (w < wave) before += n;
      base += n;
    }
    if (on) list[before + __popcll(bal & ((1ull << lane) - 1ull))] = p;
  }
  if (tid == 0) {
    if (a.units) {
      a.list_info[list_no] = make_int2(base, lo << 16 | hi << 20 | (exact ? kUnitExact : 0));
      atomicAdd(&a.act_count[(int64_t)j * n_wide + qt], base);      // (of both lists; prefill_order_kernel has cleared it)
    } else {
      a.act_count[(int64_t)j * n_wide + qt] = base;
    }
    if (!second) {
      atomicMax(&a.act_range[0], base);
      atomicMin(&a.act_range[1], base);
    }
  }
}

// Cuts the attention launch's work over lists of very different lengths (regrouped queries: hundreds of tiles beside a handful) into
// units of about equal length: every list into equal ranges of at most U tiles, U the least for which there are k units per compute unit,
// which holds one workgroup; the k of 1 to 4 that makes k * (U + kUnitTiles) least, kUnitTiles being what a unit costs beside its tiles: its
// start, a partial result to write and one to merge.  Units of half of U or more come first, by head, range and tile, an eighth of them
// for each die, so that the workgroups of a die walk the same keys at the same time and meet in its L2; the short ones fill up behind.
// Attention launch of 4 heads over regrouped queries, ranges of 512 tiles of each list / planned, us: 4096 queries at 128K tokens, clusters at
// p = 0.9 and 0.8 1060 / 860 and 1044 / 516, a few hard queries among easy ones 1060 / 129, 333 queries 159 / 106.
constexpr int kUnitTiles = 12, kUnitLeast = 16, kUnitRounds = 4, kUnitRanges = 64;
constexpr int kExactTiles = 2;                     // what a tile of the exact pass takes
constexpr int kPlanThreads = 1024, kPlanLists = 4096;
__global__ __launch_bounds__(kPlanThreads) void prefill_plan_kernel(const PrefillArgs a, const int n_cu) {
  constexpr int NW = kPlanThreads / 64;
  __shared__ int len[kPlanLists], cut[kPlanLists];     // a list's tiles; its ranges if they are long units, else 0
  __shared__ int waves[kPlanLists];
  __shared__ int best_u[kUnitRounds], longest[NW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_wide = (a.n_q + kPwQ - 1) / kPwQ, n = 2 * a.n_heads * n_wide;
  // (a second list is there only if it has tiles)
  auto ranges_of = [&](int i, int u) __attribute__((always_inline)) { return max((len[i] + u - 1) / u, 2 * i < n ? 1 : 0); };
  int most = 1;
  {
    const int blocks = (a.n_q + a.order_block - 1) / a.order_block * a.n_heads;
    bool on = false;
    for (int i = tid; i < blocks; i += kPlanThreads) on = on || a.order_on[i] == kOrderByKept;
    if (__syncthreads_or(on ? 1 : 0) == 0) {            // nothing is regrouped
      if (tid == 0) *a.n_units = 0;
      return;
    }
  }
  for (int i = tid; i < n; i += kPlanThreads) {
    const int2 info = a.list_info[i];
    len[i] = info.y & kUnitExact ? info.x * kExactTiles : info.x;
    waves[i] = info.y;
    most = max(most, len[i]);
  }
  most = wave_max_ge_m1(most);
  if (lane == 0) longest[wave] = most;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) most = max(most, longest[w]);
  int n_more = 0;
  for (int i = n / 2 + lane; i < n; i += 64) n_more += len[i] > 0 ? 1 : 0;
  n_more = wave_sum(n_more);
  if (wave < kUnitRounds) {                             // one k for each of the first waves
    const int limit = max(min((wave + 1) * n_cu, a.part_cap), n / 2 + n_more);
    int lo = min(max(kUnitLeast, (most + kUnitRanges - 1) / kUnitRanges), most), hi = most;
    while (lo < hi) {
      const int u = (lo + hi) >> 1;
      int units = 0;
      for (int i = lane; i < n; i += 64) units += ranges_of(i, u);
      if (wave_sum(units) <= limit) hi = u;
      else lo = u + 1;
    }
    if (lane == 0) best_u[wave] = lo;
  }
  __syncthreads();
  int u = 0, cost = 0x7fffffff;
#pragma unroll
  for (int k = 0; k < kUnitRounds; ++k) {
    const int c = (k + 1) * (best_u[k] + kUnitTiles);
    if (c < cost) { cost = c; u = best_u[k]; }
  }
  // prefix sums over the lists: ranges (for the partials), ranges of long units, short units
  __shared__ int3 wave_tot[NW];
  __shared__ int long_before[kPlanLists];
  int3 carry = make_int3(0, 0, 0);
  for (int i0 = 0; i0 < n; i0 += kPlanThreads) {
    const int i = i0 + tid;
    const int r = i < n ? ranges_of(i, u) : 0;
    const bool is_long = r > 0 && 2 * len[i] >= u * r;
    const int3 mine = make_int3(r, is_long ? r : 0, r > 0 && !is_long ? 1 : 0);
    int3 upto = make_int3(wave_incl_scan(mine.x), wave_incl_scan(mine.y), wave_incl_scan(mine.z));
    if (lane == 63) wave_tot[wave] = upto;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int3 t = wave_tot[w];
      if (w < wave) { upto.x += t.x; upto.y += t.y; upto.z += t.z; }
    }
    if (i < n) {
      cut[i] = is_long ? r : 0;
      long_before[i] = carry.y + upto.y - mine.y;
      len[i] = carry.z + upto.z - mine.z;               // (from here on: the short units before)
      a.list_ranges[i] = make_int2(r | ((waves[i] >> 20) & 0xf) << 16, carry.x + upto.x - mine.x);
      if (r == 0) waves[i] = -1;                        // no list
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int3 t = wave_tot[w];
      carry.x += t.x; carry.y += t.y; carry.z += t.z;
    }
    __syncthreads();
  }
  const int n_long = carry.y, per_die = n_long / 8, rest = n_long % 8;
  if (tid == 0) *a.n_units = n_long + carry.z;
  const int share = max(kPlanThreads / n, 1), stride = n > kPlanThreads ? kPlanThreads : n;     // threads per list
  for (int i = tid / share; i < n; i += stride) {
    const int sub = tid % share, h = i / n_wide;        // (the second lists as so many heads more)
    if (waves[i] == -1) continue;
    if (cut[i] == 0) {
      if (sub == 0) a.units[n_long + len[i]] = make_int2(i, 1 << 8 | waves[i]);
      continue;
    }
    const int before = long_before[h * n_wide];
    for (int s = sub; s < cut[i]; s += share) {
      int p = before;
      for (int k = h * n_wide; k < (h + 1) * n_wide; ++k) {
        const int c = cut[k];
        p += min(c, s) + (k < i && c > s ? 1 : 0);
      }
      const bool more = p < rest * (per_die + 1);       // the first `rest` dies have one more
      const int p1 = p - rest * (per_die + 1);
      const int die = more ? p / (per_die + 1) : rest + p1 / max(per_die, 1);
      const int at = more ? p % (per_die + 1) : p1 % max(per_die, 1);
      a.units[at * 8 + die] = make_int2(i, s | cut[i] << 8 | waves[i]);
    }
  }
}

// Merges the key-range partials of a (query, head): SLICES groups of 32 lanes walk the ranges slice, slice + SLICES, ...,
// four partials in flight each, a lane owns 4 of the 128 output dims; LDS merges the slices.  8 / SLICES rows per
// workgroup: two slices where there are few ranges (24 us for 16384 rows of 4 ranges with a thread per dim going through
// the ranges one by one, 11 now), all eight where a short chunk's keys are cut into dozens (43 and 5 us for 256 rows of 64).
template <int SLICES, bool ORDERED = false>
__global__ __launch_bounds__(256) void prefill_combine_kernel(const PrefillArgs a) {
  __shared__ float sh_m[8], sh_l[8];
  __shared__ int sh_kept[8];
  __shared__ __attribute__((aligned(16))) float sh_acc[8][kHeadDim];
  const int tid = threadIdx.x, d4 = tid & 31, grp = tid >> 5, slice = grp % SLICES, hs = blockIdx.y;
  const int place = blockIdx.x * (8 / SLICES) + grp / SLICES;
  const bool row = place < a.n_q;
  int t = place, n_splits;
  const float* part = a.part;
  int64_t step;                                                         // from one range's partials to the next
  if (ORDERED && *a.n_units > 0) {                       // (partials lie by place)
    const int n_wide = (a.n_q + kPwQ - 1) / kPwQ, at = min(place, a.n_q - 1), list = hs * n_wide + at / kPwQ;
    int2 ranges = a.list_ranges[list];
    if (at % kPwQ / 32 >= ranges.x >> 16) ranges = a.list_ranges[a.n_heads * n_wide + list];
    n_splits = ranges.x & 0xffff;
    if (n_splits == 1) return;                           // (the same for the whole workgroup: the attention launch has written the rows)
    part += ((int64_t)ranges.y * kPwQ + place % kPwQ) * kPfPart;
    step = (int64_t)kPwQ * kPfPart;
    if (row) t = a.order[(int64_t)hs * a.n_q + place];
  } else {                                               // (by query, which is the place)
    n_splits = (a.act_range ? listed_splits(a) : a.n_splits) * a.n_sub;   // (a listed launch decides on the device)
    part += ((int64_t)hs * a.n_q + (row ? t : 0)) * kPfPart;
    step = (int64_t)a.n_heads * a.n_q * kPfPart;
  }
  const float ninf = -__builtin_huge_valf();
  float M = ninf, L = 0.f;
  float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
  int kept = 0;
  for (int s0 = slice; row && s0 < n_splits; s0 += 4 * SLICES) {
    float pm[4], pl[4];
    int pk[4];
    float4 pv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int s = s0 + u * SLICES;
      pm[u] = ninf; pl[u] = 0.f; pk[u] = 0; pv[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (s < n_splits) {
        const float* p = part + s * step;
        const float4 h = *reinterpret_cast<const float4*>(p);
        pm[u] = h.x; pl[u] = h.y; pk[u] = __float_as_int(h.z);
        pv[u] = *reinterpret_cast<const float4*>(p + 4 + d4 * 4);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      kept += pk[u];
      const float Mn = fmaxf(M, pm[u]);
      if (Mn != ninf) {
        const float c0 = fast_exp2((M - Mn) * a.scale_log2), c1 = fast_exp2((pm[u] - Mn) * a.scale_log2);
        L = L * c0 + pl[u] * c1;
        A.x = A.x * c0 + pv[u].x * c1; A.y = A.y * c0 + pv[u].y * c1;
        A.z = A.z * c0 + pv[u].z * c1; A.w = A.w * c0 + pv[u].w * c1;
        M = Mn;
      }
    }
  }
  if (d4 == 0) { sh_m[grp] = M; sh_l[grp] = L; sh_kept[grp] = kept; }
  *reinterpret_cast<float4*>(&sh_acc[grp][d4 * 4]) = A;
  __syncthreads();
  if (slice != 0 || !row) return;
  float Mt = ninf, Lt = 0.f;
  float4 At = make_float4(0.f, 0.f, 0.f, 0.f);
  kept = 0;
#pragma unroll
  for (int k = 0; k < SLICES; ++k) { Mt = fmaxf(Mt, sh_m[grp + k]); kept += sh_kept[grp + k]; }
  if (Mt != ninf) {
#pragma unroll
    for (int k = 0; k < SLICES; ++k) {
      const float cw = fast_exp2((sh_m[grp + k] - Mt) * a.scale_log2);
      const float4 v = *reinterpret_cast<const float4*>(&sh_acc[grp + k][d4 * 4]);
      Lt += sh_l[grp + k] * cw;
      At.x += v.x * cw; At.y += v.y * cw; At.z += v.z * cw; At.w += v.w * cw;
    }
  }
  const int h = a.heads[hs];
  const int64_t o = (int64_t)t * a.n_q_heads + h;        // single sequence
  const float inv = Lt > 0.f ? 1.f / Lt : 0.f;
  const u32x2 w = a.f16 ? (u32x2){pack16<true>(At.x * inv, At.y * inv), pack16<true>(At.z * inv, At.w * inv)}
                        : (u32x2){pack16<false>(At.x * inv, At.y * inv), pack16<false>(At.z * inv, At.w * inv)};
  *reinterpret_cast<u32x2*>(a.out + o * kHeadDim + d4 * 4) = w;
  if (d4 != 0) return;
  if (a.lse) a.lse[o] = Lt > 0.f ? Mt * a.scale + logf(Lt) : ninf;
  if (a.act_range && a.count) a.count[(int64_t)hs * a.n_q + t] = kept;   // selecting mode: kept keys over all key ranges
}

// Compute units of the current device (256 on the target; also the answer where no device is visible,
// as when only a workspace size is asked for).
static int compute_units() {
  static const int v = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
      (void)hipGetLastError();
      n = 256;
    }
    return n;
  }();
  return v;
}

static void launch_prefill_combine(const PrefillArgs& a, hipStream_t s) {
  // (planned ranges: two units per compute unit over lists of about equal length; the partials there can be are far more)
  const int expected = a.units ? std::min<int>(kUnitRanges, 2 * compute_units() / (a.n_heads * ((a.n_q + kPwQ - 1) / kPwQ))) : a.n_splits * a.n_sub;
  const dim3 grid8((unsigned)a.n_q, (unsigned)a.n_heads), grid2((unsigned)((a.n_q + 3) / 4), (unsigned)a.n_heads);
  if (a.order && expected > 8) RTP_LAUNCH((prefill_combine_kernel<8, true>), grid8, dim3(256), 0, s, a);
  else if (a.order) RTP_LAUNCH((prefill_combine_kernel<2, true>), grid2, dim3(256), 0, s, a);
  else if (expected > 8) RTP_LAUNCH(prefill_combine_kernel<8>, grid8, dim3(256), 0, s, a);
  else RTP_LAUNCH(prefill_combine_kernel<2>, grid2, dim3(256), 0, s, a);
}

// Number of key-range splits for a dense launch with few workgroups (long context, few heads).  A
// compute unit holds ONE workgroup of the wide kernel (its LDS), so a launch runs in rounds of as many
// workgroups as there are compute units: the split count is the one that fills its last round best (at
// most 8, at least 32 key tiles per part), a smaller count winning near-ties because every part costs a
// partial result to write and merge.  Measured on the 131072- and 1048576-token configurations (64 and 128
// query-tile workgroups): 4 and 2 parts beat the former 8 by 4 and 2 %, 3 or 6 parts lose 15 to 20 %.
static int choose_splits(int n_heads, int32_t T, int64_t chunk_start) {
  const int64_t wgs = (int64_t)n_heads * ((T + kPwQ - 1) / kPwQ);
  const int64_t avg_tiles = (chunk_start + T / 2) / kPfK + 1;
  int64_t smax = avg_tiles / 32;
  if (smax > 8) smax = 8;
  if (wgs <= 0 || smax <= 1) return 1;
  const int64_t cus = compute_units();
  int best = 1;
  double best_cost = 0.0;
  for (int s = 1; s <= (int)smax; ++s) {
    const int64_t total = wgs * s, rounds = (total + cus - 1) / cus;
    const double cost = (double)(rounds * cus) / (double)total * (1.0 + 0.02 * (s - 1));
    if (s == 1 || cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}

// Key ranges of a selecting launch that follows a threshold search: the query tiles' lists differ in length by
// orders of magnitude (a tile with one hard query visits everything, its neighbour a few dozen tiles), and the
// host does not see the lengths.  Ranges of at most ~512 listed tiles, many more workgroups than compute units:
// the hardware's workgroup dispatch does the balancing, a workgroup with an empty range leaves at once.
static int choose_splits_listed(int n_heads, int32_t T, int64_t chunk_start) {
  const int64_t max_tiles = (chunk_start + T - 1) / kPfK + 1;
  int64_t s = (max_tiles + 511) / 512;
  if (s > 32) s = 32;
  const int base = choose_splits(n_heads, T, chunk_start);
  return s > base ? (int)s : base;
}

// Sub-ranges per key range for launches that leave compute units idle all the same (short chunks): as many as fill
// them, of at least 8 tiles, at most 64 ranges in all.  A sub-range repeats the score product of one tile for its
// reference and leaves one more partial to merge.  Chunks of 64 queries behind 60000 tokens: 113 -> 26 us for the
// attention launch, 333 queries behind 131072 (search and lists): 453 -> 145, a 2037-query prompt: 65 -> 25.
static int choose_sub(int n_heads, int32_t T, int64_t chunk_start, int n_base, int n_splits) {
  const int64_t wgs = (int64_t)n_heads * ((T + kPwQ - 1) / kPwQ) * n_base;
  const int64_t max_tiles = (chunk_start + T - 1) / kPfK + 1;
  if (wgs <= 0) return 1;
  const int64_t s = std::min(std::min((int64_t)compute_units() / wgs, max_tiles / (8 * n_base)), (int64_t)64 / n_splits);
  return s > 1 ? (int)s : 1;
}

// The most key tiles that the band of a query tile can have: sinks apart from the window, and no position from max_ctx on.  (Where
// max_ctx is far above the contexts there are, the bands of their first 192 queries take two groups all the same: 1 to 2 us.)
static int64_t band_tiles(const PrefillArgs& a, int64_t max_ctx) {
  const int64_t span = std::max<int64_t>(a.window, 1) - 1 + std::min(a.n_q, kPfQ);       // window of the first query to the last query
  return std::min((max_ctx + kPfK - 1) / kPfK, ((int64_t)a.sink + kPfK - 1) / kPfK + (span + kPfK - 2) / kPfK + 1);
}

// Ranges of a band's key tiles, of at least eight tiles each, for launches of one sequence that leave compute units idle: a workgroup's way
// through its tiles is a chain of 2.5 us a step, whoever else is there.  28 heads, window 2048, behind 131072 tokens, launch / with the merge: 32
// queries 44 / 21 us, 256 (four ranges) 54 / 31, 333 (three) 57 / 36, 512 (two) 54 / 44.
static int band_splits(const PrefillArgs& a, int32_t B, int64_t max_ctx) {
  const int64_t units = (int64_t)a.n_heads * ((a.n_q + kPfQ - 1) / kPfQ);
  if (B != 1 || units <= 0) return 1;
  const int64_t s = std::min(compute_units() / units, band_tiles(a, max_ctx) / 8);
  return s > 1 ? (int)std::min<int64_t>(s, 8) : 1;
}
static size_t band_bytes(int n_heads, int32_t n_q, int splits) { return align_up((size_t)splits * n_heads * n_q * kPfPart * sizeof(float), 256); }

static int32_t launch_prefill(const char* who, bool local, PrefillArgs& a, int32_t B, int64_t max_ctx, hipStream_t s) {
  if (a.n_heads == 0) return RTP_OK;
  if (a.n_splits < 1) a.n_splits = 1;
  if (a.n_sub < 1) a.n_sub = 1;
  // dense launches take the wide kernel; the local band (a few dozen key tiles per query tile, many of
  // them masked) stays on the 128-query kernel, whose masked tiles cost less (4096 queries, 28 heads, window 2048:
  // 205 us against 480 on the wide kernel)
  const int qt = local ? kPfQ : kPwQ;
  dim3 grid((unsigned)a.n_heads, (unsigned)((a.n_q + qt - 1) / qt), (unsigned)(B * (local ? 1 : a.n_splits * a.n_sub)));
  if (grid.y > 65535 || grid.z > 65535) return fail(RTP_ERR_INVALID_ARG, "%s: n_q / B too large for one launch", who);
  if (local) {
    const int64_t n_unit = (int64_t)grid.x * grid.y * grid.z;
    if (n_unit <= compute_units() && band_tiles(a, max_ctx) >= 4) {
      grid.z *= a.n_splits;
      if (a.f16) RTP_LAUNCH((flash_prefill_local_kernel<true, 2>), grid, dim3(2 * kPfThreads), 0, s, a);
      else RTP_LAUNCH((flash_prefill_local_kernel<false, 2>), grid, dim3(2 * kPfThreads), 0, s, a);
      if (a.n_splits > 1) launch_prefill_combine(a, s);
    } else {
      // Query tiles whose whole window lies before the chunk take equally long; of a prompt's, the early ones are short, and an eighth in one
      // piece is not an eighth of the work (calls with a prompt's 4096 queries, 28 local heads, window 2048: 247 us, 264 by die; 1024, 61 heads,
      // window 512: 89 and 93).
      a.by_die = B == 1 && max_ctx - a.n_q >= a.window;
      if (a.by_die) grid = dim3((unsigned)((n_unit + 7) / 8 * 8));
      if (a.f16) RTP_LAUNCH((flash_prefill_local_kernel<true, 1>), grid, dim3(kPfThreads), 0, s, a);
      else RTP_LAUNCH((flash_prefill_local_kernel<false, 1>), grid, dim3(kPfThreads), 0, s, a);
    }
  } else if (a.f16) RTP_LAUNCH((flash_prefill_wide_kernel<kModeDense, true>), grid, dim3(kPwThreads), 0, s, a);
  else RTP_LAUNCH(flash_prefill_wide_kernel<kModeDense>, grid, dim3(kPwThreads), 0, s, a);
  if (!local && a.n_splits * a.n_sub > 1) launch_prefill_combine(a, s);
  return check_launch(who);
}

static int32_t check_prefill_common(const char* who, const void* q, const void* K, const void* V, int64_t row_stride,
                                    int64_t head_stride, const void* out) {
  if (!q || !K || !V || !out) return fail(RTP_ERR_INVALID_ARG, "%s: NULL tensor pointer", who);
  if (row_stride < kHeadDim || (row_stride & 7) || (head_stride & 7) || head_stride < 0)
    return fail(RTP_ERR_INVALID_ARG, "%s: kv_row_stride must be >= 128, strides multiples of 8", who);
  if (row_stride > (1 << 24))   // a 64-row tile must span less than 4 GiB (32-bit lane offsets inside a tile)
    return fail(RTP_ERR_INVALID_ARG, "%s: kv_row_stride must be at most 2^24 elements", who);
  if (((uintptr_t)q & 15) || ((uintptr_t)K & 15) || ((uintptr_t)V & 15) || ((uintptr_t)out & 15))
    return fail(RTP_ERR_INVALID_ARG, "%s: q, K, V and out must be 16-byte aligned", who);
  return RTP_OK;
}

// rtp_local_attn / rtp_dense_attn with q_start != NULL.
int32_t prefill_range_attn(const char* who, bool dense, const rtp_layer_desc* L, const void* q, const void* K,
                           const void* V, int64_t row_stride, int64_t head_stride, const int64_t* seq_start,
                           const int32_t* ctx_len, const int32_t* q_start, int32_t B, int32_t n_q, int64_t max_ctx,
                           void* out, float* lse, void* ws, size_t ws_bytes, hipStream_t s) {
  HeadTable ht;
  int32_t rc = fill_head_table(L, &ht, who);
  if (rc != RTP_OK) return rc;
  rc = check_prefill_common(who, q, K, V, row_stride, head_stride, out);
  if (rc != RTP_OK) return rc;
  if (!seq_start || !ctx_len || !q_start) return fail(RTP_ERR_INVALID_ARG, "%s: NULL seq_start/ctx_len/q_start", who);
  if (B <= 0 || n_q <= 0 || max_ctx <= 0) return fail(RTP_ERR_INVALID_ARG, "%s: B, n_q and max_ctx must be positive", who);
  if (max_ctx > 0x7fffffffLL - kPwQ) return fail(RTP_ERR_INVALID_ARG, "%s: max_ctx too large", who);
  clear_error();
  PrefillArgs a = {};
  a.q = (const uint16_t*)q;
  a.K = (const uint16_t*)K;
  a.V = (const uint16_t*)V;
  a.row_stride = row_stride;
  a.head_stride = head_stride;
  a.seq_start = seq_start;
  a.q_start = q_start;
  a.n_q = n_q;
  a.n_q_heads = L->n_q_heads;
  a.n_kv_heads = L->n_kv_heads;
  a.sink = L->sink;
  a.window = L->window;
  a.scale = softmax_scale_of(L);
  a.f16 = L->kv_dtype == RTP_DTYPE_FP16;
  a.scale_log2 = a.scale * 1.4426950408889634f;
  a.out = (uint16_t*)out;
  a.lse = lse;
  a.n_heads = 0;
  for (int h = 0; h < L->n_q_heads; ++h)
    if (dense || !ht.is_ret[h]) a.heads[a.n_heads++] = (uint8_t)h;
  if (!dense && ws && !((uintptr_t)ws & 255)) {
    const int splits = band_splits(a, B, max_ctx);
    if (splits > 1 && ws_bytes >= band_bytes(a.n_heads, n_q, splits)) {
      a.n_splits = splits;
      a.part = (float*)ws;
    }
  }
  return launch_prefill(who, !dense, a, B, max_ctx, s);
}
// What every chunk of at most n_q queries can use: a server has one workspace, and it is the short last chunk that is cut into ranges.
// (Of the chunks with as many query tiles the longest has the most ranges and the largest ones; beyond half a workgroup per compute unit there are none.)
size_t prefill_range_ws(const rtp_layer_desc* L, int32_t B, int32_t n_q, int64_t max_ctx) {
  if (!L || n_q <= 1 || B != 1 || L->n_q_heads <= L->n_ret) return 0;
  PrefillArgs a = {};
  a.n_heads = L->n_q_heads - L->n_ret;
  a.sink = L->sink;
  a.window = L->window;
  size_t most = 0;
  for (int tiles = 1; 2 * tiles * a.n_heads <= compute_units(); ++tiles) {
    a.n_q = (int32_t)std::min<int64_t>(n_q, (int64_t)tiles * kPfQ);
    const int splits = band_splits(a, B, max_ctx);
    if (splits > 1) most = std::max(most, band_bytes(a.n_heads, a.n_q, splits));
    if (a.n_q == n_q) break;
  }
  return most;
}

// Workgroups per 32-query group of the threshold search: as many as fill two workgroups per compute unit, each with at
// least 4096 keys of the longest range, at most 16.  The five launches cost about 50 us beside the sweeps, what one
// workgroup needs for 9000 keys of a broad score law: the slices have to save more than that (1 to 64 queries behind
// 60000 tokens: 82 to 93 us against some 400 in one launch; 1000 queries behind 5000 tokens stay at 62 in one).
// `room`: bytes there are for what the launches hand on; fewer slices where it holds no more.
struct SearchWs {
  size_t max_bytes, hist_bytes, state_bytes, again_bytes;
  size_t total() const { return max_bytes + hist_bytes + state_bytes + again_bytes; }
};
static SearchWs search_ws(int64_t groups, int64_t workgroups) {
  SearchWs w = {};
  w.max_bytes = align_up((size_t)workgroups * 32 * sizeof(float), 256);
  w.hist_bytes = align_up((size_t)workgroups * 2 * kSelBins * 32 * sizeof(double), 256);
  w.state_bytes = align_up((size_t)groups * 2 * 32 * sizeof(SelState), 256);       // (two per query)
  w.again_bytes = align_up((size_t)groups * sizeof(int32_t), 256);
  return w;
}
static int search_slices(int n_ret, int32_t T, int64_t chunk_start, size_t room) {
  const int64_t groups = (int64_t)n_ret * ((T + 31) / 32), keys = chunk_start + T;
  int64_t s = std::min(2 * (int64_t)compute_units() / groups, std::min(keys / 4096, (int64_t)16));
  while (s >= 2 && search_ws(groups, groups * s).total() > room) --s;
  return s >= 2 && keys - keys / s > 9000 ? (int)s : 1;
}

// Queries that prefill_order_kernel may regroup together (0: none).  A group's masked tiles reach from its first query to its last, so
// the block is at most a sixteenth of what lies before the chunk.  The launches more take 20 to 45 us, which laws with nothing to regroup lose: below
// 65536 keys, 512 queries or 1.2e9 pairs of query and key over all heads that is 2 to 3 % of the call, above up to 2 near the line.  Calls of 4 heads, us, by position /
// regrouped, clusters, projected queries (a sixth of the context kept by all) and a peaked law: 4096 queries at 128K tokens 2520 / 2200, 2445 /
// 2445, 842 / 837; 3000 there 2325 / 1853, 2232 / 2219, 831 / 814; 4096 behind 98304 1994 / 1816, 1955 / 1988, 707 / 711; 1024 behind 400000 1932 / 1743,
// 1882 / 1892, 673 / 622; on the other side of the line 4000 behind 65536 1240 / 1130, 1349 / 1394, 548 / 561; 1000 at 128K 730 / 670, 699 / 716,
// 299 / 303.
// (Which of the two it is also follows from the workspace, and the probabilities are rounded to 16 bits against different references: chunks of
// less than 512 queries are left one result whatever their workspace; 333 queries behind 131072 would gain 4 %.)
// More lists than prefill_plan_kernel holds: by position.  Without planned units the attention's ranges are as uneven as the lists, and queries that
// keep few keys lose their exact pass; 64 heads, 8193 queries behind 60000 tokens, ms, by position / regrouped without a plan: clusters 37.5 / 32.6, Zipf
// clusters 36.2 / 33.5, projected queries 36.9 / 37.7, peaked 9.9 / 10.9, a few hard queries 13.6 / 15.5.
static int order_block(int n_ret, int32_t T, int64_t chunk_start) {
  if ((int64_t)2 * n_ret * ((T + kPwQ - 1) / kPwQ) > kPlanLists) return 0;
  if (chunk_start + T < 65536 || T < 2 * kPwQ || (double)n_ret * T * (double)(chunk_start + T) < 1.2e9) return 0;
  const int64_t most = std::min<int64_t>(chunk_start / 16 / kPwQ * kPwQ, kOrderMax);
  return T <= most ? (T + kPwQ - 1) / kPwQ * kPwQ : most >= 1024 ? (int)most : 0;
}
// Workgroups per group of the last sweeps behind regrouped queries whose first sweeps took whole rows: their lengths differ by two orders of
// magnitude, so two rounds of workgroups for the chip's dispatcher to even out, of at most 262144 keys (a lone hard group's time is all of the
// launch's).  Sweeps 2 and 3 of 4096 queries at 128K tokens, p = 0.9 and 0.8, one round / two / four: 411 + 226 and 373 + 200 us / 384 + 217
// and 276 + 146 / 360 + 220 and 271 + 155.  A search that is sliced from the start keeps its one round: a workgroup's start (the order, the state, the ends
// of the member ranges: some 10 us) costs more than the evener end gives.
static int order_slices(int64_t groups, int64_t keys) {
  return (int)std::min<int64_t>(std::max<int64_t>({std::min(4 * (int64_t)compute_units() / groups, keys / 4096), keys / 262144, (int64_t)1}), 16);
}

// Sizes of the tile bookkeeping of a selecting launch.  A table row has one entry per 64 keys of the context, plus
// the entries the threshold search touches past a group's last tile (its sweeps run in whole rounds of four or eight tiles of
// 32 keys and read the table one round ahead: four entries at most, sixteen are there).
struct PrefillTileWs {
  int32_t n_t64;
  size_t table_bytes, list_bytes, count_bytes;
};
static PrefillTileWs prefill_tile_ws(int32_t n_ret, int32_t T, int64_t chunk_start) {
  PrefillTileWs w;
  w.n_t64 = (int32_t)(((chunk_start + T + 31) / 32 + 32) / 2 + 1);
  w.table_bytes = align_up((size_t)n_ret * ((T + 31) / 32) * w.n_t64 * sizeof(float), 256);
  w.list_bytes = align_up((size_t)n_ret * ((T + kPwQ - 1) / kPwQ) * w.n_t64 * sizeof(int32_t), 256);
  w.count_bytes = align_up(((size_t)n_ret * ((T + kPwQ - 1) / kPwQ) + 2) * sizeof(int32_t), 256);   // + {longest, shortest}
  return w;
}

// The order, a flag per block, and the attention launch's units with their number and the lists' ranges.
struct OrderWs {
  size_t order, flags, units, info, ranges, more;
  size_t total() const { return order + flags + units + info + ranges + more; }
};
static int order_blocks(int32_t T) { return (T + 1023) / 1024 + 1; }     // at most
static int max_units(int n_ret, int32_t T) { return std::max(kUnitRounds * compute_units(), n_ret * ((T + kPwQ - 1) / kPwQ + order_blocks(T))); }
static OrderWs order_ws(int n_ret, int32_t T, int64_t chunk_start) {
  OrderWs w;
  w.order = align_up((size_t)n_ret * T * sizeof(int32_t), 256);
  const size_t lists = (size_t)n_ret * ((T + kPwQ - 1) / kPwQ);
  w.flags = align_up((size_t)n_ret * order_blocks(T) * sizeof(int32_t), 256);
  w.units = align_up(((size_t)max_units(n_ret, T) + 1) * sizeof(int2), 256);
  w.info = w.ranges = align_up(2 * lists * sizeof(int2), 256);
  w.more = align_up((size_t)n_ret * order_blocks(T) * prefill_tile_ws(n_ret, T, chunk_start).n_t64 * sizeof(int32_t), 256);
  return w;
}
// Key ranges of a launch for the retrieval heads under either rule.
struct PrefillRanges {
  int dense, dense_sub, listed, listed_sub;
};
static PrefillRanges prefill_ranges(int n_ret, int32_t T, int64_t chunk_start) {
  PrefillRanges r;
  r.dense = choose_splits(n_ret, T, chunk_start);
  r.listed = choose_splits_listed(n_ret, T, chunk_start);
  r.dense_sub = choose_sub(n_ret, T, chunk_start, r.dense, r.dense);
  r.listed_sub = choose_sub(n_ret, T, chunk_start, r.dense, r.listed);
  return r;
}
static size_t range_bytes(int n_ret, int32_t T) { return (size_t)n_ret * T * kPfPart * sizeof(float); }   // one range's partials
static size_t partial_bytes(int ranges, int n_ret, int32_t T) { return ranges > 1 ? align_up(ranges * range_bytes(n_ret, T), 256) : 0; }

// The workspace: projected index queries | one threshold per (retrieval head, query) | tile-maximum table, tile lists and
// their lengths | scratch.  The scratch first carries what the launches of a sliced search hand on and then, when the
// search is over, the key-range partials.  A call needs room for the partials of its ranges (prefill_needed); how many
// slices and sub-ranges it takes follows from the scratch it was given, so that a short chunk runs in the workspace of a
// long one.
struct PrefillWs {
  size_t proj, state, tiles;             // bytes of the parts in front of the scratch
  PrefillTileWs tw;
  size_t front() const { return proj + state + tiles; }
};
static PrefillWs prefill_ws(int n_ret, int32_t T, int64_t chunk_start) {
  PrefillWs w;
  w.proj = align_up((size_t)n_ret * T * kIndexDim * sizeof(uint16_t), 256);
  w.state = align_up((size_t)n_ret * T * sizeof(float), 256);
  w.tw = prefill_tile_ws(n_ret, T, chunk_start);
  w.tiles = w.tw.table_bytes + w.tw.list_bytes + w.tw.count_bytes;
  return w;
}
static size_t prefill_needed(int n_ret, int32_t T, int64_t chunk_start) {
  return prefill_ws(n_ret, T, chunk_start).front() + partial_bytes(choose_splits_listed(n_ret, T, chunk_start), n_ret, T);
}
// The scratch that lets every chunk of at most T queries that ends where this one does run at full speed: the largest
// partials of any of them and the most a sliced search takes.  For as many 256-query tiles the ranges follow from the average
// depth alone, which moves by two key tiles: the first and the last such chunk show every choice.  The size function therefore
// never answers less for a longer chunk with the same end.
static size_t prefill_scratch(int n_ret, int32_t T, int64_t chunk_start) {
  const int64_t end = chunk_start + T, groups = (int64_t)n_ret * ((T + 31) / 32);
  size_t most = 0;
  for (int64_t first = 1; first <= T; first += kPwQ) {
    const int32_t last = (int32_t)std::min<int64_t>(T, first + kPwQ - 1);
    int ranges = 1;
    for (const int64_t t : {first, (int64_t)last}) {
      const PrefillRanges r = prefill_ranges(n_ret, (int32_t)t, end - t);
      ranges = std::max(ranges, std::max(r.dense * r.dense_sub, r.listed * r.listed_sub));
    }
    most = std::max(most, partial_bytes(ranges, n_ret, last));
  }
  const int64_t cus = compute_units(), wgs = std::min(groups * std::min(end / 4096, (int64_t)16), 2 * cus);
  most = std::max(most, end > 9000 ? search_ws(std::min(groups, cus), wgs).total() : 0);
  if (end >= 65536 && T >= 2 * kPwQ) {
    const int64_t regrouped = std::max(groups * std::min(std::max(end / 262144, (int64_t)1), (int64_t)16), std::min(groups * std::min(end / 4096, (int64_t)16), 4 * cus));
    most = std::max(most, search_ws(groups, regrouped).total()) + order_ws(n_ret, T, chunk_start).total();
  }
  return most;
}

}  // namespace rtp

using namespace rtp;

extern "C" size_t rtp_sparse_attn_prefill_workspace_bytes(const rtp_layer_desc* layer, int32_t T, int64_t chunk_start) {
  if (!layer || T <= 0 || layer->n_ret <= 0) return 256;
  const int64_t c0 = chunk_start < 0 ? 0 : chunk_start;
  return prefill_ws(layer->n_ret, T, c0).front() + prefill_scratch(layer->n_ret, T, c0);
}

extern "C" int32_t rtp_sparse_attn_prefill(const rtp_layer_desc* layer, const void* q_pre, const void* q, const float* WQ,
                                           const void* kI, int64_t kI_head_stride,
                                           const void* K, const void* V, int64_t kv_row_stride, int64_t kv_head_stride,
                                           int64_t chunk_start, int32_t T, float p, void* out, float* lse,
                                           float* tau, int32_t* count, float* mass,
                                           void* ws, size_t ws_bytes, void* stream) {
  const char* who = "rtp_sparse_attn_prefill";
  HeadTable ht;
  int32_t rc = fill_head_table(layer, &ht, who);
  if (rc != RTP_OK) return rc;
  rc = check_prefill_common(who, q, K, V, kv_row_stride, kv_head_stride, out);
  if (rc != RTP_OK) return rc;
  if (T <= 0 || chunk_start < 0) return fail(RTP_ERR_INVALID_ARG, "%s: T must be positive and chunk_start >= 0", who);
  if (chunk_start + T > 0x7fffffffLL - kPwQ) return fail(RTP_ERR_INVALID_ARG, "%s: context too long", who);
  if (!(p > 0.f)) return fail(RTP_ERR_INVALID_ARG, "%s: p must be > 0", who);
  if ((T + kPfQ - 1) / kPfQ > 65535) return fail(RTP_ERR_INVALID_ARG, "%s: T too large for one launch", who);
  const bool sparse = p < 1.f || tau || count || mass;
  if (sparse) {
    if (!q_pre || !kI) return fail(RTP_ERR_INVALID_ARG, "%s: NULL index tensors", who);
    if (((uintptr_t)q_pre & 15) || ((uintptr_t)kI & 15) || (kI_head_stride & 7) || kI_head_stride < 0)
      return fail(RTP_ERR_INVALID_ARG, "%s: index tensors must be 16-byte aligned, kI_head_stride a multiple of 8", who);
    if (layer->n_ret > 0) {
      const size_t need = prefill_needed(layer->n_ret, T, chunk_start);
      if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need)
        return fail(RTP_ERR_WORKSPACE, "%s: workspace of %zu bytes (256-byte aligned) required, got %zu", who, need, ws_bytes);
    }
  }
  clear_error();
  if (layer->n_ret == 0) return RTP_OK;
  PrefillArgs a = {};
  a.q = (const uint16_t*)q;
  a.K = (const uint16_t*)K;
  a.V = (const uint16_t*)V;
  a.row_stride = kv_row_stride;
  a.head_stride = kv_head_stride;
  a.seq_start = nullptr;
  a.q_start = nullptr;
  a.q_start_host = chunk_start;
  a.n_q = T;
  a.n_q_heads = layer->n_q_heads;
  a.n_kv_heads = layer->n_kv_heads;
  a.sink = layer->sink;
  a.window = layer->window;
  a.scale = softmax_scale_of(layer);
  a.f16 = layer->kv_dtype == RTP_DTYPE_FP16;
  a.scale_log2 = a.scale * 1.4426950408889634f;
  a.out = (uint16_t*)out;
  a.lse = lse;
  a.n_heads = layer->n_ret;
  for (int j = 0; j < layer->n_ret; ++j) a.heads[j] = (uint8_t)layer->ret_heads[j];
  a.tau = tau;
  a.count = count;
  a.mass = mass;
  const PrefillRanges ranges = prefill_ranges(layer->n_ret, T, chunk_start);
  if (!(p < 1.f)) {                                  // the paper's dense prefill rule: nothing to score, nothing to select
    // (the partials are all this rule keeps in the workspace; without room for them: one range)
    const size_t room = ws && !((uintptr_t)ws & 255) ? ws_bytes / range_bytes(layer->n_ret, T) : 0;
    const bool split = room >= (size_t)ranges.dense;
    a.n_splits = split ? ranges.dense : 1;
    a.n_sub = split ? (int32_t)std::min<size_t>(ranges.dense_sub, room / ranges.dense) : 1;
    a.part = (float*)ws;
    return launch_prefill(who, false, a, 1, chunk_start + T, (hipStream_t)stream);
  }

  // index queries: given, or projected in fp64 into the workspace first
  const uint16_t* qI = (const uint16_t*)q_pre;
  if (WQ) {
    IndexProjectArgs pa;
    pa.W = WQ;
    pa.x = (const uint16_t*)q_pre;
    pa.out = (uint16_t*)ws;
    pa.out_head_stride = (int64_t)T * kIndexDim;
    pa.out_t0 = 0;
    pa.T = T;
    pa.n_x_heads = layer->n_q_heads;
    for (int j = 0; j < 64; ++j) pa.x_head[j] = j < layer->n_ret ? layer->ret_heads[j] : 0;
    launch_index_project(pa, layer->n_ret, (hipStream_t)stream);
    qI = (const uint16_t*)ws;
  }
  a.qI = qI;
  a.kI = (const uint16_t*)kI;
  a.kI_head_stride = kI_head_stride;
  a.p = p;
  a.index_scale = index_scale_of(layer);
  const PrefillWs w = prefill_ws(layer->n_ret, T, chunk_start);
  char* const tiles = (char*)ws + w.proj + w.state;
  char* scratch = (char*)ws + w.front();
  size_t room = ws_bytes - w.front();
  const int64_t groups = (int64_t)layer->n_ret * ((T + 31) / 32), keys = chunk_start + T;
  a.sel_thr = (float*)((char*)ws + w.proj);
  a.n_splits = ranges.listed;
  a.n_slice = search_slices(layer->n_ret, T, chunk_start, room);
  // regrouped queries: where the scratch has room for the order beside the partials of the ranges and what the sweeps leave
  int last_slices = a.n_slice;
  if (const int block = order_block(layer->n_ret, T, chunk_start)) {
    const OrderWs ow = order_ws(layer->n_ret, T, chunk_start);
    const size_t ob = ow.total();
    // (the sweeps before the order keep their slices as well, for which there is room already without it)
    const size_t parts = partial_bytes(ranges.listed, layer->n_ret, T);
    int first = a.n_slice, last = a.n_slice > 1 ? a.n_slice : order_slices(groups, keys);
    while (first > 1 && search_ws(groups, groups * first).total() + ob > room) --first;
    while (last > 1 && search_ws(groups, groups * last).total() + ob > room) --last;
    if (std::max({search_ws(groups, groups * std::max(first, last)).total(), parts}) + ob <= room && (first > 1 || a.n_slice == 1)) {
      last_slices = last;
      a.order_whole = a.n_slice == 1;
      a.n_slice = first;
      a.order = (int32_t*)scratch;
      a.order_on = (int32_t*)(scratch + ow.order);
      char* const at = scratch + ow.order + ow.flags;
      a.units = (int2*)at + 1;
      a.n_units = (int32_t*)at;
      a.list_info = (int2*)(at + ow.units);
      a.list_ranges = (int2*)(at + ow.units + ow.info);
      a.more_list = (int32_t*)(at + ow.units + ow.info + ow.ranges);
      a.order_block = block;
      a.one_round = 2 * compute_units();
      scratch += ob;
      room -= ob;
    }
  }
  a.part = (float*)scratch;
  a.n_sub = (int32_t)std::max<size_t>(std::min<size_t>(ranges.listed_sub, room / range_bytes(layer->n_ret, T) / ranges.listed), 1);
  if (a.units) {
    a.part_cap = (int32_t)std::min<size_t>(room / ((size_t)kPwQ * kPfPart * sizeof(float)), kUnitRounds * compute_units());
  }
  {
    const SearchWs sw = search_ws(groups, groups * std::max(a.n_slice, last_slices));
    a.sl_max = (float*)scratch;
    a.sl_hist = (double*)(scratch + sw.max_bytes);
    a.sl_state = (SelState*)(scratch + sw.max_bytes + sw.hist_bytes);
    a.sl_again = (int32_t*)(scratch + sw.max_bytes + sw.hist_bytes + sw.state_bytes);
    a.n_t64 = w.tw.n_t64;
    a.tile_max = (float*)tiles;
    a.act_list = (int32_t*)(tiles + w.tw.table_bytes);
    a.act_count = (int32_t*)(tiles + w.tw.table_bytes + w.tw.list_bytes);
    // (the last two ints of the counts' region)
    a.act_range = a.act_count + (w.tw.count_bytes / sizeof(int32_t) - 2);
    a.n_splits_even = std::max(2, ranges.dense);
  }
  const unsigned n_qtiles = (unsigned)((T + 31) / 32);
  // 1-D grid, padded so that every die gets whole (head, query tile, slice) columns (see the kernel's decoding)
  auto search_grid = [&](unsigned slices) {
    if (a.n_heads > 8 || 8 % a.n_heads != 0) return dim3((unsigned)a.n_heads * n_qtiles * slices);
    const unsigned per_head = 8u / (unsigned)a.n_heads;
    return dim3(8u * ((n_qtiles * slices + per_head - 1) / per_head));
  };
  hipStream_t s = (hipStream_t)stream;
  if (a.n_slice > 1) {
    const dim3 grid = search_grid((unsigned)a.n_slice);
    RTP_LAUNCH(prefill_select_kernel<0>, grid, dim3(kSelThreads), 0, s, a);
    RTP_LAUNCH(prefill_select_kernel<1>, grid, dim3(kSelThreads), 0, s, a);
    if (!a.order) {
      RTP_LAUNCH(prefill_select_kernel<2>, grid, dim3(kSelThreads), 0, s, a);
      RTP_LAUNCH(prefill_select_kernel<3>, grid, dim3(kSelThreads), 0, s, a);
      RTP_LAUNCH(prefill_select_kernel<kSelFinish>, search_grid(1), dim3(kSelThreads), 0, s, a);
    }
  } else if (!a.order) {
    // At most one workgroup per compute unit: sixteen waves each, four per SIMD, where eight leave it two.  What every wave does
    // by itself (its first loads, the ends of the member ranges) then takes twice the issue slots, which a peaked score law, whose
    // last two sweeps are a few tiles, does not win back on short contexts: the line lies where no law lost by them.  Calls of 4
    // heads, us, eight waves (as they were when sixteen came) / sixteen, clusters and a peaked law: 1000 queries at 6200 keys 111.0 / 104.8
    // and 70.4 / 73.0, at 9000 130.1 / 120.2 and 77.3 / 78.8, 200 at 11200 133.1 / 121.6 and 68.8 / 70.4; beyond the line, 200 at 11600
    // 139.9 / 122.6 and 71.9 / 70.7, 1000 at 12400 160.5 / 143.4 and 88.3 / 87.1, 2000 at 17000 230.8 / 205.8 and 99.7 / 98.5.
    const int64_t rounds = (keys + 32 * kSelRing - 1) / (32 * kSelRing);
    if (groups <= compute_units() && rounds > kSelFewRounds)
      RTP_LAUNCH((prefill_select_kernel<kSelAll, kSelThreadsFew>), search_grid(1), dim3(kSelThreadsFew), 0, s, a);
    else
      RTP_LAUNCH(prefill_select_kernel<kSelAll>, search_grid(1), dim3(kSelThreads), 0, s, a);
  }
  if (a.order) {
    if (a.n_slice > 1) RTP_LAUNCH(prefill_first_digit, search_grid(1), dim3(kSelThreads), 0, s, a);
    else RTP_LAUNCH(prefill_select_kernel<kSelFirst>, search_grid(1), dim3(kSelThreads), 0, s, a);
    RTP_LAUNCH(prefill_order_kernel, dim3((unsigned)((T + a.order_block - 1) / a.order_block), (unsigned)a.n_heads), dim3(kOrderThreads), 0, s, a);
    a.n_slice = last_slices;
    const dim3 grid = search_grid((unsigned)last_slices);
    RTP_LAUNCH((prefill_select_kernel<2, kSelThreads, true>), grid, dim3(kSelThreads), 0, s, a);
    RTP_LAUNCH((prefill_select_kernel<3, kSelThreads, true>), grid, dim3(kSelThreads), 0, s, a);
    RTP_LAUNCH((prefill_select_kernel<kSelFinish, kSelThreads, true>), search_grid(1), dim3(kSelThreads), 0, s, a);
  }
  const unsigned n_wide = (unsigned)((T + kPwQ - 1) / kPwQ);
  if (keys > 128 * kListThreadsFew) RTP_LAUNCH(prefill_active_tiles_kernel<kListThreads>, dim3(n_wide, (unsigned)a.n_heads, a.units ? 2u : 1u), dim3(kListThreads), 0, s, a);
  else RTP_LAUNCH(prefill_active_tiles_kernel<kListThreadsFew>, dim3(n_wide, (unsigned)a.n_heads), dim3(kListThreadsFew), 0, s, a);
  if (a.units) RTP_LAUNCH(prefill_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, a, compute_units());
  const dim3 grid = a.units ? dim3(std::max((unsigned)max_units(a.n_heads, T), (unsigned)(a.n_splits * a.n_sub * a.n_heads) * n_wide)) : dim3((unsigned)(a.n_splits * a.n_sub), n_wide, (unsigned)a.n_heads);
  if (a.order && a.f16) RTP_LAUNCH((flash_prefill_wide_kernel<kModeSparse, true, true>), grid, dim3(kPwThreads), 0, s, a);
  else if (a.order) RTP_LAUNCH((flash_prefill_wide_kernel<kModeSparse, false, true>), grid, dim3(kPwThreads), 0, s, a);
  else if (a.f16) RTP_LAUNCH((flash_prefill_wide_kernel<kModeSparse, true>), grid, dim3(kPwThreads), 0, (hipStream_t)stream, a);
  else RTP_LAUNCH(flash_prefill_wide_kernel<kModeSparse>, grid, dim3(kPwThreads), 0, (hipStream_t)stream, a);
  if (a.units || a.n_splits * a.n_sub > 1) launch_prefill_combine(a, (hipStream_t)stream);
  return check_launch(who);
}

extern "C" int32_t rtp_sparse_attn_prefill_tile_stats(const rtp_layer_desc* layer, int32_t T, int64_t chunk_start,
                                                      const void* ws, size_t ws_bytes, void* stream,
                                                      int64_t* tiles_visited, int64_t* tiles_causal) {
  const char* who = "rtp_sparse_attn_prefill_tile_stats";
  HeadTable ht;
  int32_t rc = fill_head_table(layer, &ht, who);
  if (rc != RTP_OK) return rc;
  if (T <= 0 || chunk_start < 0 || !tiles_visited || !tiles_causal)
    return fail(RTP_ERR_INVALID_ARG, "%s: T must be positive, chunk_start >= 0, outputs non-NULL", who);
  if (layer->n_ret <= 0) {
    *tiles_visited = *tiles_causal = 0;
    return RTP_OK;
  }
  const size_t need = rtp_sparse_attn_prefill_workspace_bytes(layer, T, chunk_start);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need)
    return fail(RTP_ERR_WORKSPACE, "%s: the workspace of the rtp_sparse_attn_prefill call (%zu bytes) is required", who, need);
  clear_error();
  const PrefillWs w = prefill_ws(layer->n_ret, T, chunk_start);
  const int n_qt = (T + kPwQ - 1) / kPwQ;
  std::vector<int32_t> counts((size_t)layer->n_ret * n_qt);
  const char* at = (const char*)ws + w.front() - w.tw.count_bytes;       // the lists' lengths end the part in front of the scratch
  hipError_t e = hipStreamSynchronize((hipStream_t)stream);
  if (e == hipSuccess) e = hipMemcpy(counts.data(), at, counts.size() * sizeof(int32_t), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail(RTP_ERR_HIP, "%s: %s", who, hipGetErrorString(e));
  int64_t vis = 0, causal = 0;
  for (size_t i = 0; i < counts.size(); ++i) vis += counts[i];
  for (int qt = 0; qt < n_qt; ++qt) {
    const int64_t m_hi = chunk_start + (int64_t)std::min(qt * kPwQ + kPwQ, T) - 1;
    causal += (m_hi / kPfK + 1) * layer->n_ret;
  }
  *tiles_visited = vis;
  *tiles_causal = causal;
  return RTP_OK;
}
