// rtp_index_project: the low-rank indexer projections of the paper's Sec. 3.2 (indexer equation),
//   kI[j, n, :] = bf16( W^K_{h_j} k^pre_{n, kv(h_j)} )     (key side: appended tokens, once per token)
//   qI[j, t, :] = bf16( W^Q_{h_j} q^pre_{t, h_j} )          (query side)
// for the j-th retrieval query head h_j.  The 128-term sums run in fp64 (every bf16 x fp32 product is
// exact there) and are rounded to bf16 ONCE, so the bits do not depend on the summation order and equal
// a correctly rounded reference.
//
// The contraction runs on the fp64 matrix cores: a wave takes 16 tokens of one retrieval head and walks the 128 terms with
// 32 v_mfma_f64_16x16x4.  The four terms of a step are spread over the four 16-lane rows of the wave, and which terms these
// are is free as long as both operands agree: row g takes terms 32 g .. 32 g + 31, so a lane reads one run of 64 bytes
// of its token and one of 128 bytes of its W row straight from memory and every load goes out at once.  (Result register i
// of lane row g is operand row 4 i + g, so operand row r holds output 4 (r % 4) + r / 4 and a lane ends with four adjacent outputs.)
// Bound by launch and load latency: 8192 tokens of 4 heads are 0.9 us per wave on the matrix cores, two waves per SIMD.
// With W staged through LDS as fp64 and vector FMAs (256 16-byte LDS reads per thread behind a barrier) that call's kernel
// took 8.5 us, now 5.1; the projection of a prompt's 2037 queries for 2 heads 6 us, now 4.2.
#include "common.h"
#include "index_project.h"

namespace rtp {

constexpr int kIbThreads = 256;
constexpr int kIbTokens = 16 * kIbThreads / 64;     // tokens per workgroup

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4a4 __attribute__((ext_vector_type(4), aligned(4)));     // (W is only known to be float-aligned)
typedef double f64x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kIbThreads) void index_build_kernel(const IndexProjectArgs a) {
  const int j = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, r = lane & 15;
  const int64_t t0 = (int64_t)blockIdx.x * kIbTokens + wave * 16;
  if (t0 >= a.T) return;
  const int64_t t = min(t0 + r, (int64_t)a.T - 1);                   // lanes past the last token repeat it
  const uint16_t* row = a.x + (t * a.n_x_heads + a.x_head[j]) * kHeadDim + g * 32;
  const float* w = a.W + ((int64_t)j * kIndexDim + 4 * (r & 3) + (r >> 2)) * kHeadDim + g * 32;
  u32x4 xr[4];
  f32x4a4 wr[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) xr[i] = *reinterpret_cast<const u32x4*>(row + i * 8);
#pragma unroll
  for (int i = 0; i < 8; ++i) wr[i] = *reinterpret_cast<const f32x4a4*>(w + i * 4);
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float xf[8] = {bf16_lo(xr[i].x), bf16_hi(xr[i].x), bf16_lo(xr[i].y), bf16_hi(xr[i].y),
                         bf16_lo(xr[i].z), bf16_hi(xr[i].z), bf16_lo(xr[i].w), bf16_hi(xr[i].w)};
#pragma unroll
    for (int k = 0; k < 8; ++k)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)wr[2 * i + (k >> 2)][k & 3], (double)xf[k], acc, 0, 0, 0);
  }
  if (t0 + r >= a.T) return;
  uint16_t* o = a.out + (int64_t)j * a.out_head_stride + (a.out_t0 + t) * kIndexDim + g * 4;
  const uint32_t lo = (uint32_t)f64_to_bf16_rne(acc[0]) | ((uint32_t)f64_to_bf16_rne(acc[1]) << 16);
  const uint32_t hi = (uint32_t)f64_to_bf16_rne(acc[2]) | ((uint32_t)f64_to_bf16_rne(acc[3]) << 16);
  *reinterpret_cast<uint2*>(o) = make_uint2(lo, hi);
}

void launch_index_project(const IndexProjectArgs& a, int32_t n_ret, hipStream_t s) {
  RTP_LAUNCH(index_build_kernel, dim3((unsigned)(((int64_t)a.T + kIbTokens - 1) / kIbTokens), (unsigned)n_ret), dim3(kIbThreads), 0, s, a);
}

}  // namespace rtp

using namespace rtp;

extern "C" int32_t rtp_index_project(const rtp_layer_desc* layer, const float* W, const void* x_pre, int32_t side,
                                     int32_t T, void* xI_out, int64_t out_head_stride, int64_t out_t0, void* stream) {
  const char* who = "rtp_index_project";
  HeadTable ht;
  int32_t rc = fill_head_table(layer, &ht, who);
  if (rc != RTP_OK) return rc;
  if (!W || !x_pre || !xI_out) return fail(RTP_ERR_INVALID_ARG, "%s: NULL tensor pointer", who);
  if (side != RTP_SIDE_QUERY && side != RTP_SIDE_KEY) return fail(RTP_ERR_INVALID_ARG, "%s: side must be RTP_SIDE_QUERY or RTP_SIDE_KEY", who);
  if (T <= 0 || out_t0 < 0) return fail(RTP_ERR_INVALID_ARG, "%s: T must be positive and out_t0 >= 0", who);
  if (out_head_stride < 0 || (out_head_stride & 3)) return fail(RTP_ERR_INVALID_ARG, "%s: out_head_stride must be a non-negative multiple of 4", who);
  if (((uintptr_t)x_pre & 15) || ((uintptr_t)xI_out & 7) || ((uintptr_t)W & 3))
    return fail(RTP_ERR_INVALID_ARG, "%s: x_pre must be 16-byte and xI_out 8-byte aligned", who);
  clear_error();
  if (layer->n_ret == 0) return RTP_OK;
  IndexProjectArgs a;
  a.W = W;
  a.x = (const uint16_t*)x_pre;
  a.out = (uint16_t*)xI_out;
  a.out_head_stride = out_head_stride;
  a.out_t0 = out_t0;
  a.T = T;
  const int G = layer->n_q_heads / layer->n_kv_heads;
  a.n_x_heads = side == RTP_SIDE_QUERY ? layer->n_q_heads : layer->n_kv_heads;
  for (int j = 0; j < 64; ++j) {
    const int h = j < layer->n_ret ? layer->ret_heads[j] : 0;
    a.x_head[j] = side == RTP_SIDE_QUERY ? h : h / G;
  }
  launch_index_project(a, layer->n_ret, (hipStream_t)stream);
  return check_launch(who);
}
