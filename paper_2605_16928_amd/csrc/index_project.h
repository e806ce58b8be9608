// The projection launch of rtp_index_project (index_build.hip), which the prefill call uses for its index queries too.
#pragma once

#include "common.h"

namespace rtp {

struct IndexProjectArgs {
  const float* W;           // [n_ret, 16, 128]
  const uint16_t* x;        // bf16 [T, n_x_heads, 128]
  uint16_t* out;            // bf16: (j, t, i) at out[j * out_head_stride + (out_t0 + t) * 16 + i]
  int64_t out_head_stride, out_t0;
  int32_t T, n_x_heads;
  int32_t x_head[64];       // head of x that retrieval head j projects
};

void launch_index_project(const IndexProjectArgs& a, int32_t n_ret, hipStream_t s);

}  // namespace rtp
