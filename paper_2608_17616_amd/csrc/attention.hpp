// Memory injection into attention (read time): launch of the kernel in attention.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mone {

struct Attention {
  const void *qh, *kh, *vh;  // [L][q][n_heads dh], [L][q][n_kv_heads dh] x 2, act dtype
  const void* kv_mem;        // [L][q][2 d_kv]
  void* out;                 // [L][q][n_heads dh]
  int L, q, n_heads, n_kv_heads, dh, d_kv;
  float scale;
  bool act_bf16, mem_bf16, out_bf16;
};

// Validated arguments, q >= 1, dh <= 256.
hipError_t launch_attention_kernel(const Attention& a, hipStream_t s);

}  // namespace mone
