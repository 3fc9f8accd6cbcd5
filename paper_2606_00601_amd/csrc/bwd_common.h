// bwd_common.h -- what the kernels of the fused backward share: the parts of
// the workspace, element loads and stores, softplus with its derivative.
#pragma once

#include "selective_common.h"

namespace sw {

constexpr int BW_N = 16;  // states per launch (groups of 16 for N > 16)
constexpr int BW_T = 8;   // steps per tile
constexpr float BW_LOG2E = 1.4426950408889634f;

__device__ __forceinline__ float sigmoid_f32(float v) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-v * BW_LOG2E));
}

// softplus(v) and its derivative sigmoid(v) from one exp2: e = e^-|v| and w =
// 1 + e give sigmoid(|v|) = 1 / w and log1p(e) = log(w) e / (w - 1) (e where w
// rounds to 1), and softplus(v) = max(v, 0) + log1p(e).  The staging of a tile
// is bound by instruction issue, and an exp2 takes 8.5 cycles of it.
__device__ __forceinline__ void softplus_sigmoid_f32(float v, float& sp, float& sg) {
  const float e = __builtin_amdgcn_exp2f(-__builtin_fabsf(v) * BW_LOG2E);
  const float w = 1.0f + e, d = w - 1.0f;
  const float l = __builtin_amdgcn_logf(w) * 0.6931471805599453f * (e * __builtin_amdgcn_rcpf(d));
  sp = (v > 0.0f ? v : 0.0f) + (d == 0.0f ? e : l);
  const float r = __builtin_amdgcn_rcpf(w);
  sg = v > 0.0f ? r : e * r;
}

__device__ __forceinline__ void bw_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

struct BwWork {
  float* ck;       // (B*D, ntile, 16) states at tile starts
  const float* s;  // (B*D, L) pre-gate output (gated calls)
  float* rec;      // (nseg - 1, 2, B*D, 16): P and end adjoint of segments 1 ..
  float* dA_p;     // (nseg, B*D, 16)
  float* dD_p;     // (nseg, B*D)
  float* db_p;     // (nseg, B*D)
  float* dB_p;     // (B, G, L, 16)
  float* dC_p;     // (B, G, L, 16)
  float* trash;    // 1024 floats: the target of stores a lane does not need
};

template <typename T>
__device__ __forceinline__ float widen(T r) {
  if constexpr (sizeof(T) == 4)
    return r;
  else
    return __uint_as_float((uint32_t)r << 16);
}

// One element of type T at byte offset voff + soff of a raw buffer resource
// (zero past the resource's end).
template <typename T>
__device__ __forceinline__ T buf_ld(__amdgpu_buffer_rsrc_t r, int32_t voff, int32_t soff) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0));
}

// One gradient value as stored: fp32, or bf16 rounded to nearest even.
template <typename OUT>
__device__ __forceinline__ void st1(OUT* p, float v) {
  if constexpr (sizeof(OUT) == 4)
    *p = v;
  else
    *p = (OUT)bf16_rne(v);
}

// The kernel of selective_bwd16.hip on whole rows: one group of 16 states from
// n0, G = ceil(D / 16) workgroups per batch; checkpoints in w.ck, which it
// writes itself first where a.ckpt is NULL.
void launch_bwd_rows16(const BwdArgs& a, const BwWork& w, int64_t G, int64_t ntile, int n0,
                       hipStream_t s);

}  // namespace sw
