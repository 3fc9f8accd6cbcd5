// selective_step.hip -- fused selective scan, forward, for a few steps per
// call (serving: one token at a time, the state carried through h0 and
// h_last), any N in [1, 64], on gfx950.
//
// The operation is that of selective_scan.hip (Sec. 1, Sec. 3.1):
//   a_{t,n} = exp(delta_t A_n),  u_{t,n} = delta_t B_{t,n} x_t,
//   h_{t,n} = a_{t,n} h_{t-1,n} + u_{t,n},  y_t = sum_n C_{t,n} h_{t,n} + Dskip x_t.
//
// With one or a few steps the call moves the states, 8 N bytes per row (h0 in,
// h_last out), against a few bytes of x, delta, z and y: it is bound by HBM,
// and there is nothing to stage or to pipeline along t.  A row is a quad of
// lanes, lane g of the quad owning states 16j + 4g .. +3 (one float4 per 16
// states), so a wavefront reads and writes 16 consecutive rows of h0, A and
// h_last as 1 KB runs, every load of a step is issued before its arithmetic,
// and y meets in the quad with two DPP adds.  No LDS, no scratch, no ticket.
// At B=64, D=5120, N=16, L=1 (bf16, every option) the 8-lane kernel, which
// stages whole 32-step tiles, took 488 us and this one takes 11.7 us (host
// work included; its 45 MB take 9 us at the rate of a copy).
#include "selective_common.h"

namespace sw {

namespace {

constexpr int ST_ROWS = 64;  // rows of one batch per workgroup
constexpr float ST_LOG2E = 1.4426950408889634f;

template <int M>
__device__ __forceinline__ float step_quad_xor(float v) {
  // quad_perm selectors: [1,0,3,2] for M = 1, [2,3,0,1] for M = 2
  constexpr int sel =
      M == 1 ? (1 | (0 << 2) | (3 << 4) | (2 << 6)) : (2 | (3 << 2) | (0 << 4) | (1 << 6));
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), sel, 0xf, 0xf, false));
}

__device__ __forceinline__ float step_widen(float v) { return v; }
__device__ __forceinline__ float step_widen(uint16_t v) { return bf16_one(v); }

// Elements n0 .. n0+3 of a row of N at p (zeros past N).  VEC: N is a multiple
// of 4 and p is aligned for the vector load.
template <bool VEC, typename T>
__device__ __forceinline__ void load4(float (&v)[4], const T* __restrict__ p, int n0, int N) {
  if constexpr (VEC) {
    RawVec<T, 4> r;
    if (n0 < N) {
      r.load_vec(p + n0);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = r.get(i);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = 0.0f;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = n0 + i < N ? step_widen(p[n0 + i]) : 0.0f;
  }
}

// NC: float4 groups of states per lane (ceil(N / 16) of them in use).  U:
// steps whose loads are issued together.
template <typename IN, int NC, bool VEC, int U>
__global__ __launch_bounds__(256) void selective_step_kernel(
    const IN* __restrict__ x, const IN* __restrict__ delta, const float* __restrict__ A,
    const IN* __restrict__ Bm, const IN* __restrict__ Cm, const float* __restrict__ Dskip,
    const IN* __restrict__ z, const float* __restrict__ dbias, const float* __restrict__ h0,
    void* __restrict__ yv, float* __restrict__ h_last, int64_t D, int N, int L, int64_t ndb,
    uint32_t flags) {
  const int64_t b = blockIdx.x / ndb;
  const int64_t d = (blockIdx.x - b * ndb) * ST_ROWS + threadIdx.x / 4;
  const int g = threadIdx.x & 3;
  if (d >= D) return;  // whole quads leave together
  const int64_t row = b * D + d;

  float Al[NC][4], h[NC][4];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    load4<VEC>(Al[j], A + d * N, 16 * j + 4 * g, N);  // past N: a = 1 and u = 0
    if (h0) {
      load4<VEC>(h[j], h0 + row * N, 16 * j + 4 * g, N);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) h[j][i] = 0.0f;
    }
  }
#pragma unroll
  for (int j = 0; j < NC; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) Al[j][i] *= ST_LOG2E;
  const float dsk = Dskip ? Dskip[d] : 0.0f;
  const float dbv = dbias ? dbias[d] : 0.0f;
  const bool ybf = (flags & SEL_Y_BF16) != 0;

  for (int t0 = 0; t0 < L; t0 += U) {
    float xv[U], dv[U], zv[U], bq[U][NC][4], cq[U][NC][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u < L ? t0 + u : L - 1;  // loads past the end are unused
      xv[u] = step_widen(x[row * L + t]);
      dv[u] = step_widen(delta[row * L + t]);
      zv[u] = (flags & SEL_GATED) ? step_widen(z[row * L + t]) : 0.0f;
      const int64_t bc = (b * L + t) * N;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        load4<VEC>(bq[u][j], Bm + bc, 16 * j + 4 * g, N);
        load4<VEC>(cq[u][j], Cm + bc, 16 * j + 4 * g, N);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (t0 + u >= L) break;
      float dl = dv[u] + dbv;
      if (flags & SEL_SOFTPLUS) dl = softplus_f32(dl);
      const float dx = dl * xv[u];
      float acc = 0.0f;
#pragma unroll
      for (int j = 0; j < NC; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float a = __builtin_amdgcn_exp2f(dl * Al[j][i]);
          h[j][i] = __builtin_fmaf(a, h[j][i], dx * bq[u][j][i]);
          acc = __builtin_fmaf(cq[u][j][i], h[j][i], acc);
        }
      acc += step_quad_xor<1>(acc);
      acc += step_quad_xor<2>(acc);
      acc = __builtin_fmaf(dsk, xv[u], acc);
      if (flags & SEL_GATED) acc *= silu_f32(zv[u]);
      if (g == 0) {
        if (ybf)
          static_cast<uint16_t*>(yv)[row * L + t0 + u] = (uint16_t)bf16_rne(acc);
        else
          static_cast<float*>(yv)[row * L + t0 + u] = acc;
      }
    }
  }
  if (h_last) {
    float* const hp = h_last + row * N;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int n0 = 16 * j + 4 * g;
      if constexpr (VEC) {
        if (n0 < N)
          *reinterpret_cast<float4*>(hp + n0) = make_float4(h[j][0], h[j][1], h[j][2], h[j][3]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n0 + i < N) hp[n0 + i] = h[j][i];
      }
    }
  }
}

template <typename IN, int NC>
void launch_step_nc(const SelArgs& a, hipStream_t s) {
  const int64_t ndb = (a.D + ST_ROWS - 1) / ST_ROWS;
  const uint32_t flags = (a.softplus ? SEL_SOFTPLUS : 0u) | (a.y_bf16 ? SEL_Y_BF16 : 0u) |
                         (a.z ? SEL_GATED : 0u);
  const uintptr_t states = (uintptr_t)a.A | (uintptr_t)a.h0 | (uintptr_t)a.h_last;
  const uintptr_t bc = (uintptr_t)a.Bm | (uintptr_t)a.Cm;
  const bool vec = a.N % 4 == 0 && states % 16 == 0 && bc % (4 * sizeof(IN)) == 0;
  auto kern = vec ? (a.L == 1 ? selective_step_kernel<IN, NC, true, 1>
                              : selective_step_kernel<IN, NC, true, 2>)
                  : selective_step_kernel<IN, NC, false, 1>;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.B * ndb)), dim3(256), 0, s,
                     static_cast<const IN*>(a.x), static_cast<const IN*>(a.delta), a.A,
                     static_cast<const IN*>(a.Bm), static_cast<const IN*>(a.Cm), a.Dskip,
                     static_cast<const IN*>(a.z), a.delta_bias, a.h0, a.y, a.h_last, a.D,
                     (int)a.N, (int)a.L, ndb, flags);
}

}  // namespace

// Launches the few-step kernel (L at least 1, no checkpoints, no pre-gate
// output; the caller has checked that the grid fits).
template <typename IN>
int launch_step(const SelArgs& a, hipStream_t s) {
  if (a.N <= 16)
    launch_step_nc<IN, 1>(a, s);
  else if (a.N <= 32)
    launch_step_nc<IN, 2>(a, s);
  else
    launch_step_nc<IN, 4>(a, s);
  note_launch("selective_step_kernel: whole rows");
  return check_launch("selective_step_kernel");
}

template int launch_step<float>(const SelArgs&, hipStream_t);
template int launch_step<uint16_t>(const SelArgs&, hipStream_t);

}  // namespace sw
