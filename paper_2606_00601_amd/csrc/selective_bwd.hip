// selective_bwd.hip -- backward of the fused selective scan on gfx950.
//
// The gradient of sum_t dy_t y_t (+ sum_n dh_last_n h_last_n) by the chain
// rule through the forward recurrence h_t = a_t h_{t-1} + u_t (Eq. (3)),
// a_{t,n} = exp(delta_t A_n), u_{t,n} = delta_t B_{t,n} x_t,
// y_t = (sum_n C_{t,n} h_{t,n} + Dskip x_t) g_t, g_t = silu(z_t) or 1.
// The adjoint lam_t = dL/dh_t obeys the same kind of recurrence run
// backwards in time, lam_t = ds_t C_t + a_{t+1} lam_{t+1} (ds_t = dy_t g_t),
// the affine pair of Eq. (6) with the order of Eq. (7) reversed.  With
// q_t = a_t h_{t-1}:
//   ddelta_t = sum_n lam (q A_n + B x_t)        dx_t = delta_t sum_n lam B + ds_t Dskip
//   dA_n    += lam q delta_t                    dB_{t,n} += lam delta_t x_t   (over d)
//   dC_{t,n} += ds_t h_t                        (over d)
//   dh0 = a_0 lam_0,  dDskip += ds x,  dz = dy s silu'(z) with s the pre-gate y.
//
// Two kernels walk it, and plan_bwd prices them per call: the one below, on 64
// rows a workgroup, and the one of selective_bwd16.hip, on 16, for calls whose
// 16-row blocks fill the compute units where their 64-row blocks do not.
//
// The state before every 8th step (a checkpoint per row, state and tile)
// comes from the forward, from its walk without y, or from
// selective_sweep_kernel below.  selective_bwd_kernel walks the tiles of its
// rows backwards:
//   * a workgroup (4 wavefronts) owns 64 rows of one batch, a wavefront 16 of
//     them: lane (rl, nl) = (lane / 8, lane % 8) owns states 2nl, 2nl+1 of
//     rows rl and rl+8.  Four chains per lane share the loads of their row and
//     state operands, the sums over the states and over the rows are half
//     done in registers, and each wavefront has four independent chains to
//     issue from while one waits;
//   * a wavefront stages its rows' delta, delta*x and ds of the next tile in
//     its own LDS, one lane per (row, two steps); the workgroup stages B and C
//     (one element per lane);
//   * every lane reloads its checkpoints, recomputes the tile's a_t and q_t
//     forward into registers, forming ds h on the way, then walks the tile
//     backwards carrying lam;
//   * lam q A and lam B, summed over the lane's two states, meet in the
//     wavefront's LDS, and the lane that staged (row, two steps) adds the
//     eight partials and stores ddelta and dx one tile later;
//   * lam delta x and ds h, summed over the lane's two rows, are summed over
//     the wavefront's rows by lane-half exchanges (v_permlane32_swap,
//     v_permlane16_swap); one lane per (dB or dC, step, state) adds the four
//     wavefronts' sums into this workgroup's share.  One barrier per tile.
// Few rows are cut into segments of tiles: a first launch walks each segment
// but the first from a zero adjoint (the last from dh_last) without gradients
// and records its end value and the product of its a_t (as exp of A times the
// sum of delta); the main launch composes the records of the segments after
// its own into its incoming lam.  A second kernel adds the shares of dB and
// dC (over the workgroups of a batch) and of dA, dDskip and ddelta_bias (over
// batch and segments) in a fixed order: no atomics, reproducible bit for bit.
//
// Bound by instruction issue: about 12 operations and an exp2 per element
// and state (45 cycles per wavefront and SIMD), the sums over rows (9) and
// states (4) and the staging with softplus and gate (9), against the HBM
// time of the checkpoints and the (B, D, L) arrays.
#include <stdlib.h>

#include "bwd_common.h"

namespace sw {
namespace {

constexpr int BW_WROWS = 16;  // rows per wavefront
constexpr int BW_ROWS = 64;   // rows per workgroup
constexpr int BW_MAX_SEG = 32;
// LDS words of one row's [n][t] partials, and of one quantity's 16 rows: as
// 16-byte groups, 18 a row (writes: two rows of 16 lanes fill the 64 banks,
// one on the even groups, one on the odd) and 8 more for the second quantity
// (reads: 4 rows x 2 quantities x 2 halves fill them)
constexpr int BW_SPR = 72;
constexpr int BW_SPQ = BW_WROWS * BW_SPR + 32;

// (the adjoint's walk without gradients uses rv and bc only, and keeps more
// workgroups on a compute unit)
template <bool ENDS>
struct BwSmem {
  float rv[4][2][3][BW_WROWS][BW_T];     // per wavefront, two tiles: delta, delta*x, ds
  float bc[2][2][BW_N][BW_T];            // two tiles: B, C as [n][t], halves swapped for n >= 8
  float sp[4][ENDS ? 4 : 2 * BW_SPQ];    // per wavefront: lam q A, lam B (summed over n next)
  float pw[2][4][2][ENDS ? 4 : 64 * 4];  // two tiles, per wavefront and 4 steps: row sums
};

// LDS writes of this wavefront are seen by its later reads in every lane.
__device__ __forceinline__ void bw_wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Value of `v` in the lane whose index differs in bit 0.
__device__ __forceinline__ float lane_xor1(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1,
                                                               0xf, 0xf, false));
}

template <typename T>
struct Bits {
  using type = uint32_t;
};
template <>
struct Bits<uint16_t> {
  using type = uint16_t;
};

// Two consecutive elements as loaded (widened when used, so that the load is
// not waited for until then).  PAIR: one access (rows of even length, bf16
// rows on a dword).
template <typename T, bool PAIR>
struct Two {
  static constexpr int W = sizeof(T) == 2 && PAIR ? 1 : 2;
  uint32_t w[W];
  __device__ __forceinline__ void load_buf(__amdgpu_buffer_rsrc_t r, int32_t voff, int32_t soff) {
    if constexpr (!PAIR) {
      w[0] = __builtin_bit_cast(typename Bits<T>::type, buf_ld<T>(r, voff, soff));
      w[1] = __builtin_bit_cast(typename Bits<T>::type, buf_ld<T>(r, voff + (int)sizeof(T), soff));
    } else if constexpr (W == 1) {
      w[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    } else {
      const uint2 v = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
      w[0] = v.x;
      w[1] = v.y;
    }
  }
  __device__ __forceinline__ void set(T a, T b) {
    const uint32_t u = __builtin_bit_cast(typename Bits<T>::type, a);
    const uint32_t v = __builtin_bit_cast(typename Bits<T>::type, b);
    if constexpr (W == 1) {
      w[0] = u | (v << 16);
    } else {
      w[0] = u;
      w[1] = v;
    }
  }
  __device__ __forceinline__ float get(int i) const {
    if constexpr (sizeof(T) == 4)
      return __uint_as_float(w[i]);
    else if constexpr (W == 1)
      return i ? bf16_hi(w[0]) : bf16_lo(w[0]);
    else
      return __uint_as_float(w[i] << 16);
  }
};

// Launch modes: the gradients; the adjoint's walk without gradients (segments
// 1 .. nseg-1), which records each segment's end value.
enum : int { BW_MAIN = 0, BW_ENDS = 1 };

// All global loads below are unconditional, from valid addresses, with the
// unwanted values replaced afterwards, and all stores the same instructions
// for every lane: the loads of the next tile then stay in flight across the
// current one instead of being waited for inside a branch.  BUF: loads and
// stores go through raw buffer resources over the wavefront's rows (and its
// batch's B, C), a per-lane offset fixed for the whole kernel plus a scalar
// one (every offset below 2^31, checked by the host; a lane with nothing to
// store aims at the resource's end, where the store is dropped); without it,
// 64-bit addresses clamped into range, and stores aimed at trash slots.
// OUT: the type of dx, ddelta, dz (and dB, dC).
template <typename IN, typename DYT, typename OUT, bool GATED, bool PAIR, bool BUF, int MODE>
__global__ __launch_bounds__(256, MODE == BW_ENDS ? 4 : 2) void selective_bwd_kernel(const BwdArgs a, const BwWork w,
                                                               int64_t G, int64_t ntile, int n0,
                                                               int nseg, int64_t seg_tiles) {
  constexpr bool ENDS = MODE == BW_ENDS;
  constexpr int ES = (int)sizeof(IN), OS = (int)sizeof(OUT);
  __shared__ __align__(16) BwSmem<ENDS> sm;
  const IN* __restrict__ X = static_cast<const IN*>(a.x);
  const IN* __restrict__ DL = static_cast<const IN*>(a.delta);
  const IN* __restrict__ Z = static_cast<const IN*>(a.z);
  const DYT* __restrict__ DY = static_cast<const DYT*>(a.dy);
  const int64_t D = a.D, L = a.L, N = a.N, R = a.B * a.D;

  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid / 64);
  const int lane = tid % 64;
  const int nsl = ENDS ? nseg - 1 : nseg;
  const int64_t rblk = blockIdx.x / (unsigned)nsl;
  const int sg = (int)(blockIdx.x - rblk * nsl) + (ENDS ? 1 : 0);
  const int64_t b = rblk / G, g = rblk - b * G;
  const int64_t k_lo = sg * seg_tiles;
  const int64_t k_hi = sg == nseg - 1 ? ntile : k_lo + seg_tiles;

  // the wavefront's rows: nrows of them from row0 (a wavefront past D works on
  // a copy of row D-1 and stores nothing)
  const int64_t d0w = g * BW_ROWS + wv * BW_WROWS;
  const int64_t d0 = d0w < D ? d0w : D - 1;
  const int nrows = d0w < D ? (int)imin(BW_WROWS, D - d0w) : 0;
  const int64_t row0 = b * D + d0;
  const int vrows = nrows > 0 ? nrows : 1;  // rows the resources cover

  // ---- walking role: states n0 + 2nl + i of rows rl + 8j
  const int nl = lane & 7, rl = lane >> 3;
  bool dok[2], nok[2];
  int rj[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    dok[j] = rl + 8 * j < nrows;
    rj[j] = dok[j] ? rl + 8 * j : vrows - 1;
    nok[j] = n0 + 2 * nl + j < N;
  }
  float Ar[2][2], Al[2][2], lam[2][2], dA_acc[2][2];  // [state][row]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int ns = n0 + 2 * nl + i;
      const float v = a.A[(d0 + rj[j]) * N + (nok[i] ? ns : 0)];
      Ar[i][j] = nok[i] ? v : 0.0f;
      Al[i][j] = Ar[i][j] * BW_LOG2E;
      dA_acc[i][j] = 0.0f;
      const bool ok = dok[j] && nok[i];
      lam[i][j] = 0.0f;
      if (sg == nseg - 1) {
        if (a.dh_last && ok) lam[i][j] = a.dh_last[(row0 + rj[j]) * N + ns];
      } else if constexpr (!ENDS) {
        // the adjoint entering from the segments after this one
        const int64_t st = R * BW_N;
        const float* const rp = w.rec + (row0 + rj[j]) * BW_N + 2 * nl + i;
        float v2 = rp[(int64_t)(2 * (nseg - 2) + 1) * st];
#pragma unroll 8
        for (int q = nseg - 3; q >= sg; --q)
          v2 = __builtin_fmaf(rp[(int64_t)(2 * q) * st], v2, rp[(int64_t)(2 * q + 1) * st]);
        lam[i][j] = ok ? v2 : 0.0f;
      }
    }
  // records are of segments 1 .., so segment q's are rec[q - 1]

  // ---- staging role: steps 2p, 2p+1 of row sr
  const int sr = lane >> 2, pr = lane & 3;
  const bool sdok = sr < nrows;
  const int src = sdok ? sr : vrows - 1;
  const float dbias = a.delta_bias ? a.delta_bias[d0 + src] : 0.0f;
  const bool first = n0 == 0;  // the terms that do not depend on the state come with the first group
  const float Dsk = a.Dskip && first ? a.Dskip[d0 + src] : 0.0f;
  // ---- B/C role: element (step bt, state bn) of B (wavefronts 0, 1) or C
  const bool isC = wv >= 2;  // wave-uniform: it picks buffer resources
  const int bt = (tid >> 4) & 7, bn = tid & 15;
  const bool bnok = n0 + bn < N;

  const int32_t ea = src * (int32_t)(BUF ? L : 0) + 2 * pr;
  const int32_t eb = bt * (int32_t)N + (bnok ? n0 + bn : (int32_t)N - 1);
  const uint32_t rows_e = (uint32_t)(vrows * L);  // elements (BUF: below 2^29)
  const __amdgpu_buffer_rsrc_t rx = buffer_rsrc(X + row0 * L, rows_e * ES);
  const __amdgpu_buffer_rsrc_t rd = buffer_rsrc(DL + row0 * L, rows_e * ES);
  const __amdgpu_buffer_rsrc_t rz = buffer_rsrc(GATED ? Z + row0 * L : X, GATED ? rows_e * ES : 0u);
  const __amdgpu_buffer_rsrc_t rdy = buffer_rsrc(DY + row0 * L, rows_e * (uint32_t)sizeof(DYT));
  const __amdgpu_buffer_rsrc_t rs =
      buffer_rsrc(GATED ? w.s + row0 * L : w.trash, GATED ? rows_e * 4u : 0u);
  const IN* const bcp = static_cast<const IN*>(isC ? a.Cm : a.Bm) + b * L * N;
  const __amdgpu_buffer_rsrc_t rbc = buffer_rsrc(bcp, (uint32_t)(L * N * ES));
  const __amdgpu_buffer_rsrc_t rck =
      buffer_rsrc(w.ck + row0 * ntile * BW_N, (uint32_t)(vrows * ntile * BW_N * 4));
  OUT* const ddp = static_cast<OUT*>(a.ddelta) + row0 * L;
  OUT* const dxp = static_cast<OUT*>(a.dx) + row0 * L;
  OUT* const dzp = static_cast<OUT*>(GATED && a.dz ? a.dz : a.dx) + row0 * L;
  const bool want_dz = GATED && a.dz && first;
  const uint32_t out_b = rows_e * OS;
  const __amdgpu_buffer_rsrc_t rodd = buffer_rsrc(ddp, out_b);
  const __amdgpu_buffer_rsrc_t rodx = buffer_rsrc(dxp, out_b);
  const __amdgpu_buffer_rsrc_t rodz = buffer_rsrc(dzp, want_dz ? out_b : 0u);
  const uint32_t sh_b = (uint32_t)(L * BW_N * 4);
  float* const shp = (isC ? w.dC_p : w.dB_p) + (b * G + g) * L * BW_N;
  const __amdgpu_buffer_rsrc_t rsh = buffer_rsrc(shp, sh_b);

  struct Raw {
    Two<IN, PAIR> x, dl, z;
    Two<DYT, PAIR> dy;
    Two<float, PAIR> s;
    IN bc;
  };
  auto at2 = [&](auto* p, int64_t t, auto& v) {  // !BUF: steps t, t+1 of the staging row
    const int64_t t1 = t < L ? t : L - 1, t2 = t + 1 < L ? t + 1 : L - 1;
    v.set(p[(row0 + src) * L + t1], p[(row0 + src) * L + t2]);
  };
  auto load_tile = [&](int64_t k, Raw& v) {
    const int64_t kc = k < 0 ? 0 : k;  // a tile before the start: tile 0, unused
    if constexpr (BUF) {
      const int32_t tk = (int32_t)kc * BW_T;
      if constexpr (!ENDS) v.x.load_buf(rx, ea * ES, tk * ES);
      v.dl.load_buf(rd, ea * ES, tk * ES);
      v.dy.load_buf(rdy, ea * (int)sizeof(DYT), tk * (int)sizeof(DYT));
      if constexpr (GATED) {
        v.z.load_buf(rz, ea * ES, tk * ES);
        if constexpr (!ENDS) v.s.load_buf(rs, ea * 4, tk * 4);
      }
      v.bc = buf_ld<IN>(rbc, eb * ES, tk * (int32_t)N * ES);
    } else {
      const int64_t t = kc * BW_T + 2 * pr;
      if constexpr (!ENDS) at2(X, t, v.x);
      at2(DL, t, v.dl);
      at2(DY, t, v.dy);
      if constexpr (GATED) {
        at2(Z, t, v.z);
        if constexpr (!ENDS) at2(w.s, t, v.s);
      }
      const int64_t tb = kc * BW_T + bt;
      v.bc = bcp[(tb < L ? tb : L - 1) * N + (bnok ? n0 + bn : N - 1)];
    }
  };
  // both steps' values of an output row; lv: which of them are stored
  auto st2 = [&](__amdgpu_buffer_rsrc_t r, OUT* p, int64_t k, const bool (&lv)[2], float v0,
                 float v1) {
    if constexpr (BUF) {
      const int32_t o = (ea + (int32_t)k * BW_T) * OS;
      if constexpr (PAIR && OS == 4) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(sw_u32x2, make_float2(v0, v1)), r,
                                              lv[0] ? o : (int32_t)out_b, 0, 0);
      } else if constexpr (PAIR) {
        __builtin_amdgcn_raw_buffer_store_b32(bf16x2_rne(v0, v1), r, lv[0] ? o : (int32_t)out_b, 0, 0);
      } else if constexpr (OS == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v0), r, lv[0] ? o : (int32_t)out_b, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v1), r, lv[1] ? o + OS : (int32_t)out_b,
                                              0, 0);
      } else {
        const uint32_t v = bf16x2_rne(v0, v1);
        __builtin_amdgcn_raw_buffer_store_b16((short)(v & 0xffffu), r, lv[0] ? o : (int32_t)out_b, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b16((short)(v >> 16), r, lv[1] ? o + OS : (int32_t)out_b, 0, 0);
      }
    } else {
      OUT* const q = p + src * L + k * BW_T + 2 * pr;  // formed, not used, where lv is false
      OUT* const tr = reinterpret_cast<OUT*>(w.trash + tid);
      st1<OUT>(lv[0] ? q : tr, v0);
      st1<OUT>(lv[1] ? q + 1 : tr, v1);
    }
  };

  // ---- checkpoints of tile k: states 2nl, 2nl+1 of both rows
  auto load_ck = [&](int64_t k, float (&h)[2][2]) {
    const int64_t kc = k < 0 ? 0 : k;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float2 v;
      if constexpr (BUF)
        v = __builtin_bit_cast(
            float2, __builtin_amdgcn_raw_buffer_load_b64(
                        rck, (rj[j] * (int32_t)ntile * BW_N + 2 * nl) * 4, (int32_t)kc * (BW_N * 4), 0));
      else
        v = make_float2(w.ck[((row0 + rj[j]) * ntile + kc) * BW_N + 2 * nl],
                        w.ck[((row0 + rj[j]) * ntile + kc) * BW_N + 2 * nl + 1]);
      h[0][j] = v.x;
      h[1][j] = v.y;
    }
  };

  // ---- stage tile k from `v`; keeps what its ddelta and dx need
  struct Keep {
    float dl[2], sg[2], xv[2], dsD[2];
    bool lv[2];
  };
  float dD_acc = 0.0f, db_acc = 0.0f;
  auto stage = [&](int64_t k, bool live, const Raw& v, int buf, Keep& kp) {
    float dlv[2], dxv[2], dsv[2], zv2[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      kp.lv[i] = live && sdok && k * BW_T + 2 * pr + i < L;
      const bool lv = kp.lv[i];
      float dv = v.dl.get(i) + dbias;
      kp.sg[i] = 1.0f;
      if (a.softplus) softplus_sigmoid_f32(dv, dv, kp.sg[i]);
      dlv[i] = lv ? dv : 0.0f;
      const float dyv = lv ? v.dy.get(i) : 0.0f;
      float gt = 1.0f;
      if constexpr (GATED) {
        const float zv = lv ? v.z.get(i) : 0.0f;
        const float sz = sigmoid_f32(zv);
        gt = zv * sz;
        if constexpr (!ENDS)
          zv2[i] = dyv * (lv ? v.s.get(i) : 0.0f) * (sz * (1.0f + zv * (1.0f - sz)));
      }
      dsv[i] = dyv * gt;
      if constexpr (!ENDS) {
        const float xv = lv ? v.x.get(i) : 0.0f;
        dxv[i] = dlv[i] * xv;
        kp.dl[i] = dlv[i];
        kp.xv[i] = xv;
        kp.dsD[i] = dsv[i] * Dsk;
        dD_acc = __builtin_fmaf(dsv[i], xv, dD_acc);
      }
    }
    *reinterpret_cast<float2*>(&sm.rv[wv][buf][0][sr][2 * pr]) = make_float2(dlv[0], dlv[1]);
    if constexpr (!ENDS)
      *reinterpret_cast<float2*>(&sm.rv[wv][buf][1][sr][2 * pr]) = make_float2(dxv[0], dxv[1]);
    *reinterpret_cast<float2*>(&sm.rv[wv][buf][2][sr][2 * pr]) = make_float2(dsv[0], dsv[1]);
    const float bcv = bnok && k * BW_T + bt < L ? widen<IN>(v.bc) : 0.0f;
    sm.bc[buf][isC ? 1 : 0][bn][4 * ((bt >> 2) ^ (bn >> 3)) + (bt & 3)] = bcv;
    if constexpr (GATED && !ENDS) {
      if (BUF || want_dz) st2(rodz, dzp, k, kp.lv, zv2[0], zv2[1]);
    }
  };

  auto row4 = [&](int buf, int q, int j, int blk) {
    return *reinterpret_cast<const float4*>(&sm.rv[wv][buf][q][rl + 8 * j][4 * blk]);
  };
  auto bc4 = [&](int buf, int q, int i, int blk) {
    return *reinterpret_cast<const float4*>(&sm.bc[buf][q][2 * nl + i][4 * (blk ^ (nl >> 2))]);
  };
  float* const spw = sm.sp[wv];

  // ---- ddelta, dx of tile k (staging role) from the wavefront's partials
  auto finish_rows = [&](int64_t k, const Keep& kp) {
    const int q = pr & 1, tq = pr >> 1;
    const float* const p = spw + q * BW_SPQ + sr * BW_SPR + 4 * (tq ^ (sr & 1));
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float4 f = *reinterpret_cast<const float4*>(p + 8 * i);
      v[0] += f.x;
      v[1] += f.y;
      v[2] += f.z;
      v[3] += f.w;
    }
    // lane q = 0 holds lam q A of steps 4tq .. +3, q = 1 lam B: each keeps its
    // two steps (2 pr, 2 pr + 1) and takes the other quantity's from its peer
    const float r0 = lane_xor1(q ? v[0] : v[2]), r1 = lane_xor1(q ? v[1] : v[3]);
    const float sa[2] = {q ? r0 : v[0], q ? r1 : v[1]};
    const float sb[2] = {q ? v[2] : r0, q ? v[3] : r1};
    float dd[2], dx[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      dd[i] = kp.lv[i] ? __builtin_fmaf(kp.xv[i], sb[i], sa[i]) * kp.sg[i] : 0.0f;
      dx[i] = __builtin_fmaf(kp.dl[i], sb[i], kp.dsD[i]);
      db_acc += dd[i];
    }
    if constexpr (OS == 4) {
      if (!first) {  // later state groups add to the sums over the states
        const int64_t o = (int64_t)src * L + k * BW_T + 2 * pr;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (kp.lv[i]) {
            dd[i] += ddp[o + i];
            dx[i] += dxp[o + i];
          }
        }
      }
    }
    st2(rodd, ddp, k, kp.lv, dd[0], dd[1]);
    st2(rodx, dxp, k, kp.lv, dx[0], dx[1]);
  };
  // ---- this workgroup's share of dB (tid < 128) or dC at step bt, state bn
  auto finish_share = [&](int64_t k, bool live, int buf) {
    const int l = (isC ? 32 : 0) + (bn & 1) * 8 + (bn >> 1);
    float s = 0.0f;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) s += sm.pw[buf][m][bt >> 2][(l + 16 * hh) * 4 + (bt & 3)];
    const int64_t t = k * BW_T + bt;
    if constexpr (BUF)
      __builtin_amdgcn_raw_buffer_store_b32(
          __float_as_uint(s), rsh, live && t < L ? ((int32_t)t * BW_N + bn) * 4 : (int32_t)sh_b, 0, 0);
    else
      *(live && t < L ? shp + t * BW_N + bn : w.trash + tid) = s;
  };

  // ---- prologue: the last tile staged, the one before in flight
  Raw raw;
  Keep kn, kc{};  // of the tile staged, and of the tile walked
  float hc[2][2], hn[2][2];
  float dsum[2] = {0.f, 0.f};
  load_tile(k_hi - 1, raw);
  if constexpr (!ENDS) load_ck(k_hi - 1, hn);
  stage(k_hi - 1, true, raw, (int)((k_hi - 1) & 1), kn);
  load_tile(k_hi - 2, raw);

  for (int64_t k = k_hi - 1; k >= k_lo; --k) {
    const int buf = (int)(k & 1);
    bw_barrier();  // tile k is staged, tile k+1's row sums are complete
    if constexpr (!ENDS) {
      finish_rows(k + 1, kc);  // (nothing to store in the first round)
      finish_share(k + 1, k + 1 < k_hi, buf ^ 1);
      kc = kn;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) hc[i][j] = dok[j] && nok[i] ? hn[i][j] : 0.0f;
      load_ck(k - 1, hn);
    }
    stage(k - 1, k > k_lo, raw, buf ^ 1, kn);  // (past the segment: nothing kept or stored)
    load_tile(k - 2, raw);
    if constexpr (ENDS) {
#pragma unroll
      for (int blk = 1; blk >= 0; --blk) {
        float dl[2][4], ds[2][4], c[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const float4 f = row4(buf, 0, j, blk), e = row4(buf, 2, j, blk), q = bc4(buf, 1, j, blk);
          dl[j][0] = f.x, dl[j][1] = f.y, dl[j][2] = f.z, dl[j][3] = f.w;
          ds[j][0] = e.x, ds[j][1] = e.y, ds[j][2] = e.z, ds[j][3] = e.w;
          c[j][0] = q.x, c[j][1] = q.y, c[j][2] = q.z, c[j][3] = q.w;
        }
#pragma unroll
        for (int t = 3; t >= 0; --t) {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            dsum[j] += dl[j][t];
#pragma unroll
            for (int i = 0; i < 2; ++i)
              lam[i][j] = __builtin_amdgcn_exp2f(dl[j][t] * Al[i][j]) *
                          __builtin_fmaf(ds[j][t], c[i][t], lam[i][j]);
          }
        }
      }
    } else {
      // recompute a_t, q_t = a_t h_{t-1}; ds h of both states, over the two rows
      float av[2][2][BW_T], qv[2][2][BW_T], ph[2][BW_T];
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) {
        float dl[2][4], dx[2][4], ds[2][4], bb[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const float4 f = row4(buf, 0, j, blk), e = row4(buf, 1, j, blk), d = row4(buf, 2, j, blk);
          const float4 q = bc4(buf, 0, j, blk);
          dl[j][0] = f.x, dl[j][1] = f.y, dl[j][2] = f.z, dl[j][3] = f.w;
          dx[j][0] = e.x, dx[j][1] = e.y, dx[j][2] = e.z, dx[j][3] = e.w;
          ds[j][0] = d.x, ds[j][1] = d.y, ds[j][2] = d.z, ds[j][3] = d.w;
          bb[j][0] = q.x, bb[j][1] = q.y, bb[j][2] = q.z, bb[j][3] = q.w;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = 4 * blk + u;
#pragma unroll
          for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              av[i][j][t] = __builtin_amdgcn_exp2f(dl[j][u] * Al[i][j]);
              qv[i][j][t] = av[i][j][t] * hc[i][j];
              hc[i][j] = __builtin_fmaf(dx[j][u], bb[i][u], qv[i][j][t]);
            }
            ph[i][t] = __builtin_fmaf(ds[1][u], hc[i][1], ds[0][u] * hc[i][0]);
          }
        }
      }
      // walk the tile backwards
#pragma unroll
      for (int blk = 1; blk >= 0; --blk) {
        float dl[2][4], dx[2][4], ds[2][4], bb[2][4], cc[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const float4 f = row4(buf, 0, j, blk), e = row4(buf, 1, j, blk), d = row4(buf, 2, j, blk);
          const float4 q = bc4(buf, 0, j, blk), p = bc4(buf, 1, j, blk);
          dl[j][0] = f.x, dl[j][1] = f.y, dl[j][2] = f.z, dl[j][3] = f.w;
          dx[j][0] = e.x, dx[j][1] = e.y, dx[j][2] = e.z, dx[j][3] = e.w;
          ds[j][0] = d.x, ds[j][1] = d.y, ds[j][2] = d.z, ds[j][3] = d.w;
          bb[j][0] = q.x, bb[j][1] = q.y, bb[j][2] = q.z, bb[j][3] = q.w;
          cc[j][0] = p.x, cc[j][1] = p.y, cc[j][2] = p.z, cc[j][3] = p.w;
        }
        float sa[2][4], sb[2][4], px[2][4];
#pragma unroll
        for (int u = 3; u >= 0; --u) {
          const int t = 4 * blk + u;
#pragma unroll
          for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const float l = __builtin_fmaf(ds[j][u], cc[i][u], lam[i][j]);
              const float p = l * qv[i][j][t];
              dA_acc[i][j] = __builtin_fmaf(p, dl[j][u], dA_acc[i][j]);
              sa[j][u] = i == 0 ? p * Ar[0][j] : __builtin_fmaf(p, Ar[1][j], sa[j][u]);
              sb[j][u] = i == 0 ? l * bb[0][u] : __builtin_fmaf(l, bb[1][u], sb[j][u]);
              px[i][u] = j == 0 ? l * dx[0][u] : __builtin_fmaf(l, dx[1][u], px[i][u]);
              lam[i][j] = av[i][j][t] * l;
            }
          }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int r = rl + 8 * j;
          float* const p = spw + r * BW_SPR + 8 * nl + 4 * (blk ^ (r & 1));
          *reinterpret_cast<float4*>(p) = make_float4(sa[j][0], sa[j][1], sa[j][2], sa[j][3]);
          *reinterpret_cast<float4*>(p + BW_SPQ) = make_float4(sb[j][0], sb[j][1], sb[j][2], sb[j][3]);
        }
        // sums over the wavefront's rows but for lane bit 3: lanes 0-31 keep
        // lam delta x, lanes 32-63 ds h (v_permlane32_swap trades the upper
        // half of its first operand with the lower of its second), then even
        // 16-lane rows state 2nl, odd rows state 2nl+1
        float o[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float r2[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const auto v = __builtin_amdgcn_permlane32_swap(
                __float_as_uint(px[i][u]), __float_as_uint(ph[i][4 * blk + u]), false, false);
            r2[i] = __uint_as_float(v[0]) + __uint_as_float(v[1]);
          }
          const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(r2[0]),
                                                          __float_as_uint(r2[1]), false, false);
          o[u] = __uint_as_float(v[0]) + __uint_as_float(v[1]);
        }
        // slot (quantity: bit 5, row half: bit 3, state: bit 4, nl), so that the
        // 16 states of a sum are contiguous
        const int slot = (lane & 32) | ((lane & 8) << 1) | ((lane & 16) >> 1) | nl;
        *reinterpret_cast<float4*>(&sm.pw[buf][wv][blk][slot * 4]) = make_float4(o[0], o[1], o[2], o[3]);
      }
    }
    bw_wave_order();  // this wavefront's partials are written before their reads
  }

  if constexpr (ENDS) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (dok[j]) {
          float* const rp = w.rec + (int64_t)(2 * (sg - 1)) * R * BW_N + (row0 + rj[j]) * BW_N + 2 * nl + i;
          rp[0] = __builtin_amdgcn_exp2f(Al[i][j] * dsum[j]);
          rp[R * BW_N] = nok[i] ? lam[i][j] : 0.0f;
        }
      }
  } else {
    bw_barrier();  // the first tile's row sums are complete
    finish_rows(k_lo, kc);
    finish_share(k_lo, true, (int)(k_lo & 1));
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (dok[j]) {
          if (sg == 0 && a.dh0 && nok[i]) a.dh0[(row0 + rj[j]) * N + n0 + 2 * nl + i] = lam[i][j];
          w.dA_p[((int64_t)sg * R + row0 + rj[j]) * BW_N + 2 * nl + i] = dA_acc[i][j];
        }
      }
#pragma unroll
    for (int off = 1; off < 4; off *= 2) {
      dD_acc += __shfl_xor(dD_acc, off);
      db_acc += __shfl_xor(db_acc, off);
    }
    if (pr == 0 && sdok) {
      const int64_t o = (int64_t)sg * R + row0 + sr;
      if (first) {
        w.dD_p[o] = dD_acc;
        w.db_p[o] = db_acc;
      } else {
        w.db_p[o] += db_acc;
      }
    }
  }
}

// The states before every 8th step, for calls without checkpoints: one lane
// per state, 16 rows of one batch per workgroup, whole rows forward.  Raw
// inputs of tile j live in ring[j % SW_RING]: loads run SW_RING - 1 tiles
// ahead of their use, from clamped addresses.
constexpr int SW_ROWS = 16, SW_RING = 4;

struct SweepSmem {
  float rv[2][2][SW_ROWS][BW_T];  // two tile buffers: delta, delta*x
  float b[2][BW_N][BW_T];         // B as [n][t], halves swapped for n >= 8
};

template <typename IN>
__global__ __launch_bounds__(256) void selective_sweep_kernel(const BwdArgs a, float* __restrict__ ck,
                                                              int64_t G, int64_t ntile, int n0) {
  __shared__ __align__(16) SweepSmem sm;
  const IN* __restrict__ X = static_cast<const IN*>(a.x);
  const IN* __restrict__ DL = static_cast<const IN*>(a.delta);
  const IN* __restrict__ BM = static_cast<const IN*>(a.Bm);
  const int64_t D = a.D, L = a.L, N = a.N;
  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid / 64);
  const int rr = 4 * wv + (tid % 64) / 16;  // row within the workgroup
  const int n = tid % 16, ns = n0 + n;
  const int64_t b = blockIdx.x / G;
  const int64_t d0 = (blockIdx.x - b * G) * SW_ROWS;
  const int64_t d = d0 + rr;
  const bool dok = d < D, nok = ns < N;
  const int64_t row = b * D + (dok ? d : D - 1);
  // staging: wavefronts 0-1 own (row sr, step st), 2-3 (step bt, state bn)
  const bool role_a = wv < 2;
  const int sr = (tid % 128) / BW_T, st = tid % BW_T;
  const int bt = (tid % 128) / BW_N, bn = tid % BW_N;
  const int64_t sd = d0 + sr;
  const bool sdok = sd < D;
  const int64_t srow = b * D + (sdok ? sd : D - 1);
  const float Al = nok ? a.A[(dok ? d : D - 1) * N + ns] * BW_LOG2E : 0.0f;
  const float dbias = a.delta_bias ? a.delta_bias[sdok ? sd : D - 1] : 0.0f;
  struct Raw {
    IN r0, r1;
    bool ok;
  };
  // (both roles run the same loads: one inside a branch is waited for there)
  const IN* __restrict__ P0 = role_a ? X : BM;
  const IN* __restrict__ P1 = role_a ? DL : BM;
  auto load = [&](int64_t k, Raw& v) {
    const int64_t ta = k * BW_T + st, tb = k * BW_T + bt;
    const int64_t tca = ta < L ? ta : L - 1, tcb = tb < L ? tb : L - 1;
    const int64_t ib = (b * L + tcb) * N + (n0 + bn < N ? n0 + bn : N - 1);
    v.ok = role_a ? sdok && ta < L : tb < L && n0 + bn < N;
    const int64_t i = role_a ? srow * L + tca : ib;
    v.r0 = P0[i];
    v.r1 = P1[i];
  };
  Raw ring[SW_RING];
  float h = (a.h0 && dok && nok) ? a.h0[row * N + ns] : 0.0f;
#pragma unroll
  for (int u = 0; u < SW_RING - 1; ++u) load(u, ring[u]);
  for (int64_t k0 = 0; k0 < ntile; k0 += SW_RING) {
#pragma unroll
    for (int u = 0; u < SW_RING; ++u) {
      const int64_t k = k0 + u;
      if (k >= ntile) break;
      const int buf = u & 1;  // SW_RING is even, so this is k & 1
      const Raw& cur = ring[u];
      if (role_a) {
        float dv = widen<IN>(cur.r1) + dbias;
        if (a.softplus) dv = softplus_f32(dv);
        dv = cur.ok ? dv : 0.0f;
        sm.rv[buf][0][sr][st] = dv;
        sm.rv[buf][1][sr][st] = cur.ok ? dv * widen<IN>(cur.r0) : 0.0f;
      } else {
        sm.b[buf][bn][bt ^ ((bn >> 1) & 4)] = cur.ok ? widen<IN>(cur.r0) : 0.0f;
      }
      load(k + SW_RING - 1, ring[(u + SW_RING - 1) % SW_RING]);
      bw_barrier();  // one per tile: the other buffer is the one staged next
      if (dok) ck[(row * ntile + k) * BW_N + n] = h;
#pragma unroll
      for (int q = 0; q < BW_T; q += 4) {
        const float4 dl4 = *reinterpret_cast<const float4*>(&sm.rv[buf][0][rr][q]);
        const float4 dx4 = *reinterpret_cast<const float4*>(&sm.rv[buf][1][rr][q]);
        const float4 b4 = *reinterpret_cast<const float4*>(&sm.b[buf][n][q ^ ((n >> 1) & 4)]);
        const float dlq[4] = {dl4.x, dl4.y, dl4.z, dl4.w};
        const float dxq[4] = {dx4.x, dx4.y, dx4.z, dx4.w};
        const float bq[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
          h = __builtin_fmaf(__builtin_amdgcn_exp2f(dlq[j] * Al), h, dxq[j] * bq[j]);
      }
    }
  }
}

// Adds the shares in a fixed order: dB, dC over the workgroups of a batch
// (one thread per 4 states of one (b, t) and one of dB / dC, float4 loads,
// eight in flight, summed in workgroup order); dA, dDskip, ddelta_bias over
// batch and segments.
// With state groups (N > 16) it runs after each group's main kernel and
// writes that group's states n0 .. n0+15; dDskip and ddelta_bias after the
// last group (last = true).
template <typename OUT>
__global__ __launch_bounds__(256) void selective_bwd_reduce_kernel(const BwdArgs a,
                                                                   const BwWork w, int64_t G,
                                                                   int n0, bool last, int nseg) {
  const int64_t B = a.B, D = a.D, N = a.N, L = a.L;
  const int64_t ng = N - n0 < BW_N ? N - n0 : BW_N;  // states of this group
  const int64_t nq = B * L * (BW_N / 4);  // float4 chunks of one of dB / dC
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t gstep = L * (BW_N / 4);   // float4 stride between workgroup shares
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 2 * nq; i += stride) {
    const bool isC = i >= nq;
    const int64_t r = isC ? i - nq : i;  // r = (b*L + t)*4 + c
    const int64_t c = r % (BW_N / 4), bt = r / (BW_N / 4);
    const int64_t b = bt / L;
    const float4* __restrict__ src =
        reinterpret_cast<const float4*>(isC ? w.dC_p : w.dB_p) + b * G * gstep + (bt - b * L) * 4 + c;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int64_t g = 0;
    for (; g + 8 <= G; g += 8) {
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = src[(g + u) * gstep];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        acc.x += v[u].x;
        acc.y += v[u].y;
        acc.z += v[u].z;
        acc.w += v[u].w;
      }
    }
    for (; g < G; ++g) {
      const float4 v = src[g * gstep];
      acc.x += v.x;
      acc.y += v.y;
      acc.z += v.z;
      acc.w += v.w;
    }
    OUT* const dst = static_cast<OUT*>(isC ? a.dC : a.dB) + bt * N + n0;
    const float av[4] = {acc.x, acc.y, acc.z, acc.w};
    if (N == BW_N && (((uintptr_t)a.dB | (uintptr_t)a.dC) & 15) == 0) {
      if constexpr (sizeof(OUT) == 4)
        *reinterpret_cast<float4*>(dst + 4 * c) = acc;
      else
        *reinterpret_cast<uint2*>(dst + 4 * c) =
            make_uint2(bf16x2_rne(acc.x, acc.y), bf16x2_rne(acc.z, acc.w));
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (4 * c + u < ng) st1<OUT>(dst + 4 * c + u, av[u]);
    }
  }
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < D * ng; i += stride) {
    const int64_t d = i / ng, nn = i - d * ng;
    float s = 0.f;
#pragma unroll 8
    for (int64_t b = 0; b < B * nseg; ++b) s += w.dA_p[(b * D + d) * BW_N + nn];
    a.dA[d * N + n0 + nn] = s;
  }
  if (!last) return;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < D; i += stride) {
    float sd = 0.f, sbias = 0.f;
#pragma unroll 8
    for (int64_t b = 0; b < B * nseg; ++b) {
      sd += w.dD_p[b * D + i];
      sbias += w.db_p[b * D + i];
    }
    if (a.dDskip) a.dDskip[i] = sd;
    if (a.ddelta_bias) a.ddelta_bias[i] = sbias;
  }
}

// True when every byte offset of the buffer-resource path stays below 2^31:
// a wavefront's rows of x, delta, dy, z, s and its checkpoints, and a batch's
// B, C and shares, with the tiles past the end.
bool bwd_buf_fits(const BwdArgs& a, int64_t ntile) {
  const int64_t lim = (int64_t)1 << 31;
  const int64_t Lp = a.L + 4 * BW_T;
  return BW_WROWS * Lp * 4 < lim && Lp * a.N * 4 < lim && Lp * BW_N * 4 < lim &&
         BW_WROWS * (ntile + 2) * BW_N * 4 < lim;
}

// Rows whose pairs of steps are one access: even length, bf16 on a dword.
bool bwd_pairs(const BwdArgs& a) {
  uintptr_t p = 0;
  if (a.bf16_in) p |= (uintptr_t)a.x | (uintptr_t)a.delta | (uintptr_t)a.z;
  if (a.dy_bf16) p |= (uintptr_t)a.dy;
  if (a.grads_bf16) p |= (uintptr_t)a.dx | (uintptr_t)a.ddelta | (uintptr_t)a.dz;
  return a.L % 2 == 0 && p % 4 == 0;
}

struct BwdPlan {
  int nseg;
  int64_t seg_tiles;
  bool rows16;  // the kernel of selective_bwd16.hip, on whole rows
};

template <typename IN, typename DYT, typename OUT, bool GATED, bool PAIR, bool BUF>
void launch_bwd_k(const BwdArgs& a, const BwWork& w, int64_t G, int64_t ntile, const BwdPlan& p,
                  int n0, hipStream_t s) {
  if (p.nseg > 1)
    hipLaunchKernelGGL((selective_bwd_kernel<IN, DYT, OUT, GATED, PAIR, BUF, BW_ENDS>),
                       dim3((unsigned)(a.B * G * (p.nseg - 1))), dim3(256), 0, s, a, w, G, ntile,
                       n0, p.nseg, p.seg_tiles);
  hipLaunchKernelGGL((selective_bwd_kernel<IN, DYT, OUT, GATED, PAIR, BUF, BW_MAIN>),
                     dim3((unsigned)(a.B * G * p.nseg)), dim3(256), 0, s, a, w, G, ntile, n0,
                     p.nseg, p.seg_tiles);
}

template <typename IN, typename DYT, typename OUT>
void launch_bwd_t(const BwdArgs& a, const BwWork& w, int64_t G, int64_t ntile, const BwdPlan& p,
                  int n0, hipStream_t s) {
  const bool buf = bwd_buf_fits(a, ntile), pair = buf && bwd_pairs(a);
  if (a.z) {
    if (pair)
      launch_bwd_k<IN, DYT, OUT, true, true, true>(a, w, G, ntile, p, n0, s);
    else if (buf)
      launch_bwd_k<IN, DYT, OUT, true, false, true>(a, w, G, ntile, p, n0, s);
    else
      launch_bwd_k<IN, DYT, OUT, true, false, false>(a, w, G, ntile, p, n0, s);
  } else {
    if (pair)
      launch_bwd_k<IN, DYT, OUT, false, true, true>(a, w, G, ntile, p, n0, s);
    else if (buf)
      launch_bwd_k<IN, DYT, OUT, false, false, true>(a, w, G, ntile, p, n0, s);
    else
      launch_bwd_k<IN, DYT, OUT, false, false, false>(a, w, G, ntile, p, n0, s);
  }
}

void launch_bwd(const BwdArgs& a, const BwWork& w, int64_t G, int64_t ntile, const BwdPlan& p,
                int n0, hipStream_t s) {
  if (!a.bf16_in) {  // fp32 gradients
    if (a.dy_bf16)
      launch_bwd_t<float, uint16_t, float>(a, w, G, ntile, p, n0, s);
    else
      launch_bwd_t<float, float, float>(a, w, G, ntile, p, n0, s);
  } else if (a.grads_bf16) {  // fp32 dy
    launch_bwd_t<uint16_t, float, uint16_t>(a, w, G, ntile, p, n0, s);
  } else {
    if (a.dy_bf16)
      launch_bwd_t<uint16_t, uint16_t, float>(a, w, G, ntile, p, n0, s);
    else
      launch_bwd_t<uint16_t, float, float>(a, w, G, ntile, p, n0, s);
  }
}

// Which kernel a call takes, and how many segments the 64-row one cuts the
// sequence into, priced like the forward's plan.  A launch of n workgroups runs
// in rounds of at most two (64 rows) or three (16 rows) per compute unit, by
// LDS and registers; a round takes BwdCost::us per tile of 8 steps with that
// many workgroups on the busiest compute unit, and `start` tiles more to start
// and end a segment.  Rows of odd length read their steps one by one: `odd`
// times that.  Cut calls add the adjoint's walk (BWD_WALK_US per tile for each
// workgroup resident, up to seven, and once more) and 5 us for its launch and
// the records.  State groups after the first read ddelta and dx back, 1.24
// times the 64-row kernel's time (0.12 more over two groups), and have their
// checkpoints from the forward's walk before it, where the 16-row kernel sweeps
// for them.  Beside the walk come a fixed part and the reduction of the shares of
// dB and dC, of which 16 rows a workgroup leave four times as many.  No call is
// below 27 us of host time.
// The constants are fits to 900 calls of up to 160000 rows, L = 32 to 8192, N = 8
// to 64, fp32 and bf16, gate with softplus or neither (what the sizing of the
// workspace knows of a call), each timed with the 16-row kernel and with the
// 64-row one in up to a dozen cuts.  More segments, and the 16-row kernel, have
// to be 3% cheaper: near a tie the simpler launch is the safer one.  The choice is
// 1.5% from the fastest on average (2.4% with the constants before), on 500 other
// calls 1.8%.  us per call with given checkpoints, 16-row / 64-row kernel:
//   B=8 D=1536 L=1024  ungated 202 / 279, gated 252 / 312 (fp32)
//   B=8 D=1536 L=2048  ungated 398 / 402 (fp32), 387 / 369 (bf16), gated 487 / 564
//                      (fp32), 453 / 479 (bf16)
//   B=8 D=1536 L=2047  ungated 425 / 513, gated 690 / 780 (fp32)
//   B=4 D=5120 L=1024  gated 421 / 528 (fp32)
//   B=4 D=1024 L=2048  ungated 271 / 157, gated 298 / 203 (fp32)
//   B=8 D=1600 L=2048  ungated 603 / 424, gated 696 / 593 (fp32)
//   B=4 D=5120 L=64    gated 52 / 42 (bf16)
//   B=1 D=1024 L=4096  ungated 505 / 113 (fp32)
struct BwdCost {
  int cap;          // workgroups per compute unit
  double start;     // tiles
  double fixed;     // us
  double us[2][3];  // [gated][workgroups resident - 1]
  double odd[2][3];
};
constexpr BwdCost COST_ROWS16 = {
    3, 4.0, 10.0, {{0.9, 1.19, 1.39}, {1.09, 1.27, 1.7}}, {{1.0, 1.0, 1.0}, {1.0, 1.0, 1.0}}};
constexpr BwdCost COST_ROWS64 = {
    2, 4.5, 1.8, {{2.0, 2.93, 0.0}, {2.31, 3.78, 0.0}}, {{1.03, 1.19, 0.0}, {1.43, 1.43, 0.0}}};
constexpr double BWD_WALK_US[2] = {0.265, 0.37};
constexpr double BWD_SHARE_US = 2.43e-5;  // per step of a workgroup's share
constexpr double BWD_HOST_US = 27.0;

// The walk of wgs workgroups (below 2^32) over `tiles` tiles.
double bwd_launch_us(const BwdCost& c, int64_t wgs, int64_t tiles, bool gated, bool odd, uint32_t cus) {
  const uint32_t per = ((uint32_t)wgs + cus - 1) / cus;
  const auto us = [&](uint32_t o) { return c.us[gated][o - 1] * (odd ? c.odd[gated][o - 1] : 1.0); };
  const double tile = (double)(per / c.cap) * us(c.cap) + (per % c.cap ? us(per % c.cap) : 0.0);
  return ((double)tiles + c.start) * tile;
}

BwdPlan plan_bwd(int64_t B, int64_t D, int64_t N, int64_t L, bool gated, uint32_t cus) {
  const int64_t ntile = (L + BW_T - 1) / BW_T, W = B * ((D + BW_ROWS - 1) / BW_ROWS);
  const int64_t W16 = B * ((D + 15) / 16);
  const int64_t ngrp = (N + BW_N - 1) / BW_N;
  const double groups = 1.0 + 0.12 * (double)(ngrp - 1) / (double)ngrp;
  const bool odd = L % 2 != 0;
  BwdPlan best{1, ntile, false};
  double us64 = groups * bwd_launch_us(COST_ROWS64, W, ntile, gated, odd, cus);
  for (int64_t k = 2; k <= BW_MAX_SEG && k <= ntile; ++k) {
    const int64_t tiles = (ntile + k - 1) / k, n = (ntile + tiles - 1) / tiles;
    if (n < 2 || W * n > SW_MAX_WGS) continue;
    const uint32_t e = ((uint32_t)(W * (n - 1)) + cus - 1) / cus;
    const double walk = BWD_WALK_US[gated] * (double)(e / 7 * 8 + (e % 7 ? e % 7 + 1 : 0));
    const double us = groups * bwd_launch_us(COST_ROWS64, W * n, tiles, gated, odd, cus) +
                      ((double)tiles + COST_ROWS64.start) * walk + 5.0;
    if (us < 0.97 * us64) {
      us64 = us;
      best = BwdPlan{(int)n, tiles, false};
    }
  }
  double us16 = bwd_launch_us(COST_ROWS16, W16, ntile, gated, odd, cus);
  if (ngrp > 1) {
    us16 *= 1.45;
    us64 += 1.47 * row16_rows_us(W16, L, (int)cus);
  }
  const auto call_us = [&](const BwdCost& c, double us, int64_t wgs) {
    us = (us + (double)wgs * (double)L * BWD_SHARE_US) * (double)ngrp + c.fixed;
    return us > BWD_HOST_US ? us : BWD_HOST_US;
  };
  // SW_SS_BWD_ROWS=16 or 64 keeps one kernel
  const char* const v = getenv("SW_SS_BWD_ROWS");
  const int force = v && *v ? atoi(v) : 0;
  const bool rows16 = call_us(COST_ROWS16, us16, W16) < 0.97 * call_us(COST_ROWS64, us64, W);
  if (W16 <= SW_MAX_WGS && (force == 16 || (force != 64 && rows16))) best = BwdPlan{1, ntile, true};
  return best;
}

// The call's sizes: workgroups per batch, tiles, segments, and the floats of
// each part of the workspace.
struct BwdSizes {
  int64_t G, ntile;
  BwdPlan plan;
  size_t ck, bc, rec, dA, s, d, total;
  size_t planes;  // bytes
};

BwdSizes bwd_sizes(int64_t B, int64_t D, int64_t N, int64_t L, bool ckpt, bool gated, bool pre) {
  BwdSizes z;
  z.ntile = (L + BW_T - 1) / BW_T;
  int cus = 0;
  if (device_cus(&cus) != SW_OK) cus = 256;
  z.plan = plan_bwd(B, D, N, L, gated, (uint32_t)cus);
  const int64_t rows = z.plan.rows16 ? 16 : BW_ROWS;
  z.G = (D + rows - 1) / rows;
  const size_t R = (size_t)(B * D), nseg = (size_t)z.plan.nseg;
  // without the forward's checkpoints the call rebuilds them in the workspace,
  // where before that the ungated forward keeps its planes of y (N > 16)
  z.ck = ckpt ? 0 : R * (size_t)z.ntile * BW_N;
  z.planes = 0;
  for (const bool bf16 : {false, true}) {
    const size_t p = pre ? (size_t)selective_fwd_workspace(B, D, N, L, bf16, false, false) : 0;
    if (z.planes < p) z.planes = p;
  }
  const size_t pw = (z.planes / sizeof(float) + 3) / 4 * 4;
  if (z.ck < pw) z.ck = pw;
  z.bc = (size_t)(B * z.G) * (size_t)L * BW_N;
  z.rec = 2 * R * BW_N * (nseg - 1);
  z.dA = R * BW_N * nseg;
  z.s = pre ? R * (size_t)L : 0;
  z.d = R * nseg;
  // 16-byte groups first: shares and checkpoints are read as vectors
  z.total = z.ck + 2 * z.bc + z.rec + z.dA + z.s + 2 * z.d + 1024;
  return z;
}

}  // namespace

int64_t selective_bwd_workspace(int64_t B, int64_t D, int64_t N, int64_t L, bool ckpt, bool z,
                                bool s_pre) {
  return (int64_t)(bwd_sizes(B, D, N, L, ckpt, z, z && !s_pre).total * sizeof(float));
}

int selective_bwd(const BwdArgs& a) {
  if (a.ckpt && a.N > BW_N)
    return fail(SW_ERR_UNSUPPORTED, "checkpoints hold 16 states (N=%lld)", (long long)a.N);
  hipStream_t s = current_stream();
  const int64_t B = a.B, D = a.D, L = a.L;
  const int64_t G16 = (D + SW_ROWS - 1) / SW_ROWS;
  // (the sweep that rebuilds checkpoints takes 16 rows a workgroup)
  const int64_t wgs = B * (a.ckpt ? (D + BW_ROWS - 1) / BW_ROWS : G16);
  if (wgs > SW_MAX_WGS)
    return fail(SW_ERR_UNSUPPORTED, "%lld workgroups exceed the grid range", (long long)wgs);
  const BwdSizes z = bwd_sizes(B, D, a.N, L, a.ckpt != nullptr, a.z != nullptr, a.z && !a.s_pre);
  const int64_t G = z.G, ntile = z.ntile;
  const BwdPlan plan = z.plan;
  void* base = a.ws;
  int st;
  if (base) {
    if (a.ws_bytes < z.total * sizeof(float))
      return fail(SW_ERR_INVALID_ARG, "workspace of %zu bytes, %zu needed", a.ws_bytes,
                  z.total * sizeof(float));
    st = refuse_capture(s, "a workspace allocated per call");
  } else {
    st = workspace_alloc(&base, z.total * sizeof(float), s);
  }
  if (st != SW_OK) return st;
  const auto done = [&] {
    if (!a.ws) workspace_free(base, s);
  };
  float* f = static_cast<float*>(base);
  BwWork w;
  w.ck = a.ckpt ? const_cast<float*>(a.ckpt) : f;  // read-only when given
  f += z.ck;
  w.dB_p = f;
  f += z.bc;
  w.dC_p = f;
  f += z.bc;
  w.rec = f;
  f += z.rec;
  w.dA_p = f;
  f += z.dA;
  float* s_pre = (a.z && !a.s_pre) ? f : nullptr;
  w.s = a.s_pre ? a.s_pre : s_pre;
  f += z.s;
  w.dD_p = f;
  f += z.d;
  w.db_p = f;
  f += z.d;
  w.trash = f;
  // with a gate, the forward without the gate runs anyway (for the pre-gate
  // output); for N <= 16 it also writes the tile checkpoints, so the backward
  // kernel skips its own forward sweep (the checkpoints are bit-identical)
  BwdArgs ab = a;
  if (a.z && !a.s_pre) {
    // the pre-gate output: the forward pass without the gate
    SelArgs fa{};
    fa.x = a.x;
    fa.delta = a.delta;
    fa.Bm = a.Bm;
    fa.Cm = a.Cm;
    fa.A = a.A;
    fa.Dskip = a.Dskip;
    fa.delta_bias = a.delta_bias;
    fa.h0 = a.h0;
    fa.y = s_pre;
    fa.B = B;
    fa.D = D;
    fa.N = a.N;
    fa.L = L;
    fa.bf16_in = a.bf16_in;
    fa.softplus = a.softplus;
    fa.vec = a.vec;
    if (z.planes > 0) {
      fa.ws = w.ck;
      fa.ws_bytes = z.planes;
    }
    if (!a.ckpt && a.N <= BW_N) {
      fa.ckpt = w.ck;
      ab.ckpt = w.ck;
    }
    st = selective_fwd(fa);
    if (st != SW_OK) {
      done();
      return st;
    }
  }
  // still without checkpoints: where the 16-lane kernels can walk the call,
  // their walk without y writes them (the states do not depend on the gate),
  // bit-identical to a sweep.  The 64-row kernel otherwise has a sweep kernel
  // run before it; the 16-row kernel sweeps by itself, which also is faster
  // than a walk per state group where it is taken (us per call, walk / own
  // sweep: B=8 D=1536 N=64 L=64 bf16 151 / 123, B=4 D=2560 N=64 L=300 395 / 359).
  SelArgs sa{};
  sa.x = a.x;
  sa.delta = a.delta;
  sa.Bm = a.Bm;
  sa.Cm = a.Cm;
  sa.A = a.A;
  sa.delta_bias = a.delta_bias;
  sa.h0 = a.h0;
  sa.B = B;
  sa.D = D;
  sa.N = a.N;
  sa.L = L;
  sa.bf16_in = a.bf16_in;
  sa.softplus = a.softplus;
  sa.vec = a.vec;
  sa.ckpt = w.ck;
  const char* ck_from = a.ckpt ? "given" : ab.ckpt ? "from the ungated forward" : nullptr;
  // the states in groups of 16: each group's main kernel, then its reduction
  // (dA, dB, dC of its states; the sums over the states accumulate)
  for (int n0 = 0; n0 < a.N && st == SW_OK; n0 += BW_N) {
    BwdArgs ag = ab;  // of this group
    if (!ab.ckpt) {
      bool taken = false;
      if (!plan.rows16 || a.N == BW_N) st = selective_states_fwd(sa, n0 / BW_N, &taken);
      if (st != SW_OK) break;
      ck_from = taken ? "from the forward's walk without y" : "rebuilt by a sweep";
      if (taken) {
        ag.ckpt = w.ck;
      } else if (!plan.rows16) {
        auto kern = a.bf16_in ? selective_sweep_kernel<uint16_t> : selective_sweep_kernel<float>;
        hipLaunchKernelGGL(kern, dim3((unsigned)(B * G16)), dim3(256), 0, s, a, w.ck, G16, ntile, n0);
        st = check_launch("selective_sweep_kernel");
        if (st != SW_OK) break;
      }
    }
    if (plan.rows16)
      launch_bwd_rows16(ag, w, G, ntile, n0, s);
    else
      launch_bwd(ag, w, G, ntile, plan, n0, s);
    st = check_launch("selective_bwd_kernel");
    if (st != SW_OK) break;
    int64_t work = 2 * B * L * (BW_N / 4);
    if (work < D * BW_N) work = D * BW_N;
    int64_t blocks = (work + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) blocks = 1;
    auto red = a.grads_bf16 ? selective_bwd_reduce_kernel<uint16_t> : selective_bwd_reduce_kernel<float>;
    hipLaunchKernelGGL(red, dim3((unsigned)blocks), dim3(256), 0, s, a, w, G, n0, n0 + BW_N >= a.N,
                       plan.nseg);
    st = check_launch("selective_bwd_reduce_kernel");
  }
  done();
  if (st == SW_OK)
    note_launch("%s + selective_bwd_reduce_kernel (%lld state group%s, %d "
                "segment%s), checkpoints %s",
                plan.rows16 ? "selective_bwd_rows16_kernel" : "selective_bwd_kernel",
                (long long)((a.N + BW_N - 1) / BW_N), a.N > BW_N ? "s" : "", plan.nseg,
                plan.nseg > 1 ? "s" : "", ck_from);
  return st;
}

}  // namespace sw
