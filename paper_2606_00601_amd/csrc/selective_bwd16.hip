// selective_bwd16.hip -- backward of the fused selective scan on gfx950 for
// calls whose 16-row blocks fill the compute units: one state per lane, whole
// rows, no second walk.
//
// The operation and the quantities are those of selective_bwd.hip.  One
// workgroup (4 wavefronts) owns 16 rows of one batch; lane n of a 16-lane row
// owns state n0 + n (states past N are identity steps).  Without checkpoints a
// forward sweep of the same lanes first writes the state before every 8th step.
// Then it walks the tiles of its rows backwards: a tile's delta, delta*x, ds and B, C
// are staged in LDS; every lane reloads its checkpoint, recomputes the tile's
// a_t and q_t forward into registers, then walks the tile backwards carrying
// lam.  Per step it forms four partial products: lam q A and lam B (summed over
// n, per row and step, into ddelta and dx) go to LDS; lam delta x and ds h
// (summed over the 16 rows, per step and state, into this workgroup's share of
// dB and dC) are first summed over the wavefront's four rows by lane-half
// exchanges, and only those sums go to LDS.  Half of the workgroup sums the
// first pair per (row, step), the other half adds the four wavefronts' row sums
// per (step, state); selective_bwd.hip's reduction adds the shares.
//
// Against the 64-row kernel it stages B and C once per 16 rows and leaves four
// times as many shares of dB and dC, but it gives four times as many
// workgroups, three to a compute unit, so that calls of two or three of them
// per compute unit need no segments and no second walk.  The rule between the
// two, with both sides measured, is plan_bwd (selective_bwd.hip).  Bound by
// instruction issue and LDS at 149 VGPRs and 48 KB (three wavefronts a SIMD).
#include "bwd_common.h"

namespace sw {
namespace {

constexpr int B16_ROWS = 16;  // (b,d) rows per workgroup
constexpr int B16_TS = 8;     // LDS stride of one [t] run (16-byte aligned)
// stride of one row's [n][t] block: 8 mod 64 banks, so that the 64 lanes of a
// (row, step) reduce (8 rows x 8 steps) read 64 different banks
constexpr int B16_RS = BW_N * B16_TS + 8;
constexpr int B16_RING = 4;   // raw tile registers: loads run 3 tiles ahead

// Position of step t of state n inside its 8-step run: the two 4-step halves
// trade places for n >= 8, so that the 16 states of a row (float4 accesses)
// and the 16 x 4 (state, step) lanes of the reduces fall on 64 different banks.
__device__ __forceinline__ int swz(int n, int t) { return t ^ ((n >> 1) & 4); }

struct B16Smem {
  float rv[2][3][B16_ROWS][B16_TS];  // two tile buffers; per row and step: delta, delta*x, ds
  float bc[2][2][BW_N][B16_TS];      // two tile buffers; B, C of the tile as [n][t]
  // partials, two buffers (tile k uses k & 1): the sums of tile k+1 are read
  // while tile k's are written, so one barrier per tile orders both
  float sp[2][2][B16_ROWS * B16_RS];  // per row [n][t]: lam q A, lam B   (sum over n)
  float pw[2][4][64 * 4];             // per wavefront and lane: four row sums (rows4_sum)
};

// Sums over the four 16-lane rows of a wavefront, by the two lane-half
// exchanges of gfx950: v_permlane32_swap trades lanes 32-63 of its first
// operand with lanes 0-31 of its second, v_permlane16_swap the odd 16-lane
// rows of the first with the even rows of the second.  In: a lane's
// lam delta x (dx) and ds h (dh) at the tile's 8 steps.  Out: lane l holds,
// for state l % 16, the sums over the four rows of dx (l < 32) or dh
// (l >= 32) at steps 4 ((l / 16) & 1) + 0..3.
__device__ __forceinline__ void rows4_sum(const float (&dx)[8], const float (&dh)[8],
                                          float (&out)[4]) {
  float r[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    // lanes 0-31 get dx of lanes l and l+32, lanes 32-63 dh of l-32 and l
    const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(dx[t]),
                                                    __float_as_uint(dh[t]), false, false);
    r[t] = __uint_as_float(v[0]) + __uint_as_float(v[1]);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    // row 0 of the wavefront gets rows 0 + 1 of r[t], row 1 rows 0 + 1 of
    // r[t+4], rows 2 and 3 likewise from rows 2 + 3
    const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(r[t]),
                                                    __float_as_uint(r[t + 4]), false, false);
    out[t] = __uint_as_float(v[0]) + __uint_as_float(v[1]);
  }
}

// One staging thread's raw inputs of one tile.  Waves 0-1 read x, delta, dy
// (and z, s) of (row, step); waves 2-3 read B, C of (step, state) through the
// same two slots r0, r1, so that every thread runs the same straight-line
// loads (their dy, z, s slots read a valid, unused element).
template <typename IN, typename DYT>
struct TileRaw {
  IN r0, r1, z;
  DYT dy;
  float s;
  bool ok;  // role a: a step of a real row inside the sequence; role b: t < L, n < N
};

// All global loads below are unconditional, from valid addresses, with the
// unwanted values replaced afterwards: the loads of the next tile then stay in
// flight across the current one instead of being waited for inside a branch.
// BUF: loads and stores go through raw buffer resources over the workgroup's
// rows (and its batch's B, C), so that a tile's address is a per-lane offset
// fixed for the whole kernel plus a scalar one (every offset below 2^31,
// checked by the host; a lane with nothing to store aims at the resource's end,
// where the store is dropped and a load returns zero); without it, 64-bit
// addresses clamped into range, and stores aimed at trash slots.  OUT: the type
// of dx, ddelta, dz (and dB, dC).
template <typename IN, typename DYT, typename OUT, bool GATED, bool BUF>
__global__ __launch_bounds__(256) void selective_bwd_rows16_kernel(const BwdArgs a, const BwWork w,
                                                                   int64_t G, int64_t ntile, int n0) {
  constexpr int OS = (int)sizeof(OUT);
  __shared__ __align__(16) B16Smem sm;
  const IN* __restrict__ X = static_cast<const IN*>(a.x);
  const IN* __restrict__ DL = static_cast<const IN*>(a.delta);
  const IN* __restrict__ BM = static_cast<const IN*>(a.Bm);
  const IN* __restrict__ CM = static_cast<const IN*>(a.Cm);
  const IN* __restrict__ Z = static_cast<const IN*>(a.z);
  const DYT* __restrict__ DY = static_cast<const DYT*>(a.dy);
  const int64_t D = a.D, L = a.L, N = a.N;

  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid / 64);  // wave-uniform
  const int lane = tid % 64;
  const int rr = 4 * wv + lane / 16;  // compute role: row within the workgroup
  const int n = lane % 16;            // ... and state
  const int64_t b = blockIdx.x / G;
  const int64_t g = blockIdx.x - b * G;
  const int64_t d0 = g * B16_ROWS;
  const int64_t d = d0 + rr;
  const bool dok = d < D;
  // this launch's states are n0 .. n0+15 (groups of 16 for N > 16); the
  // first group also adds the terms that do not depend on the state
  const int ns = n0 + n;  // the lane's state
  const bool nok = ns < N;
  const bool first = n0 == 0;
  const int64_t row = b * D + (dok ? d : D - 1);

  // staging / reduce roles (by wavefront): waves 0-1 own (row sr, step st),
  // waves 2-3 own (step bt, state bn)
  const bool role_a = wv < 2;
  const int sr = (tid % 128) / BW_T, st = tid % BW_T;
  const int bt = (tid % 128) / BW_N, bn = tid % BW_N;
  const int64_t sd = d0 + sr;
  const bool sdok = sd < D;
  const int64_t srow = b * D + (sdok ? sd : D - 1);

  const float Ar0 = a.A[(dok ? d : D - 1) * N + (nok ? ns : 0)];
  const float Ar = nok ? Ar0 : 0.0f;
  const float Al = Ar * BW_LOG2E;
  const float dbias = a.delta_bias ? a.delta_bias[sdok ? sd : D - 1] : 0.0f;
  const float Dsk = a.Dskip && first ? a.Dskip[sdok ? sd : D - 1] : 0.0f;

  // --- staging helpers -----------------------------------------------------
  const IN* __restrict__ P0 = role_a ? X : BM;
  const IN* __restrict__ P1 = role_a ? DL : CM;
  using Raw = TileRaw<IN, DYT>;
  // BUF: resources and per-lane element offsets.  Role a (and the dy, z, s
  // loads of every lane) index (row - d0) * L + t of the workgroup's rows,
  // role b (t * N + n) of the batch's B, C.
  const int64_t row0 = b * D + d0;
  const int64_t nrows = imin(B16_ROWS, D - d0);
  const int32_t ea = (int32_t)(((sdok ? sd : D - 1) - d0) * L) + st;
  const int32_t eb = bt * (int32_t)N + (n0 + bn < N ? n0 + bn : (int32_t)N - 1);
  const int32_t e01 = role_a ? ea : eb;
  const int32_t ts01 = role_a ? BW_T : BW_T * (int32_t)N;  // elements per tile
  // (built in both variants; only BUF uses them)
  const uint32_t rows_e = (uint32_t)(nrows * L);
  const uint32_t rows_b = rows_e * (uint32_t)sizeof(IN);
  const uint32_t bc_b = (uint32_t)(L * N * (int64_t)sizeof(IN));
  const __amdgpu_buffer_rsrc_t r0s =
      buffer_rsrc(role_a ? (const void*)(X + row0 * L) : (const void*)(BM + b * L * N),
                  role_a ? rows_b : bc_b);
  const __amdgpu_buffer_rsrc_t r1s =
      buffer_rsrc(role_a ? (const void*)(DL + row0 * L) : (const void*)(CM + b * L * N),
                  role_a ? rows_b : bc_b);
  const __amdgpu_buffer_rsrc_t rdy = buffer_rsrc(DY + row0 * L, rows_e * (uint32_t)sizeof(DYT));
  const __amdgpu_buffer_rsrc_t rz = buffer_rsrc(GATED ? Z + row0 * L : X, GATED ? rows_b : 0u);
  const __amdgpu_buffer_rsrc_t rs =
      buffer_rsrc(GATED ? w.s + row0 * L : w.trash, GATED ? rows_e * 4u : 0u);
  const uint32_t ck_b = (uint32_t)(nrows * ntile * BW_N * 4);
  const __amdgpu_buffer_rsrc_t rck = buffer_rsrc(w.ck + row0 * ntile * BW_N, ck_b);
  const int32_t eck = (int32_t)(((dok ? d : D - 1) - d0) * ntile * BW_N) + n;
  // BUF: the reduce's outputs through resources too, picked by the
  // wavefront's role: role a the workgroup's rows of ddelta, dx (and dz),
  // role b this workgroup's share of dB, dC
  const bool want_dz = GATED && a.dz && first;
  OUT* const ddp = static_cast<OUT*>(a.ddelta);
  OUT* const dxp = static_cast<OUT*>(a.dx);
  OUT* const dzp = static_cast<OUT*>(want_dz ? a.dz : a.dx);
  float* const dBs = w.dB_p + (b * G + g) * L * BW_N;
  float* const dCs = w.dC_p + (b * G + g) * L * BW_N;
  const uint32_t out_b = role_a ? rows_e * (uint32_t)OS : (uint32_t)(L * BW_N * 4);
  const __amdgpu_buffer_rsrc_t ro0 =
      buffer_rsrc(role_a ? (const void*)(ddp + row0 * L) : (const void*)dBs, out_b);
  const __amdgpu_buffer_rsrc_t ro1 =
      buffer_rsrc(role_a ? (const void*)(dxp + row0 * L) : (const void*)dCs, out_b);
  const __amdgpu_buffer_rsrc_t roz = buffer_rsrc(dzp + row0 * L, want_dz && role_a ? out_b : 0u);
  auto load_tile = [&](int64_t k, Raw& v) {
    if constexpr (BUF) {
      // a tile before the start reads tile 0 (unused); past the end, the
      // offsets run out of the resources or into other rows (unused)
      const int64_t kc = k < 0 ? 0 : k;
      const int64_t rem = L - k * BW_T;
      const int32_t lim = k < 0 ? 0 : (int32_t)(rem < 0 ? 0 : (rem < BW_T ? rem : BW_T));
      v.ok = role_a ? (sdok && st < lim) : (bt < lim && n0 + bn < N);
      const int32_t tk = (int32_t)kc * BW_T;  // first step of the tile
      v.r0 = buf_ld<IN>(r0s, e01 * (int32_t)sizeof(IN), tk * (ts01 / BW_T) * (int32_t)sizeof(IN));
      v.r1 = buf_ld<IN>(r1s, e01 * (int32_t)sizeof(IN), tk * (ts01 / BW_T) * (int32_t)sizeof(IN));
      v.dy = buf_ld<DYT>(rdy, ea * (int32_t)sizeof(DYT), tk * (int32_t)sizeof(DYT));
      if constexpr (GATED) {
        v.z = buf_ld<IN>(rz, ea * (int32_t)sizeof(IN), tk * (int32_t)sizeof(IN));
        v.s = buf_ld<float>(rs, ea * 4, tk * 4);
      }
      return;
    }
    // every address is clamped into range, so tiles past either end (the
    // read-ahead) load valid, unused elements
    const int64_t ta = k * BW_T + st;
    const int64_t tca = ta < 0 ? 0 : (ta < L ? ta : L - 1);
    const int64_t ia = srow * L + tca;
    const int64_t tb = k * BW_T + bt;
    const int64_t tcb = tb < 0 ? 0 : (tb < L ? tb : L - 1);
    const int64_t ib = (b * L + tcb) * N + (n0 + bn < N ? n0 + bn : N - 1);
    v.ok = role_a ? (sdok && ta >= 0 && ta < L) : (tb >= 0 && tb < L && n0 + bn < N);
    const int64_t i01 = role_a ? ia : ib;
    v.r0 = P0[i01];
    v.r1 = P1[i01];
    v.dy = DY[ia];
    if constexpr (GATED) {
      v.z = Z[ia];
      v.s = w.s[ia];
    }
  };
  auto bc_val = [&](IN r, bool ok) { return ok ? widen<IN>(r) : 0.0f; };
  // the checkpoint of tile k (clamped into range; the ones outside are unused)
  auto ck_load = [&](int64_t k) {
    const int64_t kc = k < 0 ? 0 : (k < ntile ? k : ntile - 1);
    if constexpr (BUF)
      return buf_ld<float>(rck, eck * 4, (int32_t)kc * (BW_N * 4));
    else
      return w.ck[(row * ntile + kc) * BW_N + n];
  };

  // Raw inputs of tile j live in ring[j % B16_RING]: loads run B16_RING - 1
  // tiles ahead of their use.
  Raw ring[B16_RING];

  // --- without checkpoints: a sweep forward that writes them to w.ck
  if (!a.ckpt) {
    float h = (a.h0 && dok && nok) ? a.h0[row * N + ns] : 0.0f;
#pragma unroll
    for (int u = 0; u < B16_RING - 1; ++u) load_tile(u, ring[u]);
    for (int64_t k0 = 0; k0 < ntile; k0 += B16_RING) {
#pragma unroll
      for (int u = 0; u < B16_RING; ++u) {
        const int64_t k = k0 + u;
        if (k >= ntile) break;
        const int buf = u & 1;  // B16_RING is even, so this is k & 1
        Raw& cur = ring[u];
        if (role_a) {
          float dv = widen<IN>(cur.r1) + dbias;
          if (a.softplus) dv = softplus_f32(dv);
          dv = cur.ok ? dv : 0.0f;
          sm.rv[buf][0][sr][st] = dv;
          sm.rv[buf][1][sr][st] = cur.ok ? dv * widen<IN>(cur.r0) : 0.0f;
        } else {
          sm.bc[buf][0][bn][swz(bn, bt)] = bc_val(cur.r0, cur.ok);
        }
        load_tile(k + B16_RING - 1, ring[(u + B16_RING - 1) % B16_RING]);
        bw_barrier();  // one per tile: the other buffer is the one staged next
        if constexpr (BUF)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(h), rck, dok ? eck * 4 : (int32_t)ck_b,
                                                (int32_t)k * (BW_N * 4), 0);
        else
          *(dok ? w.ck + (row * ntile + k) * BW_N + n : w.trash + tid) = h;
#pragma unroll
        for (int q = 0; q < BW_T; q += 4) {
          const float4 dl4 = *reinterpret_cast<const float4*>(&sm.rv[buf][0][rr][q]);
          const float4 dx4 = *reinterpret_cast<const float4*>(&sm.rv[buf][1][rr][q]);
          const float4 b4 = *reinterpret_cast<const float4*>(&sm.bc[buf][0][n][swz(n, q)]);
          const float dlq[4] = {dl4.x, dl4.y, dl4.z, dl4.w};
          const float dxq[4] = {dx4.x, dx4.y, dx4.z, dx4.w};
          const float bq[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
          for (int j = 0; j < 4; ++j)
            h = __builtin_fmaf(__builtin_amdgcn_exp2f(dlq[j] * Al), h, dxq[j] * bq[j]);
        }
      }
    }
    bw_barrier();  // the walk back restages the buffers of the last tiles
  }

  // --- the walk back
  float lam = (a.dh_last && dok && nok) ? a.dh_last[row * N + ns] : 0.0f;
  float dA_acc = 0.0f;
  float dD_acc = 0.0f, db_acc = 0.0f;  // role a: this thread's (row, step slot)
  float hring[B16_RING];
#pragma unroll
  for (int u = 0; u < B16_RING - 1; ++u) {
    load_tile(ntile - 1 - u, ring[u]);
    hring[u] = ck_load(ntile - 1 - u);
  }
  // Sums of tile k from partial buffer pb (role a: over the states, ddelta
  // and dx of row sr, step st; role b: over the four wavefronts' row sums,
  // this workgroup's share of dB, dC at step bt, state bn), with the
  // role-a values saved from that tile's staging.  Both roles issue the same
  // number of stores.
  float p_dlv = 0.f, p_sg = 1.f, p_ds = 0.f, p_gp = 0.f, p_xv = 0.f, p_dyv = 0.f, p_sv = 0.f;
  bool p_live = false;
  auto reduce_tile = [&](int64_t k, int pb) {
    if (role_a) {
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int m = 0; m < BW_N; ++m) {
        s1 += sm.sp[pb][0][sr * B16_RS + m * B16_TS + swz(m, st)];
        s2 += sm.sp[pb][1][sr * B16_RS + m * B16_TS + swz(m, st)];
      }
      const float ddl = p_live ? (s1 + p_xv * s2) * p_sg : 0.0f;
      float v0 = ddl;
      float v1 = __builtin_fmaf(p_dlv, s2, p_ds * Dsk);
      const float v2 = GATED ? p_dyv * p_sv * p_gp : 0.0f;
      if (first) dD_acc = __builtin_fmaf(p_ds, p_xv, dD_acc);
      db_acc += ddl;
      if constexpr (BUF) {
        const int32_t o = p_live ? (ea + (int32_t)k * BW_T) * OS : (int32_t)out_b;
        if constexpr (OS == 4) {
          if (!first) {  // later state groups add to the sums over the states
            v0 += buf_ld<float>(ro0, o, 0);
            v1 += buf_ld<float>(ro1, o, 0);
          }
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v0), ro0, o, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v1), ro1, o, 0, 0);
          if constexpr (GATED)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v2), roz, o, 0, 0);
        } else {
          __builtin_amdgcn_raw_buffer_store_b16((short)bf16_rne(v0), ro0, o, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b16((short)bf16_rne(v1), ro1, o, 0, 0);
          if constexpr (GATED) __builtin_amdgcn_raw_buffer_store_b16((short)bf16_rne(v2), roz, o, 0, 0);
        }
      } else {
        const int64_t i = srow * L + (p_live ? k * BW_T + st : 0);
        OUT* const tr = reinterpret_cast<OUT*>(w.trash + tid);
        if constexpr (OS == 4) {
          if (!first && p_live) {
            v0 += ddp[i];
            v1 += dxp[i];
          }
        }
        st1<OUT>(p_live ? ddp + i : tr, v0);
        st1<OUT>(p_live ? dxp + i : tr, v1);
        if constexpr (GATED) st1<OUT>(p_live && want_dz ? dzp + i : tr, v2);
      }
    } else {
      // lane (bt / 4) * 16 + bn of each wavefront holds the dB sums of
      // steps 4 (bt / 4) .. +3 at state bn, lane 32 more the dC sums
      const int lb = (bt >> 2) * 16 + bn, tb = bt & 3;
      float sb = 0.f, sc = 0.f;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        sb += sm.pw[pb][m][lb * 4 + tb];
        sc += sm.pw[pb][m][(32 + lb) * 4 + tb];
      }
      const int64_t t = k * BW_T + bt;
      if constexpr (BUF) {
        const int32_t o = t < L ? ((int32_t)t * BW_N + bn) * 4 : (int32_t)out_b;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sb), ro0, o, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sc), ro1, o, 0, 0);
        if constexpr (GATED) __builtin_amdgcn_raw_buffer_store_b32(0u, roz, 0, 0, 0);  // dropped
      } else {
        *(t < L ? dBs + t * BW_N + bn : w.trash + tid) = sb;
        *(t < L ? dCs + t * BW_N + bn : w.trash + tid) = sc;
      }
    }
  };

  for (int64_t k0 = ntile - 1; k0 >= 0; k0 -= B16_RING) {
#pragma unroll
    for (int u = 0; u < B16_RING; ++u) {
      const int64_t k = k0 - u;
      if (k < 0) break;
      // tile k is in ring[u] (its index counted down from the last tile)
      const int buf = (int)(k & 1);
      Raw& cur = ring[u];
      float dlv = 0.f, sg = 1.f, ds = 0.f, gp = 0.f, xv = 0.f, dyv = 0.f, sv = 0.f;
      const bool live = role_a && cur.ok;
      if (role_a) {
        float dv = widen<IN>(cur.r1) + dbias;
        if (a.softplus) softplus_sigmoid_f32(dv, dv, sg);
        dlv = live ? dv : 0.0f;
        xv = widen<IN>(cur.r0);
        dyv = widen<DYT>(cur.dy);
        float gt = 1.0f;
        if constexpr (GATED) {
          const float zv = widen<IN>(cur.z);
          const float sz = sigmoid_f32(zv);
          gt = zv * sz;
          gp = sz * (1.0f + zv * (1.0f - sz));
          sv = cur.s;
        }
        ds = live ? dyv * gt : 0.0f;
        xv = live ? xv : 0.0f;
        sm.rv[buf][0][sr][st] = dlv;
        sm.rv[buf][1][sr][st] = dlv * xv;
        sm.rv[buf][2][sr][st] = ds;
      } else {
        sm.bc[buf][0][bn][swz(bn, bt)] = bc_val(cur.r0, cur.ok);
        sm.bc[buf][1][bn][swz(bn, bt)] = bc_val(cur.r1, cur.ok);
      }
      const float hstart = dok && nok ? hring[u] : 0.0f;
      load_tile(k - (B16_RING - 1), ring[(u + B16_RING - 1) % B16_RING]);
      hring[(u + B16_RING - 1) % B16_RING] = ck_load(k - (B16_RING - 1));
      bw_barrier();  // tile k is staged, tile k+1's partials are complete

      if (k + 1 < ntile) reduce_tile(k + 1, (int)((k + 1) & 1));
      p_dlv = dlv;
      p_sg = sg;
      p_ds = ds;
      p_gp = gp;
      p_xv = xv;
      p_dyv = dyv;
      p_sv = sv;
      p_live = live;

      // recompute a_t, q_t = a_t h_{t-1} and h_t of the tile; delta, delta*x
      // and B stay in registers for the backward walk
      float av[BW_T], qv[BW_T], hv[BW_T], dlr[BW_T], dxr[BW_T], br[BW_T];
      {
        float hh = hstart;
#pragma unroll
        for (int q = 0; q < BW_T; q += 4) {
          const float4 dl4 = *reinterpret_cast<const float4*>(&sm.rv[buf][0][rr][q]);
          const float4 dx4 = *reinterpret_cast<const float4*>(&sm.rv[buf][1][rr][q]);
          const float4 b4 = *reinterpret_cast<const float4*>(&sm.bc[buf][0][n][swz(n, q)]);
          const float dlq[4] = {dl4.x, dl4.y, dl4.z, dl4.w};
          const float dxq[4] = {dx4.x, dx4.y, dx4.z, dx4.w};
          const float bq[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            dlr[q + j] = dlq[j];
            dxr[q + j] = dxq[j];
            br[q + j] = bq[j];
            av[q + j] = __builtin_amdgcn_exp2f(dlq[j] * Al);
            qv[q + j] = av[q + j] * hh;
            hh = __builtin_fmaf(dxq[j], bq[j], qv[q + j]);
            hv[q + j] = hh;
          }
        }
      }
      // walk the tile backwards
      float* const sp0 = &sm.sp[buf][0][rr * B16_RS + n * B16_TS];
      float* const sp1 = &sm.sp[buf][1][rr * B16_RS + n * B16_TS];
      float pdx[BW_T], pdh[BW_T];  // lam delta x and ds h, summed over rows below
#pragma unroll
      for (int q = BW_T - 4; q >= 0; q -= 4) {
        const float4 ds4 = *reinterpret_cast<const float4*>(&sm.rv[buf][2][rr][q]);
        const float4 c4 = *reinterpret_cast<const float4*>(&sm.bc[buf][1][n][swz(n, q)]);
        const float dsq[4] = {ds4.x, ds4.y, ds4.z, ds4.w};
        const float cq[4] = {c4.x, c4.y, c4.z, c4.w};
        float o0[4], o1[4];
#pragma unroll
        for (int j = 3; j >= 0; --j) {
          const int t = q + j;
          const float l = __builtin_fmaf(dsq[j], cq[j], lam);
          const float p = l * qv[t];
          dA_acc = __builtin_fmaf(p, dlr[t], dA_acc);
          o0[j] = p * Ar;
          o1[j] = l * br[t];
          pdx[t] = l * dxr[t];
          pdh[t] = dsq[j] * hv[t];
          lam = av[t] * l;
        }
        const int qs = swz(n, q);
        *reinterpret_cast<float4*>(sp0 + qs) = make_float4(o0[0], o0[1], o0[2], o0[3]);
        *reinterpret_cast<float4*>(sp1 + qs) = make_float4(o1[0], o1[1], o1[2], o1[3]);
      }
      {
        float o[4];
        rows4_sum(pdx, pdh, o);
        *reinterpret_cast<float4*>(&sm.pw[buf][wv][lane * 4]) =
            make_float4(o[0], o[1], o[2], o[3]);
      }
    }
  }
  bw_barrier();  // tile 0's partials are complete
  reduce_tile(0, 0);

  if (dok) {
    if (nok && a.dh0) a.dh0[row * N + ns] = lam;
    w.dA_p[row * BW_N + n] = dA_acc;
  }
  // per-row sums of the step slots (8 consecutive lanes of role a)
  if (role_a) {
#pragma unroll
    for (int off = 1; off < BW_T; off *= 2) {
      dD_acc += __shfl_xor(dD_acc, off);
      db_acc += __shfl_xor(db_acc, off);
    }
    if (st == 0 && sdok) {
      if (first) {
        w.dD_p[srow] = dD_acc;
        w.db_p[srow] = db_acc;
      } else {
        w.db_p[srow] += db_acc;
      }
    }
  }
}

// True when every byte offset of the buffer-resource path stays below 2^31:
// a workgroup's rows of x, delta, dy, z and s, a batch's B and C, and a
// workgroup's checkpoints, with the read-ahead tiles past the end.
bool rows16_buf_fits(const BwdArgs& a, int64_t ntile) {
  const int64_t lim = (int64_t)1 << 31;
  const int64_t Lp = a.L + 4 * B16_RING * BW_T;
  return B16_ROWS * Lp * 4 < lim && Lp * a.N * 4 < lim && Lp * BW_N * 4 < lim &&
         B16_ROWS * (ntile + 2 * B16_RING) * BW_N * 4 < lim;
}

template <typename IN, typename DYT, typename OUT>
void launch_rows16_t(const BwdArgs& a, const BwWork& w, int64_t G, int64_t ntile, int n0,
                     hipStream_t s) {
  const bool buf = rows16_buf_fits(a, ntile);
  auto kern = a.z ? (buf ? selective_bwd_rows16_kernel<IN, DYT, OUT, true, true>
                         : selective_bwd_rows16_kernel<IN, DYT, OUT, true, false>)
                  : (buf ? selective_bwd_rows16_kernel<IN, DYT, OUT, false, true>
                         : selective_bwd_rows16_kernel<IN, DYT, OUT, false, false>);
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.B * G)), dim3(256), 0, s, a, w, G, ntile, n0);
}

}  // namespace

void launch_bwd_rows16(const BwdArgs& a, const BwWork& w, int64_t G, int64_t ntile, int n0,
                       hipStream_t s) {
  if (!a.bf16_in) {  // fp32 gradients
    if (a.dy_bf16)
      launch_rows16_t<float, uint16_t, float>(a, w, G, ntile, n0, s);
    else
      launch_rows16_t<float, float, float>(a, w, G, ntile, n0, s);
  } else if (a.grads_bf16) {  // fp32 dy
    launch_rows16_t<uint16_t, float, uint16_t>(a, w, G, ntile, n0, s);
  } else {
    if (a.dy_bf16)
      launch_rows16_t<uint16_t, uint16_t, float>(a, w, G, ntile, n0, s);
    else
      launch_rows16_t<uint16_t, float, float>(a, w, G, ntile, n0, s);
  }
}

}  // namespace sw
