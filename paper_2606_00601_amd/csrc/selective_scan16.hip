// selective_scan16.hip -- fused selective scan, forward, N = 16, on gfx950.
//
// The same operation as selective_scan.hip (the Mamba-style instance of the
// affine recurrence, Sec. 1 and Sec. 3.1; chunk composition Eq. (7)):
//   a_{t,n} = exp(delta_t A_n),  u_{t,n} = delta_t B_{t,n} x_t,
//   h_{t,n} = a_{t,n} h_{t-1,n} + u_{t,n},
//   y_t     = sum_n C_{t,n} h_{t,n} + Dskip x_t,
// for the state size of Mamba (N = 16), laid out so that the machine is full
// at Mamba shapes.  One lane owns ONE state of one (b,d) row and walks the
// whole sequence; a row is a 16-lane DPP row, a wavefront holds 4 rows and a
// workgroup 16 rows of one batch.  At B=8, D=1536 that is 3072 wavefronts,
// three per SIMD, all doing the same work, so every SIMD has other
// wavefronts to issue from while one waits, and none is left with extra work.
//
// Per step a lane issues exactly the method's work: delta*A*log2e, exp2,
// (delta*x)*B, the state FMA and C*h -- four VALU operations and one
// transcendental.  The per-row operands cost nothing per step:
//   * delta and delta*x live in registers in a transposed layout: in a
//     super-tile of 16*V steps (V = 16/sizeof(IN)), lane m of a row holds
//     steps V*m .. V*m+V-1 (one 16-byte load per lane), and each step takes
//     its value from lane m with a row_newbcast DPP operand of the multiply,
//     i.e. for free;
//   * B_{t,n} and C_{t,n} are shared by the 16 rows of the workgroup: the
//     workgroup widens each 32-step tile once into LDS (three rotating
//     buffers, one barrier per tile), transposed to [n][t] so that a lane
//     reads its state's four steps with one 16-byte LDS read;
//   * the 16 partials C_{t,n} h_{t,n} of a row meet in a per-wavefront LDS
//     transpose and are summed one tile later: lane n adds 8 states over 4
//     steps, the two halves of the row meet through a row_ror:8 DPP add, and
//     the first 8 lanes add Dskip*x and store y (16-byte stores along t).
// All global loads go through buffer resources and run ahead of use: a
// super-tile of delta/x, two tiles of B/C; lanes past the end read zeros or
// are masked.  There is no carry between workgroups: each workgroup walks
// its rows over the whole sequence.
//
// Narrow shapes (too few rows to give every SIMD a wavefront) split each row
// into segments instead, composed with Eq. (7) in three launches that need no
// memory beyond y, in one of two forms; plan_n16 below prices these choices,
// and the quad layout of selective_scan_quad.hip, per call.
// Records form: (1) each segment but the last walks from a zero state (the
// first from h0) and records its end state U and the product P of its a_t,
// formed as exp(A * the segment's sum of delta); (2) a fold turns these into
// each segment's initial state, h_in(s+1) = P_s h_in(s) + U_s; (3) every
// segment walks from its initial state and stores y.  The records of segment
// s live in y's first 32 words of segment s+1 (P in 16, U in 16; the fold
// leaves h_in in the first 16), which launch (3) reads before it overwrites
// them with y.
// Correction form (fp32 y): (1) every segment walks from a
// zero state (the first from h0), stores y except in its first super-tile,
// and records P and U as above (the last segment its P beside the records
// of its own first words, its U in h_last); (2) the fold composes them and
// corrects h_last; (3) each later segment walks again from its initial
// state, rewriting y, until the part of every state carried in from the
// segment's start has faded against the segment's own terms.  By Eq. (5)
// the state is that carried part, P_t h_in, plus the walk from zero, so y
// beyond that point already holds the result to within 2^-26 of its
// magnitude; with the decay of Mamba-like parameters the third launch walks
// a small part of each segment, and the first runs every segment at once.
#include <stdlib.h>

#include <type_traits>

#include "selective_common.h"

namespace sw {

namespace {

constexpr int R16_N = 16;                   // states per row = lanes per DPP row
constexpr int R16_WAVES = 4;                // wavefronts per workgroup
constexpr int R16_RPW = 4;                  // rows per wavefront
constexpr int R16_ROWS = R16_WAVES * R16_RPW;
constexpr int R16_T = 32;                   // steps per tile
constexpr int R16_NB = R16_T / 4;           // 4-step blocks per tile
constexpr int R16_TS = R16_T + 4;           // LDS stride of one state's B (or C) tile row
constexpr int R16_NBUF = 3;                 // B/C tile buffers
constexpr int R16_PRS = R16_N * R16_TS + 32;  // partials: row stride (rows 32 banks apart)
constexpr int R16_LA = 2;                   // read-ahead, in 4-step blocks
constexpr int R16_NS = 4;                   // rotating operand sets
constexpr float R16_LOG2E = 1.4426950408889634f;
// A byte offset past the end of every buffer resource of the kernel (their
// sizes stay below 2^31 - 2^14): a load there returns zeros and moves no
// memory.  The super-tile of delta and x run ahead of the walk takes it for
// steps past the segment, so that no row reads the start of the next one
// (6% of those bytes at L = 2048 in bf16).  The tiles of B, C and of x for
// the D skip run ahead too, but only a tile, and mostly hit L2.
constexpr int32_t R16_OOB = 0x7FFFFF00;
static_assert(R16_NB == 8 && R16_NB % R16_NS == 0 && R16_LA < R16_NS,
              "operand sets must rotate over a tile");

struct R16Smem {
  float bc[R16_NBUF][2][R16_N * R16_TS];     // [buf][B, C][n * TS + t]
  float p[R16_WAVES][R16_RPW * R16_PRS];     // per wavefront: [row][n * TS + t]
  int vote[R16_WAVES];                       // correction walk: wavefronts not yet done
};

// Value of `v` in lane M of this lane's 16-lane row.
template <int M>
__device__ __forceinline__ float row_bcast(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + M, 0xf, 0xf,
                                         false));
}

// Value of `v` in lane n ^ 8 of this lane's 16-lane row (rotate by 8).
__device__ __forceinline__ float row_ror8(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xf, 0xf, false));
}

__device__ __forceinline__ void wg_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// B and C of one lane's state for one 4-step block.
struct R16Ops {
  float4 b, c;
};

// Raw registers for COUNT consecutive elements at any element of a row, for
// calls whose rows are not 16-byte aligned (RAG below).  fp32: the elements
// from a 4-byte aligned address.  bf16: the COUNT / 2 + 1 dwords that cover
// them.  A vector that would cross the row's end is read from COUNT elements
// before it instead, so no load leaves the tensor; get() shifts it back by
// `sh`: the elements stepped back, plus 1 (bf16) where the first element sits
// in the high half of its dword.
template <typename IN, int COUNT>
struct RagVec {
  static constexpr bool F32 = sizeof(IN) == 4;
  static constexpr int NW = F32 ? COUNT : COUNT / 2 + 1;
  uint32_t w[NW];
  // from the (4-byte aligned) byte offset `off`
  template <int POL = 0>
  __device__ __forceinline__ void load_buf(__amdgpu_buffer_rsrc_t rs, int32_t off) {
    if constexpr (COUNT == 4 && !F32) {
      const uint2 v =
          __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, POL));
      w[0] = v.x;
      w[1] = v.y;
    } else {
#pragma unroll
      for (int q = 0; q < NW / 4; ++q) {
        const uint4 v = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 * q, 0, POL));
        w[4 * q] = v.x;
        w[4 * q + 1] = v.y;
        w[4 * q + 2] = v.z;
        w[4 * q + 3] = v.w;
      }
    }
    if constexpr (!F32)
      w[NW - 1] = __builtin_bit_cast(
          uint32_t, __builtin_amdgcn_raw_buffer_load_b32(rs, off + 4 * (NW - 1), 0, POL));
  }
  // the elements as fp32; tail (wave-uniform): some lane's sh may exceed 1
  __device__ __forceinline__ void get(float (&out)[COUNT], int sh, bool tail) const {
    uint32_t v[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) v[i] = w[i];
    constexpr int UNIT = F32 ? 1 : 2;  // elements per dword
    if (tail) {
#pragma unroll
      for (int m = 4; m >= 1; m /= 2) {  // dwords
        const bool on = (sh & (m * UNIT)) != 0;
#pragma unroll
        for (int i = 0; i + m < NW; ++i) v[i] = on ? v[i + m] : v[i];
      }
    }
#pragma unroll
    for (int i = 0; i < COUNT / UNIT; ++i) {
      if constexpr (F32) {
        out[i] = __uint_as_float(v[i]);
      } else {
        const uint32_t o = __builtin_amdgcn_alignbit(v[i + 1], v[i], 16u * ((uint32_t)sh & 1u));
        out[2 * i] = bf16_lo(o);
        out[2 * i + 1] = bf16_hi(o);
      }
    }
  }
};

// The resource over `bytes` bytes from `p` for RagVec loads: it starts and
// ends on a dword (a dword that holds an element of the tensor is inside its
// allocation); *h: the element `p` is at, from the resource's start.
template <typename IN>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rag_rsrc(const IN* p, uint32_t bytes, int* h) {
  const uintptr_t at = (uintptr_t)p;
  *h = (int)((at & 3) / sizeof(IN));
  return buffer_rsrc((const void*)(at & ~(uintptr_t)3),
                     (bytes + (uint32_t)(at & 3) + 3u) & ~3u);
}

// Segment modes of the kernel (see the top of the file).
//   R16_SEG_ENDS, R16_SEG_FWD: launches (1) and (3) of the records form;
//   R16_SEG_ALL, R16_SEG_CORR: launches (1) and (3) of the correction form.
//   R16_STATES: a whole-row walk that writes only the states (the 8-step
//   checkpoints and h_last), for a backward call without them.
enum : int {
  R16_WHOLE = 0,
  R16_SEG_ENDS = 1,
  R16_SEG_FWD = 2,
  R16_SEG_ALL = 3,
  R16_SEG_CORR = 4,
  R16_STATES = 5
};
constexpr int R16_MAX_SEG = 16;  // segments per row at most
// The correction walk of a segment stops once, for every state of its
// workgroup, the part of the state carried in from the segment's start,
// P_t h_in (P_t the product of the a since the start), is at most this
// fraction of the magnitude m_t of the segment's own terms (the sum of their
// absolute values, tracked by the walk).  Both P_t |h_in| and every later
// carried part shrink or grow by the same factors |a| as m_t's terms, so
// from then on the part left out is at most R16_CORR_EPS times the
// magnitude of the state, and of y (an fp32 walk rounds at 2^-24 of it).
constexpr float R16_CORR_EPS = 1.4901161193847656e-08f;  // 2^-26

// Word i of the records of the segment starting at step t of a row, in y's
// memory (fp32 or bf16 elements; a bf16 row of odd length starts at an odd
// element, so there a word is two 2-byte accesses).
__device__ __forceinline__ float rec_load(const void* yv, bool ybf, int64_t row, int64_t L,
                                          int64_t t, int i) {
  if (!ybf) return static_cast<const float*>(yv)[row * L + t + i];
  const uint16_t* const p = static_cast<const uint16_t*>(yv) + row * L + t + 2 * i;
  return __uint_as_float((uint32_t)p[0] | ((uint32_t)p[1] << 16));
}
__device__ __forceinline__ void rec_store(void* yv, bool ybf, int64_t row, int64_t L, int64_t t,
                                          int i, float v) {
  if (!ybf) {
    static_cast<float*>(yv)[row * L + t + i] = v;
  } else {
    uint16_t* const p = static_cast<uint16_t*>(yv) + row * L + t + 2 * i;
    p[0] = (uint16_t)(__float_as_uint(v) & 0xffffu);
    p[1] = (uint16_t)(__float_as_uint(v) >> 16);
  }
}

// OPT: the optional Mamba-block inputs (flags, z, delta bias) are read;
// without it the kernel is the plain form (an initial state is always taken).
// CK: the state at every 8-step boundary goes to ck, laid out as
// (B*D, nT8, 16), for the backward pass.
// SEG: R16_WHOLE walks whole rows; R16_SEG_ENDS and R16_SEG_FWD are launches
// (1) and (3) of the segmented form, whose workgroups are (row block,
// segment) pairs, logical workgroup = row block * segments of the launch +
// segment (the logical order is spread over the XCDs in contiguous ranges);
// a row has nseg segments of Lseg steps, the last one taking the rest
// (shorter than Lseg, or up to a super-tile longer).
// RAG: rows of any length at any element alignment (L at least a lane's V
// steps): loads through RagVec, steps past the row's end made identity steps
// one by one, y stored by element in the last tile (bf16 y in every tile).
// KIND: R16_VEC whole aligned vectors, R16_RAG as above, R16_GRP as R16_RAG for
// N other than 16 (even): the states in ngrp groups of 16, a
// workgroup per (row block, group), states past N masked to identity steps.
// With several groups each writes its part of y (no skip, no gate, fp32) to
// its own plane of B*D*L elements from yv, added up by row16_groups_kernel.
enum : int { R16_VEC = 0, R16_RAG = 1, R16_GRP = 2 };
template <typename IN, bool OPT, bool CK, int SEG, int KIND>
__global__ __launch_bounds__(256) void selective_row16_kernel(
    const IN* __restrict__ x, const IN* __restrict__ delta, const float* __restrict__ A,
    const IN* __restrict__ Bm, const IN* __restrict__ Cm, const float* __restrict__ Dskip,
    const IN* __restrict__ z, const float* __restrict__ dbias, const float* __restrict__ h0,
    void* __restrict__ yv_in, float* __restrict__ h_last, int64_t D, int64_t L, int64_t ndb,
    uint32_t flags_in, float* __restrict__ ck, int64_t nT8, float* __restrict__ s_out,
    int64_t nseg, int64_t Lseg, int Nst, int ngrp, int64_t plane) {
  constexpr bool RAG = KIND != R16_VEC, GRP = KIND == R16_GRP;
  constexpr bool WHOLE = SEG == R16_WHOLE || SEG == R16_STATES;  // one walk per row
  static_assert(!CK || WHOLE || SEG == R16_SEG_FWD, "checkpoints come from walks from the true state");
  constexpr bool ENDS = SEG == R16_SEG_ENDS;  // no y: the segment's P and end state
  constexpr bool NOY = ENDS || SEG == R16_STATES;  // no C, no y
  constexpr bool ALL = SEG == R16_SEG_ALL;    // y from a zero state, and the segment's records
  constexpr bool CORR = SEG == R16_SEG_CORR;  // the walk from the composed initial state
  constexpr bool DSUM = ENDS || ALL || CORR;  // sum of delta over the segment
  constexpr int ES = (int)sizeof(IN);
  const uint32_t flags = OPT ? flags_in : 0u;
  constexpr int V = 16 / ES;              // steps a lane holds of a super-tile
  constexpr int ST = R16_N * V;           // steps per super-tile
  constexpr int TPS = ST / R16_T;         // tiles per super-tile
  static_assert(TPS * R16_T == ST, "a super-tile is a whole number of tiles");
  __shared__ __align__(16) R16Smem sm;

  const int tid = threadIdx.x;
  const int w = tid / 64, lane = tid % 64;
  const int r = lane / R16_N, n = lane % R16_N;
  // segment of this workgroup (launch (1) of the records form covers
  // segments 0 .. nseg-2, launch (3) of the correction form 1 .. nseg-1)
  const int64_t nsl = (ENDS || CORR) ? nseg - 1 : nseg;
  const int64_t bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int64_t sg = !WHOLE ? bid % nsl + (CORR ? 1 : 0) : 0;
  const int64_t rblk_g = !WHOLE ? bid / nsl : bid;
  // (R16_STATES walks one group, whose number is ngrp)
  constexpr bool ONE = SEG == R16_STATES;
  const int64_t rblk = GRP && !ONE ? rblk_g / ngrp : rblk_g;
  const int grp = GRP ? (ONE ? ngrp : (int)(rblk_g - rblk * ngrp)) : 0;
  const int N = GRP ? Nst : R16_N, n0 = R16_N * grp;
  void* const yv = GRP && !ONE ? static_cast<void*>(static_cast<float*>(yv_in) + grp * plane) : yv_in;
  const int64_t ts = !WHOLE ? sg * Lseg : 0;  // first step of the segment
  const int64_t Ls = !WHOLE ? (sg == nseg - 1 ? L - ts : Lseg) : L;  // its steps
  const int32_t Ls32 = (int32_t)Ls;  // below 2^31 / 16 (row16_fits)
  const int64_t b = rblk / ndb;
  const int64_t d0 = (rblk - b * ndb) * R16_ROWS;
  const int64_t d = d0 + R16_RPW * w + r;
  const bool dok = d < D;
  const int64_t dcl = dok ? d : D - 1;  // rows past D compute a copy of row D-1, never stored
  const int64_t rows = imin(R16_ROWS, D - d0);
  const int64_t row0 = b * D + d0;

  // resources start at the segment's first step (row strides stay L)
  const uint32_t rows_bytes = (uint32_t)((rows * L - ts) * ES);
  const uint32_t bc_bytes = (uint32_t)((L - ts) * N * ES);
  int hx = 0, hd = 0, hz = 0;  // RAG: where x, delta and z start in their resources
  const __amdgpu_buffer_rsrc_t rx = RAG ? rag_rsrc(x + row0 * L + ts, rows_bytes, &hx)
                                        : buffer_rsrc(x + row0 * L + ts, rows_bytes);
  const __amdgpu_buffer_rsrc_t rd = RAG ? rag_rsrc(delta + row0 * L + ts, rows_bytes, &hd)
                                        : buffer_rsrc(delta + row0 * L + ts, rows_bytes);
  const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(Bm + (b * L + ts) * N, bc_bytes);
  const __amdgpu_buffer_rsrc_t rc = buffer_rsrc(Cm + (b * L + ts) * N, bc_bytes);
  // the gate's input; without a gate (OPT set) the same loads read x (cached),
  // so that every path of one instantiation issues the same loads
  const IN* const zsrc = ((flags & SEL_GATED) ? z : x) + row0 * L + ts;
  const __amdgpu_buffer_rsrc_t rz =
      RAG ? rag_rsrc(zsrc, rows_bytes, &hz) : buffer_rsrc(zsrc, rows_bytes);
  const int32_t lrow = (int32_t)((dcl - d0) * L * ES);  // byte offset of this lane's row
  // RAG: the row's elements from the segment's start, and the byte offset and
  // the shift of a vector of cnt elements at step t in an array that starts
  // at element h of its resource
  const int32_t Lr32 = (int32_t)(L - ts);
  const int32_t lrow_e = (int32_t)((dcl - d0) * L);
  auto rag_at = [&](int32_t t, int cnt, int h) { return lrow_e + h + (t < Lr32 - cnt ? t : Lr32 - cnt); };
  auto rag_off = [&](int32_t t, int cnt, int h) {
    const int32_t e = rag_at(t, cnt, h);
    return ES == 4 ? e * 4 : (e & ~1) * 2;
  };
  auto rag_shift = [&](int32_t t, int cnt, int h) {
    const int32_t back = t < Lr32 - cnt ? 0 : t - (Lr32 - cnt);
    return back + (ES == 4 ? 0 : (rag_at(t, cnt, h) & 1));
  };

  const bool nok = !GRP || n0 + n < N;
  const float Al = nok ? A[dcl * N + n0 + n] * R16_LOG2E : 0.0f;
  const float dsk = Dskip ? Dskip[dcl] : 0.0f;
  const float dbv = (OPT && dbias) ? dbias[dcl] : 0.0f;
  const bool ybf = (flags & SEL_Y_BF16) != 0;
  float h = (h0 && sg == 0 && nok) ? h0[(b * D + dcl) * N + n0 + n] : 0.0f;
  if constexpr (SEG == R16_SEG_FWD || CORR) {
    // the initial state the fold left in this segment's first words of y
    if (sg > 0) h = rec_load(yv, ybf, b * D + dcl, L, ts, n);
  }
  // CORR: the initial state, and the magnitude of the segment's own terms
  const float hin = h;
  float mag = 0.0f;
  // ENDS: this lane's share of the sum of delta over the segment; the product
  // of the segment's a_t is exp2(Al * that sum over the row's 16 lanes)
  float dsum = 0.0f;

  const int64_t nsup = (Ls + ST - 1) / ST;
  const int64_t ntile = nsup * TPS;  // tiles past L are identity steps, never stored

  // ---- B/C staging: thread tid widens steps tt = tid/8 of a tile, states
  // 2*(tid%8) and 2*(tid%8)+1, from one B pair and one C pair.
  const int stt = tid / 8, sn = 2 * (tid % 8);
  RawVec<IN, 2> sbr[2], scr[2];  // raw pairs of tiles kt+1 and kt+2 (by tile parity)
  auto fetch_bc = [&](RawVec<IN, 2>& rbv, RawVec<IN, 2>& rcv, int64_t kt) {
    const int32_t off = (int32_t)(((kt * R16_T + stt) * N + n0 + sn) * ES);
    rbv.load_buf(rb, off);
    if constexpr (!NOY) rcv.load_buf(rc, off);  // NOY: C is not read
  };
  auto stage_bc = [&](const RawVec<IN, 2>& rbv, const RawVec<IN, 2>& rcv, int buf) {
    float* bb = &sm.bc[buf][0][sn * R16_TS + stt];
    float* cc = &sm.bc[buf][1][sn * R16_TS + stt];
    const bool ok = !GRP || n0 + sn < N;  // N is even: both states or neither
    bb[0] = ok ? rbv.get(0) : 0.0f;
    bb[R16_TS] = ok ? rbv.get(1) : 0.0f;
    if constexpr (!NOY) {
      cc[0] = ok ? rcv.get(0) : 0.0f;
      cc[R16_TS] = ok ? rcv.get(1) : 0.0f;
    }
  };

  // ---- delta / x of a super-tile: this lane's V steps starting at V*n
  // raw bits of the next super-tile
  typename std::conditional<RAG, RagVec<IN, V>, RawVec<IN, V>>::type dlr, xr;
  float dl[V], dx[V];     // delta and delta*x of the current one
  auto fetch_dx = [&](int64_t sup) {
    // Ls is a multiple of V: a lane's V steps are all in or all out
    const int32_t t = (int32_t)(sup * ST) + V * n;
    // delta is read once (non-temporal); x is read again for the y of its
    // tiles (fetch_yx), so this read keeps the default policy
    if constexpr (RAG) {
      dlr.template load_buf<SW_NT>(rd, t < Ls32 ? rag_off(t, V, hd) : R16_OOB);
      xr.load_buf(rx, t < Ls32 ? rag_off(t, V, hx) : R16_OOB);
    } else {
      const int32_t off = t < Ls32 ? lrow + t * ES : R16_OOB;
      dlr.template load_buf<SW_NT>(rd, off);
      xr.load_buf(rx, off);
    }
  };
  auto widen_dx = [&](int64_t sup) {
    // steps past the segment are identity steps (a = 1, u = 0): the loads
    // there returned zeros (fetch_dx), which is that already, unless the
    // options turn delta = 0 into something else; Ls is a multiple of V, so
    // a lane's V steps are all inside or all past
    const bool past = OPT && (int32_t)(sup * ST) + V * n >= Ls32;
    float draw[V], xraw[V];
    if constexpr (RAG) {
      const int32_t t = (int32_t)(sup * ST) + V * n;
      const bool tail = (int32_t)(sup * ST) + ST > Lr32;
      dlr.get(draw, rag_shift(t, V, hd), tail);
      xr.get(xraw, rag_shift(t, V, hx), tail);
    } else {
#pragma unroll
      for (int k = 0; k < V; ++k) {
        draw[k] = dlr.get(k);
        xraw[k] = xr.get(k);
      }
    }
#pragma unroll
    for (int k = 0; k < V; ++k) {
      float dv = draw[k], xv = xraw[k];
      if constexpr (OPT) {
        dv += dbv;
        if (flags & SEL_SOFTPLUS) dv = softplus_f32(dv);
        if (past) dv = xv = 0.0f;
      }
      // a lane's steps may straddle the row's end here
      if (RAG && (int32_t)(sup * ST) + V * n + k >= Ls32) dv = xv = 0.0f;
      dl[k] = dv;
      dx[k] = dv * xv;
      if constexpr (DSUM) dsum += dv;
    }
  };

  // ---- y: the 16 lanes of a row split the reduce of a tile: lane n sums
  // states 8*(n/8) .. +7 over steps 4*(n%8) .. +3 with 16-byte LDS reads,
  // the two halves meet through a row_ror:8 DPP add, and lanes n < 8 store.
  const int rq = n % 8, rh = n / 8;
  // raw x and z of those four steps, for the tile awaiting its reduce
  typename std::conditional<RAG, RagVec<IN, 4>, RawVec<IN, 4>>::type yxr, yzr;
  auto fetch_yx = [&](int64_t kt) {
    if constexpr (NOY) return;
    const int32_t t = (int32_t)(kt * R16_T) + 4 * rq;
    if constexpr (RAG) {
      yxr.template load_buf<SW_NT>(rx, rag_off(t, 4, hx));
      if constexpr (OPT) yzr.template load_buf<SW_NT>(rz, rag_off(t, 4, hz));
    } else {
      const int32_t off = lrow + t * ES;
      yxr.template load_buf<SW_NT>(rx, off);  // the last read of x
      if constexpr (OPT) yzr.template load_buf<SW_NT>(rz, off);
    }
  };
  float* const p_w = &sm.p[w][r * R16_PRS + n * R16_TS];
  const float* const p_r = &sm.p[w][r * R16_PRS + 8 * rh * R16_TS + 4 * rq];
  // y (and, OPT, y before the output gate, for the backward of a gated call)
  // leave through buffer resources over the workgroup's rows from the
  // segment's start: a 32-bit offset per lane, and lanes with nothing to
  // store aim at the resource's end, where the hardware drops the store.
  // Sizes fit 32 bits: 16 rows of L < 2^26 steps of at most 4 bytes.  Both
  // are written once, with the non-temporal policy.
  const uint32_t ys = ybf ? 2u : 4u;
  const uint32_t y_bytes = (uint32_t)((rows * L - ts) * ys);
  const __amdgpu_buffer_rsrc_t ry =
      ybf ? buffer_rsrc(static_cast<uint16_t*>(yv) + row0 * L + ts, y_bytes)
          : buffer_rsrc(static_cast<float*>(yv) + row0 * L + ts, y_bytes);
  const uint32_t y_lrow = (uint32_t)((dcl - d0) * L) * ys;
  const uint32_t s_bytes = (uint32_t)((rows * L - ts) * 4);
  const __amdgpu_buffer_rsrc_t rs =
      buffer_rsrc((OPT && s_out) ? s_out + row0 * L + ts : static_cast<float*>(yv), s_bytes);
  const uint32_t s_lrow = (uint32_t)((dcl - d0) * L) * 4u;

  auto read_partials = [&](float4 (&pr)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) pr[i] = *reinterpret_cast<const float4*>(p_r + i * R16_TS);
  };
  auto finish_reduce = [&](int64_t kt, const float4 (&pr)[8], const float (&yx)[4],
                           const float (&gt)[4]) {
    float s4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      s4[0] += pr[i].x;
      s4[1] += pr[i].y;
      s4[2] += pr[i].z;
      s4[3] += pr[i].w;
    }
    // add the other half of the row (lane n ^ 8), then Dskip*x, then the gate
#pragma unroll
    for (int q = 0; q < 4; ++q) s4[q] = __builtin_fmaf(dsk, yx[q], s4[q] + row_ror8(s4[q]));
    const int32_t t = (int32_t)(kt * R16_T) + 4 * rq;
    const bool mine = dok && rh == 0 && t < Ls32;
    // ALL: the first super-tile of every segment but the first holds the
    // records until the correction walk writes its y
    const bool skip = ALL && sg > 0 && t < ST;
    // RAG: the tile that holds the row's end stores by element, and so does
    // bf16 y, whose rows may start at an odd element
    const bool by_elem = RAG && (int32_t)(kt * R16_T) + R16_T > Ls32;
    if constexpr (OPT) {
      if (s_out && by_elem) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          __builtin_amdgcn_raw_buffer_store_b32(
              __float_as_uint(s4[q]), rs,
              (int)(mine && t + q < Ls32 ? s_lrow + 4u * (uint32_t)(t + q) : s_bytes), 0, 0);
      } else if (s_out) {
        const uint32_t so = mine ? s_lrow + 4u * (uint32_t)t : s_bytes;
        __builtin_amdgcn_raw_buffer_store_b128(
            __builtin_bit_cast(sw_u32x4, make_float4(s4[0], s4[1], s4[2], s4[3])), rs, (int)so,
            0, SW_NT);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) s4[q] *= gt[q];
    const uint32_t yo = (mine && !skip) ? y_lrow + ys * (uint32_t)t : y_bytes;
    if (RAG && ybf) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        __builtin_amdgcn_raw_buffer_store_b16(
            (short)bf16_rne(s4[q]), ry,
            (int)(mine && t + q < Ls32 ? yo + 2u * (uint32_t)q : y_bytes), 0, 0);
    } else if (by_elem) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        __builtin_amdgcn_raw_buffer_store_b32(
            __float_as_uint(s4[q]), ry,
            (int)(mine && !skip && t + q < Ls32 ? yo + 4u * (uint32_t)q : y_bytes), 0, 0);
    } else if (ybf)
      __builtin_amdgcn_raw_buffer_store_b64(
          __builtin_bit_cast(sw_u32x2, make_uint2(bf16x2_rne(s4[0], s4[1]), bf16x2_rne(s4[2], s4[3]))),
          ry, (int)yo, 0, SW_NT);
    else
      __builtin_amdgcn_raw_buffer_store_b128(
          __builtin_bit_cast(sw_u32x4, make_float4(s4[0], s4[1], s4[2], s4[3])), ry, (int)yo, 0,
          SW_NT);
  };

  auto read_ops = [&](R16Ops& o, int buf, int bi) {
    o.b = *reinterpret_cast<const float4*>(&sm.bc[buf][0][n * R16_TS + 4 * bi]);
    if constexpr (!NOY) o.c = *reinterpret_cast<const float4*>(&sm.bc[buf][1][n * R16_TS + 4 * bi]);
  };

  // ---- prologue: delta/x of super-tile 0, B/C of tiles 0..2, y-x of tile 0
  fetch_dx(0);
  fetch_bc(sbr[0], scr[0], 0);
  fetch_bc(sbr[1], scr[1], 1);
  stage_bc(sbr[0], scr[0], 0);
  fetch_bc(sbr[0], scr[0], 2);
  fetch_yx(0);
  wg_barrier();
  R16Ops ops[R16_NS];
#pragma unroll
  for (int i = 0; i < R16_LA; ++i) read_ops(ops[i], 0, i);

  float yx_prev[4] = {0.f, 0.f, 0.f, 0.f};  // x of the tile awaiting its reduce
  float gt_prev[4] = {1.f, 1.f, 1.f, 1.f};  // ... and its output gate
  int buf = 0;                             // B/C buffer of the tile being computed

  // One tile: stage B/C of tile kt+1, issue the reads of tile kt-1's
  // partials, wait for the workgroup, then compute the 8 blocks with the
  // operands of block i+LA read ahead (into tile kt+1's buffer at the end).
  auto tile = [&](int64_t kt, auto ttc) {
    constexpr int TT = decltype(ttc)::value;  // tile within the super-tile
    const int nbuf = buf == R16_NBUF - 1 ? 0 : buf + 1;
    const bool has_next = kt + 1 < ntile;
    stage_bc(sbr[(TT + 1) & 1], scr[(TT + 1) & 1], nbuf);
    fetch_bc(sbr[(TT + 1) & 1], scr[(TT + 1) & 1], kt + 3);
    float yx[4], yz[4], gt[4];
    if constexpr (RAG && !NOY) {
      const int32_t t = (int32_t)(kt * R16_T) + 4 * rq;
      const bool tail = (int32_t)(kt * R16_T) + R16_T > Lr32;
      yxr.get(yx, rag_shift(t, 4, hx), tail);
      if constexpr (OPT) yzr.get(yz, rag_shift(t, 4, hz), tail);
    } else if constexpr (!RAG) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        yx[q] = yxr.get(q);
        if constexpr (OPT) yz[q] = yzr.get(q);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (RAG && NOY) yx[q] = 0.0f;
      gt[q] = (OPT && !NOY && (flags & SEL_GATED)) ? silu_f32(yz[q]) : 1.0f;
    }
    fetch_yx(kt + 1);
    wg_barrier();
    // this wavefront's own partials: after the barrier, so that the barrier
    // only drains the staging writes
    float4 pr[8];
    if (!NOY && kt > 0) read_partials(pr);
#pragma unroll
    for (int bi = 0; bi < R16_NB; ++bi) {
      const int nb = bi + R16_LA;
      if (nb < R16_NB)
        read_ops(ops[nb % R16_NS], buf, nb);
      else if (has_next)
        read_ops(ops[nb % R16_NS], nbuf, nb - R16_NB);
      if constexpr (CK) {
        // the state before step kt*T + 4*bi; rows past D write the same
        // values as row D-1 to row D-1's slots
        const int64_t t8 = (ts + kt * R16_T + 4 * bi) / 8;
        if ((bi & 1) == 0 && t8 < nT8) ck[((b * D + dcl) * nT8 + t8) * R16_N + n] = h;
      }
      const R16Ops& o = ops[bi % R16_NS];
      const float bq[4] = {o.b.x, o.b.y, o.b.z, o.b.w};
      const float cq[4] = {o.c.x, o.c.y, o.c.z, o.c.w};
      float p4[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        constexpr int S0 = TT * R16_T;  // step of the super-tile at block 0
        const int s = S0 + 4 * bi + q;
        float dlv, dxv;
        // the source lane and register are compile-time constants
        switch (s / V) {
#define SW_R16_CASE(M)             \
  case M:                          \
    dlv = row_bcast<M>(dl[s % V]); \
    dxv = row_bcast<M>(dx[s % V]); \
    break;
          SW_R16_CASE(0) SW_R16_CASE(1) SW_R16_CASE(2) SW_R16_CASE(3)
          SW_R16_CASE(4) SW_R16_CASE(5) SW_R16_CASE(6) SW_R16_CASE(7)
          SW_R16_CASE(8) SW_R16_CASE(9) SW_R16_CASE(10) SW_R16_CASE(11)
          SW_R16_CASE(12) SW_R16_CASE(13) SW_R16_CASE(14) SW_R16_CASE(15)
#undef SW_R16_CASE
          default:
            dlv = dxv = 0.0f;
        }
        const float a = __builtin_amdgcn_exp2f(dlv * Al);
        const float u = dxv * bq[q];
        h = __builtin_fmaf(a, h, u);
        if constexpr (CORR) mag = __builtin_fmaf(a, mag, __builtin_fabsf(u));
        if constexpr (NOY) {
          p4[q] = 0.0f;
        } else {
          p4[q] = cq[q] * h;
        }
      }
      if constexpr (!NOY) {
        *reinterpret_cast<float4*>(p_w + 4 * bi) = make_float4(p4[0], p4[1], p4[2], p4[3]);
        if (bi == 0 && kt > 0) finish_reduce(kt - 1, pr, yx_prev, gt_prev);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      yx_prev[q] = yx[q];
      gt_prev[q] = gt[q];
    }
    buf = nbuf;
    wave_order();  // this wavefront's partials are written before its next reads
  };

  int64_t kt_end = ntile;  // tiles walked
  for (int64_t sup = 0; sup < nsup; ++sup) {
#pragma unroll
    for (int tt = 0; tt < TPS; ++tt) {
      // the delta/x registers switch to this super-tile at its first tile,
      // and the next super-tile is loaded (every super-tile, so that each
      // path has the same loads in flight)
      if (tt == 0) {
        widen_dx(sup);
        fetch_dx(sup + 1);
      }
      switch (tt) {
        case 0: tile(sup * TPS + 0, std::integral_constant<int, 0>()); break;
        case 1: tile(sup * TPS + 1, std::integral_constant<int, 1>()); break;
        case 2: if constexpr (TPS > 2) tile(sup * TPS + 2, std::integral_constant<int, 2>()); break;
        case 3: if constexpr (TPS > 3) tile(sup * TPS + 3, std::integral_constant<int, 3>()); break;
        default: break;
      }
    }
    if constexpr (CORR) {
      // the carried part of each state, P h_in with P = exp2(A log2e * the
      // row's sum of delta so far), against the walk's own magnitude; the
      // workgroup stops together (its wavefronts share the B/C staging)
      float srow = dsum;
#pragma unroll
      for (int mm = 8; mm >= 1; mm /= 2) srow += __shfl_xor(srow, mm, R16_N);
      const float carried = __builtin_amdgcn_exp2f(Al * srow) * hin;
      const bool done = !dok || __builtin_fabsf(carried) <= R16_CORR_EPS * mag;
      const uint64_t open = __builtin_amdgcn_ballot_w64(!done);
      if (lane == 0) sm.vote[w] = open != 0;
      wg_barrier();
      const bool stop = (sm.vote[0] | sm.vote[1] | sm.vote[2] | sm.vote[3]) == 0;
      if (stop) {
        kt_end = (sup + 1) * TPS;
        break;
      }
    }
  }
  if constexpr (ENDS) {
    // the records of this segment, in the first words of the next one
#pragma unroll
    for (int m = 8; m >= 1; m /= 2) dsum += __shfl_xor(dsum, m, R16_N);
    if (dok) {
      rec_store(yv, ybf, b * D + d, L, ts + Ls, n, __builtin_amdgcn_exp2f(Al * dsum));
      rec_store(yv, ybf, b * D + d, L, ts + Ls, R16_N + n, h);
    }
  } else if constexpr (SEG == R16_STATES) {
    if (h_last && dok && nok) h_last[(b * D + d) * N + n0 + n] = h;
  } else {
    float4 pr[8];
    read_partials(pr);
    finish_reduce(kt_end - 1, pr, yx_prev, gt_prev);
    if constexpr (ALL) {
      // the records of this segment: its P and end state in the first words
      // of the next segment; the last segment's P beside the records there,
      // its end state in h_last (the fold composes both)
#pragma unroll
      for (int mm = 8; mm >= 1; mm /= 2) dsum += __shfl_xor(dsum, mm, R16_N);
      if (dok) {
        const float P = __builtin_amdgcn_exp2f(Al * dsum);
        if (sg < nseg - 1) {
          rec_store(yv, false, b * D + d, L, ts + Ls, n, P);
          rec_store(yv, false, b * D + d, L, ts + Ls, R16_N + n, h);
        } else {
          rec_store(yv, false, b * D + d, L, ts, 2 * R16_N + n, P);
        }
      }
    }
    if constexpr (!CORR) {
      if (h_last && dok && nok && (WHOLE || sg == nseg - 1))
        h_last[(b * D + d) * N + n0 + n] = h;
    }
  }
}

// Launch (2) of the segmented form: one lane per (row, state) walks the
// segments' records in order and leaves each segment's initial state in its
// first words: h_in(1) = U_0 (segment 0 started from h0), then
// h_in(s+1) = P_s h_in(s) + U_s.
__global__ __launch_bounds__(256) void row16_fold_kernel(void* __restrict__ yv, bool ybf,
                                                         int64_t R, int64_t L, int64_t nseg,
                                                         int64_t Lseg) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= R * R16_N) return;
  const int64_t row = i / R16_N;
  const int n = (int)(i % R16_N);
  // all records first (independent loads in flight together), then the fold
  float P[R16_MAX_SEG], U[R16_MAX_SEG];
#pragma unroll
  for (int sgi = 1; sgi < R16_MAX_SEG; ++sgi) {
    if (sgi < nseg) {
      P[sgi] = rec_load(yv, ybf, row, L, sgi * Lseg, n);
      U[sgi] = rec_load(yv, ybf, row, L, sgi * Lseg, R16_N + n);
    }
  }
  float h = 0.0f;
#pragma unroll
  for (int sgi = 1; sgi < R16_MAX_SEG; ++sgi) {
    if (sgi < nseg) {
      h = sgi == 1 ? U[sgi] : __builtin_fmaf(P[sgi], h, U[sgi]);
      rec_store(yv, ybf, row, L, sgi * Lseg, n, h);
    }
  }
}

// Launch (2) of the correction form: one lane per (row, state) composes the
// segments' records in order, h_in(1) = U_0 (segment 0 started from h0),
// h_in(s+1) = P_s h_in(s) + U_s, leaves h_in(s) in the first words of segment
// s, and corrects the final state: h_last = P_last h_in(last) + U_last.
__global__ __launch_bounds__(256) void row16_fold_corr_kernel(float* __restrict__ y,
                                                              float* __restrict__ h_last,
                                                              int64_t R, int64_t L, int64_t nseg,
                                                              int64_t Lseg, int N, int64_t Rg) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= R * R16_N) return;
  const int64_t row = i / R16_N;
  const int n = (int)(i % R16_N);
  float P[R16_MAX_SEG], U[R16_MAX_SEG];
#pragma unroll
  for (int sgi = 1; sgi < R16_MAX_SEG; ++sgi) {
    if (sgi < nseg) {
      P[sgi] = rec_load(y, false, row, L, sgi * Lseg, n);  // of segment sgi - 1
      U[sgi] = rec_load(y, false, row, L, sgi * Lseg, R16_N + n);
    }
  }
  float h = 0.0f;
#pragma unroll
  for (int sgi = 1; sgi < R16_MAX_SEG; ++sgi) {
    if (sgi < nseg) {
      h = sgi == 1 ? U[sgi] : __builtin_fmaf(P[sgi], h, U[sgi]);
      rec_store(y, false, row, L, sgi * Lseg, n, h);
    }
  }
  // row r of plane g (Rg rows a plane) holds states 16g .. of the call's row r
  const int64_t g = row / Rg, ns = R16_N * g + n, at = (row - g * Rg) * N + ns;
  if (h_last && ns < N) {
    const float Pl = rec_load(y, false, row, L, (nseg - 1) * Lseg, 2 * R16_N + n);
    h_last[at] = __builtin_fmaf(Pl, h, h_last[at]);
  }
}

// y of a call whose states were walked in groups: the groups' planes added in
// order, Dskip x, the pre-gate output, the gate, and y in its type.  One
// workgroup per row and 1024 steps; bound by HBM (the planes, x, z and y).
template <typename IN>
__global__ __launch_bounds__(256) void row16_groups_kernel(
    const float* __restrict__ planes, int ngrp, const IN* __restrict__ x,
    const IN* __restrict__ z, const float* __restrict__ Dskip, void* __restrict__ y,
    float* __restrict__ s_out, int64_t R, int64_t D, int64_t L, int64_t nch, bool ybf) {
  const int64_t row = blockIdx.x / nch;
  const int64_t t0 = (blockIdx.x - row * nch) * 1024 + threadIdx.x;
  const float dsk = Dskip ? Dskip[row % D] : 0.0f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t t = t0 + 256 * q;
    if (t >= L) break;
    const int64_t i = row * L + t;
    float s = planes[i];
    for (int g = 1; g < ngrp; ++g) s += planes[g * R * L + i];
    if (Dskip) s = __builtin_fmaf(dsk, __uint_as_float(Elt<IN>::raw(x, i) << (sizeof(IN) == 2 ? 16 : 0)), s);
    if (s_out) s_out[i] = s;
    if (z) s *= silu_f32(__uint_as_float(Elt<IN>::raw(z, i) << (sizeof(IN) == 2 ? 16 : 0)));
    if (ybf)
      static_cast<uint16_t*>(y)[i] = (uint16_t)bf16_rne(s);
    else
      static_cast<float*>(y)[i] = s;
  }
}

}  // namespace

// The fold of the correction form over ngrp planes of R rows, shared with the
// quad layout (selective_scan_quad.hip), which keeps its records in the same places.
void launch_fold_corr(float* y, float* h_last, int64_t R, int64_t L, int64_t nseg, int64_t Lseg,
                      int N, int ngrp, hipStream_t s) {
  const int64_t lanes = R * ngrp * R16_N;
  hipLaunchKernelGGL(row16_fold_corr_kernel, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0,
                     s, y, h_last, R * ngrp, L, nseg, Lseg, N, R);
}

template <typename IN>
bool quad_fits(const SelArgs& a);
template <typename IN>
int launch_quad(const SelArgs& a, int64_t nseg, int64_t Lseg, hipStream_t s);

// True when the N = 16 layout can take the call: rows of at least a lane's
// vector of steps, and every byte offset of a workgroup (including loads run
// ahead past the end) below 2^31.
// (N other than 16: the state groups of R16_GRP, which read B and C in pairs.)
bool row16_fits(int64_t D, int64_t N, int64_t L, size_t es) {
  if (N % 2 != 0) return false;
  const int64_t vstep = 16 / (int64_t)es;
  if (L < vstep) return false;
  const int64_t pad = 4 * R16_N * vstep;
  return R16_ROWS * (L + pad) * (int64_t)es < ((int64_t)1 << 31) &&
         (L + pad) * (N > R16_N ? N : R16_N) * (int64_t)es < ((int64_t)1 << 31) && D > 0;
}

// ---- which layout, how many segments and which form an N = 16 call takes
//
// The candidates: the 16-lane layout walking whole rows; the 16-lane layout
// with 2..16 segments per row, in the records or the correction form; the
// quad layout (four lanes per row, selective_scan_quad.hip) on whole rows or
// with 2..16 segments, correction form.  (Whole rows of the quad layout win
// from about 32768 rows on: B=16, D=5120, L=256 110 / 81 us, 16-lane / quad,
// B=32, D=1024, L=512 76 / 65, but B=4, D=5120, L=1024 95 / 117.)  Each is priced with a model of its launches
// and the cheapest is taken.  A launch of G workgroups on `cus` CUs runs in
// rounds: its busiest CU holds ceil(G / cus) workgroups, at most `cap` at a
// time (three of the 16-lane layout, four of the quad layout, by LDS), and a
// round with o workgroups resident per CU takes `ns[o]` per step of its walk
// -- the per-step times of each layout measured on MI355X with one to four
// workgroups per CU, fp32 inputs (the quad layout is 8% faster with bf16
// inputs; its four-per-CU time, 226 ns with every CU at four, is set at 220
// ns, what B=1, D=5120, L=65536 measures with three quarters of the CUs at
// four).  Every segment of a launch walks at once, so a launch is priced at
// its longest segment.  A correction walk is priced at the fading length of Mamba-like
// decay, 1024 steps plus one check (slower decay walks further, up to the
// whole segment: slower, never wrong); a segmented call adds 8 us for its
// fold and two more launches; the first walk of the records form (no C, no
// y) is priced at 0.85 of a walk.  Over 42 shapes (B = 1..4, D = 1280..8192,
// L = 4096..65536, fp32 and bf16 inputs) the model's choice came within 1.2%
// of the fastest measured candidate on average and 10% at worst, where
// fixed occupancy bands had been 29% and 150% off.
// SW_SS_QUAD=0 leaves the quad layout out, =1 takes it whenever the call
// allows; SW_SS_SEGMENTS=k keeps only the candidates with k segments (1:
// whole rows; the 16-lane layout unless SW_SS_QUAD=1); SW_SS_SEGFORM=1 or 2
// keeps only the records or the correction form of the 16-lane layout.
struct StepCost {
  int cap;
  float ns[5];
};
constexpr StepCost R16_COST = {3, {0.0f, 28.8f, 42.3f, 57.1f, 0.0f}};
constexpr StepCost QUAD_COST = {4, {0.0f, 98.6f, 135.8f, 171.6f, 220.0f}};
constexpr int64_t PLAN_CORR_STEPS = 1024;
constexpr double PLAN_SEG_US = 8.0;
constexpr double PLAN_ENDS_SHARE = 0.85;
constexpr int64_t QUAD_SKIP = 64;  // the quad layout's segment granularity and check interval

double launch_us(int64_t G, int64_t steps, int cus, const StepCost& c, double scale) {
  const int64_t per = (G + cus - 1) / cus;  // workgroups on the busiest CU
  const int64_t full = per / c.cap, rest = per % c.cap;
  const double ns = (double)full * c.ns[c.cap] + (rest > 0 ? c.ns[rest] : 0.0);
  return (double)steps * ns * scale * 1e-3;
}

int64_t env_i64(const char* name) {
  const char* v = getenv(name);
  return (v && *v) ? atoll(v) : -1;
}

struct N16Plan {
  bool quad = false;
  int64_t nseg = 1;  // 1: whole rows
  int64_t Lseg = 0;
  bool corr = false;
  double us = 0.0;  // its price
};

// Segments of the 16-lane layout for a count k: L / k rounded up to whole
// super-tiles of st steps, as many segments as that takes, the last one the
// rest; a rest shorter than a super-tile (too short for the records the
// segment before leaves in its first words) joins the segment before.  n = 0
// when k gives fewer than two.
void r16_geometry(int64_t L, int64_t st, int64_t k, int64_t* n, int64_t* Lseg) {
  *n = 0;
  if (k < 2 || k > R16_MAX_SEG || L / st < 2) return;
  const int64_t per = (L + k - 1) / k;
  *Lseg = (per + st - 1) / st * st;
  int64_t m = (L + *Lseg - 1) / *Lseg;
  if (L - (m - 1) * *Lseg < st) --m;
  if (m >= 2 && m <= R16_MAX_SEG) *n = m;
}

// Segments of the quad layout for a count k: k - 1 segments of Lseg steps (a
// multiple of QUAD_SKIP) and the last taking the rest.  Lseg is L / k rounded
// up, which leaves the last segment the shortest, unless that leaves it fewer
// than QUAD_SKIP steps (its first words hold 48 words of records); then
// rounded down (the last the longest).  Lseg < QUAD_SKIP: no such geometry.
void quad_geometry(int64_t L, int64_t k, int64_t* Lseg, int64_t* last) {
  const int64_t per = (L + k - 1) / k;
  *Lseg = (per + QUAD_SKIP - 1) / QUAD_SKIP * QUAD_SKIP;
  if (L - (k - 1) * *Lseg < QUAD_SKIP) *Lseg = (L / k) / QUAD_SKIP * QUAD_SKIP;
  *last = L - (k - 1) * *Lseg;
}

// `cus`: the compute units the launches are priced for.
template <typename IN>
N16Plan plan_n16(const SelArgs& a, int64_t ndb, int cus) {
  N16Plan best;
  // checkpoints come from whole-row walks, or where the caller allows
  // segments, from the records form (whose last launch walks every segment
  // from its composed state)
  const int64_t G16 = a.B * ndb;
  best.us = launch_us(G16, a.L, cus, R16_COST, 1.0);
  if (a.ckpt && !a.ckpt_seg) return best;
  const int64_t L = a.L, st = R16_N * (16 / (int64_t)sizeof(IN));
  const int64_t quad_env = env_i64("SW_SS_QUAD"), seg_env = env_i64("SW_SS_SEGMENTS");
  const int64_t form_env = env_i64("SW_SS_SEGFORM");
  const bool qfits = a.vec && quad_fits<IN>(a);
  const bool quad_only = quad_env == 1 && qfits;
  const bool with_quad = qfits && quad_env != 0 && (seg_env < 0 || quad_only);
  const bool corr_ok = !a.y_bf16 && !a.ckpt;
  const double qscale = sizeof(IN) == 2 ? 0.92 : 1.0;
  const int64_t Gq = a.B * ((a.D + 63) / 64);
  double best_us = 1e300;
  auto consider = [&](double us, bool quad, int64_t nseg, int64_t Lseg, bool corr) {
    if (us < best_us) {
      best_us = us;
      best.quad = quad;
      best.nseg = nseg;
      best.Lseg = Lseg;
      best.corr = corr;
      best.us = us;
    }
  };
  const int64_t kmin = seg_env > 0 ? (seg_env < 16 ? seg_env : 16) : 1;
  const int64_t kmax = seg_env > 0 ? kmin : 16;
  if (!quad_only) {
    if (kmin == 1) consider(launch_us(G16, L, cus, R16_COST, 1.0), false, 1, L, false);
    for (int64_t k = (kmin > 2 ? kmin : 2); k <= kmax; ++k) {
      int64_t n, Lseg;
      r16_geometry(L, st, k, &n, &Lseg);
      if (n < 2 || G16 * n > SW_MAX_WGS) continue;
      // every segment walks at once: the longest sets the launch's time
      const int64_t last = L - (n - 1) * Lseg;
      const int64_t longest = last > Lseg ? last : Lseg;
      const double first = launch_us(G16 * n, longest, cus, R16_COST, 1.0);
      if (corr_ok && form_env != 1) {
        const int64_t walk = longest < PLAN_CORR_STEPS + st ? longest : PLAN_CORR_STEPS + st;
        consider(first + launch_us(G16 * (n - 1), walk, cus, R16_COST, 1.0) + PLAN_SEG_US, false,
                 n, Lseg, true);
      }
      if (form_env != 2)
        consider(PLAN_ENDS_SHARE * launch_us(G16 * (n - 1), Lseg, cus, R16_COST, 1.0) + first +
                     PLAN_SEG_US,
                 false, n, Lseg, false);
    }
    // a forced count that gives fewer than two segments walks whole rows
    if (best_us == 1e300) consider(0.0, false, 1, L, false);
  }
  if (with_quad) {
    // a forced count is capped at one segment per QUAD_SKIP steps
    const int64_t kcap = L / QUAD_SKIP;
    if (kmin == 1 || (quad_only && seg_env > 0 && kcap < 2))
      consider(launch_us(Gq, L, cus, QUAD_COST, qscale), true, 1, L, false);
    const int64_t qmin = seg_env > 0 && kmin > kcap ? kcap : kmin;
    // bf16 y has no room for the segments' records of the correction form
    const int64_t qmax = a.y_bf16 ? 1 : seg_env > 0 && kmax > kcap ? kcap : kmax;
    for (int64_t k = (qmin > 2 ? qmin : 2); k <= qmax; ++k) {
      int64_t Lseg, last;
      quad_geometry(L, k, &Lseg, &last);
      if (Lseg < QUAD_SKIP || Gq * k > SW_MAX_WGS) continue;
      // every segment walks at once: the longest sets the launch's time
      const int64_t longest = last > Lseg ? last : Lseg;
      const int64_t walk =
          longest < PLAN_CORR_STEPS + QUAD_SKIP ? longest : PLAN_CORR_STEPS + QUAD_SKIP;
      consider(launch_us(Gq * k, longest, cus, QUAD_COST, qscale) +
                   launch_us(Gq * (k - 1), walk, cus, QUAD_COST, qscale) + PLAN_SEG_US,
               true, k, Lseg, true);
    }
    if (quad_only && best_us == 1e300) consider(0.0, true, 1, L, false);
  }
  return best;
}

// Groups of 16 states of a call of that kind.
template <int KIND>
int r16_groups(int64_t N) {
  return KIND == R16_GRP ? (int)((N + R16_N - 1) / R16_N) : 1;
}

template <typename IN, bool OPT, int KIND>
void launch_row16_segments(const SelArgs& a, int64_t ndb, uint32_t flags, int64_t nseg,
                           int64_t Lseg, hipStream_t s) {
  const int64_t R = a.B * a.D;
  const int ngrp = r16_groups<KIND>(a.N);
  const int64_t rblocks = a.B * ndb * ngrp;
  hipLaunchKernelGGL((selective_row16_kernel<IN, OPT, false, R16_SEG_ENDS, KIND>),
                     dim3((unsigned)(rblocks * (nseg - 1))), dim3(256), 0, s,
                     static_cast<const IN*>(a.x), static_cast<const IN*>(a.delta), a.A,
                     static_cast<const IN*>(a.Bm), static_cast<const IN*>(a.Cm), a.Dskip,
                     static_cast<const IN*>(a.z), a.delta_bias, a.h0, a.y, nullptr, a.D, a.L,
                     ndb, flags, nullptr, (int64_t)0, nullptr, nseg, Lseg, (int)a.N, ngrp, R * a.L);
  const int64_t lanes = R * ngrp * R16_N;
  hipLaunchKernelGGL(row16_fold_kernel, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, s,
                     a.y, a.y_bf16, R * ngrp, a.L, nseg, Lseg);
  auto kern = a.ckpt ? selective_row16_kernel<IN, OPT, true, R16_SEG_FWD, KIND>
                     : selective_row16_kernel<IN, OPT, false, R16_SEG_FWD, KIND>;
  hipLaunchKernelGGL(kern, dim3((unsigned)(rblocks * nseg)), dim3(256), 0, s,
                     static_cast<const IN*>(a.x), static_cast<const IN*>(a.delta), a.A,
                     static_cast<const IN*>(a.Bm), static_cast<const IN*>(a.Cm), a.Dskip,
                     static_cast<const IN*>(a.z), a.delta_bias, a.h0, a.y, a.h_last, a.D, a.L,
                     ndb, flags, a.ckpt, (a.L + 7) / 8, a.s_out, nseg, Lseg, (int)a.N, ngrp, R * a.L);
}

// The correction form: (1) every segment walks from a zero state (the first
// from h0), stores y (all but its first super-tile) and records its P and
// end state; (2) the fold composes the records into each segment's initial
// state and corrects h_last; (3) every segment but the first walks again from
// its initial state, rewriting y, until the part carried in from the start
// is negligible against the segment's own terms (R16_CORR_EPS).
template <typename IN, bool OPT, int KIND>
void launch_row16_corr(const SelArgs& a, int64_t ndb, uint32_t flags, int64_t nseg,
                       int64_t Lseg, hipStream_t s) {
  const int64_t R = a.B * a.D;
  const int ngrp = r16_groups<KIND>(a.N);
  const int64_t rblocks = a.B * ndb * ngrp;
  hipLaunchKernelGGL((selective_row16_kernel<IN, OPT, false, R16_SEG_ALL, KIND>),
                     dim3((unsigned)(rblocks * nseg)), dim3(256), 0, s,
                     static_cast<const IN*>(a.x), static_cast<const IN*>(a.delta), a.A,
                     static_cast<const IN*>(a.Bm), static_cast<const IN*>(a.Cm), a.Dskip,
                     static_cast<const IN*>(a.z), a.delta_bias, a.h0, a.y, a.h_last, a.D, a.L,
                     ndb, flags, nullptr, (int64_t)0, a.s_out, nseg, Lseg, (int)a.N, ngrp, R * a.L);
  launch_fold_corr(static_cast<float*>(a.y), a.h_last, R, a.L, nseg, Lseg, (int)a.N, ngrp, s);
  hipLaunchKernelGGL((selective_row16_kernel<IN, OPT, false, R16_SEG_CORR, KIND>),
                     dim3((unsigned)(rblocks * (nseg - 1))), dim3(256), 0, s,
                     static_cast<const IN*>(a.x), static_cast<const IN*>(a.delta), a.A,
                     static_cast<const IN*>(a.Bm), static_cast<const IN*>(a.Cm), a.Dskip,
                     static_cast<const IN*>(a.z), a.delta_bias, a.h0, a.y, nullptr, a.D, a.L,
                     ndb, flags, nullptr, (int64_t)0, a.s_out, nseg, Lseg, (int)a.N, ngrp, R * a.L);
}

// Whether the call's rows are whole 16-byte vectors: otherwise it takes the
// RAG variant of the kernels.
template <typename IN>
bool row16_aligned(const SelArgs& a) {
  return a.vec && a.L % (16 / (int64_t)sizeof(IN)) == 0;
}

template <typename IN, bool OPT, int KIND>
int launch_row16_t(const SelArgs& a, const N16Plan& p, int64_t ndb, hipStream_t s) {
  const uint32_t flags = (a.softplus ? SEL_SOFTPLUS : 0u) | (a.y_bf16 ? SEL_Y_BF16 : 0u) |
                         (a.z ? SEL_GATED : 0u);
  const int64_t nseg = p.nseg, Lseg = p.Lseg;
  if (nseg > 1) {
    if (p.corr)
      launch_row16_corr<IN, OPT, KIND>(a, ndb, flags, nseg, Lseg, s);
    else
      launch_row16_segments<IN, OPT, KIND>(a, ndb, flags, nseg, Lseg, s);
    note_launch("selective_row16_kernel: %lld segments of %lld steps, %s form (3 launches)",
                (long long)nseg, (long long)Lseg, p.corr ? "correction" : "records");
    return check_launch("selective_row16_kernel (segments)");
  }
  const int ngrp = r16_groups<KIND>(a.N);
  auto kern = a.ckpt ? selective_row16_kernel<IN, OPT, true, R16_WHOLE, KIND>
                     : selective_row16_kernel<IN, OPT, false, R16_WHOLE, KIND>;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.B * ndb * ngrp)), dim3(256), 0, s,
                     static_cast<const IN*>(a.x), static_cast<const IN*>(a.delta), a.A,
                     static_cast<const IN*>(a.Bm), static_cast<const IN*>(a.Cm), a.Dskip,
                     static_cast<const IN*>(a.z), a.delta_bias, a.h0, a.y, a.h_last, a.D, a.L,
                     ndb, flags, a.ckpt, (a.L + 7) / 8, a.s_out, (int64_t)1, a.L, (int)a.N, ngrp,
                     a.B * a.D * a.L);
  note_launch("selective_row16_kernel: whole rows");
  return check_launch("selective_row16_kernel");
}

template <typename IN>
int launch_row16(const SelArgs& a, hipStream_t s) {
  const bool opt = a.z || a.delta_bias || a.softplus || a.y_bf16 || a.s_out;
  const int64_t ndb = (a.D + R16_ROWS - 1) / R16_ROWS;
  const int64_t grid = a.B * ndb;
  if (grid > SW_MAX_WGS)
    return fail(SW_ERR_UNSUPPORTED, "%lld workgroups exceed the grid range", (long long)grid);
  int cus = 0;
  if (device_cus(&cus) != SW_OK) cus = 256;  // a forced choice needs no device facts
  const N16Plan p = plan_n16<IN>(a, ndb, cus);
  if (p.quad) return launch_quad<IN>(a, p.nseg, p.Lseg, s);
  if (row16_aligned<IN>(a))
    return opt ? launch_row16_t<IN, true, R16_VEC>(a, p, ndb, s)
               : launch_row16_t<IN, false, R16_VEC>(a, p, ndb, s);
  return opt ? launch_row16_t<IN, true, R16_RAG>(a, p, ndb, s)
             : launch_row16_t<IN, false, R16_RAG>(a, p, ndb, s);
}

double row16_rows_us(int64_t wgs, int64_t L, int cus) {
  return launch_us(wgs, L, cus, R16_COST, 1.0);
}

// The planned price of the groups' walk on `cus` compute units.
template <typename IN>
double row16_groups_us(const SelArgs& a, int cus) {
  return plan_n16<IN>(a, (a.D + R16_ROWS - 1) / R16_ROWS * r16_groups<R16_GRP>(a.N), cus).us;
}

// N other than 16 (row16_fits): one group of up to 16 states writes y itself;
// several write planes of a workspace (the caller's, or one taken for the call)
// that a last kernel adds up.
// At B=2, D=1024, N=64, L=1024 (fp32) the 8-lane kernel, with 256 wavefronts
// for the GPU's 1024 SIMDs, took 125 us.
template <typename IN>
int launch_row16_groups(const SelArgs& a, hipStream_t s) {
  const int64_t ndb = (a.D + R16_ROWS - 1) / R16_ROWS, R = a.B * a.D;
  const int ngrp = r16_groups<R16_GRP>(a.N);
  if (a.B * ndb * ngrp > SW_MAX_WGS || (ngrp > 1 && R * ((a.L + 1023) / 1024) > SW_MAX_WGS))
    return fail(SW_ERR_UNSUPPORTED, "%lld workgroups exceed the grid range",
                (long long)(a.B * ndb * ngrp));
  int cus = 0;
  if (device_cus(&cus) != SW_OK) cus = 256;
  int st = refuse_capture(s, "the per-stream scratch (tickets and carries)");
  if (st != SW_OK) return st;
  SelArgs g = a;
  if (ngrp > 1) {
    const size_t need = (size_t)ngrp * (size_t)R * (size_t)a.L * sizeof(float);
    if (a.ws && a.ws_bytes < need)
      return fail(SW_ERR_INVALID_ARG, "workspace of %zu bytes, %zu needed", a.ws_bytes, need);
    g.y = a.ws;
    if (!a.ws && (st = workspace_alloc(&g.y, need, s)) != SW_OK) return st;
    g.Dskip = nullptr;
    g.z = nullptr;
    g.s_out = nullptr;
    g.y_bf16 = false;
  }
  const N16Plan p = plan_n16<IN>(g, ndb * ngrp, cus);
  const bool opt = g.z || g.delta_bias || g.softplus || g.y_bf16 || g.s_out;
  st = opt ? launch_row16_t<IN, true, R16_GRP>(g, p, ndb, s)
           : launch_row16_t<IN, false, R16_GRP>(g, p, ndb, s);
  if (ngrp > 1) {
    if (st == SW_OK) {
      const int64_t nch = (a.L + 1023) / 1024;
      hipLaunchKernelGGL((row16_groups_kernel<IN>), dim3((unsigned)(R * nch)), dim3(256), 0, s,
                         static_cast<const float*>(g.y), ngrp, static_cast<const IN*>(a.x),
                         static_cast<const IN*>(a.z), a.Dskip, a.y, a.s_out, R, a.D, a.L, nch, a.y_bf16);
      st = check_launch("row16_groups_kernel");
    }
    if (!a.ws) workspace_free(g.y, s);
  }
  return st;
}

// The states of a whole-row walk without y (R16_STATES): the 8-step
// checkpoints of state group grp (16 states, 0 for N = 16) into a.ckpt and, if given, h_last; x, delta, B, A, h0 and the
// delta options are read, C, Dskip, z and y are not.  The call must satisfy
// row16_fits and, for N = 16, have whole, aligned vectors in its rows.
template <typename IN>
int launch_row16_states(const SelArgs& a, int grp, hipStream_t s) {
  const int64_t ndb = (a.D + R16_ROWS - 1) / R16_ROWS;
  const int64_t grid = a.B * ndb;
  if (grid > SW_MAX_WGS)
    return fail(SW_ERR_UNSUPPORTED, "%lld workgroups exceed the grid range", (long long)grid);
  const bool opt = a.delta_bias || a.softplus;
  const uint32_t flags = a.softplus ? SEL_SOFTPLUS : 0u;
  auto kern = a.N == R16_N ? (opt ? selective_row16_kernel<IN, true, true, R16_STATES, R16_VEC>
                                  : selective_row16_kernel<IN, false, true, R16_STATES, R16_VEC>)
                           : (opt ? selective_row16_kernel<IN, true, true, R16_STATES, R16_GRP>
                                  : selective_row16_kernel<IN, false, true, R16_STATES, R16_GRP>);
  // y is never written in this mode: x stands in for its pointer
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), 0, s, static_cast<const IN*>(a.x),
                     static_cast<const IN*>(a.delta), a.A, static_cast<const IN*>(a.Bm),
                     static_cast<const IN*>(a.Cm), a.Dskip, static_cast<const IN*>(nullptr),
                     a.delta_bias, a.h0, const_cast<void*>(a.x), a.h_last, a.D, a.L, ndb, flags,
                     a.ckpt, (a.L + 7) / 8, static_cast<float*>(nullptr), (int64_t)1, a.L, (int)a.N, grp,
                     (int64_t)0);
  return check_launch("selective_row16_kernel (states)");
}

// What launch_row16 would enqueue for `a` on a part with `cus` compute units.
template <typename IN>
SelPlan plan_row16(const SelArgs& a, int cus) {
  const N16Plan p = plan_n16<IN>(a, (a.D + R16_ROWS - 1) / R16_ROWS, cus);
  SelPlan q;
  q.layout = p.quad ? 4 : 16;
  q.nseg = p.nseg;
  q.lseg = p.nseg > 1 ? p.Lseg : a.L;
  q.form = p.nseg > 1 ? (p.corr ? 2 : 1) : 0;
  return q;
}

template int launch_row16<float>(const SelArgs&, hipStream_t);
template int launch_row16<uint16_t>(const SelArgs&, hipStream_t);
template double row16_groups_us<float>(const SelArgs&, int);
template double row16_groups_us<uint16_t>(const SelArgs&, int);
template int launch_row16_groups<float>(const SelArgs&, hipStream_t);
template int launch_row16_groups<uint16_t>(const SelArgs&, hipStream_t);
template SelPlan plan_row16<float>(const SelArgs&, int);
template SelPlan plan_row16<uint16_t>(const SelArgs&, int);
template int launch_row16_states<float>(const SelArgs&, int, hipStream_t);
template int launch_row16_states<uint16_t>(const SelArgs&, int, hipStream_t);

}  // namespace sw
