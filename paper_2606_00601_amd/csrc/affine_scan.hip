// affine_scan.hip -- bare affine scan h_t = a_t h_{t-1} + bx_t (Eq. (3)) on
// gfx950, as a prefix scan over the affine pairs of Eq. (6) under the
// composition of Eq. (7), for fp32 and for the int32 wraparound ring.
//
// One workgroup (4 wavefronts, 256 lanes) walks a row in chunks of 256*K
// consecutive steps:
//   1. each lane loads K consecutive (a, bx) with 16-byte vector loads (a
//      wavefront reads one contiguous run) and composes them sequentially
//      into its local inclusive prefixes;
//   2. the 64 lane totals of a wavefront are scanned with DPP lane moves
//      (wave_inclusive_scan) and shifted to exclusive prefixes;
//   3. the four wavefront totals go through LDS and every lane folds them,
//      so every lane knows its prefix and the state leaving the chunk;
//   4. every lane rebuilds its states as h = A_pre * h_in + U_pre (Sec. 3.2)
//      and stores them with 16-byte vector stores.
// The carry stays in a register from chunk to chunk, and the next chunk's
// loads are in flight while the current one is scanned.  Rows may have any
// length and any element alignment: gfx950 takes 16-byte accesses at 4-byte
// alignment, and a vector that would cross the row's end is read from before
// it and shifted.  The elementwise form of Eq. (3)-(4) (IO variant) forms bx =
// b * x, stores y = c * h instead of h and can write the final state h_last.
//
// Few long rows are cut into segments of whole chunks, one workgroup each: it
// composes its segment into a total pair and publishes it, waits for the
// pairs of the row's segments before it (a lane per segment), composes them
// into its incoming state and walks the segment again as above, its inputs
// still in the L2 (a segment of one chunk stays in registers).  Segments are
// handed out by a ticket counter per row, so a workgroup only waits for
// workgroups that already run, and the counters do not queue the rows behind
// each other.  Pairs are composed in a fixed order: the result does not
// depend on timing.
//
// Rows of at most 512 steps take one wavefront each (no LDS, no barrier).
// The long walks run at the rate of a copy (R=512, L=65536 in fp32: 79 us,
// 5.1 TB/s), the ragged ones too: B=2, D=1000, L=3001 with x, c and h0 takes
// 21 us, and took 125 us when rows off the 16-byte grid were gathered by
// element; R=16384, L=100: 5.5 us against 20.7 with a workgroup per row.
#include <mutex>

#include "sw_internal.h"

// Scratch of the entry point that allocates nothing (sw_affine_scan_noalloc):
// the ticket counters of a call's rows, directly followed by its segments'
// records (two words each, at most AS_MAX_SEG segments of SW_ROW_TICKETS rows;
// room for three words per chunk of SW_NOALLOC_MAX_CHUNKS chunks).  Each call
// clears what it uses of both.  Each GPU holds its own copy, found by
// hipGetSymbolAddress once per device; host code uses only that address,
// never the array's name.
static __device__ __align__(256) unsigned long long
    scratch[sw::SW_ROW_TICKETS * sw::SW_TICKET_STRIDE / 2 + 3 * (int64_t)SW_NOALLOC_MAX_CHUNKS];

namespace sw {
namespace {

constexpr int AS_THREADS = 256;
constexpr int AS_K = 8;
constexpr int AS_WAVES = AS_THREADS / 64;
constexpr int AS_MAX_SEG = AS_THREADS;  // segments per row at most: a record per lane
constexpr int AS_TICKET_STRIDE = SW_TICKET_STRIDE;

// Operands of one call.  The plain scan has b = bx, y = h and no x, c or
// h_last; the IO variant reads x (NULL: 1) and c (NULL: 1) and writes h_last
// (NULL: not written).
template <typename T>
struct AffIO {
  const T *a, *b, *x, *c, *h0;
  T *y, *h_last;
};

// 2 or 4 elements at 4-byte alignment (one memory instruction on gfx950)
struct __attribute__((packed, aligned(4))) Words2 {
  uint32_t w[2];
};
struct __attribute__((packed, aligned(4))) Words4 {
  uint32_t w[4];
};

// Raw bits of K consecutive elements from element t of a run of n (both
// 32-bit: a run is the rest of a row from a chunk's start, cut at twice the
// chunk), in vectors of V = min(K, 4).  A vector that would cross the run's
// end is read from V elements before it: fix() shifts it back.  Elements past
// the end are left over from the row: they only reach states past the end.
// (n may be below V, or negative, for a later chunk of a row of at least V
// elements: the address then falls before the run, still inside the row.)
template <int K>
struct RowRegs {
  static constexpr int V = K < 4 ? K : 4;
  uint32_t w[K];
  template <typename T>
  __device__ __forceinline__ void load(const T* __restrict__ r, int t, int n) {
#pragma unroll
    for (int q = 0; q < K; q += V) {
      const int at = min(t + q, n - V);
      if constexpr (V == 4) {
        const Words4 v = *reinterpret_cast<const Words4*>(r + at);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[q + i] = v.w[i];
      } else if constexpr (V == 2) {
        const Words2 v = *reinterpret_cast<const Words2*>(r + at);
        w[q] = v.w[0];
        w[q + 1] = v.w[1];
      } else {
        w[q] = *reinterpret_cast<const uint32_t*>(r + at);
      }
    }
  }
  __device__ __forceinline__ void fix(int t, int n) {
#pragma unroll
    for (int q = 0; q < K; q += V) {
      const int back = t + q - (n - V);
      const int sh = back > 0 && back < V ? back : 0;
#pragma unroll
      for (int m = V / 2; m >= 1; m /= 2) {
        // (as masks: selects of array elements became indexed private memory)
        const uint32_t on = (sh & m) ? ~0u : 0u;
#pragma unroll
        for (int i = 0; i + m < V; ++i) w[q + i] = (w[q + i] & ~on) | (w[q + i + m] & on);
      }
    }
  }
};

// a, b (and, IO, x and c) of one lane's K steps
template <typename T, int K, bool IO>
struct StepRegs {
  RowRegs<K> a, b, x, c;
  // steps t .. t+K-1 of the run of n at element `at`
  __device__ __forceinline__ void load(const AffIO<T>& io, int64_t at, int t, int n) {
    a.load(io.a + at, t, n);
    b.load(io.b + at, t, n);
    if constexpr (IO) {
      if (io.x) x.load(io.x + at, t, n);
      if (io.c) c.load(io.c + at, t, n);
    }
  }
  __device__ __forceinline__ void fix(const AffIO<T>& io, int t, int n) {
    a.fix(t, n);
    b.fix(t, n);
    if constexpr (IO) {
      if (io.x) x.fix(t, n);
      if (io.c) c.fix(t, n);
    }
  }
  // the pairs (a, b x), composed sequentially into inclusive prefixes
  __device__ __forceinline__ void prefixes(const AffIO<T>& io, T (&pa)[K], T (&pu)[K]) const {
    using Rg = Ring<T>;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      pa[k] = Rg::from_bits(a.w[k]);
      pu[k] = Rg::from_bits(b.w[k]);
      if (IO && io.x) pu[k] = Rg::mul(pu[k], Rg::from_bits(x.w[k]));
    }
#pragma unroll
    for (int k = 1; k < K; ++k) absorb_earlier(pa[k], pu[k], pa[k - 1], pu[k - 1]);
  }
  // y of the K steps from the state hs before them; the state of step
  // n-1 also goes to h_last, where the run ends the row (last)
  __device__ __forceinline__ void store(const AffIO<T>& io, const T (&pa)[K], const T (&pu)[K], T hs,
                                        int64_t row, int64_t at, int t0, int n, bool last) const {
    using Rg = Ring<T>;
    T* __restrict__ yr = io.y + at;
    uint32_t o[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      T hv = Rg::mad(pa[k], hs, pu[k]);
      if constexpr (IO) {
        if (last && io.h_last && t0 + k == n - 1) io.h_last[row] = hv;
        if (io.c) hv = Rg::mul(Rg::from_bits(c.w[k]), hv);
      }
      o[k] = Rg::bits(hv);
    }
    if (t0 + K <= n) {
#pragma unroll
      for (int q = 0; q < K; q += RowRegs<K>::V) {
        if constexpr (K >= 4)
          *reinterpret_cast<Words4*>(yr + t0 + q) = Words4{{o[q], o[q + 1], o[q + 2], o[q + 3]}};
        else if constexpr (K == 2)
          *reinterpret_cast<Words2*>(yr + t0) = Words2{{o[0], o[1]}};
        else
          yr[t0] = Rg::from_bits(o[0]);
      }
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (t0 + k < n) yr[t0 + k] = Rg::from_bits(o[k]);
    }
  }
};

// Totals of the four wavefronts, from LDS: this lane's prefix of the
// wavefronts before its own, and the total of all.
template <typename T>
__device__ __forceinline__ void fold_waves(const T (&sA)[AS_WAVES], const T (&sU)[AS_WAVES],
                                           int wave, T& pA, T& pU, T& cA, T& cU) {
  pA = cA = Ring<T>::one();
  pU = cU = Ring<T>::zero();
#pragma unroll
  for (int w = 0; w < AS_WAVES; ++w) {
    if (w == wave) {
      pA = cA;
      pU = cU;
    }
    T nA = sA[w], nU = sU[w];
    absorb_earlier(nA, nU, cA, cU);
    cA = nA;
    cU = nU;
  }
}

// One workgroup per row, or (LOOK) per segment of a row: rows of nseg segments
// of seg_chunks chunks, the last taking the rest.  rec holds two carry words
// per segment but the last, its pair's A and U; ticket a counter per row,
// AS_TICKET_STRIDE words apart, zero before and after the launch.
template <typename T, int K, bool IO, bool LOOK>
__global__ __launch_bounds__(AS_THREADS) void affine_rows_kernel(
    const AffIO<T> io, int64_t R, int64_t L, int64_t nseg, int64_t seg_chunks,
    unsigned long long* __restrict__ rec, uint32_t* __restrict__ ticket, uint32_t epoch) {
  constexpr int64_t CH = (int64_t)AS_THREADS * K;
  using Rg = Ring<T>;
  __shared__ T sA[2][AS_WAVES], sU[2][AS_WAVES];
  __shared__ uint32_t s_seg;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t nch = (L + CH - 1) / CH;
  const int t0 = tid * K;
  // elements left in the row from chunk c on, as a 32-bit run
  auto left = [&](int64_t c) {
    const int64_t n = L - c * CH;
    return (int)(n < 2 * CH ? n : 2 * CH);
  };

  for (int64_t id = blockIdx.x; id < (LOOK ? R * nseg : R); id += gridDim.x) {
    const int64_t row = LOOK ? id % R : id;
    int64_t sg = 0, c0 = 0, c1 = nch;
    if constexpr (LOOK) {
      // segments of a row are taken in order of its tickets, so a segment only
      // waits for segments that running workgroups hold
      if (tid == 0) {
        uint32_t* const tk = ticket + row * AS_TICKET_STRIDE;
        s_seg = atomicAdd(tk, 1u);
        if (s_seg == (uint32_t)nseg - 1u)  // the row's last: ready for the next launch
          __hip_atomic_store(tk, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      sg = s_seg;
      c0 = sg * seg_chunks;
      if (c0 + seg_chunks < nch) c1 = c0 + seg_chunks;
    }
    const int64_t base = row * L;
    StepRegs<T, K, IO> cur, nxt;
    cur.load(io, base + c0 * CH, t0, left(c0));
    T carry = io.h0 ? io.h0[row] : Rg::zero();
    T pa[K], pu[K];
    // the wavefronts' totals of the chunk in cur into buffer buf; wA, wU: the
    // lane's inclusive prefix
    auto scan_chunk = [&](int buf, T& wA, T& wU) {
      cur.prefixes(io, pa, pu);
      wA = pa[K - 1];
      wU = pu[K - 1];
      wave_inclusive_scan(wA, wU);
      if (lane == 63) {
        sA[buf][wave] = wA;
        sU[buf][wave] = wU;
      }
    };
    T wA, wU, pA, pU, cA, cU;
    int buf = 0;  // one barrier per chunk: the totals alternate between two buffers
    if (LOOK && sg + 1 < nseg) {
      // the segment's total pair, for the segments after it
      T totA = Rg::one(), totU = Rg::zero();
      for (int64_t c = c0; c < c1; ++c) {
        if (c + 1 < c1) nxt.load(io, base + (c + 1) * CH, t0, left(c + 1));
        scan_chunk(buf, wA, wU);
        __syncthreads();
        fold_waves(sA[buf], sU[buf], wave, pA, pU, cA, cU);
        absorb_earlier(cA, cU, totA, totU);
        totA = cA;
        totU = cU;
        if (c + 1 < c1) cur = nxt;
        buf ^= 1;
      }
      if (tid == 0) {
        unsigned long long* const w = rec + (row * (nseg - 1) + sg) * 2;
        const uint32_t st = carry_status(epoch, CARRY_AGG);
        carry_put(w, st, Rg::bits(totA));
        carry_put(w + 1, st, Rg::bits(totU));
      }
      // a segment of one chunk is still in cur, a longer one is walked again
      // (from the L2 this compute unit just filled)
      if (c1 - c0 > 1) cur.load(io, base + c0 * CH, t0, left(c0));
    }
    if (LOOK && sg > 0) {
      // the state entering the segment: lane l holds the pair of segment l
      wA = Rg::one();
      wU = Rg::zero();
      if (tid < sg) {
        const unsigned long long* const w = rec + (row * (nseg - 1) + tid) * 2;
        const uint32_t st = carry_status(epoch, CARRY_AGG);
        unsigned long long a, u;
        while (a = carry_get(w), u = carry_get(w + 1),
               (uint32_t)(a >> 32) != st || (uint32_t)(u >> 32) != st)
          __builtin_amdgcn_s_sleep(1);
        wA = Rg::from_bits((uint32_t)a);
        wU = Rg::from_bits((uint32_t)u);
      }
      wave_inclusive_scan(wA, wU);
      if (lane == 63) {
        sA[buf][wave] = wA;
        sU[buf][wave] = wU;
      }
      __syncthreads();
      fold_waves(sA[buf], sU[buf], wave, pA, pU, cA, cU);
      carry = Rg::mad(cA, carry, cU);
      buf ^= 1;
    }
    for (int64_t c = c0; c < c1; ++c) {
      const int n = left(c);
      if (c + 1 < c1) nxt.load(io, base + (c + 1) * CH, t0, left(c + 1));  // in flight during the scan
      if (n < CH) cur.fix(io, t0, n);
      scan_chunk(buf, wA, wU);
      wave_shift_exclusive(wA, wU);
      __syncthreads();
      fold_waves(sA[buf], sU[buf], wave, pA, pU, cA, cU);
      absorb_earlier(wA, wU, pA, pU);
      cur.store(io, pa, pu, Rg::mad(wA, carry, wU), row, base + c * CH, t0, n, n <= CH);
      carry = Rg::mad(cA, carry, cU);
      cur = nxt;
      buf ^= 1;
    }
    __syncthreads();  // the totals buffers are reused by the next row
  }
}

// Rows of at most 64*K steps: one wavefront per row.
template <typename T, int K, bool IO>
__global__ __launch_bounds__(AS_THREADS) void affine_wave_kernel(const AffIO<T> io, int64_t R,
                                                                 int64_t L) {
  using Rg = Ring<T>;
  const int t0 = (int)(threadIdx.x & 63) * K, n = (int)L;
  for (int64_t row = (int64_t)blockIdx.x * AS_WAVES + (threadIdx.x >> 6); row < R;
       row += (int64_t)gridDim.x * AS_WAVES) {
    StepRegs<T, K, IO> cur;
    cur.load(io, row * L, t0, n);
    const T h0 = io.h0 ? io.h0[row] : Rg::zero();
    if (n < 64 * K) cur.fix(io, t0, n);
    T pa[K], pu[K];
    cur.prefixes(io, pa, pu);
    T wA = pa[K - 1], wU = pu[K - 1];
    wave_inclusive_scan(wA, wU);
    wave_shift_exclusive(wA, wU);
    cur.store(io, pa, pu, Rg::mad(wA, h0, wU), row, row * L, t0, n, true);
  }
}

std::mutex scratch_addr_mu;
unsigned long long* scratch_addr[64] = {};  // per device, guarded by scratch_addr_mu

// The device address of `scratch` on device `dev` (the current device).
int static_scratch(int dev, unsigned long long** out) {
  *out = nullptr;
  if (dev < 0 || dev >= 64)
    return fail(SW_ERR_UNSUPPORTED, "device %d: the static scratch table holds 64 devices", dev);
  std::lock_guard<std::mutex> g(scratch_addr_mu);
  if (!scratch_addr[dev]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      (void)hipGetLastError();
      return fail(SW_ERR_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                  hipGetErrorString(e));
    }
    scratch_addr[dev] = static_cast<unsigned long long*>(p);
  }
  *out = scratch_addr[dev];
  return SW_OK;
}

// Segments of a row of nch chunks when R rows are scanned on cus compute
// units (1: whole rows).  One compute unit walks a chunk in about 0.8 us (27
// GB/s: what its outstanding misses hold), so few rows leave the bandwidth
// idle; segments read the inputs a second time, from L2.  They pay where half
// of the compute units or fewer have a row and a row has more than 5 chunks;
// about three segments per compute unit measured best or within 10% of it.
// us per call, whole rows / segments: R=64 L=65536 27.5 / 13, L=20000 9.0 /
// 6.4, L=12288 6.1 / 6.4; R=128 L=65536 28.8 / 24, R=192 31.6 / 34; R=1
// L=262144 83 / 6.5.  (The look-back over 2048-step chunks that both forms
// replaced was bound by its one ticket counter, 16 ns a chunk: R=64 L=65536
// 52, R=512 381 against 79.)
int64_t affine_segments(int64_t R, int64_t nch, int cus) {
  if (2 * R > cus || R > SW_ROW_TICKETS || nch <= 5) return 1;
  int64_t n = 3 * (int64_t)cus / R;
  if (n > nch) n = nch;
  return n < AS_MAX_SEG ? n : AS_MAX_SEG;
}

template <typename T, int K, bool IO>
int launch_rows(const AffIO<T>& io, int64_t R, int64_t L, hipStream_t s) {
  hipLaunchKernelGGL((affine_rows_kernel<T, K, IO, false>),
                     dim3((unsigned)(R < SW_MAX_WGS ? R : SW_MAX_WGS)), dim3(AS_THREADS), 0, s, io, R, L,
                     (int64_t)1, (int64_t)0, nullptr, nullptr, 0u);
  return check_launch("affine_rows_kernel");
}

template <typename T, bool IO>
int launch_segments(const AffIO<T>& io, int64_t R, int64_t L, int64_t nseg, int64_t seg_chunks,
                    unsigned long long* rec, uint32_t* ticket, uint32_t epoch, hipStream_t s) {
  hipLaunchKernelGGL((affine_rows_kernel<T, AS_K, IO, true>), dim3((unsigned)(R * nseg)),
                     dim3(AS_THREADS), 0, s, io, R, L, nseg, seg_chunks, rec, ticket, epoch);
  return check_launch("affine_rows_kernel (segments)");
}

template <typename T, int K, bool IO>
int launch_wave(const AffIO<T>& io, int64_t R, int64_t L, hipStream_t s) {
  const int64_t wgs = (R + AS_WAVES - 1) / AS_WAVES;
  hipLaunchKernelGGL((affine_wave_kernel<T, K, IO>),
                     dim3((unsigned)(wgs < SW_MAX_WGS ? wgs : SW_MAX_WGS)), dim3(AS_THREADS), 0, s, io, R,
                     L);
  return check_launch("affine_wave_kernel");
}

// `fixed`: take the records' scratch from the static array instead of the
// per-stream allocation.
template <typename T, bool IO>
int launch_affine(const AffIO<T>& io, int64_t R, int64_t L, bool fixed = false) {
  hipStream_t s = current_stream();
  if (L <= 64) return launch_wave<T, 1, IO>(io, R, L, s);
  if (L <= 128) return launch_wave<T, 2, IO>(io, R, L, s);
  if (L <= 256) return launch_wave<T, 4, IO>(io, R, L, s);
  if (L <= 512) return launch_wave<T, 8, IO>(io, R, L, s);
  constexpr int64_t CH = (int64_t)AS_THREADS * AS_K;
  if (L <= CH / 2) return launch_rows<T, AS_K / 2, IO>(io, R, L, s);
  int cus = 0;
  int st = device_cus(&cus);
  if (st != SW_OK) return st;
  const int64_t nch = (L + CH - 1) / CH;
  // calls of several chunks on fewer than 8 rows per compute unit: the
  // scratch limits and the refusal while capturing are those of this rule,
  // whether or not the call is cut into segments
  const bool scratched = nch > 1 && R < 8 * (int64_t)cus;
  const int64_t total = R * nch;
  if (!scratched) return launch_rows<T, AS_K, IO>(io, R, L, s);
  if (fixed && total > (int64_t)SW_NOALLOC_MAX_CHUNKS)
    return fail(SW_ERR_UNSUPPORTED, "%lld chunks of %lld steps exceed the %d the static scratch holds",
                (long long)total, (long long)CH, (int)SW_NOALLOC_MAX_CHUNKS);
  if (!fixed) {
    if (total >= ((int64_t)1 << 31))
      return fail(SW_ERR_UNSUPPORTED, "%lld chunks exceed the supported range", (long long)total);
    st = refuse_capture(s, "the per-stream scratch (tickets and carries)");
    if (st != SW_OK) return st;
  }
  const int64_t want = affine_segments(R, nch, cus);
  const int64_t per = (nch + want - 1) / want, nseg = (nch + per - 1) / per;
  if (nseg <= 1) return launch_rows<T, AS_K, IO>(io, R, L, s);
  if (fixed) {
    int cur = 0;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return fail(SW_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    unsigned long long* base = nullptr;
    st = static_scratch(cur, &base);
    if (st != SW_OK) return st;
    // The records of the call before carry the same epoch, and its counters
    // may hold anything if it did not run alone: a segment that no workgroup
    // ever takes would be waited for forever.  So each call starts from
    // cleared counters and records, whatever came before it.
    unsigned long long* const rec = base + R * SW_TICKET_STRIDE / 2;
    st = zero_words(reinterpret_cast<uint32_t*>(base),
                    (size_t)(R * SW_TICKET_STRIDE + R * (nseg - 1) * 4), s);
    if (st != SW_OK) return st;
    return launch_segments<T, IO>(io, R, L, nseg, per, rec, reinterpret_cast<uint32_t*>(base), 1u, s);
  }
  ScratchSession ss;
  st = ss.reserve((size_t)(R * (nseg - 1) * 2), 0, s);
  if (st != SW_OK) return st;
  st = launch_segments<T, IO>(io, R, L, nseg, per, ss.carry, ss.row_tickets, ss.epoch, s);
  if (st != SW_OK) ss.invalidate();
  return st;
}

}  // namespace

int affine_scan_f32(const float* a, const float* bx, const float* h0, float* h, int64_t R,
                    int64_t L) {
  return launch_affine<float, false>(AffIO<float>{a, bx, nullptr, nullptr, h0, h, nullptr}, R, L);
}

int affine_scan_f32_noalloc(const float* a, const float* bx, const float* h0, float* h,
                            int64_t R, int64_t L) {
  return launch_affine<float, false>(AffIO<float>{a, bx, nullptr, nullptr, h0, h, nullptr}, R, L, true);
}

int affine_scan_u32(const uint32_t* a, const uint32_t* bx, const uint32_t* h0, uint32_t* h,
                    int64_t R, int64_t L) {
  return launch_affine<uint32_t, false>(
      AffIO<uint32_t>{a, bx, nullptr, nullptr, h0, h, nullptr}, R, L);
}

int affine_scan_io_f32(const float* a, const float* b, const float* x, const float* c,
                       const float* h0, float* y, float* h_last, int64_t R, int64_t L) {
  return launch_affine<float, true>(AffIO<float>{a, b, x, c, h0, y, h_last}, R, L);
}

int affine_scan_io_u32(const uint32_t* a, const uint32_t* b, const uint32_t* x, const uint32_t* c,
                       const uint32_t* h0, uint32_t* y, uint32_t* h_last, int64_t R, int64_t L) {
  return launch_affine<uint32_t, true>(AffIO<uint32_t>{a, b, x, c, h0, y, h_last}, R, L);
}

}  // namespace sw
