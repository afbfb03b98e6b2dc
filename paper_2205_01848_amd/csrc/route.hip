// Load counting, capacities, slot assignment + dispatch (GroupBy with the
// Section 4.1 capacity/drop rule), combine (Aggregate) and their backward.
//
// Slot assignment is a stable counting sort of the T*k assignments in
// priority order q = j*T + t (all first choices in token order, then all
// second choices, ...):
//   1. per-chunk expert histograms (4096 assignments per workgroup),
//   2. one workgroup scans them into per-chunk bases and applies capacity,
//   3. each chunk re-ranks its assignments with wavefront ballots (expert id
//      equality masks from 6 ballots, rank = popcount below the lane),
//      giving pos, keep, dest_row and src - all integer, bit-exact.
// The row copies (dispatch gather, combine, their backward) are token-major:
// one wavefront per token, 16-byte vector loads/stores along the row, so x
// is read once even when k rows are written.

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.hpp"
#include "route.hpp"
#include "sched.hpp"
#include "validate.hpp"

namespace moe {
namespace {

constexpr int kChunk = 1024;  // assignments per workgroup in the routing kernels

// Is assignment (t, j) live?  Sets status bits when `status` is non-null.
__device__ __forceinline__ bool live_assignment(const int32_t* __restrict__ ids, int t,
                                                int j, int k, int E, int32_t* status) {
  const int32_t* row = ids + static_cast<size_t>(t) * k;
  const int e = row[j];
  if (e < 0 || e >= E) {
    if (status) atomicOr(status, MOE_STATUS_BAD_ID);
    return false;
  }
  for (int jj = 0; jj < j; ++jj) {
    if (row[jj] == e) {
      if (status) atomicOr(status, MOE_STATUS_DUP_ID);
      return false;
    }
  }
  return true;
}

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// counts[e] += live assignments of this block's chunk (counts zeroed before)
__global__ __launch_bounds__(256) void count_kernel(const int32_t* __restrict__ ids, int T,
                                                    int E, int k, int32_t* counts,
                                                    int32_t* status) {
  __shared__ int h[kMaxE];
  if (threadIdx.x < kMaxE) h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t n = static_cast<int64_t>(T) * k;
  const int64_t q0 = static_cast<int64_t>(blockIdx.x) * kChunk;
  const int64_t q1 = min(n, q0 + kChunk);
  for (int64_t q = q0 + threadIdx.x; q < q1; q += 256) {
    const int j = static_cast<int>(q / T), t = static_cast<int>(q - static_cast<int64_t>(j) * T);
    if (live_assignment(ids, t, j, k, E, status)) atomicAdd(&h[ids[static_cast<size_t>(t) * k + j]], 1);
  }
  __syncthreads();
  if (threadIdx.x < E && h[threadIdx.x]) atomicAdd(&counts[threadIdx.x], h[threadIdx.x]);
}

__device__ __forceinline__ int capacity_of(const CapRule& c, int T, int k, int E, int count) {
  int64_t v;
  if (c.dynamic) {
    const uint64_t n = static_cast<uint64_t>(c.num) * static_cast<uint32_t>(max(count, 0)) +
                       static_cast<uint32_t>(c.den - 1);
    v = n >> 32 ? static_cast<int64_t>(n / static_cast<uint32_t>(c.den))
                : static_cast<int64_t>(static_cast<uint32_t>(n) / static_cast<uint32_t>(c.den));
  } else {
    v = (static_cast<int64_t>(c.num) * T * k + static_cast<int64_t>(c.den) * E - 1) /
        (static_cast<int64_t>(c.den) * E);
  }
  v = max(v, static_cast<int64_t>(c.cap_min));
  return static_cast<int>(min(v, static_cast<int64_t>(T)));
}

// First row of expert lane's region (lanes below E of one wavefront, their
// capacities in cap): the sum of the earlier capacities, each rounded up to
// a multiple of the alignment; `total` gets the end of the last region.
__device__ __forceinline__ int region_start(const CapRule& c, int cap, int E, int& total) {
  const int lane = threadIdx.x & 63;
  const int mine = lane < E ? (cap + c.align - 1) / c.align * c.align : 0;
  int v = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  total = __shfl(v, 63, 64);
  return v - mine;
}

__global__ __launch_bounds__(64) void capacity_kernel(int T, int k, int E,
                                                      const int32_t* __restrict__ counts,
                                                      const CapRule rule,
                                                      int32_t* __restrict__ capacity,
                                                      int32_t* __restrict__ offsets) {
  const int e = threadIdx.x;
  const int cap = e < E ? capacity_of(rule, T, k, E, counts ? counts[e] : 0) : 0;
  int total;
  const int off = region_start(rule, cap, E, total);
  if (e < E) {
    capacity[e] = cap;
    offsets[e] = off;
  }
  if (e == 0) offsets[E] = total;
}

// Dispatch step 1: chunk histograms; also initialises src[] to -1.
__global__ __launch_bounds__(256) void route_hist_kernel(
    const int32_t* __restrict__ ids, int T, int E, int k, int nblk, int64_t rows_alloc,
    int32_t* __restrict__ hist, int32_t* __restrict__ src, int32_t* status) {
  __shared__ int h[kMaxE];
  if (threadIdx.x < kMaxE) h[threadIdx.x] = 0;
  const int64_t rs = (rows_alloc + nblk - 1) / nblk;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * rs;
  const int64_t r1 = min(rows_alloc, r0 + rs);
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) src[r] = -1;
  __syncthreads();
  const int64_t n = static_cast<int64_t>(T) * k;
  const int64_t q0 = static_cast<int64_t>(blockIdx.x) * kChunk;
  const int64_t q1 = min(n, q0 + kChunk);
  for (int64_t q = q0 + threadIdx.x; q < q1; q += 256) {
    const int j = static_cast<int>(q / T), t = static_cast<int>(q - static_cast<int64_t>(j) * T);
    if (live_assignment(ids, t, j, k, E, status)) atomicAdd(&h[ids[static_cast<size_t>(t) * k + j]], 1);
  }
  __syncthreads();
  if (threadIdx.x < E) hist[static_cast<size_t>(blockIdx.x) * E + threadIdx.x] = h[threadIdx.x];
}

// Usable rows of a region of `cap` rows that starts at row `off` of a buffer
// of rows_alloc.
__device__ __forceinline__ int own_room(int cap, int off, int64_t rows_alloc) {
  return static_cast<int>(max(int64_t(0), min(static_cast<int64_t>(cap), rows_alloc - off)));
}

// Usable rows of expert e's region: its capacity, clamped to the region the
// offsets give it and to rows_alloc (0 for a region starting out of range).
__device__ __forceinline__ int64_t region_room(const int32_t* __restrict__ capacity,
                                               const int32_t* __restrict__ offsets,
                                               int64_t rows_alloc, int e) {
  const int64_t off = offsets[e];
  int64_t room = 0;
  if (off >= 0) {
    room = capacity[e];
    room = min(room, static_cast<int64_t>(offsets[e + 1]) - off);
    room = min(room, rows_alloc - off);
    room = max(room, int64_t(0));
  }
  return room;
}

// Dispatch step 2: per-expert exclusive scan over chunks, counts, the usable
// capacity of each region, fill.  OWN: the capacities and offsets follow from
// the counts just summed, and are written too.
template <bool OWN>
__global__ __launch_bounds__(64) void route_scan_kernel(
    const int32_t* __restrict__ hist, int nblk, int T, int k, int E, const CapRule rule,
    int32_t* __restrict__ capacity, int32_t* __restrict__ offsets, int64_t rows_alloc,
    int32_t* __restrict__ base, int32_t* __restrict__ cap_eff, int32_t* __restrict__ counts,
    int32_t* __restrict__ fill, int32_t* status) {
  const int lane = threadIdx.x;
  const int e = min(lane, E - 1);   // lanes past E repeat expert E - 1 (same values written)
  int run = 0;
  int b = 0;
  for (; b + 8 <= nblk; b += 8) {   // loads of 8 chunks issued before their adds
    int h[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) h[u] = hist[static_cast<size_t>(b + u) * E + e];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      base[static_cast<size_t>(b + u) * E + e] = run;
      run += h[u];
    }
  }
  for (; b < nblk; ++b) {
    base[static_cast<size_t>(b) * E + e] = run;
    run += hist[static_cast<size_t>(b) * E + e];
  }
  int64_t room;
  int cap;
  if constexpr (OWN) {
    cap = capacity_of(rule, T, k, E, run);
    int total;
    const int off = region_start(rule, cap, E, total);
    room = own_room(cap, off, rows_alloc);
    if (lane < E) {
      capacity[e] = cap;
      offsets[e] = off;
    }
    if (lane == 0) offsets[E] = total;
  } else {
    cap = capacity[e];
    room = region_room(capacity, offsets, rows_alloc, e);
  }
  if (lane >= E) return;
  counts[e] = run;
  if (room < cap) atomicOr(status, MOE_STATUS_REGION);
  cap_eff[e] = static_cast<int32_t>(room);
  fill[e] = static_cast<int32_t>(min(static_cast<int64_t>(run), room));
}

// Dispatch step 3: rank within chunk (wavefront ballots), keep/dest/src.
// SCAN: small batches (at most kScanChunks chunks) skip step 2; every
// workgroup sums the histograms of the chunks before its own, and workgroup
// 0 writes counts, fill and the region status bit.
// OWN (with SCAN): every workgroup also derives the capacities and offsets
// from the counts, and workgroup 0 writes them.
constexpr int kScanChunks = 64;
template <bool SCAN, bool OWN>
__global__ __launch_bounds__(256) void route_rank_kernel(
    const int32_t* __restrict__ ids, int T, int E, int k, const int32_t* __restrict__ base,
    const int32_t* __restrict__ cap_eff, int32_t* __restrict__ offsets,
    int32_t* __restrict__ dest_row, int32_t* __restrict__ src,
    const int32_t* __restrict__ hist, int nblk, const CapRule rule,
    int32_t* __restrict__ capacity, int64_t rows_alloc, int32_t* __restrict__ counts,
    int32_t* __restrict__ fill, int32_t* status) {
  __shared__ int run[kMaxE];
  __shared__ int wcnt[4][kMaxE];
  __shared__ int capv[kMaxE];
  __shared__ int offv[kMaxE];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if constexpr (SCAN) {
    // wave w sums chunks w, w + 4, ...: those before this one (wcnt) and
    // all of them (tot)
    __shared__ int tot[4][kMaxE];
    if (lane < E) {
      int lo = 0, all = 0;
      for (int b = wave; b < nblk; b += 4) {
        const int v = hist[static_cast<size_t>(b) * E + lane];
        all += v;
        lo += b < static_cast<int>(blockIdx.x) ? v : 0;
      }
      wcnt[wave][lane] = lo;
      tot[wave][lane] = all;
    }
    __syncthreads();
    if (wave == 0) {
      const int e = min(lane, E - 1);
      const int total = tot[0][e] + tot[1][e] + tot[2][e] + tot[3][e];
      int cap, off;
      int64_t room;
      if constexpr (OWN) {
        cap = capacity_of(rule, T, k, E, total);
        int end;
        off = region_start(rule, cap, E, end);
        room = own_room(cap, off, rows_alloc);
        if (blockIdx.x == 0 && lane < E) {
          capacity[e] = cap;
          offsets[e] = off;
          if (e == E - 1) offsets[E] = end;
        }
      } else {
        cap = capacity[e];
        off = offsets[e];
        room = region_room(capacity, offsets, rows_alloc, e);
      }
      if (lane < E) {
        run[e] = wcnt[0][e] + wcnt[1][e] + wcnt[2][e] + wcnt[3][e];
        if (blockIdx.x == 0) {
          counts[e] = total;
          fill[e] = static_cast<int32_t>(min(static_cast<int64_t>(total), room));
          if (room < cap) atomicOr(status, MOE_STATUS_REGION);
        }
        capv[e] = static_cast<int32_t>(room);
        offv[e] = off;
      }
    }
  } else {
    if (threadIdx.x < E) {
      run[threadIdx.x] = base[static_cast<size_t>(blockIdx.x) * E + threadIdx.x];
      capv[threadIdx.x] = cap_eff[threadIdx.x];
      offv[threadIdx.x] = offsets[threadIdx.x];
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 4 * kMaxE; i += 256) (&wcnt[0][0])[i] = 0;
  __syncthreads();
  const int64_t n = static_cast<int64_t>(T) * k;
  const int64_t q0 = static_cast<int64_t>(blockIdx.x) * kChunk;
  const int64_t q1 = min(n, q0 + kChunk);
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  for (int64_t qb = q0; qb < q1; qb += 256) {
    const int64_t q = qb + threadIdx.x;
    int e = -1, t = 0, j = 0;
    if (q < q1) {
      j = static_cast<int>(q / T);
      t = static_cast<int>(q - static_cast<int64_t>(j) * T);
      if (live_assignment(ids, t, j, k, E, nullptr)) e = ids[static_cast<size_t>(t) * k + j];
    }
    const bool live = e >= 0;
    uint64_t eq = __ballot(live);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
      const bool bit = live && ((e >> b) & 1);
      const uint64_t m = __ballot(bit);
      eq &= bit ? m : ~m;
    }
    int rank = 0;
    if (live) {
      rank = __popcll(eq & lt_mask);
      if (rank == 0) wcnt[wave][e] = __popcll(eq);
    }
    __syncthreads();
    if (live) {
      int pos = run[e] + rank;
      for (int w = 0; w < wave; ++w) pos += wcnt[w][e];
      const size_t a = static_cast<size_t>(t) * k + j;
      if (pos < capv[e]) {
        const int r = offv[e] + pos;
        dest_row[a] = r;
        src[r] = static_cast<int32_t>(a);
      } else {
        dest_row[a] = -1;
      }
    } else if (q < q1) {
      dest_row[static_cast<size_t>(t) * k + j] = -1;
    }
    __syncthreads();
    if (threadIdx.x < E) {
      run[threadIdx.x] += wcnt[0][threadIdx.x] + wcnt[1][threadIdx.x] +
                          wcnt[2][threadIdx.x] + wcnt[3][threadIdx.x];
      wcnt[0][threadIdx.x] = wcnt[1][threadIdx.x] = 0;
      wcnt[2][threadIdx.x] = wcnt[3][threadIdx.x] = 0;
    }
    __syncthreads();
  }
}

// Token-major row kernels: one wavefront per token, `nvec` 16-byte vectors
// per row (row bytes / 16), lanes stride over the row. The token index and
// its picks are wave-uniform (scalar registers, scalar branches); each lane
// loads a batch of its vectors before it uses any of them (one memory
// latency per batch instead of one per 1 KB of the row), the ragged end of a
// row in smaller batches.
constexpr int kRowWaves = 4;
constexpr int kRowBatch = 4;

__device__ __forceinline__ int row_token() {
  return __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x) * kRowWaves +
                                        (static_cast<int>(threadIdx.x) >> 6));
}

// Makes a loaded value opaque to the optimiser, so that the copies below
// store the registers the batch loaded rather than loading them again per
// kept pick.
__device__ __forceinline__ void hold(uint4& v) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  u32x4 r = __builtin_bit_cast(u32x4, v);
  asm volatile("" : "+v"(r));
  v = __builtin_bit_cast(uint4, r);
}

// Walks a lane's vectors v = lane, lane+64, ... < nvec in batches: f(NB, v)
// takes vectors v, v+64, ..., v+64*(NB-1), all in range. Batches of UB while
// they fit, then one of 2 (UB > 2), then single vectors.
template <int UB, typename F>
__device__ __forceinline__ void for_row_batches(int nvec, int lane, F&& f) {
  int v = lane;
  for (; v + 64 * (UB - 1) < nvec; v += 64 * UB) f(std::integral_constant<int, UB>{}, v);
  if constexpr (UB > 2) {
    if (v + 64 < nvec) {
      f(std::integral_constant<int, 2>{}, v);
      v += 128;
    }
  }
  for (; v < nvec; v += 64) f(std::integral_constant<int, 1>{}, v);
}

template <int NB>
__device__ __forceinline__ void gather_vecs(const uint4* __restrict__ xr, const int (&dst)[kMaxK],
                                            int nvec, int v, uint4* __restrict__ x_disp) {
  uint4 val[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) val[u] = xr[v + 64 * u];
#pragma unroll
  for (int u = 0; u < NB; ++u) hold(val[u]);
#pragma unroll
  for (int j = 0; j < kMaxK; ++j) {
    if (dst[j] >= 0) {
      uint4* o = x_disp + static_cast<size_t>(dst[j]) * nvec + v;
#pragma unroll
      for (int u = 0; u < NB; ++u) o[64 * u] = val[u];
    }
  }
}

// Dispatch step 4: x_disp[dest_row[t,j]] = x[t] for every kept j.
__global__ __launch_bounds__(256) void gather_rows_kernel(
    const uint4* __restrict__ x, const int32_t* __restrict__ dest_row, int T, int k,
    int nvec, uint4* __restrict__ x_disp) {
  const int t = row_token();
  const int lane = threadIdx.x & 63;
  if (t >= T) return;
  int dst[kMaxK];
  bool any = false;
#pragma unroll
  for (int j = 0; j < kMaxK; ++j) {
    dst[j] = __builtin_amdgcn_readfirstlane(j < k ? dest_row[static_cast<size_t>(t) * k + j] : -1);
    any |= dst[j] >= 0;
  }
  if (!any) return;
  const uint4* xr = x + static_cast<size_t>(t) * nvec;
  for_row_batches<kRowBatch>(nvec, lane, [&](auto nb, int v) {
    gather_vecs<decltype(nb)::value>(xr, dst, nvec, v, x_disp);
  });
}

// ---- count + capacity + dispatch of small batches --------------------------
// At a few thousand tokens each of the routing kernels costs its launch (about
// 4.7 us between dependent kernels) and little else, so moe_route does the
// whole of it in two launches, or one for the smallest batches.  Tokens come
// in chunks of CT, one workgroup each; per chunk and choice j the histogram
// kernel counts the live assignments to every expert (hist[chunk][j * E +
// e]); then every workgroup of the second kernel sums the histograms of all
// chunks and of those before its own, derives capacities, offsets and the
// first position of each of its (j, e) groups, ranks its tokens with one
// wavefront per choice, and copies their rows.  Up to kTinyAssign
// assignments every workgroup counts the ids itself instead of reading
// histograms, and a workgroup takes four tokens.  The first rows are loaded
// before the routing they do not depend on.  One workgroup more, if asked,
// derives the fills as the others do and builds the expert products' schedule
// from them, which saves that kernel's launch.
constexpr int kTinyAssign = 2048;     // 8 ids per thread
constexpr int kMaxHist = 16384;       // histogram entries every workgroup reads (64 KB)
constexpr int kMaxPairs = kMaxK * kMaxE;

// Lane's assignment among the same choice of the wavefront's tokens: eq =
// lanes with the same expert (0 for a lane without a live assignment).
__device__ __forceinline__ uint64_t same_expert(int e, bool live) {
  uint64_t eq = __ballot(live);
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    const bool bit = live && ((e >> b) & 1);
    const uint64_t m = __ballot(bit);
    eq &= bit ? m : ~m;
  }
  return live ? eq : 0;
}

// One wavefront per chunk of CT tokens.
template <int CT>
__global__ __launch_bounds__(256) void route_chunk_hist_kernel(
    const int32_t* __restrict__ ids, int T, int E, int k, int nchunk, int32_t* __restrict__ hist,
    int32_t* status) {
  __shared__ int h[4][kMaxPairs];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int chunk = blockIdx.x * 4 + wave;
  const int P = k * E;
  for (int i = lane; i < P; i += 64) h[wave][i] = 0;
  __builtin_amdgcn_wave_barrier();
  const int t = chunk * CT + lane;
  for (int j = 0; j < k; ++j) {
    const bool live = lane < CT && t < T && live_assignment(ids, t, j, k, E, status);
    const int e = live ? ids[static_cast<size_t>(t) * k + j] : 0;
    const uint64_t eq = same_expert(e, live);
    if (live && (eq & ((uint64_t(1) << lane) - 1)) == 0) h[wave][j * E + e] = __popcll(eq);
  }
  __builtin_amdgcn_wave_barrier();
  if (chunk >= nchunk) return;
  for (int i = lane; i < P; i += 64) hist[static_cast<size_t>(chunk) * P + i] = h[wave][i];
}

struct RouteArgs {
  const uint4* x;
  const int32_t* ids;
  const int32_t* hist;   // null: counted from the ids
  int T, E, k, nvec, nchunk;
  CapRule rule;
  int64_t rows_alloc;
  int32_t *capacity, *offsets, *counts, *fill, *dest_row, *src;
  uint4* x_disp;
  int32_t* status;
  SchedArgs sched;       // built by workgroup nchunk, where the grid has it
};

template <int CT>
__global__ __launch_bounds__(256) void route_fused_kernel(const RouteArgs a) {
  __shared__ int tot[kMaxPairs], bef[kMaxPairs];   // then bef: first position of (j, e) here
  __shared__ int capv[kMaxE], offv[kMaxE], fillv[kMaxE];
  __shared__ int dst[CT][kMaxK];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int E = a.E, k = a.k, P = k * E;
  const int chunk = blockIdx.x, t0 = chunk * CT;
  // wavefront w copies the rows of tokens t0 + w, t0 + w + 4, ...: UB of them
  // and VB vectors of each per lane at a time
  constexpr int NT = CT / 4, UB = NT < 8 ? NT : 8, VB = UB == 1 ? 4 : 1;
  uint4 val[UB][VB];
  auto load = [&](int first, int v) {
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
      for (int w = 0; w < VB; ++w)
        if (v + 64 * w < a.nvec)
          val[u][w] = a.x[static_cast<size_t>(min(first + 4 * u, a.T - 1)) * a.nvec + v + 64 * w];
  };
  const bool scheduler = chunk == a.nchunk;   // has no tokens
  if (!scheduler) load(t0 + wave, lane);
  for (int i = tid; i < P; i += 256) tot[i] = bef[i] = 0;
  for (int i = tid; i < CT * kMaxK; i += 256) (&dst[0][0])[i] = -1;
  __syncthreads();
  if (a.hist) {
    // threads in groups of P (or more pairs than threads: one group), each
    // group every G-th chunk, eight loads in flight per thread
    const int Pt = min(P, 256), G = 256 / Pt, grp = tid / Pt;
    if (grp < G) {
      for (int p = tid - grp * Pt; p < P; p += Pt) {
        int all = 0, lo = 0;
        for (int c0 = grp; c0 < a.nchunk; c0 += 8 * G) {
          int v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int c = c0 + u * G;
            v[u] = c < a.nchunk ? a.hist[static_cast<size_t>(c) * P + p] : 0;
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            all += v[u];
            lo += c0 + u * G < chunk ? v[u] : 0;
          }
        }
        atomicAdd(&tot[p], all);
        atomicAdd(&bef[p], lo);
      }
    }
  } else {
    const int n = a.T * k;
    for (int q = tid; q < n; q += 256) {
      const int t = q / k, j = q - t * k;
      if (live_assignment(a.ids, t, j, k, E, chunk == 0 ? a.status : nullptr)) {
        const int p = j * E + a.ids[q];
        atomicAdd(&tot[p], 1);
        if (t < t0) atomicAdd(&bef[p], 1);
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    const int e = min(lane, E - 1);
    int count = 0;
    for (int j = 0; j < k; ++j) count += tot[j * E + e];
    const int cap = capacity_of(a.rule, a.T, k, E, count);
    int end;
    const int off = region_start(a.rule, cap, E, end);
    const int room = own_room(cap, off, a.rows_alloc);
    if (lane < E) {
      int run = 0;
      for (int j = 0; j < k; ++j) {
        bef[j * E + e] += run;
        run += tot[j * E + e];
      }
      capv[e] = room;
      offv[e] = off;
      fillv[e] = min(count, room);
      if (chunk == 0) {
        a.counts[e] = count;
        a.capacity[e] = cap;
        a.offsets[e] = off;
        if (e == E - 1) a.offsets[E] = end;
        a.fill[e] = min(count, room);
        if (room < cap) atomicOr(a.status, MOE_STATUS_REGION);
      }
    }
  }
  __syncthreads();
  if (scheduler) {
    build_schedule<4>(lane < E ? fillv[lane] : 0, a.sched);
    return;
  }
  // ranks: one wavefront per choice, lane = token
  for (int j = wave; j < k; j += 4) {
    const int t = t0 + lane;
    const bool in = lane < CT && t < a.T;
    const bool live = in && live_assignment(a.ids, t, j, k, E, nullptr);
    const size_t as = static_cast<size_t>(t) * k + j;
    const int e = live ? a.ids[as] : 0;
    const uint64_t eq = same_expert(e, live);
    int r = -1;
    if (live) {
      const int pos = bef[j * E + e] + __popcll(eq & ((uint64_t(1) << lane) - 1));
      if (pos < capv[e]) {
        r = offv[e] + pos;
        a.src[r] = static_cast<int32_t>(as);
        dst[lane][j] = r;
      }
    }
    if (in) a.dest_row[as] = r;
  }
  // rows that hold no assignment: past the kept ones of their region, or past
  // the last region
  for (int64_t r = static_cast<int64_t>(chunk) * 256 + tid; r < a.rows_alloc;
       r += static_cast<int64_t>(a.nchunk) * 256) {
    int lo = 0, hi = E - 1;   // last expert whose region starts at or before r
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (offv[mid] <= r) lo = mid;
      else hi = mid - 1;
    }
    if (r - offv[lo] >= fillv[lo]) a.src[r] = -1;
  }
  __syncthreads();
#pragma unroll 1
  for (int i0 = 0; i0 < NT; i0 += UB) {
    const int first = t0 + wave + 4 * i0;
    if (first >= a.T) break;
    for (int v = lane; v < a.nvec; v += 64 * VB) {
      if (i0 > 0 || v >= 64 * VB) load(first, v);   // the first batch is there already
#pragma unroll
      for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int w = 0; w < VB; ++w) hold(val[u][w]);
      for (int j = 0; j < k; ++j)
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int r = __builtin_amdgcn_readfirstlane(dst[wave + 4 * (i0 + u)][j]);
          if (r < 0) continue;
#pragma unroll
          for (int w = 0; w < VB; ++w)
            if (v + 64 * w < a.nvec) a.x_disp[static_cast<size_t>(r) * a.nvec + v + 64 * w] = val[u][w];
        }
    }
  }
}

// dx is the layer's last output of a step and is not read again by the
// library: it is stored non-temporally, so its lines do not stay dirty in
// the caches, to be written back while the next kernels stream their inputs.
__device__ __forceinline__ void store_stream(uint4* p, const uint4& v) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), reinterpret_cast<u32x4*>(p));
}

// Batch of the combine below: NB vectors of the row (v, v+64, ...), all
// kept rows' loads issued first, each output element summed in order j;
// STREAM stores the result non-temporally.
template <typename T, int KT, int NB, bool STREAM = false>
__device__ __forceinline__ void combine_vecs(const uint4* __restrict__ yd, const int (&dst)[KT],
                                             const float (&w)[KT], int nvec, int v,
                                             uint4* __restrict__ yr) {
  constexpr int V = Elem<T>::kVec;
  uint4 raw[NB][KT];
#pragma unroll
  for (int j = 0; j < KT; ++j) {
    if (dst[j] >= 0) {
      const uint4* src = yd + static_cast<size_t>(dst[j]) * nvec + v;
#pragma unroll
      for (int u = 0; u < NB; ++u) raw[u][j] = src[64 * u];
    }
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    float acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = 0.f;
#pragma unroll
    for (int j = 0; j < KT; ++j) {
      if (dst[j] >= 0) {
        float f[V];
        Elem<T>::load(raw[u][j], f);
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = fmaf(w[j], f[i], acc[i]);
      }
    }
    if (STREAM)
      store_stream(yr + v + 64 * u, Elem<T>::store(acc));
    else
      yr[v + 64 * u] = Elem<T>::store(acc);
  }
}

// y[t] = sum_j kept w[t,j] * y_disp[dest_row[t,j]]  (fp32 sum in order j);
// KT >= k bounds the picks held in registers, and the batch shrinks as KT
// grows (KT rows' vectors per batch element).
template <typename T, int KT>
__global__ __launch_bounds__(256) void combine_kernel(
    const uint4* __restrict__ yd, const int32_t* __restrict__ dest_row,
    const float* __restrict__ wts, int Ttok, int k, int nvec, int64_t rows_alloc,
    uint4* __restrict__ y) {
  const int t = row_token();
  const int lane = threadIdx.x & 63;
  if (t >= Ttok) return;
  int dst[KT];
  float w[KT];
#pragma unroll
  for (int j = 0; j < KT; ++j) {
    int r = j < k ? dest_row[static_cast<size_t>(t) * k + j] : -1;
    if (r >= rows_alloc) r = -1;  // not a row of y_disp: treated as dropped
    dst[j] = __builtin_amdgcn_readfirstlane(r);
    w[j] = j < k ? wts[static_cast<size_t>(t) * k + j] : 0.f;
  }
  uint4* yr = y + static_cast<size_t>(t) * nvec;
  constexpr int UB = KT <= 2 ? kRowBatch : (KT <= 4 ? 2 : 1);
  for_row_batches<UB>(nvec, lane, [&](auto nb, int v) {
    combine_vecs<T, KT, decltype(nb)::value>(yd, dst, w, nvec, v, yr);
  });
}

// Batch of the combine backward below: NB vectors of dy[t] and of each kept
// row of y_disp, loads first; dot[j] accumulates in the lane's vector order.
template <typename T, int KT, int NB>
__device__ __forceinline__ void combine_bwd_vecs(const uint4* __restrict__ dr,
                                                 const uint4* __restrict__ yd,
                                                 const int (&dst)[KT], const float (&w)[KT],
                                                 float (&dot)[KT], int nvec, int v,
                                                 uint4* __restrict__ dyd) {
  constexpr int V = Elem<T>::kVec;
  uint4 rg[NB], ry[NB][KT];
#pragma unroll
  for (int u = 0; u < NB; ++u) rg[u] = dr[v + 64 * u];
#pragma unroll
  for (int j = 0; j < KT; ++j) {
    if (dst[j] >= 0) {
      const uint4* src = yd + static_cast<size_t>(dst[j]) * nvec + v;
#pragma unroll
      for (int u = 0; u < NB; ++u) ry[u][j] = src[64 * u];
    }
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    float g[V];
    Elem<T>::load(rg[u], g);
#pragma unroll
    for (int j = 0; j < KT; ++j) {
      if (dst[j] >= 0) {
        float f[V], o[V];
        Elem<T>::load(ry[u][j], f);
#pragma unroll
        for (int i = 0; i < V; ++i) {
          dot[j] = fmaf(g[i], f[i], dot[j]);
          o[i] = w[j] * g[i];
        }
        dyd[static_cast<size_t>(dst[j]) * nvec + v + 64 * u] = Elem<T>::store(o);
      }
    }
  }
}

// dweights[t,j] = <dy[t], y_disp[r]>; dy_disp[r] = w[t,j] * dy[t]
template <typename T, int KT>
__global__ __launch_bounds__(256) void combine_bwd_kernel(
    const uint4* __restrict__ dy, const uint4* __restrict__ yd,
    const int32_t* __restrict__ dest_row, const float* __restrict__ wts, int Ttok, int k,
    int nvec, int64_t rows_alloc, uint4* __restrict__ dyd, float* __restrict__ dweights) {
  const int t = row_token();
  const int lane = threadIdx.x & 63;
  if (t >= Ttok) return;
  int dst[KT];
  float w[KT], dot[KT];
#pragma unroll
  for (int j = 0; j < KT; ++j) {
    int r = j < k ? dest_row[static_cast<size_t>(t) * k + j] : -1;
    if (r >= rows_alloc) r = -1;  // not a row of the grouped buffers
    dst[j] = __builtin_amdgcn_readfirstlane(r);
    w[j] = j < k ? wts[static_cast<size_t>(t) * k + j] : 0.f;
    dot[j] = 0.f;
  }
  const uint4* dr = dy + static_cast<size_t>(t) * nvec;
  constexpr int UB = KT <= 2 ? kRowBatch : (KT <= 4 ? 2 : 1);
  for_row_batches<UB>(nvec, lane, [&](auto nb, int v) {
    combine_bwd_vecs<T, KT, decltype(nb)::value>(dr, yd, dst, w, dot, nvec, v, dyd);
  });
#pragma unroll
  for (int j = 0; j < KT; ++j) {
    if (j < k) {
      const float s = wave_sum(dot[j]);
      if (lane == 0) dweights[static_cast<size_t>(t) * k + j] = dst[j] >= 0 ? s : 0.f;
    }
  }
}

// dx[t] = sum_j kept dx_disp[r_j] on the cached path (no gate term): the
// combine with unit weights (fmaf(1, f, acc) rounds as acc + f does), summed
// in float32 in order j, one rounding, stored non-temporally.
template <typename T, int KT>
__global__ __launch_bounds__(256) void row_sum_kernel(
    const uint4* __restrict__ dxd, const int32_t* __restrict__ dest_row, int Ttok, int k,
    int nvec, int64_t rows_alloc, uint4* __restrict__ dx) {
  const int t = row_token();
  const int lane = threadIdx.x & 63;
  if (t >= Ttok) return;
  int dst[KT];
  float w[KT];
#pragma unroll
  for (int j = 0; j < KT; ++j) {
    int r = j < k ? dest_row[static_cast<size_t>(t) * k + j] : -1;
    if (r >= rows_alloc) r = -1;
    dst[j] = __builtin_amdgcn_readfirstlane(r);
    w[j] = 1.f;
  }
  uint4* o = dx + static_cast<size_t>(t) * nvec;
  constexpr int UB = KT <= 2 ? kRowBatch : (KT <= 4 ? 2 : 1);
  for_row_batches<UB>(nvec, lane, [&](auto nb, int v) {
    combine_vecs<T, KT, decltype(nb)::value, true>(dxd, dst, w, nvec, v, o);
  });
}

// dx[t] = sum_j kept dx_disp[r_j] + dl[t] . w_g.  A wavefront takes a group
// of TG tokens (k <= KT) and one 64-vector column chunk of their rows
// (blockIdx.y), so each w_g vector is loaded once per group rather than once
// per token, and issues all of the group's row gathers at once.
template <int KT> struct DispatchBwdShape {
  static constexpr int TG = KT <= 2 ? 8 : 16 / KT;   // tokens per wavefront
};

template <typename T, int KT>
__global__ __launch_bounds__(256) void dispatch_bwd_kernel(
    const uint4* __restrict__ dxd, const int32_t* __restrict__ dest_row,
    const float* __restrict__ dl, const uint4* __restrict__ wg, int Ttok, int E, int k,
    int nvec, int64_t rows_alloc, uint4* __restrict__ dx) {
  constexpr int V = Elem<T>::kVec;
  constexpr int kTokGroup = DispatchBwdShape<KT>::TG;
  constexpr int kMaxK = KT;
  // wave-uniform token group: its routing values and dlogits come in through
  // scalar loads, read once per group rather than once per row vector
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int tg = (static_cast<int>(blockIdx.x) * kRowWaves + wave) * kTokGroup;
  const int lane = threadIdx.x & 63;
  if (tg >= Ttok) return;
  int rows[kTokGroup][kMaxK];
#pragma unroll
  for (int u = 0; u < kTokGroup; ++u)
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) {
      int r = -1;
      if (j < k && tg + u < Ttok) r = dest_row[static_cast<size_t>(tg + u) * k + j];
      rows[u][j] = r >= 0 && r < rows_alloc ? r : -1;
    }
  const int v = static_cast<int>(blockIdx.y) * 64 + lane;
  if (v >= nvec) return;
  {
    float acc[kTokGroup][V];
    // issue every gather of the group before summing
    uint4 raw[kTokGroup][kMaxK];
#pragma unroll
    for (int u = 0; u < kTokGroup; ++u)
#pragma unroll
      for (int j = 0; j < kMaxK; ++j)
        if (j < k && rows[u][j] >= 0) raw[u][j] = dxd[static_cast<size_t>(rows[u][j]) * nvec + v];
#pragma unroll
    for (int u = 0; u < kTokGroup; ++u) {
#pragma unroll
      for (int i = 0; i < V; ++i) acc[u][i] = 0.f;
#pragma unroll
      for (int j = 0; j < kMaxK; ++j)
        if (j < k && rows[u][j] >= 0) {
          float f[V];
          Elem<T>::load(raw[u][j], f);
#pragma unroll
          for (int i = 0; i < V; ++i) acc[u][i] += f[i];
        }
    }
    {
      // four w_g vectors in flight per step
      constexpr int kEu = 4;
      for (int e0 = 0; e0 < E; e0 += kEu) {
        uint4 gv[kEu];
#pragma unroll
        for (int q = 0; q < kEu; ++q)
          if (e0 + q < E) gv[q] = wg[static_cast<size_t>(e0 + q) * nvec + v];
#pragma unroll
        for (int q = 0; q < kEu; ++q) {
          if (e0 + q >= E) break;
          float f[V];
          Elem<T>::load(gv[q], f);
#pragma unroll
          for (int u = 0; u < kTokGroup; ++u) {
            const int t = tg + u;
            const float g = t < Ttok ? dl[static_cast<size_t>(t) * E + e0 + q] : 0.f;
#pragma unroll
            for (int i = 0; i < V; ++i) acc[u][i] = fmaf(g, f[i], acc[u][i]);
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kTokGroup; ++u)
      if (tg + u < Ttok) store_stream(dx + static_cast<size_t>(tg + u) * nvec + v, Elem<T>::store(acc[u]));
  }
}

// The same for wide gates (E > 16) of bf16 layers, where E multiply-adds per
// element take longer than the memory traffic (T = 16384, d = 1024, E = 64, k
// = 1: 51 us, here 36 us; see wide_gate_pays): dl . w_g on bf16 matrix cores, dl as three bf16
// parts (split8).  A wavefront takes 16 tokens by 128 columns: lane l = 16 G +
// n supplies token n, experts 32 s + 8 G .. +7 of step s, and of each of those
// experts columns 8 n .. +7, which an 8 x 8 transpose in registers turns into
// the fragments of eight column blocks (block j's column n stands for column
// 8 n + j), so it ends with 8 consecutive columns of tokens 4 G + q and adds
// and stores whole vectors.  The w_g fragments stay in registers over kMmTiles
// token tiles; the column groups of a row run next to each other (one grid
// dimension: HIP allows 65,536 blocks in the others, 8.4M tokens here).
constexpr int kMmTiles = 2;

template <int KT, int KS>   // KS: steps of 32 experts
__global__ __launch_bounds__(256) void dispatch_bwd_wide_kernel(
    const uint4* __restrict__ dxd, const int32_t* __restrict__ dest_row,
    const float* __restrict__ dl, const uint4* __restrict__ wg, int Ttok, int E, int k,
    int nvec, int64_t rows_alloc, uint4* __restrict__ dx) {
  using T = uint16_t;
  constexpr int V = Elem<T>::kVec;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int n = lane & 15, G = lane >> 4;
  const int ncol = (nvec + 15) / 16;
  const int tb = static_cast<int>(blockIdx.x) / ncol;
  const int v = (static_cast<int>(blockIdx.x) - tb * ncol) * 16 + n;
  const bool colok = v < nvec;
  const int vc = min(v, nvec - 1);
  const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
  const bool vec4 = E % 4 == 0 && (reinterpret_cast<uintptr_t>(dl) & 15) == 0;
  uint4 w[KS][V];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    uint4 raw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = 32 * s + 8 * G + i;
      const uint4 x = wg[static_cast<size_t>(min(e, E - 1)) * nvec + vc];
      raw[i] = e < E ? x : zero;
    }
    transpose8(raw, w[s]);
  }
#pragma unroll 1
  for (int tile = 0; tile < kMmTiles; ++tile) {
    const int t0 = ((tb * kMmTiles + tile) * kRowWaves + wave) * 16;
    if (t0 >= Ttok) break;
    // the rows of the lane's output tokens 4 G + q: their gathers are issued
    // ahead of the MFMAs while they fit in registers
    constexpr bool kHold = KT <= 2;
    int rows[4][KT];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < KT; ++j) {
        const int t = t0 + 4 * G + q;
        const int r = dest_row[static_cast<size_t>(min(t, Ttok - 1)) * k + min(j, k - 1)];
        rows[q][j] = t < Ttok && j < k && r >= 0 && r < rows_alloc ? r : -1;
      }
    const float* dr = dl + static_cast<size_t>(min(t0 + n, Ttok - 1)) * E;
    float a[KS][8];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int e = 32 * s + 8 * G + 4 * h;
        float4 x;
        if (vec4) {
          x = *reinterpret_cast<const float4*>(dr + min(e, E - 4));
        } else {
          x = make_float4(dr[min(e, E - 1)], dr[min(e + 1, E - 1)], dr[min(e + 2, E - 1)],
                          dr[min(e + 3, E - 1)]);
        }
        a[s][4 * h] = e < E ? x.x : 0.f;
        a[s][4 * h + 1] = e + 1 < E ? x.y : 0.f;
        a[s][4 * h + 2] = e + 2 < E ? x.z : 0.f;
        a[s][4 * h + 3] = e + 3 < E ? x.w : 0.f;
      }
    // a dropped pick counts as zero
    auto row = [&](int q, int j) {
      return rows[q][j] >= 0 ? dxd[static_cast<size_t>(rows[q][j]) * nvec + vc] : zero;
    };
    uint4 held[kHold ? 4 : 1][KT];
    if constexpr (kHold) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < KT; ++j) held[q][j] = row(q, j);
    }
    floatx4 acc[V];
#pragma unroll
    for (int j = 0; j < V; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const Split8 g = split8(a[s]);
#pragma unroll
      for (int j = 0; j < V; ++j) mma_split(acc[j], g, w[s][j]);
    }
    if (any_nan(acc)) {
      // non-finite inputs: the wavefront's sums by FMAs (see split8)
#pragma unroll
      for (int j = 0; j < V; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int e = 0; e < E; ++e) {
        float f[V];
        Elem<T>::load(wg[static_cast<size_t>(e) * nvec + vc], f);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float g = dl[static_cast<size_t>(min(t0 + 4 * G + q, Ttok - 1)) * E + e];
#pragma unroll
          for (int j = 0; j < V; ++j) acc[j][q] = __builtin_fmaf(g, f[j], acc[j][q]);
        }
      }
    }
    if (!colok) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + 4 * G + q;
      if (t >= Ttok) continue;
      float o[V];
#pragma unroll
      for (int i = 0; i < V; ++i) o[i] = 0.f;
#pragma unroll
      for (int j = 0; j < KT; ++j) {
        float f[V];
        Elem<T>::load(kHold ? held[kHold ? q : 0][j] : row(q, j), f);
#pragma unroll
        for (int i = 0; i < V; ++i) o[i] += f[i];
      }
#pragma unroll
      for (int i = 0; i < V; ++i) o[i] += acc[i][q];
      store_stream(dx + static_cast<size_t>(t) * nvec + v, Elem<T>::store(o));
    }
  }
}

// Padded static baseline: zero rows [offsets[e] + fill[e], offsets[e] + rows[e])
// of a grouped buffer, rows[e] clamped to the expert's region and to
// rows_alloc exactly as the FFN schedule clamps it.  A wavefront takes one
// row; lane e tests expert e's unfilled range and a ballot decides.
constexpr int kPadRowsPerBlock = 16;

__global__ __launch_bounds__(256) void zero_pad_rows_kernel(
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ fill,
    const int32_t* __restrict__ rows, int E, int64_t rows_alloc, int nvec,
    uint4* __restrict__ buf) {
  __shared__ int64_t lo[kMaxE], hi[kMaxE];
  if (threadIdx.x < kMaxE) {
    const int e = threadIdx.x;
    int64_t a = 0, b = 0;
    if (e < E) {
      const int64_t off = offsets[e];
      int64_t m = rows[e];
      if (off < 0 || off >= rows_alloc) m = 0;
      m = min(m, static_cast<int64_t>(offsets[e + 1]) - off);
      m = min(m, rows_alloc - off);
      m = max(m, int64_t(0));
      const int64_t fl = min(max(static_cast<int64_t>(fill[e]), int64_t(0)), m);
      a = off + fl;
      b = off + m;
    }
    lo[e] = a;
    hi[e] = b;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  for (int i = wave; i < kPadRowsPerBlock; i += kRowWaves) {
    const int64_t r = static_cast<int64_t>(blockIdx.x) * kPadRowsPerBlock + i;
    if (r >= rows_alloc) break;
    const bool mine = lane < E && r >= lo[lane] && r < hi[lane];
    if (__ballot(mine) == 0) continue;
    uint4* row = buf + static_cast<size_t>(r) * nvec;
    for (int v = lane; v < nvec; v += 64) row[v] = make_uint4(0u, 0u, 0u, 0u);
  }
}

inline int nblocks(int64_t n, int per) { return static_cast<int>((n + per - 1) / per); }

}  // namespace
}  // namespace moe

using namespace moe;

extern "C" moe_status moe_count(void* stream, int T, int E, int k, const int32_t* ids,
                                int32_t* counts, int32_t* status) {
  if (!shape_ok(T, E, k) || !counts || !status) return MOE_EINVAL;
  if (T > 0 && !ids) return MOE_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  MOE_TIMED("count", s);
  fill_i32_kernel<<<1, 64, 0, s>>>(counts, E, 0);
  MOE_LAUNCH_CHECK();
  const int64_t n = static_cast<int64_t>(T) * k;
  if (n > 0) {
    count_kernel<<<nblocks(n, kChunk), 256, 0, s>>>(ids, T, E, k, counts, status);
    MOE_LAUNCH_CHECK();
  }
  return MOE_OK;
}

static bool cap_rule_ok(int T, int E, int k, int num, int den, int cap_min, int row_align) {
  if (!shape_ok(T, E, k) || num < 1 || den < 1 || cap_min < 0) return false;
  if (row_align < 1 || row_align > kMaxRowAlign) return false;
  return static_cast<int64_t>(T) * E + static_cast<int64_t>(row_align - 1) * E < (int64_t(1) << 31);
}

extern "C" moe_status moe_update_capacity(void* stream, int T, int k, int E,
                                          const int32_t* counts, int num, int den,
                                          int cap_min, int row_align, int32_t* capacity,
                                          int32_t* offsets) {
  if (!cap_rule_ok(T, E, k, num, den, cap_min, row_align) || !capacity || !offsets)
    return MOE_EINVAL;
  MOE_TIMED("capacity", static_cast<hipStream_t>(stream));
  const CapRule rule = {counts != nullptr, num, den, cap_min, row_align};
  capacity_kernel<<<1, 64, 0, static_cast<hipStream_t>(stream)>>>(T, k, E, counts, rule, capacity,
                                                                  offsets);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

static int route_nblk(int T, int k) {
  const int64_t n = static_cast<int64_t>(T) * k;
  return n > 0 ? nblocks(n, kChunk) : 1;
}

extern "C" size_t moe_dispatch_workspace_bytes(int T, int E, int k) {
  if (!shape_ok(T, E, k)) return 0;
  const size_t nblk = route_nblk(T, k);
  return align_up((2 * nblk * E + E) * sizeof(int32_t), 256);
}

static moe_status dispatch_args_ok(moe_dtype dt, int T, int d, int E, int k, const void* x,
                                   const int32_t* ids, const int32_t* capacity,
                                   const int32_t* offsets, int64_t rows_alloc,
                                   const int32_t* counts, const int32_t* fill,
                                   const int32_t* dest_row, const int32_t* src,
                                   const void* x_disp, const int32_t* status) {
  if (!dtype_ok(dt) || !shape_ok(T, E, k) || !width_ok(d) || !rows_ok(rows_alloc))
    return MOE_EINVAL;
  if (!capacity || !offsets || !counts || !fill || !status) return MOE_EINVAL;
  if (rows_alloc > 0 && (!src || !x_disp)) return MOE_EINVAL;
  if (T > 0 && (!x || !ids || !dest_row)) return MOE_EINVAL;
  if ((x && !aligned16(x)) || (x_disp && !aligned16(x_disp))) return MOE_EINVAL;
  return MOE_OK;
}

// The launches of moe_dispatch (rule null) or, with a capacity rule, of
// moe_route; `workspace` holds moe_dispatch_workspace_bytes.
static moe_status dispatch_launch(hipStream_t s, moe_dtype dt, int T, int d, int E, int k,
                                  const void* x, const int32_t* ids, const CapRule* rule,
                                  int32_t* capacity, int32_t* offsets, int64_t rows_alloc,
                                  int32_t* counts, int32_t* fill, int32_t* dest_row, int32_t* src,
                                  void* x_disp, int32_t* status, void* workspace);

extern "C" moe_status moe_dispatch(void* stream, moe_dtype dt, int T, int d, int E, int k,
                                   const void* x, const int32_t* ids,
                                   const int32_t* capacity, const int32_t* offsets,
                                   int64_t rows_alloc, int32_t* counts, int32_t* fill,
                                   int32_t* dest_row, int32_t* src, void* x_disp,
                                   int32_t* status, void* workspace, size_t workspace_bytes) {
  const moe_status st = dispatch_args_ok(dt, T, d, E, k, x, ids, capacity, offsets, rows_alloc,
                                         counts, fill, dest_row, src, x_disp, status);
  if (st != MOE_OK) return st;
  const size_t need = moe_dispatch_workspace_bytes(T, E, k);
  if (!workspace || workspace_bytes < need) return MOE_EWORKSPACE;
  return dispatch_launch(static_cast<hipStream_t>(stream), dt, T, d, E, k, x, ids, nullptr,
                         const_cast<int32_t*>(capacity), const_cast<int32_t*>(offsets), rows_alloc,
                         counts, fill, dest_row, src, x_disp, status, workspace);
}

static moe_status dispatch_launch(hipStream_t s, moe_dtype dt, int T, int d, int E, int k,
                                  const void* x, const int32_t* ids, const CapRule* rule,
                                  int32_t* capacity, int32_t* offsets, int64_t rows_alloc,
                                  int32_t* counts, int32_t* fill, int32_t* dest_row, int32_t* src,
                                  void* x_disp, int32_t* status, void* workspace) {
  const int nblk = route_nblk(T, k);
  int32_t* hist = static_cast<int32_t*>(workspace);
  int32_t* base = hist + static_cast<size_t>(nblk) * E;
  int32_t* cap_eff = base + static_cast<size_t>(nblk) * E;
  const CapRule cr = rule ? *rule : CapRule{};
  {
    MOE_TIMED("route_hist", s);
    route_hist_kernel<<<nblk, 256, 0, s>>>(ids, T, E, k, nblk, rows_alloc, hist, src, status);
    MOE_LAUNCH_CHECK();
  }
  if (nblk <= kScanChunks) {
    // the rank kernel does the scan too (and writes counts and fill)
    MOE_TIMED("route_rank", s);
    (rule ? route_rank_kernel<true, true> : route_rank_kernel<true, false>)<<<nblk, 256, 0, s>>>(
        ids, T, E, k, nullptr, nullptr, offsets, dest_row, src, hist, nblk, cr, capacity,
        rows_alloc, counts, fill, status);
    MOE_LAUNCH_CHECK();
  } else {
    {
      MOE_TIMED("route_scan", s);
      (rule ? route_scan_kernel<true> : route_scan_kernel<false>)<<<1, 64, 0, s>>>(
          hist, nblk, T, k, E, cr, capacity, offsets, rows_alloc, base, cap_eff, counts, fill,
          status);
      MOE_LAUNCH_CHECK();
    }
    MOE_TIMED("route_rank", s);
    route_rank_kernel<false, false><<<nblk, 256, 0, s>>>(
        ids, T, E, k, base, cap_eff, offsets, dest_row, src, nullptr, nblk, cr, nullptr,
        rows_alloc, nullptr, nullptr, nullptr);
    MOE_LAUNCH_CHECK();
  }
  if (T == 0) return MOE_OK;
  MOE_TIMED("dispatch_gather", s);
  const int nvec = static_cast<int>(static_cast<int64_t>(d) * esize(dt) / 16);
  gather_rows_kernel<<<nblocks(T, kRowWaves), 256, 0, s>>>(
      static_cast<const uint4*>(x), dest_row, T, k, nvec, static_cast<uint4*>(x_disp));
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

// ---- count + capacity + dispatch in one call ---------------------------------
// Tokens per chunk of the fused kernels (32 or 64), or 0 for the general path
// (chunks of kChunk assignments, a scan and a gather of their own): the
// histogram entries every workgroup sums bound the batch.  The smaller chunk
// gives the row copies more workgroups.  The two kernels against the six (fill,
// count, capacity, histogram, rank, gather): T = 8192, k = 2, E = 16, d = 512:
// 14 us against 32 us; T = 16384, k = 1, E = 64, d = 1024: 23 us against 42 us;
// T = 32, k = 2, E = 8, d = 4096 (one kernel): 5.6 us against 29 us; at the
// bound with short rows, T = 262144, k = 1, E = 2, d = 64: 54 us against 92 us,
// T = 1048576, k = 1, E = 1, d = 8: 121 us against 314 us.
static int route_chunk_tokens(int T, int E, int k) {
  for (int ct = 32; ct <= 64; ct *= 2)
    if (T > 0 && static_cast<int64_t>(nblocks(T, ct)) * k * E <= kMaxHist) return ct;
  return 0;
}

constexpr bool route_tiny(int T, int k) { return static_cast<int64_t>(T) * k <= kTinyAssign; }

// Whether the fused kernels are faster than the general path, where they are
// possible.  A chunk is copied by one workgroup, the general path's rows by a
// wavefront per token: long rows of many picks take the few workgroups of a
// short batch longer, and past the last-level cache the gather alone keeps
// more loads in flight.  Fused / general, us: T = 512, k = 8, E = 8, d = 256 20
// / 19, d = 4096 55 / 25; T = 8192, k = 1, E = 1, d = 2048 21 / 21, d = 4096 43 /
// 31; T = 32768, k = 2, E = 8, d = 1024 41 / 45, d = 2048 108 / 93.  Where the
// expert products' schedule is built on the way, the general path pays that
// kernel's launch too, about 5 us.
static bool route_fused_pays(const Route& r, int ct, bool sched) {
  const int64_t row = static_cast<int64_t>(r.d) * esize(r.dt) * (r.k + 1);   // moved per token
  const int64_t chunk = row * (route_tiny(r.T, r.k) ? 4 : ct);
  return chunk <= (sched ? 800 : 400) * 1024 &&
         (chunk <= 200 * 1024 || row * r.T <= 300 * int64_t(1000000));
}

extern "C" size_t moe_route_workspace_bytes(int T, int E, int k) {
  const size_t general = moe_dispatch_workspace_bytes(T, E, k);
  return general && route_chunk_tokens(T, E, k)
             ? std::max(general, static_cast<size_t>(kMaxHist) * sizeof(int32_t))
             : general;
}

namespace moe {

moe_status route_check(const Route& a, size_t workspace_bytes) {
  const moe_status st = dispatch_args_ok(a.dt, a.T, a.d, a.E, a.k, a.x, a.ids, a.capacity,
                                         a.offsets, a.rows_alloc, a.counts, a.fill, a.dest_row,
                                         a.src, a.x_disp, a.status);
  if (st != MOE_OK) return st;
  if (!cap_rule_ok(a.T, a.E, a.k, a.rule.num, a.rule.den, a.rule.cap_min, a.rule.align))
    return MOE_EINVAL;
  return !a.workspace || workspace_bytes < moe_route_workspace_bytes(a.T, a.E, a.k) ? MOE_EWORKSPACE
                                                                                     : MOE_OK;
}

moe_status route_launch(hipStream_t s, const Route& r, const SchedArgs* sched, bool* scheduled) {
  const int T = r.T, E = r.E, k = r.k;
  const int ct = route_chunk_tokens(T, E, k);
  const bool fused = ct && route_fused_pays(r, ct, sched != nullptr);
  if (scheduled) *scheduled = sched && fused;
  if (!fused)
    return dispatch_launch(s, r.dt, T, r.d, E, k, r.x, r.ids, &r.rule, r.capacity, r.offsets,
                           r.rows_alloc, r.counts, r.fill, r.dest_row, r.src, r.x_disp, r.status,
                           r.workspace);
  const bool tiny = route_tiny(T, k);
  const int nchunk = nblocks(T, tiny ? 4 : ct);
  int32_t* hist = nullptr;
  if (!tiny) {
    hist = static_cast<int32_t*>(r.workspace);
    MOE_TIMED("route_hist", s);
    (ct == 32 ? route_chunk_hist_kernel<32> : route_chunk_hist_kernel<64>)<<<
        nblocks(nchunk, 4), 256, 0, s>>>(r.ids, T, E, k, nchunk, hist, r.status);
    MOE_LAUNCH_CHECK();
  }
  const RouteArgs a = {static_cast<const uint4*>(r.x), r.ids, hist, T, E, k,
                       static_cast<int>(static_cast<int64_t>(r.d) * esize(r.dt) / 16), nchunk,
                       r.rule, r.rows_alloc, r.capacity, r.offsets, r.counts, r.fill, r.dest_row,
                       r.src, static_cast<uint4*>(r.x_disp), r.status,
                       sched ? *sched : SchedArgs{}};
  MOE_TIMED("dispatch_gather", s);
  (tiny ? route_fused_kernel<4> : ct == 32 ? route_fused_kernel<32> : route_fused_kernel<64>)<<<
      nchunk + (sched ? 1 : 0), 256, 0, s>>>(a);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

}  // namespace moe

extern "C" moe_status moe_route(void* stream, moe_dtype dt, int T, int d, int E, int k,
                                const void* x, const int32_t* ids, int dynamic, int num, int den,
                                int cap_min, int row_align, int64_t rows_alloc, int32_t* capacity,
                                int32_t* offsets, int32_t* counts, int32_t* fill,
                                int32_t* dest_row, int32_t* src, void* x_disp, int32_t* status,
                                void* workspace, size_t workspace_bytes) {
  const Route r = {dt, T, d, E, k, x, ids, {dynamic != 0, num, den, cap_min, row_align}, rows_alloc,
                   capacity, offsets, counts, fill, dest_row, src, x_disp, status, workspace};
  const moe_status st = route_check(r, workspace_bytes);
  return st != MOE_OK ? st : route_launch(static_cast<hipStream_t>(stream), r, nullptr, nullptr);
}

// ---- allocation-free dispatch ------------------------------------------------
// moe_dispatch_noalloc keeps the routing histograms in `scratch`, a fixed
// device array of this library, instead of a caller workspace.  Each GPU
// holds its own copy at its own address; the host looks that address up once
// per device and passes it to the kernels (the array's name in host code is
// only a host-side stand-in).  Every call on one GPU shares the array, so
// calls that overlap on one GPU race.  Nothing in it needs clearing: the
// histogram kernel writes every entry the scan and rank kernels read.
constexpr int64_t kNoAllocMaxAssignments = int64_t(1) << 21;  // T*k limit
constexpr size_t kNoAllocScratchBytes =
    (2 * static_cast<size_t>(kNoAllocMaxAssignments / kChunk) * kMaxE + kMaxE) * sizeof(int32_t);
static_assert(kNoAllocScratchBytes % 256 == 0, "scratch size is whole 256-byte blocks");

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_dev[kMaxDevices];  // device address of `scratch`, per device

// Device address of this device's `scratch` (looked up on the first call
// made with that device current).
static moe_status scratch_address(hipStream_t s, void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MOE_EHIP;
  if (s != nullptr) {
    hipDevice_t sdev = -1;
    if (hipStreamGetDevice(s, &sdev) != hipSuccess) return MOE_EHIP;
    if (sdev != dev) return MOE_EINVAL;  // the stream must belong to the current device
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_dev[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr)
      return MOE_EHIP;
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return MOE_OK;
}

extern "C" size_t moe_dispatch_noalloc_max_assignments(void) {
  return static_cast<size_t>(kNoAllocMaxAssignments);
}

extern "C" moe_status moe_dispatch_noalloc(void* stream, moe_dtype dt, int T, int d, int E,
                                           int k, const void* x, const int32_t* ids,
                                           const int32_t* capacity, const int32_t* offsets,
                                           int64_t rows_alloc, int32_t* counts, int32_t* fill,
                                           int32_t* dest_row, int32_t* src, void* x_disp,
                                           int32_t* status) {
  const moe_status st = dispatch_args_ok(dt, T, d, E, k, x, ids, capacity, offsets, rows_alloc,
                                         counts, fill, dest_row, src, x_disp, status);
  if (st != MOE_OK) return st;
  if (static_cast<int64_t>(T) * k > kNoAllocMaxAssignments ||
      moe_dispatch_workspace_bytes(T, E, k) > kNoAllocScratchBytes)
    return MOE_EWORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  void* ws = nullptr;
  const moe_status sa = scratch_address(s, &ws);
  if (sa != MOE_OK) return sa;
  return dispatch_launch(s, dt, T, d, E, k, x, ids, nullptr, const_cast<int32_t*>(capacity),
                         const_cast<int32_t*>(offsets), rows_alloc, counts, fill, dest_row, src,
                         x_disp, status, ws);
}

// Calls f with std::integral_constant<int, KT> for the smallest pick bound
// KT in {1, 2, 4, 8} with k <= KT (templated row kernels size their per-pick
// registers by KT).
template <typename F>
static void with_pick_bound(int k, F&& f) {
  if (k <= 1) f(std::integral_constant<int, 1>{});
  else if (k <= 2) f(std::integral_constant<int, 2>{});
  else if (k <= 4) f(std::integral_constant<int, 4>{});
  else f(std::integral_constant<int, 8>{});
}

extern "C" moe_status moe_combine(void* stream, moe_dtype dt, int T, int d, int k,
                                  int64_t rows_alloc, const void* y_disp,
                                  const int32_t* dest_row, const float* weights, void* y) {
  if (!dtype_ok(dt) || T < 0 || k < 1 || k > kMaxK || !width_ok(d) || !rows_ok(rows_alloc))
    return MOE_EINVAL;
  if (T == 0) return MOE_OK;
  if (!y_disp || !dest_row || !weights || !y) return MOE_EINVAL;
  if (!aligned16(y_disp) || !aligned16(y)) return MOE_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nvec = static_cast<int>(static_cast<int64_t>(d) * esize(dt) / 16);
  MOE_TIMED("combine", s);
  with_pick_bound(k, [&](auto kt_tag) {
    constexpr int KT = decltype(kt_tag)::value;
    if (dt == MOE_BF16)
      combine_kernel<uint16_t, KT><<<nblocks(T, kRowWaves), 256, 0, s>>>(
          static_cast<const uint4*>(y_disp), dest_row, weights, T, k, nvec, rows_alloc,
          static_cast<uint4*>(y));
    else
      combine_kernel<float, KT><<<nblocks(T, kRowWaves), 256, 0, s>>>(
          static_cast<const uint4*>(y_disp), dest_row, weights, T, k, nvec, rows_alloc,
          static_cast<uint4*>(y));
  });
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

extern "C" moe_status moe_combine_bwd(void* stream, moe_dtype dt, int T, int d, int k,
                                      int64_t rows_alloc, const void* dy, const void* y_disp,
                                      const int32_t* dest_row, const float* weights,
                                      void* dy_disp, float* dweights) {
  if (!dtype_ok(dt) || T < 0 || k < 1 || k > kMaxK || !width_ok(d) || !rows_ok(rows_alloc))
    return MOE_EINVAL;
  if (T == 0) return MOE_OK;
  if (!dy || !y_disp || !dest_row || !weights || !dy_disp || !dweights) return MOE_EINVAL;
  if (!aligned16(dy) || !aligned16(y_disp) || !aligned16(dy_disp)) return MOE_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nvec = static_cast<int>(static_cast<int64_t>(d) * esize(dt) / 16);
  MOE_TIMED("combine_bwd", s);
  with_pick_bound(k, [&](auto kt_tag) {
    constexpr int KT = decltype(kt_tag)::value;
    if (dt == MOE_BF16)
      combine_bwd_kernel<uint16_t, KT><<<nblocks(T, kRowWaves), 256, 0, s>>>(
          static_cast<const uint4*>(dy), static_cast<const uint4*>(y_disp), dest_row, weights,
          T, k, nvec, rows_alloc, static_cast<uint4*>(dy_disp), dweights);
    else
      combine_bwd_kernel<float, KT><<<nblocks(T, kRowWaves), 256, 0, s>>>(
          static_cast<const uint4*>(dy), static_cast<const uint4*>(y_disp), dest_row, weights,
          T, k, nvec, rows_alloc, static_cast<uint4*>(dy_disp), dweights);
  });
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

// Whether dispatch_bwd_wide_kernel is the faster one (bf16, E > 16).  It has
// the multiply-adds on matrix cores but takes 256 bytes of a row at a time
// where the other takes 1 KB, so it moves rows at 3.6 to 4 TB/s against 4.9
// (2.7 against 4.4 where its gathers no longer fit in registers, k > 2).  A
// multiply-add costs the other about 1/22 ps, more where the last 64 vectors
// of a row are partly filled, and a row element moved 0.4 ps: the line lies at
// about 10 experts per row moved (13 past the last-level cache), 20 with a
// second step of 32 experts, 17 for k > 2.  Below 16 MB both wait on
// latencies, the other on E of them in series.
// Other / wide kernel, us: T = 65536, d = 1024: E = 17, k = 2 75 / 100, E = 24,
// k = 1 74 / 77, E = 32, k = 1 89 / 78, E = 64, k = 2 165 / 137, k = 3 179 /
// 209; T = 8192, d = 2048, E = 32, k = 2 32 / 24; T = 65536, d = 64, E = 17, k =
// 2 32 / 11; T = 2000, d = 64, E = 20: k = 2 18 / 7.9, k = 8 9.7 / 14; T =
// 2000, d = 1000, E = 24, k = 3 9.8 / 13.
static bool wide_gate_pays(int T, int d, int E, int k) {
  constexpr int64_t MB = 1 << 20;
  const int64_t bytes = static_cast<int64_t>(T) * d * 2 * (k + 1);
  if (bytes < 16 * MB) return k <= 2 || (k <= 4 && bytes < 4 * MB);
  const int64_t nvec = d / 8, lanes = (nvec + 63) / 64 * 64;
  const int per_row = k > 2 ? 17 : E > 32 ? 20 : bytes >= 256 * MB ? 13 : 10;
  return E * lanes > per_row * (k + 1) * nvec;
}

extern "C" moe_status moe_dispatch_bwd(void* stream, moe_dtype dt, int T, int d, int E, int k,
                                       int64_t rows_alloc, const void* dx_disp,
                                       const int32_t* dest_row, const float* dlogits,
                                       const void* w_g, void* dx) {
  if (!dtype_ok(dt) || !shape_ok(T, E, k) || !width_ok(d) || !rows_ok(rows_alloc))
    return MOE_EINVAL;
  if (T == 0) return MOE_OK;
  if (!dx_disp || !dest_row || !dx) return MOE_EINVAL;
  if ((dlogits == nullptr) != (w_g == nullptr)) return MOE_EINVAL;
  if (!aligned16(dx_disp) || !aligned16(dx) || (w_g && !aligned16(w_g))) return MOE_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nvec = static_cast<int>(static_cast<int64_t>(d) * esize(dt) / 16);
  const uint4* a = static_cast<const uint4*>(dx_disp);
  const uint4* g = static_cast<const uint4*>(w_g);
  uint4* o = static_cast<uint4*>(dx);
  MOE_TIMED("dispatch_bwd", s);
  if (!dlogits) {
    with_pick_bound(k, [&](auto kt_tag) {
      constexpr int KT = decltype(kt_tag)::value;
      if (dt == MOE_BF16)
        row_sum_kernel<uint16_t, KT><<<nblocks(T, kRowWaves), 256, 0, s>>>(a, dest_row, T, k,
                                                                          nvec, rows_alloc, o);
      else
        row_sum_kernel<float, KT><<<nblocks(T, kRowWaves), 256, 0, s>>>(a, dest_row, T, k,
                                                                       nvec, rows_alloc, o);
    });
    MOE_LAUNCH_CHECK();
    return MOE_OK;
  }
  if (dt == MOE_BF16 && E > 16 && wide_gate_pays(T, d, E, k)) {
    const int grid = nblocks(nvec, 16) * nblocks(T, kRowWaves * kMmTiles * 16);
    with_pick_bound(k, [&](auto kt_tag) {
      constexpr int KT = decltype(kt_tag)::value;
      (E <= 32 ? dispatch_bwd_wide_kernel<KT, 1> : dispatch_bwd_wide_kernel<KT, 2>)<<<grid, 256, 0, s>>>(
          a, dest_row, dlogits, g, T, E, k, nvec, rows_alloc, o);
    });
    MOE_LAUNCH_CHECK();
    return MOE_OK;
  }
  auto go = [&](auto kt_tag) {
    constexpr int KT = decltype(kt_tag)::value;
    const dim3 grid(nblocks(T, kRowWaves * DispatchBwdShape<KT>::TG), nblocks(nvec, 64));
    if (dt == MOE_BF16)
      dispatch_bwd_kernel<uint16_t, KT><<<grid, 256, 0, s>>>(a, dest_row, dlogits, g, T, E, k, nvec, rows_alloc, o);
    else
      dispatch_bwd_kernel<float, KT><<<grid, 256, 0, s>>>(a, dest_row, dlogits, g, T, E, k, nvec, rows_alloc, o);
  };
  with_pick_bound(k, go);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

extern "C" moe_status moe_zero_pad_rows(void* stream, moe_dtype dt, int E, int d,
                                        const int32_t* offsets, const int32_t* fill,
                                        const int32_t* rows, int64_t rows_alloc, void* buf) {
  if (!dtype_ok(dt) || E < 1 || E > kMaxE || !width_ok(d) || !rows_ok(rows_alloc))
    return MOE_EINVAL;
  if (rows_alloc == 0) return MOE_OK;
  if (!offsets || !fill || !rows || !buf || !aligned16(buf)) return MOE_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nvec = static_cast<int>(static_cast<int64_t>(d) * esize(dt) / 16);
  MOE_TIMED("zero_pad_rows", s);
  zero_pad_rows_kernel<<<nblocks(rows_alloc, kPadRowsPerBlock), 256, 0, s>>>(
      offsets, fill, rows, E, rows_alloc, nvec, static_cast<uint4*>(buf));
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}
