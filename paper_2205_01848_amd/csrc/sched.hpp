// The tile schedule of the expert products: built on the device from the rows
// of every expert, by a kernel of its own (ffn.hip) or by one workgroup of
// the fused routing kernel (route.hip), and read by the GEMM kernels.
#pragma once

#include "common.hpp"
#include "tiles.hpp"
#include "validate.hpp"

namespace moe {

constexpr int kSplitFloor = 512;  // smallest K chunk of a split dW product
constexpr int kKc = 64;           // split chunks are multiples of this many rows
constexpr int kSplitItems = 256;  // work items the split aims at: one 256x256 tile per CU

// Device-side schedule written by schedule_kernel.
struct Sched {
  int n_mtiles;    // (expert, m0) tiles of BM rows
  int n_mid[2];    // tiles of the two-workgroups-per-CU kernel, per list
  int n_segs;      // (expert, k range) segments of the dW products
  int n_slots;     // partial-sum slots used
  int rows[kMaxE];    // clamped rows per expert
  int slot0[kMaxE];   // first partial slot of expert e (split experts)
  int nsplit[kMaxE];  // K segments of expert e (0: no rows, its gradients are zero)
};

// Inclusive prefix sum over the 64 lanes of a wavefront.
__device__ __forceinline__ int wave_incl_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  return v;
}

// ceil(v / unit); v may lie just below 2^31
__device__ __forceinline__ int ceil_units(int v, int unit) {
  return static_cast<int>((static_cast<uint32_t>(v) + unit - 1) / unit);
}

// Entry of a mid tile list: tile i of the n tiles an expert's `rows` rows are
// spread over: x = expert | height in units << 8, y = first row.
__device__ __forceinline__ int2 mid_tile(int rows, int n, int i, int e) {
  const int units = ceil_units(rows, kMidUnit);
  const int h = units / n, more = units - h * n;
  return make_int2(e | ((h + (i < more ? 1 : 0)) << 8), (i * h + min(i, more)) * kMidUnit);
}

// First index g < E whose inclusive prefix exceeds t.
__device__ __forceinline__ int find_expert(const int* incl, int E, int t) {
  int lo = 0, hi = E - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (incl[mid] > t) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

struct SchedArgs {
  int E;
  int64_t rows_alloc;
  int max_mtiles, max_mid, max_segs, tmn_min, max_slots;
  int nt[2], steps[2];   // column tiles and K steps of the products of the two mid lists
  int slots_mid;         // workgroups of the mid kernel's persistent grid
  StepCost cost[2];      // of the two mid lists' products
  Sched* s;              // outputs: the schedule and its lists
  int2 *mtile, *mtile_mid;
  int4* seg;
};
constexpr int kSchedTasks = kMidMaxH + 2;

// Writes the schedule of m rows of expert g in lane g of every one of WAVES
// wavefronts (a whole workgroup; rows clamped to their regions).  The
// wavefronts number the experts' tiles and segments in expert order by prefix
// sums, one list per task, and then all threads write the lists, each entry
// finding its expert by bisection.
//  * mtile: 256-row tiles (task kMidMaxH).  mtile_mid[i], i = 0, 1 (the
//    products with N = f and with N = d columns): the tiles of the
//    two-workgroups-per-CU kernel.  Its rounds on the persistent grid decide
//    their height: for each largest height h (task h - 1) the experts
//    need ceil(units / h) tiles of at most h units, and the h whose rounds
//    take the least time wins, so a few rows more than a whole number of
//    tiles make tiles a little higher rather than one more round of tiles.
//    An expert's units are spread evenly over its tiles.
//  * the weight-gradient products (last task) split an expert's rows
//    into K segments only when few experts carry most rows: an expert's rows
//    over the share of all 256x256 tile work that one of kSplitItems CUs
//    would get, rounded, is its number of segments.  A segment costs the
//    write and the read of its partial sums: 8 experts of 2048 rows, 1024 x
//    2816 and 5632 x 1024 gradients, took 154 + 77 and 264 + 77 us (products
//    + reductions) in two segments each, 123 and 212 us in one; 15,650 of
//    16,384 rows in one of 64 experts, 4096 x 1024, 343 + 54 us in eight
//    segments, 325 + 29 us in four.  Experts without rows get no segment:
//    split_reduce_kernel writes their zeros.
// Should a list be longer than the workspace has room for (inconsistent
// offsets), one thread walks the experts in order and cuts the lists there.
template <int WAVES>
__device__ __forceinline__ void build_schedule(int m, const SchedArgs& A) {
  Sched* const s = A.s;
  int2 *const mtile = A.mtile, *const mtile_mid = A.mtile_mid;
  int4* const seg = A.seg;
  __shared__ int ti[kMaxE], si[kMaxE], mid_incl[kMidMaxH][kMaxE], rw[kMaxE], q0s[kMaxE];
  __shared__ int64_t cost[2][kMidMaxH];
  __shared__ int fit_rows, fit_segs;
  const int E = A.E;
  const int g = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  for (int task = wave; task < kSchedTasks; task += WAVES) {
    if (task < kMidMaxH) {
      const int h = task + 1;
      const int units = ceil_units(m, kMidUnit);
      const int n = (units + h - 1) / h;
      int hm = n ? (units + n - 1) / n : 0;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) hm = max(hm, __shfl_xor(hm, o, 64));
      const int incl = wave_incl_scan(n);
      const int tot = __shfl(incl, 63, 64);
      mid_incl[task][g] = incl;
      if (g < 2)
        cost[g][task] = mid_time(static_cast<int64_t>(tot) * A.nt[g], hm, A.slots_mid, A.steps[g], A.cost[g]);
    } else if (task == kMidMaxH) {
      ti[g] = wave_incl_scan(ceil_units(m, BM));
      rw[g] = m;
      // the rows of consistent regions add up to at most rows_alloc; then no
      // 32-bit sum here overflows
      int64_t sum = m;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
      if (g == 0) fit_rows = sum <= A.rows_alloc;
    } else {
      const int64_t kw = (static_cast<int64_t>(m) + kKc - 1) / kKc * kKc;
      int64_t kwork = kw;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) kwork += __shfl_xor(kwork, o, 64);
      const int64_t kc = (kwork * A.tmn_min + kSplitItems - 1) / kSplitItems;
      const int kci = static_cast<int>(min(max(kc, static_cast<int64_t>(kSplitFloor)),
                                           static_cast<int64_t>(1 << 29)));
      const int q = m / kci;
      const int nsp = m > 0 ? max(1, q + (2 * (m - q * kci) >= kci ? 1 : 0)) : 0;
      const int segs_incl = wave_incl_scan(nsp);
      const int slots_incl = wave_incl_scan(nsp > 1 ? nsp : 0);
      const int slots_total = __shfl(slots_incl, 63, 64);
      si[g] = segs_incl;
      q0s[g] = nsp > 1 ? slots_incl - nsp : -1;
      if (g == 63) {
        fit_segs = segs_incl <= A.max_segs && slots_total <= A.max_slots;
        s->n_slots = slots_total;
      }
    }
  }
  __syncthreads();
  // the heights: the least time, the larger height on a tie
  int best[2];
#pragma unroll
  for (int l = 0; l < 2; ++l) {
    best[l] = 0;
#pragma unroll
    for (int h = 1; h < kMidMaxH; ++h)
      if (cost[l][h] <= cost[l][best[l]]) best[l] = h;
  }
  const int* mi2[2] = {mid_incl[best[0]], mid_incl[best[1]]};
  const bool fits = fit_rows && fit_segs && ti[E - 1] <= A.max_mtiles &&
                    mi2[0][E - 1] <= A.max_mid && mi2[1][E - 1] <= A.max_mid;
  const int max_mid = A.max_mid;
  const int tid = threadIdx.x, nthreads = 64 * WAVES;
  if (fits) {
    if (tid < E) {
      s->rows[tid] = rw[tid];
      s->nsplit[tid] = si[tid] - (tid ? si[tid - 1] : 0);
      s->slot0[tid] = q0s[tid];
    }
    if (tid == 0) {
      s->n_mtiles = ti[E - 1];
      s->n_mid[0] = mi2[0][E - 1];
      s->n_mid[1] = mi2[1][E - 1];
      s->n_segs = si[E - 1];
    }
    for (int t = tid; t < ti[E - 1]; t += nthreads) {
      const int e = find_expert(ti, E, t);
      mtile[t] = make_int2(e, (t - (e ? ti[e - 1] : 0)) * BM);
    }
#pragma unroll
    for (int l = 0; l < 2; ++l)
      for (int t = tid; t < mi2[l][E - 1]; t += nthreads) {
        const int e = find_expert(mi2[l], E, t);
        const int first = e ? mi2[l][e - 1] : 0;
        mtile_mid[l * max_mid + t] = mid_tile(rw[e], mi2[l][e] - first, t - first, e);
      }
    for (int t = tid; t < si[E - 1]; t += nthreads) {
      const int e = find_expert(si, E, t);
      const int first = e ? si[e - 1] : 0, n = si[e] - first, i = t - first;
      // equal segments, in whole K steps; the last ones may be short or empty
      const int64_t len = static_cast<int64_t>(ceil_units(ceil_units(rw[e], n), kKc)) * kKc;
      const int64_t me = rw[e];
      seg[t] = make_int4(e, static_cast<int>(min(i * len, me)),
                         n > 1 ? static_cast<int>(min((i + 1) * len, me)) : rw[e],
                         n > 1 ? q0s[e] + i : -1);
    }
  }
  if (fits || tid != 0) return;
  int nm = 0, nmid = 0;
  int64_t kwork_c = 0;
  for (int e = 0; e < E; ++e) {
    int64_t me = rw[e];
    me = min(me, static_cast<int64_t>(A.max_mtiles - nm) * BM);
    me = min(me, static_cast<int64_t>(max_mid - nmid) * kMidMaxH * kMidUnit);
    const int mi = static_cast<int>(me);
    s->rows[e] = mi;
    for (int m0 = 0; m0 < mi; m0 += BM) mtile[nm++] = make_int2(e, m0);
    const int n = ceil_units(mi, kMidMaxH * kMidUnit);
    for (int i = 0; i < n; ++i, ++nmid)
      mtile_mid[nmid] = mtile_mid[max_mid + nmid] = mid_tile(mi, n, i, e);
    kwork_c += static_cast<int64_t>(ceil_units(mi, kKc)) * kKc;
  }
  s->n_mtiles = nm;
  s->n_mid[0] = s->n_mid[1] = nmid;
  int64_t kcc = (kwork_c * A.tmn_min + kSplitItems - 1) / kSplitItems;
  kcc = (kcc + kKc - 1) / kKc * kKc;
  kcc = max(kcc, static_cast<int64_t>(kSplitFloor));
  int ns = 0, slots = 0;
  for (int e = 0; e < E; ++e) {
    const int kp = s->rows[e];
    int ne = kp > kcc ? static_cast<int>((kp + kcc - 1) / kcc) : (kp > 0 ? 1 : 0);
    if (ne > 1 && (slots + ne > A.max_slots || ns + ne > A.max_segs)) ne = 1;
    if (ns + ne > A.max_segs) ne = 0;
    s->nsplit[e] = ne;
    s->slot0[e] = ne > 1 ? slots : -1;
    for (int i = 0; i < ne; ++i) {
      const int k0 = static_cast<int>(min(static_cast<int64_t>(i) * kcc, static_cast<int64_t>(kp)));
      const int k1 = static_cast<int>(min(static_cast<int64_t>(i + 1) * kcc, static_cast<int64_t>(kp)));
      seg[ns++] = make_int4(e, ne > 1 ? k0 : 0, ne > 1 ? k1 : kp, ne > 1 ? slots + i : -1);
    }
    if (ne > 1) slots += ne;
  }
  s->n_segs = ns;
  s->n_slots = slots;
}

}  // namespace moe
