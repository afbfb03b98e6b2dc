// Tile shapes of the expert products and the times they are chosen by.  Plain
// C++: the host picks the kernel of a bf16 product, the device schedule the
// heights of the two-workgroups-per-CU tiles, both from mid_time.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define MOE_HD __host__ __device__
#else
#define MOE_HD
#endif

namespace moe {

constexpr int BM = 256;                           // 256x256 tiles
constexpr int BN = 256;
// Tiles of the two-workgroups-per-CU kernels: kMidN columns, and 1 to
// kMidMaxH units of kMidUnit rows, chosen per tile.
constexpr int kMidUnit = 32;
constexpr int kMidMaxH = 6;
constexpr int kMidN = 128;
constexpr int kMidDwH = 4;      // its units in the bf16 weight-gradient products

// Time (ns) of the two-workgroups-per-CU kernel on `tiles` tiles of at most h
// units of rows and `steps` K steps each: rounds of `slots` tiles, each as
// long as its K steps and its prologue and epilogue, which the other
// workgroup of the CU overlaps in part.  A K step takes the longer of
//  * its MFMAs, operand reads and waits: 0.87 us at h = 4 and 1.21 us at h = 6
//    for both workgroups of a CU with operands in the caches, about a tenth
//    more in a layer (1024- to 8192-row products, K = 512 .. 8192); fp32 (K
//    steps of 32): the 16 h MFMAs of a step and wave, 64 cycles each;
//  * the cache lines its loads touch, about 640 per us and CU: a row's 128
//    bytes are one line where the row pitch is a multiple of 128 bytes and up
//    to two elsewhere (152,000 rows, K = 12064, N = 536: 2.0 us per step at h = 6,
//    the product 3276 us against 2356 us on 256x256 tiles, which touch 0.6
//    times as many lines per MFMA).
// A round of K = 512 at h = 4 takes 3.2 us more than its 8 steps.  A last round
// that leaves at least one of the two places of every CU empty takes about
// 0.65 of a full one.
struct StepCost {
  int fixed, per_unit;               // ns per K step, ns per K step and unit of rows
  int lines_fixed, lines_per_unit;   // the same for the cache lines
};
constexpr StepCost kStepF32 = {60, 890, 0, 0};
MOE_HD inline int64_t mid_time(int64_t tiles, int h, int slots, int steps, const StepCost& c) {
  const int64_t full = tiles / slots, rem = tiles - full * slots;
  const int a = c.fixed + c.per_unit * h, b = c.lines_fixed + c.lines_per_unit * h;
  return (20 * full + (rem == 0 ? 0 : 2 * rem <= slots ? 13 : 20)) *
         (static_cast<int64_t>(steps) * (a > b ? a : b) + 3200) / 20;
}

// Cache lines per 128-byte row segment, in sixteenths, of rows `pitch` bytes
// apart: 1 where every segment starts on a line, else 2 for all but those
// that do.
inline int lines16(int64_t pitch) {
  const int64_t g = pitch & -pitch;   // largest power of two in the pitch
  return g >= 128 ? 16 : 32 - static_cast<int>(g / 8);
}

// bf16 K step of the two-workgroups-per-CU kernel (both workgroups): A rows
// pa bytes apart, B K-contiguous with rows pb apart or K-major (64 k-rows of
// 256 bytes: 2 lines, or up to 3).
inline StepCost step16(int64_t pa, int64_t pb, bool b_km) {
  // 2 x 32 x lines16 / 16 lines a unit, 1000 / 640 ns a line
  return {210, 185, b_km ? (pb % 128 ? 600 : 400) : 25 * lines16(pb), 100 * lines16(pa) / 16};
}

// And of the 256x256 kernel, ns; few: at most half the CUs have a tile.
inline int big_step16(int64_t pa, int64_t pb, bool b_km, bool few) {
  if (few) return b_km ? 1400 : 1200;
  const int lines = 16 * lines16(pa) + (b_km ? (pb % 128 ? 320 : 256) : 16 * lines16(pb));
  const int t = lines * 25 / 16, least = b_km ? 1700 : 1400;
  return t > least ? t : least;
}

// One bf16 product of the forward or the data gradients (var-M).
struct VarM {
  int E;
  int64_t rows_alloc;
  int64_t rows;        // at most this many of them hold a token (rows_alloc if not known)
  int N, K;
  bool gated;          // W1 and W3 share a tile
  bool act;            // an activation or its derivative in the epilogue
  bool b_km;           // weights read K-major
  int64_t pa, pb;      // row pitches, bytes
};

// Whether the two-workgroups-per-CU kernel is the faster one on `cus` CUs.
// Its smaller tiles leave fewer CUs idle in the last round and overlap one
// tile's prologue and epilogue with the other's MFMAs, but read more operand
// bytes per flop.  The host knows N, K and the rows at most, not the rows per
// expert, so it takes every expert to hold rows / E rows and half a
// tile's raggedness (but no fewer tiles than experts that can hold a row), and
// compares the two kernels' estimated times: rounds of 256x256 tiles, each its
// K steps and 10 us of prologue and epilogue, 13 with an activation, against
// the least mid_time over the heights.  That estimate counts 0.8 where the
// 256x256 tiles are one round and a tenth more for every round up to six: the
// smaller tiles' operand bytes tell once their panels no longer stay in the
// caches.  A budget of whole 256-row tiles per expert is read as a static
// capacity of that size, filled, where the rows can fill it: no raggedness,
// and a factor from 1 to 1.18.  The layer
// forward passes its number of picks: a static capacity of twice that counts
// as half filled and ragged (8 experts of 1024 rows, 1024 -> 4096: 75 / 41 us;
// over 236 such products 1.005 of the better kernel's time, against 1.16 with
// the capacity read as filled).
// Fitted on 2900 products (1 to 64 experts of 1 to 20,000 rows, d and f from
// 64 to 14336): the choice takes 0.6 % more than the better kernel on average;
// with 6/5 throughout, 1400 ns a K-major step, raggedness always and the tiles
// of all experts together rounded down it took 6.7 % more (1 expert of 86 rows,
// 2048 -> 512 51 us on 256x256 tiles, 13 on the smaller).  Whole products,
// 256x256 / smaller tiles, us: 4 experts of 2210 rows, 5000 -> 536 134 / 74; 4
// of 4073, K-major 4096 -> 4096 592 / 510; 32 of 512 exactly, 4096 -> 1024 117
// / 162; 8 of 16,000, 4096 -> 2 x 14336 23598 / 40342; 32 of about 2048, 8192
// -> 2048 1809 / 2064, K-major 2048 -> 8192 2342 / 2547.
inline bool mid_pays(const VarM& p, int cus) {
  auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int steps = static_cast<int>(cdiv(p.K, 64));
  const int64_t per = cdiv(p.rows, p.E);
  const bool whole = p.rows == p.rows_alloc && p.rows % (static_cast<int64_t>(BM) * p.E) == 0;
  int64_t m = whole ? p.rows / BM : p.E * (2 * per + BM) / (2 * BM);
  const int64_t least = p.rows < p.E ? p.rows : p.E;
  if (m < least) m = least;
  const int64_t big = m * cdiv(p.N, p.gated ? BN / 2 : BN);
  const int64_t rounds = cdiv(big, cus);
  const int64_t t_big = rounds * (static_cast<int64_t>(big_step16(p.pa, p.pb, p.b_km, 2 * big <= cus)) * steps +
                                  (p.act ? 13000 : 10000));
  const StepCost c = step16(p.pa, p.pb, p.b_km);
  int64_t t_mid = 0;
  for (int h = 1; h <= kMidMaxH; ++h) {
    const int64_t n = cdiv(2 * per + (whole ? 0 : kMidUnit), 2 * kMidUnit * h);
    const int64_t t = mid_time(n * p.E * cdiv(p.N, p.gated ? kMidN / 2 : kMidN), h, 2 * cus, steps, c);
    if (h == 1 || t < t_mid) t_mid = t;
  }
  const int64_t r = rounds < 6 ? rounds : 6;
  return (whole ? 47 + 3 * r : 35 + 5 * r) * t_mid < 50 * t_big;
}

}  // namespace moe
