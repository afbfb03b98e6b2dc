// Shared device helpers of libmoe (gfx950 / CDNA4 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "../../include/moe.h"

namespace moe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

// Compute units of the current device (cached per device; 256 if unknown).
inline int num_cus() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cache[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cache[dev] = n;
  }
  return cache[dev];
}

// bf16 bit pattern -> float (exact)
__device__ __forceinline__ float bf2f(uint16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}

// float -> bf16 bit pattern, round to nearest even (hardware v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t f2bf(float f) {
  __bf16 b = static_cast<__bf16>(f);
  return __builtin_bit_cast(uint16_t, b);
}

// two floats -> packed bf16x2 (lo in bits 0..15)
__device__ __forceinline__ uint32_t pack2bf(float lo, float hi) {
  bf16x2 v;
  v.x = static_cast<__bf16>(lo);
  v.y = static_cast<__bf16>(hi);
  return __builtin_bit_cast(uint32_t, v);
}

// 16 bytes = 8 bf16 <-> 8 floats
__device__ __forceinline__ void unpack8(const uint4& v, float* f) {
  f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xFFFF0000u);
  f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xFFFF0000u);
  f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xFFFF0000u);
  f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xFFFF0000u);
}
__device__ __forceinline__ uint4 pack8(const float* f) {
  uint4 v;
  v.x = pack2bf(f[0], f[1]); v.y = pack2bf(f[2], f[3]);
  v.z = pack2bf(f[4], f[5]); v.w = pack2bf(f[6], f[7]);
  return v;
}

// Element traits: the kernels move 16-byte vectors, 8 bf16 or 4 fp32 values.
template <typename T> struct Elem;
template <> struct Elem<uint16_t> {
  static constexpr int kVec = 8;  // elements per 16 bytes
  __device__ static __forceinline__ void load(const uint4& v, float* f) { unpack8(v, f); }
  __device__ static __forceinline__ uint4 store(const float* f) { return pack8(f); }
  __device__ static __forceinline__ float to_f(uint16_t h) { return bf2f(h); }
  __device__ static __forceinline__ uint16_t from_f(float x) { return f2bf(x); }
};
template <> struct Elem<float> {
  static constexpr int kVec = 4;
  __device__ static __forceinline__ void load(const uint4& v, float* f) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y);
    f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
  }
  __device__ static __forceinline__ uint4 store(const float* f) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]),
                      __float_as_uint(f[2]), __float_as_uint(f[3]));
  }
  __device__ static __forceinline__ float to_f(float x) { return x; }
  __device__ static __forceinline__ float from_f(float x) { return x; }
};

// Wave-wide sums (64 lanes) via cross-lane shuffles.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ---- fp32 x bf16 products on bf16 matrix cores --------------------------------
// A float is the sum of three bf16 values (its top 8 significant bits, the
// next 8, the last 8: each the truncation of what the ones before leave), so
// a product with a bf16 value is the sum of three exact bf16 products, and
// three bf16 MFMAs with fp32 sums give what fp32 FMAs give, at 16 / 3 times
// the rate of fp32 MFMAs.  An infinity keeps to the first part.  An infinity
// on the bf16 side meets parts that are zero (those of 0.5, say), and 0 x inf
// is NaN where the FMA gives inf: callers look for NaNs among their sums and form
// those again with FMAs.
struct Split8 {
  uint4 part[3];   // 8 values each, packed bf16
};
__device__ __forceinline__ uint32_t high_halves(uint32_t lo, uint32_t hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}
__device__ __forceinline__ uint32_t low_halves(uint32_t lo, uint32_t hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
__device__ __forceinline__ Split8 split8(const float (&g)[8]) {
  Split8 o;
  uint32_t* const p[3] = {&o.part[0].x, &o.part[1].x, &o.part[2].x};
  uint32_t h[8], m[8], l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    h[i] = __float_as_uint(g[i]);
    const float r1 = __builtin_isinf(g[i]) ? 0.f : g[i] - __uint_as_float(h[i] & 0xFFFF0000u);
    m[i] = __float_as_uint(r1);
    l[i] = __float_as_uint(r1 - __uint_as_float(m[i] & 0xFFFF0000u));
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[0][i] = high_halves(h[2 * i], h[2 * i + 1]);
    p[1][i] = high_halves(m[2 * i], m[2 * i + 1]);
    p[2][i] = high_halves(l[2 * i], l[2 * i + 1]);
  }
  return o;
}
// 8 x 8 transpose: out[j] = element j of each of the 8 rows (bf16).
__device__ __forceinline__ void transpose8(const uint4 (&in)[8], uint4 (&out)[8]) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    uint32_t d[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) d[i] = c == 0 ? in[i].x : c == 1 ? in[i].y : c == 2 ? in[i].z : in[i].w;
    out[2 * c] = make_uint4(low_halves(d[0], d[1]), low_halves(d[2], d[3]),
                            low_halves(d[4], d[5]), low_halves(d[6], d[7]));
    out[2 * c + 1] = make_uint4(high_halves(d[0], d[1]), high_halves(d[2], d[3]),
                                high_halves(d[4], d[5]), high_halves(d[6], d[7]));
  }
}
// c += a * b over 32 k: lane l = 16 G + n holds row (column) n at k = 8 G .. +7
__device__ __forceinline__ void mma_split(floatx4& c, const Split8& a, const uint4& b) {
  const bf16x8 bv = __builtin_bit_cast(bf16x8, b);
#pragma unroll
  for (int i = 2; i >= 0; --i)
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.part[i]), bv, c, 0, 0, 0);
}
// Whether one of the wavefront's sums is NaN.
template <int N> __device__ __forceinline__ bool any_nan(const floatx4 (&c)[N]) {
  bool bad = false;
#pragma unroll
  for (int j = 0; j < N; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) bad |= c[j][q] != c[j][q];
  return __any(bad);
}

// Eight lanes (8i .. 8i+7 of a wavefront) share one token's experts: lane
// `sub` of them holds experts sub, sub + 8, .., at most kGroupE of them.  A
// thread per token evaluates up to 64 exponentials in series; the group takes
// an eighth of them each and adds them in expert order, as a thread per token
// does.  Every kernel that evaluates the gate's softmax uses that order, so
// the same logits give the same probabilities bit for bit everywhere.
constexpr int kGroupE = 8;
__device__ __forceinline__ float group8_sum(float v) {
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float group8_max(float v) {
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
// The value of the group's lane J, in all its lanes (row_newbcast copies one
// lane to its row of 16, a group being half a row: two bank masks).
template <int J> __device__ __forceinline__ float group8_lane(float v) {
  const int x = __float_as_int(v);
  const int lo = __builtin_amdgcn_update_dpp(x, x, 0x150 + J, 0xF, 0x3, false);
  return __int_as_float(__builtin_amdgcn_update_dpp(lo, x, 0x158 + J, 0xF, 0xC, false));
}
// f(integral_constant J) for the group's lanes J = 0 .. 7 in order
template <typename F> __device__ __forceinline__ void for_group8(F&& f) {
  f(std::integral_constant<int, 0>{}); f(std::integral_constant<int, 1>{});
  f(std::integral_constant<int, 2>{}); f(std::integral_constant<int, 3>{});
  f(std::integral_constant<int, 4>{}); f(std::integral_constant<int, 5>{});
  f(std::integral_constant<int, 6>{}); f(std::integral_constant<int, 7>{});
}
// z[i] = exp(l[sub + 8 i] - m) (0 past E), m the largest logit, s the sum of
// all z in expert order.
__device__ __forceinline__ void group8_softmax(const float* l, int E, int sub, float (&z)[kGroupE],
                                               float& m, float& s) {
  m = -INFINITY;
#pragma unroll
  for (int i = 0; i < kGroupE; ++i) {
    const int e = sub + 8 * i;
    z[i] = e < E ? l[e] : -INFINITY;
    m = fmaxf(m, z[i]);
  }
  m = group8_max(m);
  s = 0.f;
#pragma unroll
  for (int i = 0; i < kGroupE; ++i) {
    if (8 * i >= E) {
      z[i] = 0.f;
      continue;
    }
    z[i] = sub + 8 * i < E ? expf(z[i] - m) : 0.f;
    for_group8([&](auto j) { s += group8_lane<decltype(j)::value>(z[i]); });
  }
}

__device__ __forceinline__ int ceil_div_i(int a, int b) { return (a + b - 1) / b; }

// ---- opt-in kernel timing (moe_timing_enable / moe_timing_report) ---------
// While enabled, each library kernel launch is bracketed by two HIP events
// recorded on the launch stream; the report aggregates them by kernel name.
bool timing_enabled();
void timing_record(const char* name, hipStream_t s, bool start);

struct TimedLaunch {
  const char* name;
  hipStream_t s;
  bool on;
  TimedLaunch(const char* n, hipStream_t st) : name(n), s(st), on(timing_enabled()) {
    if (on) timing_record(name, s, true);
  }
  ~TimedLaunch() {
    if (on) timing_record(name, s, false);
  }
};

}  // namespace moe

#define MOE_TIMED(name, stream) ::moe::TimedLaunch moe_timed_scope_(name, stream)

// Host-side launch check: returns MOE_EHIP from the calling entry point.
#define MOE_LAUNCH_CHECK()                                   \
  do {                                                       \
    if (hipGetLastError() != hipSuccess) return MOE_EHIP;    \
  } while (0)
