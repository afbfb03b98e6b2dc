// One layer forward in one call: the gate (or caller-given picks), count,
// capacity and dispatch, the expert FFN, the combine.  The same kernels as the
// separate calls, except that on small batches the expert products' schedule
// is built inside the routing kernel.  The host checks every argument first,
// so an error enqueues nothing, and then only launches: a caller in Python
// pays for one library call instead of four, which on the smallest layers
// takes longer than the kernels (T = 256, d = 64: 49 us of host work per
// forward against 26 us).

#include <algorithm>

#include "ffn.hpp"
#include "route.hpp"

using namespace moe;

extern "C" moe_status moe_layer_fwd(void* stream, const moe_layer_fwd_args* p) {
  if (!p) return MOE_EINVAL;
  const moe_layer_fwd_args& a = *p;
  const bool gate = a.cached_ids == nullptr;
  const int32_t* ids = gate ? a.ids : a.cached_ids;
  if (!dtype_ok(a.dtype) || !shape_ok(a.T, a.E, a.k) || !width_ok(a.d)) return MOE_EINVAL;
  if (gate && a.T > 0) {   // as moe_gate_topk
    if (!a.x || !a.w_g || !a.logits || !a.ids || !a.weights) return MOE_EINVAL;
    if (!aligned16(a.x) || !aligned16(a.w_g)) return MOE_EINVAL;
    if (a.dtype == MOE_BF16 && static_cast<int64_t>(a.d) * 2 * kMaxE >= (int64_t(1) << 31))
      return MOE_EINVAL;
  }
  if (a.y && a.T > 0) {    // as moe_combine
    if (!a.y_disp || !a.weights || !aligned16(a.y_disp) || !aligned16(a.y)) return MOE_EINVAL;
  }
  const Route r = {a.dtype, a.T, a.d, a.E, a.k, a.x, ids,
                   {a.dynamic != 0, a.num, a.den, a.cap_min, a.row_align}, a.rows_alloc,
                   a.capacity, a.offsets, a.counts, a.fill, a.dest_row, a.src, a.x_disp, a.status,
                   a.route_ws};
  moe_status st = route_check(r, a.route_ws_bytes);
  if (st != MOE_OK) return st;
  const FfnFwd f = {a.dtype, a.act, a.E, a.d, a.f, a.offsets, a.fill, a.rows_alloc, a.x_disp, a.w1,
                    a.w3, a.w2, a.h_save, a.y_disp, a.ffn_ws,
                    std::min<int64_t>(a.rows_alloc, static_cast<int64_t>(a.T) * a.k)};
  st = ffn_fwd_check(f, a.ffn_ws_bytes);
  if (st != MOE_OK) return st;

  if (gate) {
    st = moe_gate_topk(stream, a.dtype, a.T, a.d, a.E, a.k, a.renorm, a.x, a.w_g, a.bias, a.logits,
                       a.ids, a.weights);
    if (st != MOE_OK) return st;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  bool scheduled = false;
  SchedArgs sched;
  if (a.rows_alloc > 0) sched = ffn_fwd_sched(f);
  st = route_launch(s, r, a.rows_alloc > 0 ? &sched : nullptr, &scheduled);
  if (st != MOE_OK) return st;
  st = ffn_fwd_launch(s, f, scheduled);
  if (st != MOE_OK || !a.y) return st;
  return moe_combine(stream, a.dtype, a.T, a.d, a.k, a.rows_alloc, a.y_disp, a.dest_row, a.weights,
                     a.y);
}
