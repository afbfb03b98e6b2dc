// Count, capacity and dispatch in one call, and the combine, as the fused
// layer forward calls them.
#pragma once

#include "sched.hpp"

namespace moe {

// The capacity rule of a call: Eq. 4 (num / den = alpha) or, when dynamic,
// ceil(num / den * count), in exact 64-bit integer arithmetic, clamped to
// [cap_min, T]; regions start at multiples of align rows.
struct CapRule {
  int dynamic, num, den, cap_min, align;
};

struct Route {   // arguments of moe_route
  moe_dtype dt;
  int T, d, E, k;
  const void* x;
  const int32_t* ids;
  CapRule rule;
  int64_t rows_alloc;
  int32_t *capacity, *offsets, *counts, *fill, *dest_row, *src;
  void* x_disp;
  int32_t* status;
  void* workspace;
};
moe_status route_check(const Route& a, size_t workspace_bytes);
// sched: the expert products' schedule to build on the way (their rows: the
// fill), or null; *scheduled tells whether it was (the fused kernel only).
moe_status route_launch(hipStream_t s, const Route& a, const SchedArgs* sched, bool* scheduled);

}  // namespace moe
