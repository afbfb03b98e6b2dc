// The expert FFN forward, as the fused layer forward calls it.
#pragma once

#include "sched.hpp"

namespace moe {

struct FfnFwd {   // arguments of moe_expert_ffn_fwd
  moe_dtype dt;
  moe_act act;
  int E, d, f;
  const int32_t *offsets, *rows;
  int64_t rows_alloc;
  const void *x_disp, *w1, *w3, *w2;
  void *h_save, *y_disp, *workspace;
  int64_t rows_most;   // at most this many rows hold a token: rows_alloc if not known
};
moe_status ffn_fwd_check(const FfnFwd& a, size_t workspace_bytes);
// Arguments for a schedule of this call built elsewhere (a.rows_alloc > 0).
SchedArgs ffn_fwd_sched(const FfnFwd& a);
// scheduled: the schedule is in the workspace already.
moe_status ffn_fwd_launch(hipStream_t s, const FfnFwd& a, bool scheduled);

}  // namespace moe
