// Device half of split items (split.hip), as transform.hip uses it.
#pragma once

#include <hip/hip_runtime.h>

#include "rocket_internal.h"

namespace rocket {

struct FusedArgs;    // arguments of the fp32 items (tiles.h)
struct SplitDevice;  // a SplitPlan's tables on the device and its launch shape

// Whether one row of length L fits a workgroup's LDS.
bool split_fits(int32_t L, int64_t lds_limit);
hipError_t split_create(SplitPlan &&plan, int device, int n_cu, int64_t lds_limit, bool mpv, SplitDevice **out);
void split_destroy(SplitDevice *d);
// Series-lane layout: LDS per workgroup; the kernel of each slot (-1: empty);
// S[slot][s_rows] features <- X[n, L], n <= s_rows, asynchronous on s.
int64_t split_series_lds(int32_t L);
const std::vector<int32_t> &split_slot_kernels(const SplitDevice *d);
rocket_status split_launch_series(const SplitDevice *d, const float *X, int64_t n, int32_t K, float *S, int64_t s_rows,
                                  hipStream_t s);
int64_t split_lds_bytes(const SplitDevice *d);
int split_rows_per_block(const SplitDevice *d);
// Items; kernels left to fp32 items; distinct (length, dilation, padding) of the set.
int64_t split_n_items(const SplitDevice *d);
int64_t split_n_rest(const SplitDevice *d);
int64_t split_n_buckets(const SplitDevice *d);
// Dynamic LDS that the kernels are allowed.
int64_t split_lds_room(const SplitDevice *d);
// Rows above 40 KB: one workgroup per CU.
bool split_one_per_cu(const SplitDevice *d);
// Issue cycles per series of the kernels left to fp32 items.
double split_rest_cost(const SplitDevice *d);
// F[n, K * (2 or 3)] of the plan's kernels <- X[n, L], asynchronous on s; rest
// (or null): MFMA and VALU items of padded rows to run in the same launch,
// with rest_lds bytes of LDS (its row fields are set here).
rocket_status split_launch(const SplitDevice *d, const float *X, int64_t n, int32_t K, float *F, const FusedArgs *rest,
                           int64_t rest_lds, hipStream_t s);
// ORs the failed checks since the last call into *flags and clears them (checked builds).
rocket_status split_check_flags(uint32_t *flags);

}  // namespace rocket
