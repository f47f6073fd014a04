// What the plan of a split forward (split_plan.cpp), its kernel and its launcher (sparse_attn_split.hip) agree on.
#pragma once
#include <stdint.h>

#include "calibatt.h"

// bytes that one part leaves in the workspace: fp32 sums of its rows, a reference and a row sum per thread (two per row)
constexpr int64_t calibatt_part_bytes(int block_q, int D) { return ((int64_t)block_q * D + 4 * block_q) * 4; }
constexpr int CALIBATT_MAX_PARTS = 16;    // parts of one row: their weights lie in LDS
constexpr int CALIBATT_PART_WORDS = 12;   // int32 of a part's record (attn_kernel_split.h)

#ifdef __HIP__
#include "attn_common.h"
#include "launch.h"
// sparse_attn_split.hip
template <int D, int BQ, int BK>
int launch_split(const calibatt_host::FwdPtrs &a, const calibatt_dev::FwdDims &p, const calibatt_split &split,
                 float *workspace, hipStream_t stream);
#endif
