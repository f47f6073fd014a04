// Launcher of the forward whose rows are cut along the keys (attn_kernel_split.h).
#include "attn_kernel_split.h"
#include "launch.h"
#include "split_plan.h"

using namespace calibatt_dev;
using namespace calibatt_host;

template <int D, int BQ, int BK, bool IV, typename T>
static int launch_split_typed(const FwdPtrs &a, const FwdDims &p, const calibatt_split &split, float *workspace,
                 hipStream_t stream) {
  using Part = IlPart<D, BQ, BK, T>;
  static_assert(Part::FLOATS * 4 == calibatt_part_bytes(BQ, D), "plan and kernel disagree");
  static_assert(Part::LDS_BYTES >= CALIBATT_MAX_PARTS * Part::NT * 8, "the weights of the parts do not fit");
  constexpr int SMEM = Part::LDS_BYTES + 64 + (IV ? il_iv_cols(BQ) * 4 : 0);
  static DevInfo info;
  int slots = 0;
  auto kernel = sparse_attn_fwd_split_kernel<D, BQ, BK, IV, T>;
  if (int st = prepare(kernel, BQ * 2, SMEM, info, slots)) return st;
  const FwdSplit s = {split.arrivals, workspace};
  return launch_kernel(kernel, (unsigned)split.n_parts, BQ * 2, SMEM, stream, a.q, a.k, a.v, a.out,
                       (const int4 *)split.parts, a.col_idx, a.iv, a.fan_dst, a.head_map, a.lse, p, s);
}

template <int D, int BQ, int BK>
int launch_split(const FwdPtrs &a, const FwdDims &p, const calibatt_split &split, float *workspace,
                 hipStream_t stream) {
  auto with = [&](auto iv, auto type) {
    return launch_split_typed<D, BQ, BK, iv, decltype(type)>(a, p, split, workspace, stream);
  };
  if (a.dtype == CALIBATT_F16) return a.iv ? with(std::true_type{}, F16{}) : with(std::false_type{}, F16{});
  return a.iv ? with(std::true_type{}, Bf16{}) : with(std::false_type{}, Bf16{});
}

#define CALIBATT_CASE(d, bq, bk) \
  template int launch_split<d, bq, bk>(const FwdPtrs &, const FwdDims &, const calibatt_split &, float *, hipStream_t);
CALIBATT_CASE(128, 128, 128)
CALIBATT_CASE(128, 128, 64)
CALIBATT_CASE(128, 128, 96)
CALIBATT_CASE(128, 128, 160)
CALIBATT_CASE(128, 128, 192)
CALIBATT_CASE(128, 64, 128)
CALIBATT_CASE(128, 64, 64)
CALIBATT_CASE(64, 128, 128)
CALIBATT_CASE(64, 128, 64)
CALIBATT_CASE(64, 64, 128)
CALIBATT_CASE(64, 64, 64)
