// Host side of a kernel launch, shared by the files that hold kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "calibatt.h"

namespace calibatt_host {

struct FwdPtrs {
  const uint16_t *q, *k, *v;
  uint16_t *out;
  const int32_t *row_ptr, *col_idx, *work, *fan_ptr, *fan_dst;
  int32_t *counter;
  const int32_t *iv_ptr;  // interval form of the kept-block lists, or NULL
  const uint32_t *iv;
  const int32_t *head_map;  // tensor head of each pattern head, or NULL
  float *lse;               // log-sum-exp output, or NULL
  int dtype;                // CALIBATT_BF16 or CALIBATT_F16
};

// Per-device launch facts of one kernel: how many workgroups the whole device holds at a time.
// Looked up on the first call per device.  Concurrent first calls all compute the same figure, so
// the slot is a plain atomic (0 = not known yet) and no lock is taken.
struct DevInfo {
  std::atomic<int> slots[64];
};

template <typename Kernel>
int prepare(Kernel kernel, int threads, int smem, DevInfo &info, int &slots) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return CALIBATT_ERR_LAUNCH;
  slots = info.slots[dev].load(std::memory_order_acquire);
  if (slots > 0) return CALIBATT_OK;
  int cus = 0, per_cu = 0;
  if (hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kernel, threads, smem) != hipSuccess ||
      cus <= 0 || per_cu <= 0)
    return CALIBATT_ERR_LAUNCH;
  slots = cus * per_cu;
  info.slots[dev].store(slots, std::memory_order_release);
  return CALIBATT_OK;
}

// Launches through the call that reports its own status: the runtime's "last error" may still hold
// an unrelated error left by earlier calls of the host program.
template <typename Kernel, typename... Args>
int launch_kernel(Kernel kernel, unsigned grid, int threads, int smem, hipStream_t stream, Args... args) {
  void *argv[] = {(void *)&args...};
  return hipLaunchKernel((const void *)kernel, dim3(grid), dim3(threads), argv, smem, stream) == hipSuccess
             ? CALIBATT_OK
             : CALIBATT_ERR_LAUNCH;
}

}  // namespace calibatt_host
