// ee_sweep_whole.hip -- the on-chip sweep kernel with the whole-region protocol.
#define EE_WHOLE 1
#define EE_SWEEP_KERNEL sweep_whole_kernel
#include "ee_sweep.hpp"

extern "C" int ee_k_sweep_whole_ptr(const void** fn) {
  *fn = reinterpret_cast<const void*>(&sweep_whole_kernel);
  return (int)hipFuncSetAttribute(*fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  ee_k_max_lds_bytes() + ee::kSweepTailBytes);
}
