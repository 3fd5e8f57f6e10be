// ee_sweep.hip -- the on-chip sweep kernel without the whole-region protocol.
#define EE_WHOLE 0
#define EE_SWEEP_KERNEL sweep_kernel
#include "ee_sweep.hpp"

extern "C" int ee_k_sweep_plain_ptr(const void** fn) {
  *fn = reinterpret_cast<const void*>(&sweep_kernel);
  return (int)hipFuncSetAttribute(*fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  ee_k_max_lds_bytes() + ee::kSweepTailBytes);
}
