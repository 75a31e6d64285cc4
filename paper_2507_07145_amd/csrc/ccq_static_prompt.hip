// The partial tiles of ccq_gemm_static's prompts, as large as any plan of the block kernel asks for.  A source file, and with it a code object,
// of its own: a process that makes no such call does not hold the array.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ccq_internal.h"

namespace ccq {

// In host code this name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char prompt_scratch[kPromptPartialMost];

static SymbolAddresses prompt_scratch_addr;

int prompt_scratch_of_current_device(void** out) { return symbol_of_current_device(HIP_SYMBOL(prompt_scratch), prompt_scratch_addr, out); }

}  // namespace ccq
