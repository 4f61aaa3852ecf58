// Softmax kernel instances, bf16, for plans whose rows all start and end on 16-byte vectors, on
// 16-byte aligned buffers.
#include <hip/hip_runtime.h>

#include "bsm_kernel_set.hpp"

namespace bsm {

const void* softmax_fn_bf16(int kclass, bool temporal, bool bwd) {
    return kernel_set<bsm_dev::BF16, false>(kclass, temporal, bwd);
}

}  // namespace bsm
