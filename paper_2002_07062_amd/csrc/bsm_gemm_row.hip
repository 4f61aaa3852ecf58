// Host launch wrapper of the row-tile matrix products (device code in bsm_gemm_row.hpp).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "bsm.h"
#include "bsm_gemm_row.hpp"
#include "bsm_launch.hpp"

namespace {

using namespace bsm_mm;

struct Launch {
    const uint16_t* a;
    const uint16_t* b;
    void* c;
    Shape s;
    const int32_t* worker_ptr;
    const bsm_item* items;
    bsm_trace_rec* trace;
    int n_wg;
    hipStream_t stream;
};

template <bool BF16OUT, int OPS, bool TEMPORAL, int NK, int Q>
hipError_t launch_softmax_rows(Launch& l) {
    void* args[] = {&l.a, &l.b, &l.c, &l.s, &l.worker_ptr, &l.items, &l.trace};
    return hipLaunchKernel(reinterpret_cast<const void*>(&bsm_gemm_row_kernel<BF16OUT, OPS, TEMPORAL, NK, Q>),
                           dim3(l.n_wg), dim3(64 * Q), args, row_lds_bytes(Q), l.stream);
}

template <bool BF16OUT, int OPS, bool TEMPORAL>
hipError_t pick_shape(Launch& l, int q) {
    const bool one = l.s.k <= kChunkK;
    if (q == 8)
        return one ? launch_softmax_rows<BF16OUT, OPS, TEMPORAL, 1, 8>(l) : launch_softmax_rows<BF16OUT, OPS, TEMPORAL, 2, 8>(l);
    return one ? launch_softmax_rows<BF16OUT, OPS, TEMPORAL, 1, 4>(l) : launch_softmax_rows<BF16OUT, OPS, TEMPORAL, 2, 4>(l);
}
template <bool BF16OUT, int OPS>
hipError_t pick_temporal(Launch& l, int q, bool temporal) {
    return temporal ? pick_shape<BF16OUT, OPS, true>(l, q) : pick_shape<BF16OUT, OPS, false>(l, q);
}
template <bool BF16OUT>
hipError_t pick_ops(Launch& l, int q, bool temporal, bool vec) {
    return vec ? pick_temporal<BF16OUT, kVec>(l, q, temporal) : pick_temporal<BF16OUT, kAny>(l, q, temporal);
}

}  // namespace

namespace bsm {

int gemm_row_lds_bytes_per_wg(int q) { return row_lds_bytes(q); }
int gemm_row_max_cols(int q) { return row_max_cols(q); }

hipError_t launch_gemm_row(int q, bool bf16_out, bool temporal, const void* a, const void* b, void* c, int64_t batch,
                           int m, int n, int k, float alpha, const int32_t* d_worker_ptr, const bsm_item* d_items,
                           int n_wg, void* trace, hipStream_t stream) {
    Launch l{static_cast<const uint16_t*>(a), static_cast<const uint16_t*>(b), c,
             product_shape(batch, m, n, k, alpha), d_worker_ptr, d_items,
             static_cast<bsm_trace_rec*>(trace), n_wg, stream};
    const bool vec = aligned_pieces(a, b, k);
    return bf16_out ? pick_ops<true>(l, q, temporal, vec) : pick_ops<false>(l, q, temporal, vec);
}

}  // namespace bsm
