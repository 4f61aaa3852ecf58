// Host launch wrappers of the batched matrix-product kernels (device code in bsm_gemm.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "bsm.h"
#include "bsm_gemm.hpp"
#include "bsm_launch.hpp"

namespace {

using bsm_mm::Shape;

template <int MODE, bool BF16OUT, int OPS, bool TEMPORAL, int FORM>
hipError_t launch_g(const void* a, const void* b, void* c, const Shape& s, const int32_t* worker_ptr,
                    const bsm_item* items, int n_wg, void* trace, hipStream_t stream) {
    const uint16_t* a_a = static_cast<const uint16_t*>(a);
    const uint16_t* a_b = static_cast<const uint16_t*>(b);
    void* a_c = c;
    Shape a_s = s;
    bsm_trace_rec* a_trace = static_cast<bsm_trace_rec*>(trace);
    void* args[] = {&a_a, &a_b, &a_c, &a_s, &worker_ptr, &items, &a_trace};
    constexpr int layout = MODE == bsm_mm::kModeNn ? bsm_mm::kNN : bsm_mm::kNT;
    const size_t lds = static_cast<size_t>(MODE == bsm_mm::kModeNtSoftmax1
                                               ? bsm_mm::s1_lds_bytes(BF16OUT, FORM == bsm_mm::kFormA2)
                                               : bsm_mm::wg_bytes<layout, FORM>(BF16OUT));
    return hipLaunchKernel(reinterpret_cast<const void*>(&bsm_mm::bsm_gemm_kernel<MODE, BF16OUT, OPS, TEMPORAL, FORM>),
                           dim3(n_wg), dim3(bsm_mm::kGemmThreads), args, lds, stream);
}

}  // namespace

namespace bsm {

int gemm_wg_threads() { return bsm_mm::kGemmThreads; }
bool gemm_single_pass_shape(int n, int k) { return bsm_mm::single_pass_shape(n, k); }
int gemm_lds_bytes_per_wg(bool bf16_out, bool single_pass) {
    return single_pass ? bsm_mm::s1_lds_bytes(bf16_out, true)
                       : bsm_mm::wg_bytes<bsm_mm::kNT, bsm_mm::kFormStep>(bf16_out);
}
int gemm_wide_lds_bytes_per_wg(bool bf16_out) {
    return std::max(bsm_mm::wg_bytes<bsm_mm::kNT, bsm_mm::kFormA2>(bf16_out),
                    bsm_mm::wg_bytes<bsm_mm::kNN, bsm_mm::kFormWide>(bf16_out));
}
// NN's rounds of 128 rows come to between two and three per CU: three workgroups per CU of the
// 64-column form then take one each, where two of the 128-column form leave some CUs a second
// turn.  us, two -> three: 192 x (512 x 512)(512 x 128) 41.8 -> 39.3, 192 x (512 x 128)(128 x 128)
// 16.7 -> 12.9, 150 x (512 x 333)(333 x 128) 36.7 -> 35.3; past the lines 129 x (512 x 512)(512 x 128)
// 31.7 -> 36.5, 225 x (512 x 512)(512 x 128) 43 -> 75, 192 x (512 x 512)(512 x 80) 39.5 -> 40.9, 96 x (1024 x
// 1024)(1024 x 128) 64 -> 72; n = 512 gains too (192 x (512 x 512)(512 x 512) 145 -> 138) unless every
// round has a batch index of its own (768 x (128 x 512)(512 x 256) 83 -> 93).
static bool nn_three_per_cu(int64_t batch, int m, int n, int k, int n_cu) {
    const int64_t rounds = batch * ((m + 127) / 128);
    return n > 80 && (n <= 128 || m > 128) && k <= 768 && 10 * rounds > 22 * n_cu && rounds <= 3 * n_cu;
}
// kFormWide is compiled for two workgroups per CU.  With a third, which waits, it still pays over
// several reduction steps (32 x (2048 x 2048)(2048 x 128) 105 us against kFormStep's 113), but not
// over one (384 x (512 x 64)(64 x 100) 27.8 against 25.2; two per CU 23.9), nor where three is the
// better number.
//
// fp32 plain scores of whole rounds, 64 < k <= 128: kFormA2 stores the same bits, later (its step is
// the whole reduction, of which k <= 96 leaves a quarter or more empty).  It loses where a workgroup
// takes its only round, and after that where two of few columns, a short reduction and long slices
// meet; more columns read A more often, and each new batch index starts over at every step.  us,
// kFormA2 -> kFormStep: 92 x 1024 x 128 (k = 128) 16.8 -> 14.5, 175 x 512 x 128 (k = 96) 15.3 -> 13.4, 92 x
// 1024 x 256 (k = 80) 25.1 -> 21.3, 190 x 1024 x 512 (k = 80) 88.5 -> 80.5, 1100 x 128 x 128 (k = 72) 24.0 ->
// 23.3; past the lines 175 x 512 x 512 (k = 128) 42.6 -> 44.6, 700 x 128 x 160 (k = 128) 20.9 -> 23.3, 575 x
// 512 x 256 (k = 128) 76 -> 87.
bool gemm_wide_pays(int layout, bool bf16_out, int64_t batch, int m, int n, int k, int n_cu, int wgs_per_cu) {
    if (wgs_per_cu <= bsm_mm::kS1WavesPerSimd) return true;
    if (layout == bsm_mm::kNT && !bf16_out && m % 128 == 0 && n <= (k <= 96 ? 512 : 256)) {
        const bool one_round = batch * m <= 128 * static_cast<int64_t>(bsm_mm::kWavesPerSimd) * n_cu;
        if (one_round ? m >= 512 || n <= 128 : (m >= 1024) + (k <= 96) + (n <= 128) >= 2) return false;
    }
    return k > bsm_mm::kChunkK && !(layout == bsm_mm::kNN && nn_three_per_cu(batch, m, n, k, n_cu));
}
int gemm_waves_per_simd(bool single_pass) {
    return single_pass ? bsm_mm::kS1WavesPerSimd : bsm_mm::kWavesPerSimd;
}
int gemm_default_wgs_per_cu(int layout, int64_t batch, int m, int n, int k, int n_cu, bool single_pass) {
    if (single_pass) return bsm_mm::kS1WavesPerSimd;
    const bool vec = k % 8 == 0 && (layout != bsm_mm::kNN || n % 8 == 0);  // as launch_gemm, aligned operands
    const int form = bsm_mm::form_of(layout, vec, true, n, k);
    if (form == bsm_mm::kFormWide && nn_three_per_cu(batch, m, n, k, n_cu)) return bsm_mm::kWavesPerSimd;
    return form == bsm_mm::kFormStep ? bsm_mm::kWavesPerSimd : bsm_mm::waves_per_simd(layout, form);
}
int gemm_rows_per_wg(bool single_pass) {
    return single_pass ? bsm_mm::kS1Rows : bsm_mm::kWaves * bsm_mm::kTileM;
}

hipError_t launch_gemm(int layout, bool bf16_out, bool temporal, bool single_pass, bool wide, const void* a,
                       const void* b, void* c, int64_t batch, int m, int n, int k, float alpha,
                       const int32_t* d_worker_ptr, const bsm_item* d_items, int n_wg, void* trace,
                       hipStream_t stream) {
    const Shape s = bsm_mm::product_shape(batch, m, n, k, alpha);
    // rows of A (and NT's B) have k elements, rows of NN's B n; C is stored at any boundary
    const bool vec = bsm_mm::aligned_pieces(a, b, k) && (layout != bsm_mm::kNN || n % 8 == 0);
    const int form = bsm_mm::form_of(layout, vec, wide, n, k);
    const int out = (bf16_out ? 1 : 0) | (temporal ? 2 : 0);
#define BSM_G(M, V, F)                                                                                        \
    switch (out) {                                                                                            \
        case 0: return launch_g<M, false, V, false, F>(a, b, c, s, d_worker_ptr, d_items, n_wg, trace, stream); \
        case 1: return launch_g<M, true, V, false, F>(a, b, c, s, d_worker_ptr, d_items, n_wg, trace, stream);  \
        case 2: return launch_g<M, false, V, true, F>(a, b, c, s, d_worker_ptr, d_items, n_wg, trace, stream);  \
        default: return launch_g<M, true, V, true, F>(a, b, c, s, d_worker_ptr, d_items, n_wg, trace, stream);  \
    }
    using namespace bsm_mm;
    // the one-pass softmax takes alpha != 0 only (with alpha = 0 every logit is 0, which the
    // two-pass form handles)
    if (layout == kModeNtSoftmax && single_pass && vec && alpha != 0.0f && single_pass_shape(n, k)) {
        if (k > kChunkK) BSM_G(kModeNtSoftmax1, kVec, kFormA2)
        BSM_G(kModeNtSoftmax1, kVec, kFormA1)
    }
    if (s.k > 0 && (s.a_total < 8 || s.b_total < 8)) {
#define BSM_GT(M)                                                                                              \
    return bf16_out ? launch_g<M, true, kTiny, false, kFormStep>(a, b, c, s, d_worker_ptr, d_items, n_wg, trace, stream) \
                    : launch_g<M, false, kTiny, false, kFormStep>(a, b, c, s, d_worker_ptr, d_items, n_wg, trace, stream)
        if (layout == kNN) BSM_GT(kModeNn);
        if (layout == kModeNtSoftmax) BSM_GT(kModeNtSoftmax);
        BSM_GT(kModeNt);
#undef BSM_GT
    }
    if (layout == kNN) {
        if (form == kFormA1) BSM_G(kModeNn, kVec, kFormA1)
        if (form == kFormWide) {
            if (vec) BSM_G(kModeNn, kVec, kFormWide)
            BSM_G(kModeNn, kAny, kFormWide)
        }
        if (vec) BSM_G(kModeNn, kVec, kFormStep)
        BSM_G(kModeNn, kAny, kFormStep)
    }
    if (layout == kModeNtSoftmax) {
        if (form == kFormA1) BSM_G(kModeNtSoftmax, kVec, kFormA1)
        if (form == kFormA2) BSM_G(kModeNtSoftmax, kVec, kFormA2)
        if (vec) BSM_G(kModeNtSoftmax, kVec, kFormStep)
        BSM_G(kModeNtSoftmax, kAny, kFormStep)
    }
    if (form == kFormA1) BSM_G(kModeNt, kVec, kFormA1)
    if (form == kFormA2) BSM_G(kModeNt, kVec, kFormA2)
    if (vec) BSM_G(kModeNt, kVec, kFormStep)
    BSM_G(kModeNt, kAny, kFormStep)
#undef BSM_G
}

}  // namespace bsm
