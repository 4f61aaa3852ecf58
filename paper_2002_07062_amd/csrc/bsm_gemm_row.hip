// Host launch wrapper of the row-tile matrix products (device code in bsm_gemm_row.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
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

template <int LAYOUT, bool BF16OUT, int OPS, bool TEMPORAL, int NK>
hipError_t launch_few(Launch& l, int parts, int lds_bytes) {
    void* args[] = {&l.a, &l.b, &l.c, &l.s, &l.worker_ptr, &l.items, &l.trace};
    return hipLaunchKernel(reinterpret_cast<const void*>(&bsm_gemm_few_rows_kernel<LAYOUT, BF16OUT, OPS, TEMPORAL, NK>),
                           dim3(l.n_wg, parts), dim3(64 * kRowWaves), args, lds_bytes, l.stream);
}
template <bool BF16OUT, int OPS, bool TEMPORAL>
hipError_t pick_layout(Launch& l, int parts, int layout, int lds) {
    if (layout == kNN) return launch_few<kNN, BF16OUT, OPS, TEMPORAL, 1>(l, parts, lds);
    return l.s.k <= kChunkK ? launch_few<kNT, BF16OUT, OPS, TEMPORAL, 1>(l, parts, lds)
                            : launch_few<kNT, BF16OUT, OPS, TEMPORAL, 2>(l, parts, lds);
}
template <bool BF16OUT>
hipError_t pick_few(Launch& l, int parts, int layout, int lds, bool temporal, bool vec) {
    if (vec)
        return temporal ? pick_layout<BF16OUT, kVec, true>(l, parts, layout, lds) : pick_layout<BF16OUT, kVec, false>(l, parts, layout, lds);
    return temporal ? pick_layout<BF16OUT, kAny, true>(l, parts, layout, lds) : pick_layout<BF16OUT, kAny, false>(l, parts, layout, lds);
}

}  // namespace

namespace bsm {

int gemm_row_lds_bytes_per_wg(int q) { return row_lds_bytes(q); }
int gemm_few_rows_lds_bytes_per_wg(int layout) { return few_rows_lds_bytes(layout); }
int gemm_few_rows_lds_bytes_two_per_cu(int layout) { return std::max(few_rows_lds_bytes(layout), kTwoPerCuBytes); }
int gemm_few_rows_wgs_per_cu(int layout) { return few_rows_wgs_per_cu(layout); }

// us below: the other form -> row tiles.
int gemm_row_softmax_waves(int64_t batch, int m, int n, int k) {
    // the 16-byte loads need eight elements per operand
    if (k > 2 * kChunkK || n > row_max_cols(8) || batch * std::min(m, n) * k < 8) return 0;
    const int64_t tiles = batch * ((m + kTileM - 1) / kTileM);  // of 32 rows
    const int blocks = (n + kBlockN - 1) / kBlockN;             // of 64 columns
    // Past 512 columns, and where k is no whole number of 16-byte pieces, the other form takes two
    // passes (384 x 512 x 512 (k = 100) 303 -> 114, 9469 x 33 x 128 (k = 100) 269 -> 203).
    if (n > kBlockN && (k % 8 != 0 || !single_pass_shape(n, k))) return n <= row_max_cols(4) ? 4 : 8;
    // One column block (the other form: two passes of 128-row rounds; here one wave of four
    // works): where the chip is not full of rounds, or they are mostly empty.  1000 x 30 x 60
    // 23.6 -> 8.5, 40 x 500 x 60 (k = 128) 20.9 -> 9.3, 100 x 500 x 40 20.1 -> 13.9; past the line
    // 100 x 1000 x 50 25.8 -> 28.4, 2000 x 200 x 64 58 -> 67.
    if (n <= kBlockN) return m <= kTileM || batch * ((m + 127) / 128) <= 512 ? 4 : 0;
    // Up to 512 columns the other form is one pass of 64-row rounds by wave pairs, which splits
    // the columns over two waves.  Four must not leave more of them idle (1000 x 33 x 300
    // 22.4 -> 27.5, 2000 x 128 x 128 34 -> 43), and win where the rounds do not fill the chip a few times
    // (16 x 512 x 512 13.4 -> 8.7, 96 x 512 x 512 20.6 -> 17.1, 300 x 90 x 448 (k = 128) 29.9 -> 22.2; 192 x 512 x 512
    // (k = 128) 40 -> 45, 384 x 512 x 512 65 -> 71) or where rows are not whole 128-byte lines, whose
    // halves the waves then store at about the same time, and the rounds are mostly full
    // (1000 x 128 x 500 77 -> 61, 1000 x 64 x 200 19.0 -> 17.4; 969 x 33 x 500 28.6 -> 31.0).  With two
    // slices of k, and as many column blocks to a wave, few rows do not make up for B read once
    // per 32 of them (488 x 64 x 512 (k = 128) 21.2 -> 27.1, 200 x 100 x 440 (k = 96) 20.4 -> 23.1).
    const int64_t rounds = batch * ((m + kS1Rows - 1) / kS1Rows);
    const int64_t work = tiles * ((blocks + 3) / 4), other = rounds * ((blocks + 1) / 2);
    if (work > other) return 0;
    if (m <= kTileM) return 4;
    const bool full = 5 * batch * m > 4 * rounds * kS1Rows, lines = n % kBlockN == 0;
    if (rounds > 800) return !lines && full ? 4 : 0;
    const bool b_twice = k > kChunkK && n > 4 * kBlockN && rounds > 256 && 10 * work > 9 * other;
    return b_twice && (lines ? m <= 2 * kS1Rows : !full) ? 0 : 4;
}

// Lines that decide the last bits of a result (row tiles or not, for NN and the score softmax) are
// those of a 256-CU card whatever n_cu the topology names, so that the bits do not depend on it.
int gemm_row_parts(int layout, bool bf16_out, int64_t batch, int m, int n, int k, int n_cu) {
    if (batch * std::min(m, n) * k < 8 || (layout == kNT && k > 2 * kChunkK)) return 0;
    const int64_t tiles = batch * ((m + kTileM - 1) / kTileM);
    const int64_t blocks = (n + kBlockN - 1) / kBlockN;
    // column parts until three workgroups per CU have rows, at least four blocks (NN: one) to a part
    const int64_t most = layout == kNT ? (blocks + kRowWaves - 1) / kRowWaves : blocks;
    const int64_t parts = std::max<int64_t>(1, std::min<int64_t>({most, 8, 3 * n_cu / tiles}));
    if (layout == kNT) {
        // Both forms' time by what their workgroups do, three to a CU, in steps of one 64-column
        // block.  The general form's units are 128 rows of the row stream, dealt whole; a unit
        // starts over in every batch index that it meets.  Its steps take longer in fp32, and
        // where two blocks share 64 bytes of a line (which row tiles store at about the same time;
        // halves of a line cost nothing: bf16 846 x 640 x 160 (k = 72) 53 -> 82, 253 x 1024 x 96 (k = 96)
        // 25 -> 36).
        // A row tile takes 0.9 steps and 0.75 for every four blocks, a quarter more with two
        // slices of k.  Fitted to 4840 shapes (n 16 .. 2048, m 8 .. 2048, 1 to 60 million outputs,
        // both types): 95% get the faster form, or one within 5% of it, the worst one of 1.43
        // times its time.  us, general -> row tiles: 384 x 512 x 512 44 -> 54 (fp32 78.7 -> 72.8), 190 x
        // 512 x 512 (k = 128) 27.5 -> 36.6, 7324 x 512 x 16 120 -> 299, fp32 384 x 512 x 64 13.7 -> 19.1;
        // 4 x 2048 x 2048 (k = 128) 48 -> 12, 512 x 16 x 936 142 -> 30, 1000 x 128 x 300 62 -> 38, 473 x 33 x
        // 64 14.5 -> 8.7.
        const double resident = 3.0 * n_cu;  // either form: the same bits
        const int64_t units = (batch * m + 127) / 128;
        const double per_unit = m % 128 == 0 ? 1.0 : 128 % m == 0 ? 128.0 / m : 1.0 + 128.0 / m;
        const bool shared_lines = blocks > 1 && n % (bf16_out ? 32 : 16) != 0;
        const double general = std::ceil(units / resident) * per_unit * (0.6 + (bf16_out ? 1.0 : 1.5) * blocks) *
                               (shared_lines ? 3.0 : 1.0);
        const double row = std::max(1.0, tiles * parts / resident) * (k > kChunkK ? 1.25 : 1.0) *
                           (0.9 + 0.75 * static_cast<double>((blocks + 4 * parts - 1) / (4 * parts)));
        if (general <= row) return 0;
    } else {
        // NN's waves split the reduction, A is read once per 64 columns and B once per 32 rows:
        // for few tiles.  us at tiles x blocks: 504 (4 x (2000 x 2000)(2000 x 128)) 58 -> 20, 800
        // (200 x (128 x 500)(500 x 64)) 24.6 -> 13.7, 876 33.6 -> 29.9, 1000 16.5 -> 19.5, 1024 27 -> 31, 1512 32 -> 37.
        if (tiles * blocks > 896) return 0;
    }
    return static_cast<int>(parts);
}

hipError_t launch_gemm_row(int q, bool bf16_out, bool temporal, const void* a, const void* b, void* c, int64_t batch,
                           int m, int n, int k, float alpha, const int32_t* d_worker_ptr, const bsm_item* d_items,
                           int n_wg, void* trace, hipStream_t stream) {
    Launch l{static_cast<const uint16_t*>(a), static_cast<const uint16_t*>(b), c,
             product_shape(batch, m, n, k, alpha), d_worker_ptr, d_items,
             static_cast<bsm_trace_rec*>(trace), n_wg, stream};
    const bool vec = aligned_pieces(a, b, k);
    return bf16_out ? pick_ops<true>(l, q, temporal, vec) : pick_ops<false>(l, q, temporal, vec);
}

hipError_t launch_gemm_few_rows(int layout, int parts, int lds_bytes, bool bf16_out, bool temporal, const void* a,
                                const void* b, void* c, int64_t batch, int m, int n, int k, float alpha, const int32_t* d_worker_ptr,
                                const bsm_item* d_items, int n_wg, void* trace, hipStream_t stream) {
    Launch l{static_cast<const uint16_t*>(a), static_cast<const uint16_t*>(b), c,
             product_shape(batch, m, n, k, alpha), d_worker_ptr, d_items,
             static_cast<bsm_trace_rec*>(trace), n_wg, stream};
    const bool vec = aligned_pieces(a, b, k) && (layout != kNN || n % 8 == 0);
    return bf16_out ? pick_few<true>(l, parts, layout, lds_bytes, temporal, vec) : pick_few<false>(l, parts, layout, lds_bytes, temporal, vec);
}

}  // namespace bsm
