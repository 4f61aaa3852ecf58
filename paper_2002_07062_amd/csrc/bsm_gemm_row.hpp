// Matrix products by row-tile workgroups: the Q waves of a workgroup share one 32-row tile of
// the output and split its columns; wave q takes the 64-column blocks q, q + Q, ..  Each wave
// streams its own columns of B through its own LDS region (no other wave reads them, so the
// stream meets no barrier) against the tile's rows of A; k <= 128.  The 32-row tiles make four times the
// workgroups of the general form's 128-row rounds, and the four waves work on any of them.
//
//   NT: each block is stored as it comes.
//   NN: the waves split the reduction instead and add their sums at the end.
//   NT + softmax: the products of a row stay in registers until it is done, for n <= 256 Q.
//   The two-pass form forms every product and every exponential twice, with a barrier at every
//   64 columns.  us, two passes -> this, calls back to back: 237 x (241 x 64)(64 x 920) bf16 100 ->
//   57, 64 x (1000 x 64)(64 x 777) 103 -> 53, 32 x (1024 x 128)(128 x 2048) fp32 126 -> 74, 32 x
//   (2048 x 128)(128 x 2048) bf16 127 -> 105 (the profiler's kernel times are 119 to 152 there);
//   16 x (24 x 96)(96 x 560), where 128-row rounds leave most of the chip idle, 24.3 -> 9.4.  At Q = 8 the round's 28k clocks go to the waves' LDS traffic and exponentials
//   (15k) and to the output's staging and stores (8k); skipping the stores changes nothing.
#pragma once

#include "bsm_gemm.hpp"

namespace bsm_mm {

constexpr int kRowMaxBlocks = 4;  // 64-column blocks a wave holds (128 registers)
constexpr int kRowPieces = kBlockN * kChunkK / 8 / 64;  // 16-byte pieces per lane of a 64 x 64 chunk of B
constexpr int kRowWaves = 4;      // waves of the plain products' workgroups
// a wave's LDS: the chunk; A's and the output's staging reuse it
constexpr int kRowWaveBytes = kBlockN * kLdk * 2;
static_assert(kRowWaveBytes >= kTileM * Geo<kNT, kFormA1>::kLdc * 4, "fp32 output staging fits the chunk");
template <int NK>
constexpr int kRowLda = NK * kChunkK + 8;  // padded LDS row of A
constexpr int row_lds_bytes(int q) { return q * (kRowWaveBytes + 2 * kTileM * 4) + kTileM * kRowLda<2> * 2; }
constexpr int row_max_cols(int q) { return q * kRowMaxBlocks * kBlockN; }

// The rounds of a worker, one after the other: rows [i, i + rows) of batch index bidx, at most
// `most`, cut where a batch index ends.
struct Rounds {
    const bsm_item* __restrict__ items;
    int it, it_end, most;
    int rep = 0, left = 0;
    int64_t g = 0;  // row of the stack of outputs
    __device__ __forceinline__ bool next(const Shape& s, int64_t& bidx, int& i, int& rows) {
        if (left == 0) {
            if (it >= it_end) return false;
            g = (items[it].elem_offset + static_cast<int64_t>(rep) * items[it].rep_stride * s.n) / s.n;
            left = items[it].nrows;
            if (++rep >= items[it].reps) {
                rep = 0;
                ++it;
            }
        }
        bidx = g / s.m;
        i = static_cast<int>(g - bidx * s.m);
        rows = s.m - i < left ? s.m - i : left;
        rows = rows > most ? most : rows;
        g += rows;
        left -= rows;
        return true;
    }
};

// The lane index as a value the compiler knows nothing about: what is computed from it stays
// where it is used.  Offsets and masks of every block and slice, kept over a worker's rounds as
// invariants, spilled up to 186 registers.
__device__ __forceinline__ int here(int lane) {
    asm volatile("" : "+v"(lane));
    return lane;
}

// A 64 x 64 chunk of B: rows [j0, j0 + 64) of a batch index, reduction [k0, k0 + 64), into
// registers and from there to the wave's LDS.  All offsets are 32-bit and relative to `base`,
// element (j0, 0) of the batch index (the same for the wave): eight 64-bit addresses per lane
// and their clamps, kept over the rounds, spilled.  Rows past n are row n - 1 again: they give
// columns that nobody takes.  Columns past k are zeroed.  kVec and kAny as in load8 and keep8;
// `end` is the offset of the last whole piece of the operand.
template <int OPS>
__device__ __forceinline__ void row_load(const uint16_t* base, const Shape& s, int j0, int k0, int end, int lane,
                                         u16x8 (&p)[kRowPieces]) {
    const int c = k0 + (lane & 7) * 8;
    const int r0 = lane >> 3, r_last = s.n - 1 - j0;
    if (OPS == kVec && r_last >= kBlockN - 1) {  // one lane offset, the row steps on the scalar unit
        const unsigned off = __umul24(r0, 2 * s.k) + 2 * (c < s.k ? c : s.k - 8);
        const char* at = reinterpret_cast<const char*>(base);
#pragma unroll
        for (int q = 0; q < kRowPieces; ++q) p[q] = *reinterpret_cast<const u16x8*>(at + 16 * s.k * q + off);
        return;
    }
#pragma unroll
    for (int q = 0; q < kRowPieces; ++q) {
        const int r = r0 + 8 * q < r_last ? r0 + 8 * q : r_last;
        if constexpr (OPS == kVec) {
            const unsigned off = __umul24(r, 2 * s.k) + 2 * (c < s.k ? c : s.k - 8);
            p[q] = *reinterpret_cast<const u16x8*>(reinterpret_cast<const char*>(base) + off);
        } else {
            const int off = __mul24(r, s.k) + c;
            p[q] = *reinterpret_cast<const u16x8_any*>(base + (off < end ? off : end));
        }
    }
}

template <int OPS>
__device__ __forceinline__ void row_write(u16x8 (&p)[kRowPieces], const Shape& s, int j0, int k0, int end,
                                          int lane, uint16_t* lb) {
    const int c = k0 + (lane & 7) * 8;
    const int r0 = lane >> 3, r_last = s.n - 1 - j0;
    uint16_t* const at = lb + r0 * kLdk + (lane & 7) * 8;
    const bool whole = k0 + kChunkK <= s.k;  // wave-uniform
    if (OPS != kVec || !whole) {
        const int cc = here(c);  // keeps this a branch: as selects it cost every write
#pragma unroll
        for (int q = 0; q < kRowPieces; ++q) {
            const int row = __mul24(r0 + 8 * q < r_last ? r0 + 8 * q : r_last, s.k);
            p[q] = keep8<OPS>(p[q], row, cc, s.k, end + 8, true, whole && row + cc <= end);
        }
    }
#pragma unroll
    for (int q = 0; q < kRowPieces; ++q) *reinterpret_cast<u16x8*>(at + 8 * q * kLdk) = p[q];
}

// Worker of the score softmax.  NK 64-deep slices cover k.  lstat: [2][Q][32] floats, the waves'
// row maxima and sums.  The next round's A and first chunk of B are loaded while this round's
// rows are stored: with one workgroup per CU (Q = 8) nothing else covers their latency.
template <bool BF16OUT, int OPS, bool TEMPORAL, int NK, int Q>
__device__ __forceinline__ uint32_t row_softmax_worker(const uint16_t* a, const uint16_t* b, void* c, const Shape& s,
                                                       Rounds rounds, int wave, int lane, uint16_t* lw,
                                                       uint16_t* la, float* lstat) {
    const int li = lane & 31;
    const int h = lane >> 5;
    const int nj = (s.n + kBlockN - 1) / kBlockN;
    const int ns = nj > wave ? (nj - wave + Q - 1) / Q : 0;  // this wave's blocks, 0 .. kRowMaxBlocks
    const int last = ns * NK - 1;                            // its last chunk
    float* const lmax = lstat;
    float* const lsum = lstat + Q * kTileM;
    // Logits in base-2 units, y = c2 * product with c2 > 0: for alpha <= 0 the products are first
    // multiplied by -1 or 0.  Columns past n get the product -inf, so that the maximum, the
    // exponentials and the sums take every held value as it is.
    const float sign = s.alpha < 0.0f ? -1.0f : (s.alpha == 0.0f ? 0.0f : 1.0f);
    const float c2 = s.alpha == 0.0f ? 1.0f : sign * s.alpha * kLog2eF;
    auto higher = [](float u, float v) { return __builtin_elementwise_maximum(u, v); };
    uint32_t done = 0;

    int64_t bidx;
    int i0, rows;
    if (!rounds.next(s, bidx, i0, rows)) return 0;
    // A's 32 rows, dealt to all threads
    constexpr int kAll = 8 * NK * kTileM, kThreads = 64 * Q;
    constexpr int kMine = (kAll + kThreads - 1) / kThreads;
    u16x8 pa[kMine];
    auto a_piece = [&](int q, auto f) {  // f(row, column) of the thread's piece q
        const int e = here(lane) + 64 * wave + kThreads * q;
        if (kAll >= kThreads || e < kAll) f(e / (8 * NK), e % (8 * NK) * 8);
    };
    auto load_a_rows = [&]() {
#pragma unroll
        for (int q = 0; q < kMine; ++q)
            a_piece(q, [&](int r, int col) {
                pa[q] = load8<OPS>(a, bidx * s.a_batch + static_cast<int64_t>(i0 + (r < rows ? r : rows - 1)) * s.k,
                                   col, s.k, s.a_total);
            });
    };
    u16x8 p[kRowPieces];
    const uint16_t* base;  // of the chunk in flight: element (j0, 0)
    int end;
    auto load_b = [&](int u) {
        const int j0 = (wave + Q * (u / NK)) * kBlockN;
        const int64_t at = bidx * s.b_batch + static_cast<int64_t>(j0) * s.k;
        base = b + at;
        const int64_t to_end = s.b_total - 8 - at;  // below 0 in a last block of under 8 elements
        end = to_end < (1 << 24) ? static_cast<int>(to_end) : (1 << 24);
        row_load<OPS>(base, s, j0, (u % NK) * kChunkK, end, here(lane), p);
    };
    load_a_rows();
    if (ns > 0) load_b(0);
    while (true) {
#pragma unroll
        for (int q = 0; q < kMine; ++q)
            a_piece(q, [&](int r, int col) {
                *reinterpret_cast<u16x8*>(la + r * kRowLda<NK> + col) =
                    keep8<OPS>(pa[q], bidx * s.a_batch + static_cast<int64_t>(i0 + r) * s.k, col, s.k, s.a_total,
                               r < rows, NK * kChunkK <= s.k);
            });
        __syncthreads();
        u16x8 a_reg[NK * (kChunkK / kTileK)];
#pragma unroll
        for (int q = 0; q < NK * (kChunkK / kTileK); ++q)
            a_reg[q] = *reinterpret_cast<const u16x8*>(la + li * kRowLda<NK> + q * kTileK + 8 * h);
        // Tile t of block st, lane (li, h): row li, columns 64 (wave + Q st) + 32 t + 8 g + 4 h + 0..3
        // (value 4 g + e).  A block's exponentials are taken as soon as its products are there,
        // against the lane's own maximum of the block, and brought to the row's maximum by the
        // factor that divides by the sum: the waves need no common step until the row's end, so
        // that one wave's exponentials run under another's loads and products.
        f32x16 held[kRowMaxBlocks][kBlockTiles];
        float bmax[kRowMaxBlocks], bsum[kRowMaxBlocks];
#pragma unroll
        for (int st = 0; st < kRowMaxBlocks; ++st) {
            bmax[st] = kNegInfF;
            bsum[st] = 0.0f;
        }
        auto block_cols = [&](int st) {
            const int left = s.n - (wave + Q * st) * kBlockN;
            return left < kBlockN ? left : kBlockN;
        };
#pragma unroll
        for (int st = 0; st < kRowMaxBlocks; ++st) {
            if (st >= ns) break;  // wave-uniform
#pragma unroll
            for (int kc = 0; kc < NK; ++kc) {
                const int u = NK * st + kc;
                row_write<OPS>(p, s, (wave + Q * st) * kBlockN, kc * kChunkK, end, here(lane), lw);
                wave_lds_sync();
                if (u < last) load_b(u + 1);
#pragma unroll
                for (int kk = 0; kk < kChunkK; kk += kTileK) {
                    const bf16x8 av = __builtin_bit_cast(bf16x8, a_reg[(kc * kChunkK + kk) / kTileK]);
#pragma unroll
                    for (int t = 0; t < kBlockTiles; ++t) {  // a tile past n: columns that are masked below
                        const bf16x8 bv = __builtin_bit_cast(
                            bf16x8, *reinterpret_cast<const u16x8*>(lw + (t * kTileN + li) * kLdk + kk + 8 * h));
                        held[st][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            bv, av, (kc == 0 && kk == 0) ? f32x16{} : held[st][t], 0, 0, 0);
                    }
                }
                wave_lds_sync();
            }
            if (sign != 1.0f) {
#pragma unroll
                for (int t = 0; t < kBlockTiles; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i) held[st][t][i] *= sign;
            }
            const int jn = block_cols(st);
            if (jn < kBlockN) {
                const int jh = here(jn - 4 * h);
#pragma unroll
                for (int t = 0; t < kBlockTiles; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        held[st][t][i] = t * kTileN + 8 * (i / 4) + (i % 4) < jh ? held[st][t][i] : kNegInfF;
            }
            float f[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) f[i] = higher(held[st][0][i], held[st][1][i]);
#pragma unroll
            for (int w = 8; w >= 1; w /= 2)
#pragma unroll
                for (int i = 0; i < w; ++i) f[i] = higher(f[i], f[i + w]);
            bmax[st] = c2 * f[0];
            const float ms = bmax[st] == kNegInfF ? 0.0f : bmax[st];
#pragma unroll
            for (int t = 0; t < kBlockTiles; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    held[st][t][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(held[st][t][i], c2, -ms));
#pragma unroll
            for (int i = 0; i < 16; ++i) f[i] = held[st][0][i] + held[st][1][i];
#pragma unroll
            for (int w = 8; w >= 1; w /= 2)
#pragma unroll
                for (int i = 0; i < w; ++i) f[i] += f[i + w];
            bsum[st] = f[0];
        }
        // the row's maximum and sum: the lane's blocks, the row's two lanes, the Q waves
        auto to_max = [](float m, float all) { return all == kNegInfF ? 0.0f : __builtin_amdgcn_exp2f(m - all); };
        float mx = higher(higher(bmax[0], bmax[1]), higher(bmax[2], bmax[3]));
        mx = half_pair(mx, lane, higher);
        float sum = 0.0f;
#pragma unroll
        for (int st = 0; st < kRowMaxBlocks; ++st) sum = __builtin_fmaf(bsum[st], to_max(bmax[st], mx), sum);
        sum = half_pair(sum, lane, [](float u, float v) { return u + v; });
        if (h == 0) {
            lmax[wave * kTileM + li] = mx;
            lsum[wave * kTileM + li] = sum;
        }
        __syncthreads();  // these are rewritten after the next round's barrier over A
        mx = lmax[li];
#pragma unroll
        for (int q = 1; q < Q; ++q) mx = higher(mx, lmax[q * kTileM + li]);
        float tot = 0.0f;  // in the same order in every wave
#pragma unroll
        for (int q = 0; q < Q; ++q) tot = __builtin_fmaf(lsum[q * kTileM + li], to_max(lmax[q * kTileM + li], mx), tot);
        const float inv = tot == 0.0f ? 0.0f : __builtin_amdgcn_rcpf(tot);

        const int64_t out_bidx = bidx;
        const int out_i0 = i0, out_rows = rows;
        const bool more = rounds.next(s, bidx, i0, rows);
        if (more) {
            load_a_rows();
            if (ns > 0) load_b(0);
        }
#pragma unroll
        for (int st = 0; st < kRowMaxBlocks; ++st) {
            if (st >= ns) break;
            s1_store_block<BF16OUT, TEMPORAL>(held[st], to_max(bmax[st], mx) * inv, c, s, out_bidx, out_i0, out_rows,
                                              (wave + Q * st) * kBlockN, block_cols(st), here(lane), lw);
        }
        if (wave == 0) done += static_cast<uint32_t>(out_rows);
        if (!more) return done;
    }
}

// Worker of the plain scores (NT, k <= 128): as above, each block stored as soon as its products
// are there.  The columns may be split over `slots` waves of several workgroups: `slot` is this
// wave's.
template <bool BF16OUT, int OPS, bool TEMPORAL, int NK, int Q>
__device__ __forceinline__ uint32_t row_nt_worker(const uint16_t* a, const uint16_t* b, void* c, const Shape& s,
                                                  Rounds rounds, int wave, int lane, int slot, int slots,
                                                  uint16_t* lw, uint16_t* la) {
    const int li = lane & 31;
    const int h = lane >> 5;
    const int nj = (s.n + kBlockN - 1) / kBlockN;
    uint32_t done = 0;
    int64_t bidx;
    int i0, rows;
    while (rounds.next(s, bidx, i0, rows)) {
        u16x8 p[kRowPieces];
        const uint16_t* base;
        int end;
        auto load_b = [&](int jb, int kc) {
            const int64_t at = bidx * s.b_batch + static_cast<int64_t>(jb * kBlockN) * s.k;
            base = b + at;
            const int64_t to_end = s.b_total - 8 - at;
            end = to_end < (1 << 24) ? static_cast<int>(to_end) : (1 << 24);
            row_load<OPS>(base, s, jb * kBlockN, kc * kChunkK, end, here(lane), p);
        };
        if (slot < nj) load_b(slot, 0);
        __syncthreads();  // the previous round's A is consumed
#pragma unroll
        for (int q = 0; q < 8 * NK * kTileM / (64 * Q); ++q) {
            const int e = here(lane) + 64 * wave + 64 * Q * q;
            const int r = e / (8 * NK), col = e % (8 * NK) * 8;
            const int64_t row = bidx * s.a_batch + static_cast<int64_t>(i0 + (r < rows ? r : rows - 1)) * s.k;
            *reinterpret_cast<u16x8*>(la + r * kRowLda<NK> + col) =
                keep8<OPS>(load8<OPS>(a, row, col, s.k, s.a_total), row, col, s.k, s.a_total, r < rows,
                           false);
        }
        __syncthreads();
        u16x8 a_reg[NK * (kChunkK / kTileK)];
#pragma unroll
        for (int q = 0; q < NK * (kChunkK / kTileK); ++q)
            a_reg[q] = *reinterpret_cast<const u16x8*>(la + li * kRowLda<NK> + q * kTileK + 8 * h);
        for (int jb = slot; jb < nj; jb += slots) {
            f32x16 acc[kBlockTiles];
#pragma unroll
            for (int kc = 0; kc < NK; ++kc) {
                row_write<OPS>(p, s, jb * kBlockN, kc * kChunkK, end, here(lane), lw);
                wave_lds_sync();
                if (kc + 1 < NK) load_b(jb, kc + 1);
                else if (jb + slots < nj) load_b(jb + slots, 0);
#pragma unroll
                for (int kk = 0; kk < kChunkK; kk += kTileK) {
                    const bf16x8 av = __builtin_bit_cast(bf16x8, a_reg[(kc * kChunkK + kk) / kTileK]);
#pragma unroll
                    for (int t = 0; t < kBlockTiles; ++t) {
                        const bf16x8 bv = __builtin_bit_cast(
                            bf16x8, *reinterpret_cast<const u16x8*>(lw + (t * kTileN + li) * kLdk + kk + 8 * h));
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            bv, av, (kc == 0 && kk == 0) ? f32x16{} : acc[t], 0, 0, 0);
                    }
                }
                wave_lds_sync();
            }
            const int left = s.n - jb * kBlockN;
            s1_store_block<BF16OUT, TEMPORAL>(acc, s.alpha, c, s, bidx, i0, rows, jb * kBlockN,
                                              left < kBlockN ? left : kBlockN, here(lane), lw);
        }
        if (wave == 0) done += static_cast<uint32_t>(rows);
    }
    return done;
}

// Worker of the context product (NN): wave q of Q takes the 64-deep slices q, q + Q, .. of the
// reduction for all 32 rows and one 64-column block, and the Q partial sums meet in LDS.
struct RowNnGeo {
    static constexpr bool kAReg = false;
    static constexpr int kStepK = kChunkK;
    static constexpr int kN = kBlockN;
    static constexpr int kBCols = kBlockN;
    static constexpr int kLdb = kBlockN + 8;
    static constexpr int kBPieces = kRowPieces;
    // A's rows are not padded, but their 16-byte pieces permuted by the row (eight rows' reads of
    // one column still fall on eight different pieces): padded, three workgroups' LDS took 2 KB
    // more than a CU has, and the third waited (us, padded -> this: 200 x (128 x 500)(500 x 64) 15.6 ->
    // 13.7, 438 x (64 x 333)(333 x 64) 21.9 -> 16.5, 4 x (2000 x 2000)(2000 x 128), two at most, 19.3 -> 19.4)
    __device__ __forceinline__ static int a_at(int r, int c) { return r * kChunkK + (c ^ (8 * (r & 7))); }
};
constexpr int kRowNnA = kTileM * kChunkK * 2;  // bytes of a wave's A slice
constexpr int kRowNnWaveBytes = kRowNnA + kChunkK * RowNnGeo::kLdb * 2;
constexpr int kRowLdc = kBlockN + 4;        // floats, the partial sums' row
static_assert(kRowNnWaveBytes >= kTileM * kRowLdc * 4, "a wave's partial sums fit its region");

constexpr int few_rows_lds_bytes(int layout) {
    return layout == kNN ? kRowWaves * kRowNnWaveBytes : kRowWaves * kRowWaveBytes + kTileM * kRowLda<2> * 2;
}
// Workgroups of the plain products that a CU holds: three by registers (launch bounds) and by
// LDS (160 KB, given out in pieces of 1280 bytes).
constexpr int few_rows_wgs_per_cu(int layout) {
    const int by_lds = 160 * 1024 / ((few_rows_lds_bytes(layout) + 1279) / 1280 * 1280);
    return by_lds < kWavesPerSimd ? by_lds : kWavesPerSimd;
}
constexpr int kTwoPerCuBytes = 43 * 1280;  // of which a CU gives out two
static_assert(3 * kTwoPerCuBytes > 160 * 1024);
static_assert(few_rows_wgs_per_cu(kNT) == 3 && few_rows_wgs_per_cu(kNN) == 3, "the column parts count on three");

template <bool BF16OUT, int OPS, bool TEMPORAL, int Q>
__device__ __forceinline__ uint32_t row_nn_worker(const uint16_t* a, const uint16_t* b, void* c, const Shape& s,
                                                  Rounds rounds, int wave, int lane, int jb0, int jbs, uint16_t* lds) {
    const int li = lane & 31;
    const int h = lane >> 5;
    uint16_t* const la = lds + wave * (kRowNnWaveBytes / 2);
    uint16_t* const lb = la + kRowNnA / 2;
    const int nk = (s.k + kChunkK - 1) / kChunkK;
    uint32_t done = 0;
    int64_t bidx;
    int i0, rows;
    while (rounds.next(s, bidx, i0, rows)) {
        const int64_t a_row = bidx * s.a_batch + static_cast<int64_t>(i0) * s.k;
        const int64_t b_row = bidx * s.b_batch;
        for (int j0 = jb0 * kBlockN; j0 < s.n; j0 += jbs * kBlockN) {
            f32x16 acc[kBlockTiles] = {f32x16{}, f32x16{}};
            Pieces<RowNnGeo> p;
            auto load = [&](int kc) {
                load_step<kNN, OPS, RowNnGeo>(a, a_row, b, b_row, s, rows, j0, kc * kChunkK, 0, here(lane), false, p);
            };
            if (wave < nk) load(wave);
            for (int kc = wave; kc < nk; kc += Q) {
                write_step<kNN, OPS, RowNnGeo>(p, a_row, b_row, s, rows, j0, kc * kChunkK, 0, here(lane), la, lb);
                wave_lds_sync();
                if (kc + Q < nk) load(kc + Q);
#pragma unroll
                for (int kk = 0; kk < kChunkK; kk += kTileK) {
                    const bf16x8 av = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(la + RowNnGeo::a_at(li, kk + 8 * h)));
#pragma unroll
                    for (int t = 0; t < kBlockTiles; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(nn_row_operand<RowNnGeo::kLdb>(lb, t, kk, lane),
                                                                         av, acc[t], 0, 0, 0);
                }
                wave_lds_sync();
            }
            // the partial sums, as rows, over the wave's own slices
            float* const part = reinterpret_cast<float*>(la);
#pragma unroll
            for (int t = 0; t < kBlockTiles; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<f32x4*>(part + li * kRowLdc + t * kTileN + 8 * g + 4 * h) =
                        f32x4{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
            __syncthreads();
            // wave q adds rows 8 q .. 8 q + 7 (Q = 4), eight lanes of eight columns per row
            static_assert(kTileM == 8 * Q, "the waves share the tile's rows");
            const int r = 8 * wave + (lane >> 3), col = (lane & 7) * 8;
            f32x4 v[2] = {};
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const float* from = reinterpret_cast<const float*>(lds + q * (kRowNnWaveBytes / 2)) + r * kRowLdc + col;
                v[0] += *reinterpret_cast<const f32x4*>(from);
                v[1] += *reinterpret_cast<const f32x4*>(from + 4);
            }
            v[0] *= s.alpha;
            v[1] *= s.alpha;
            const int left = s.n - j0 - col;  // columns from this lane's first one on
            const int64_t at = bidx * s.c_batch + static_cast<int64_t>(i0 + r) * s.n + j0 + col;
            if (r < rows && left > 0) {
                if constexpr (BF16OUT) {
                    uint16_t* const cp = static_cast<uint16_t*>(c) + at;
                    const u32x4 w{pack_bf16(v[0][0], v[0][1]), pack_bf16(v[0][2], v[0][3]),
                                  pack_bf16(v[1][0], v[1][1]), pack_bf16(v[1][2], v[1][3])};
                    if (left >= 8) {
                        if constexpr (TEMPORAL) *reinterpret_cast<u32x4_any*>(cp) = w;
                        else __builtin_nontemporal_store(w, reinterpret_cast<u32x4_any*>(cp));
                    } else {
                        const u16x8 e8 = __builtin_bit_cast(u16x8, w);
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (e < left) cp[e] = e8[e];
                    }
                } else {
                    float* const cp = static_cast<float*>(c) + at;
                    if (left >= 8) {
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            if constexpr (TEMPORAL) reinterpret_cast<f32x4_any*>(cp)[e] = v[e];
                            else __builtin_nontemporal_store(v[e], reinterpret_cast<f32x4_any*>(cp) + e);
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (e < left) cp[e] = v[e / 4][e % 4];
                    }
                }
            }
            __syncthreads();  // the sums are read before the regions are written again
        }
        if (wave == 0) done += static_cast<uint32_t>(rows);
    }
    return done;
}

extern __shared__ uint16_t bsm_gemm_row_lds[];  // row_lds_bytes(Q)

// Two waves per SIMD: the held products take 128 registers.
template <bool BF16OUT, int OPS, bool TEMPORAL, int NK, int Q>
__global__ void __launch_bounds__(64 * Q, kS1WavesPerSimd)
bsm_gemm_row_kernel(const uint16_t* a, const uint16_t* b, void* c, Shape s,
                    const int32_t* __restrict__ worker_ptr, const bsm_item* __restrict__ items,
                    bsm_trace_rec* __restrict__ trace) {
    const int w = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const uint64_t t0 = trace ? __builtin_amdgcn_s_memrealtime() : 0;
    uint16_t* const lw = bsm_gemm_row_lds + wave * (kRowWaveBytes / 2);
    float* const lstat = reinterpret_cast<float*>(bsm_gemm_row_lds + Q * (kRowWaveBytes / 2));
    uint16_t* const la = reinterpret_cast<uint16_t*>(lstat + 2 * Q * kTileM);
    const Rounds rounds{items, worker_ptr[w], worker_ptr[w + 1], kTileM};
    const uint32_t done = row_softmax_worker<BF16OUT, OPS, TEMPORAL, NK, Q>(a, b, c, s, rounds, wave, lane, lw, la, lstat);
    if (trace && lane == 0) write_trace(trace, w, wave, Q, done, t0);
}

// The plain products: gridDim.y parts of the columns of every worker's rows.  In a trace, the
// workgroups of the first part come first and count the rows.
template <int LAYOUT, bool BF16OUT, int OPS, bool TEMPORAL, int NK>
__global__ void __launch_bounds__(64 * kRowWaves, kWavesPerSimd)
bsm_gemm_few_rows_kernel(const uint16_t* a, const uint16_t* b, void* c, Shape s,
                         const int32_t* __restrict__ worker_ptr, const bsm_item* __restrict__ items,
                         bsm_trace_rec* __restrict__ trace) {
    constexpr int Q = kRowWaves;
    const int w = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const uint64_t t0 = trace ? __builtin_amdgcn_s_memrealtime() : 0;
    const Rounds rounds{items, worker_ptr[w], worker_ptr[w + 1], kTileM};
    uint32_t done;
    if constexpr (LAYOUT == kNT)
        done = row_nt_worker<BF16OUT, OPS, TEMPORAL, NK, Q>(a, b, c, s, rounds, wave, lane, Q * blockIdx.y + wave,
                                                            Q * gridDim.y, bsm_gemm_row_lds + wave * (kRowWaveBytes / 2),
                                                            bsm_gemm_row_lds + Q * (kRowWaveBytes / 2));
    else
        done = row_nn_worker<BF16OUT, OPS, TEMPORAL, Q>(a, b, c, s, rounds, wave, lane, blockIdx.y, gridDim.y,
                                                        bsm_gemm_row_lds);
    if (trace && lane == 0)
        write_trace(trace, w + static_cast<int>(blockIdx.y * gridDim.x), wave, Q, blockIdx.y == 0 ? done : 0, t0);
}

}  // namespace bsm_mm
