// Device code of the persistent batched row-softmax kernels for gfx950 (CDNA4, wave64).
//
// One launch runs a grid of n_wg persistent workgroups.  Each worker -- a workgroup, or a
// single wave when the table is per-wave -- walks its items [worker_ptr[v], worker_ptr[v+1])
// of the host-built work table (the mapping table of the paper's Section 5: geometry is read
// per item, the instructions are the same for every patch).  A row up to the register tile is
// owned by one group of lanes of one wave (no barrier); a longer row is shared by all the
// waves of its workgroup (256 or 512 threads), which combine their partial max and sum through
// LDS.
//
// Per row (softmax over the row, the operation of the problem statement, Section 2):
//   128-bit loads (fp32, or bf16 widened to fp32; nontemporal unless the plan asks for cache-
//   resident accesses) -> lane max -> group max (DPP,
//   permlane) -> e = 2^((x - m) * log2 e) (v_exp_f32) -> lane sum (pairwise) -> group sum
//   -> y = e * (1/S) -> round-to-nearest-even to bf16 if needed -> 128-bit stores.
// Reductions combine each lane with a partner that combines the same two values in the other
// order; IEEE max and add are commutative, so every lane of a group ends with the same bits,
// and a row's result depends only on its values and length, never on the schedule.
//
// A group of G lanes (16, 32 or 64) owns one row and holds V 16-byte vectors per lane, so a
// wave covers 64/G rows at a time, with four 16-byte loads per lane in flight.  Rows longer
// than the largest register tile (512 vectors) are held in the registers of a whole workgroup
// (up to 32 values per lane in kernel class 4, 64 in classes 5 and 6, whose workgroups have 256
// and 512 threads) and read once, or, longer still, read twice with an online max/sum.  Rows whose
// start or length is not 16-byte aligned take the same paths with 16-byte accesses at element
// boundaries.  This is bandwidth-bound work: no MFMA.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "bsm.h"
#include "bsm_tile.hpp"

// No multiply-add contraction anywhere in this code: the same row may run through different
// instances (a tile's U-row and one-row forms), and a fused a*b+c in one of them would round
// differently from the other, so a row's bits would depend on the schedule.
#pragma clang fp contract(off)

namespace bsm_dev {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// 16-byte accesses at element boundaries (the same instructions as the aligned ones)
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));

constexpr float kLog2e = 1.44269504088896340736f;
constexpr float kNegInf = -__builtin_huge_valf();

__device__ __forceinline__ float bits_f(unsigned v) { return __builtin_bit_cast(float, v); }
__device__ __forceinline__ unsigned f_bits(float v) { return __builtin_bit_cast(unsigned, v); }

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// The row max uses IEEE 754-2019 maximum (NaN in, NaN out: gfx950's v_maximum3_f32), not
// fmaxf: fmaxf's NaN-ignoring form makes the compiler canonicalize every operand first (one
// extra instruction per value and per butterfly stage).  A NaN anywhere in the row makes the
// whole row NaN either way (through the max here, through the exponentials with fmaxf), and a
// max of -0 or +0 gives the same exponentials.
struct OpMax {
    __device__ __forceinline__ static float f(float a, float b) { return __builtin_elementwise_maximum(a, b); }
};
struct OpAdd {
    __device__ __forceinline__ static float f(float a, float b) { return a + b; }
};

// Reduction over aligned groups of G lanes; all lanes of a group end with identical bits.
template <int G, class Op>
__device__ __forceinline__ float group_reduce(float v) {
    static_assert(G == 8 || G == 16 || G == 32 || G == 64, "group size");
    v = Op::f(v, dpp<0xB1>(v));   // quad_perm [1,0,3,2]: partner lane ^ 1
    v = Op::f(v, dpp<0x4E>(v));   // quad_perm [2,3,0,1]: partner lane ^ 2
    v = Op::f(v, dpp<0x141>(v));  // row_half_mirror: partner in the other quad of 8
    if constexpr (G >= 16)
        v = Op::f(v, dpp<0x140>(v));  // row_mirror: partner in the other half of the 16-lane row
    if constexpr (G >= 32) {      // rows 2k and 2k+1 meet
        auto p = __builtin_amdgcn_permlane16_swap(f_bits(v), f_bits(v), false, false);
        v = Op::f(bits_f(p[0]), bits_f(p[1]));
    }
    if constexpr (G == 64) {      // the two 32-lane halves meet
        auto p = __builtin_amdgcn_permlane32_swap(f_bits(v), f_bits(v), false, false);
        v = Op::f(bits_f(p[0]), bits_f(p[1]));
    }
    return v;
}

// In-lane pairwise reduction of K values: neighbours combine in pairs, an odd last value is
// carried to the next level, until one is left (a fixed tree for each K).
template <int K, class Op>
__device__ __forceinline__ float lane_reduce(const float* x) {
    static_assert(K > 0, "lane_reduce needs a value");
    if constexpr (K == 1) {
        return x[0];
    } else {
        constexpr int H = (K + 1) / 2;
        float t[H];
#pragma unroll
        for (int i = 0; i < K / 2; ++i) t[i] = Op::f(x[2 * i], x[2 * i + 1]);
        if constexpr (K % 2 == 1) t[H - 1] = x[K - 1];
        return lane_reduce<H, Op>(t);
    }
}

// In-lane sum of a[k] g[k] by the same pairwise tree, its first level fused: a[2i] g[2i] +
// a[2i+1] g[2i+1] as one fma over one product, so that no product is held in a register of its
// own (with K products formed first, a backward row held by a lane needs 3K values at once).
template <int K>
__device__ __forceinline__ float lane_dot(const float* a, const float* g) {
    static_assert(K > 0, "lane_dot needs a value");
    if constexpr (K == 1) {
        return a[0] * g[0];
    } else {
        constexpr int H = (K + 1) / 2;
        float t[H];
#pragma unroll
        for (int i = 0; i < K / 2; ++i) t[i] = __builtin_fmaf(a[2 * i], g[2 * i], a[2 * i + 1] * g[2 * i + 1]);
        if constexpr (K % 2 == 1) t[H - 1] = a[K - 1] * g[K - 1];
        return lane_reduce<H, OpAdd>(t);
    }
}

// 16-byte accesses, nontemporal (streaming) or ordinary (cache-resident) by NT.
template <bool NT, class V>
__device__ __forceinline__ V load16(const V* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    return *p;
}
template <bool NT, class V>
__device__ __forceinline__ void store16(V* p, V v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <bool NT>
struct F32 {
    using T = float;
    static constexpr int kBytes = 4;
    static constexpr int kEPV = 4;  // elements per 16-byte vector
    using R = f32x4;  // one 16-byte vector as loaded
    __device__ __forceinline__ static R load_raw(const T* p) { return load16<NT>(reinterpret_cast<const R*>(p)); }
    __device__ __forceinline__ static R load_any(const T* p) {
        if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(p));
        return *reinterpret_cast<const f32x4_any*>(p);
    }
    __device__ __forceinline__ static void store_any(T* p, const float* y) {
        const f32x4 v{y[0], y[1], y[2], y[3]};
        if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<f32x4_any*>(p));
        else *reinterpret_cast<f32x4_any*>(p) = v;
    }
    __device__ __forceinline__ static R raw_fill(float f) { return R{f, f, f, f}; }
    __device__ __forceinline__ static void unpack(R v, float* x) {
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    }
    __device__ __forceinline__ static void store_vec(T* p, const float* y) {
        store16<NT>(reinterpret_cast<f32x4*>(p), f32x4{y[0], y[1], y[2], y[3]});
    }
    __device__ __forceinline__ static float load1(const T* p) { return *p; }
    __device__ __forceinline__ static void store1(T* p, float y) { *p = y; }
};

template <bool NT>
struct BF16 {
    using T = uint16_t;  // raw bf16 bit pattern
    static constexpr int kBytes = 2;
    static constexpr int kEPV = 8;
    using R = u32x4;  // one 16-byte vector as loaded: eight bf16 bit patterns
    __device__ __forceinline__ static R load_raw(const T* p) { return load16<NT>(reinterpret_cast<const R*>(p)); }
    __device__ __forceinline__ static R load_any(const T* p) {
        if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(p));
        return *reinterpret_cast<const u32x4_any*>(p);
    }
    __device__ __forceinline__ static void store_any(T* p, const float* y) {
        const u32x4 v{pack(y[0], y[1]), pack(y[2], y[3]), pack(y[4], y[5]), pack(y[6], y[7])};
        if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_any*>(p));
        else *reinterpret_cast<u32x4_any*>(p) = v;
    }
    // f's bf16 pattern twice per dword (exact for the fills used: -inf and 0)
    __device__ __forceinline__ static R raw_fill(float f) {
        const unsigned h = f_bits(f) >> 16;
        return R{h | (h << 16), h | (h << 16), h | (h << 16), h | (h << 16)};
    }
    __device__ __forceinline__ static void unpack(R v, float* x) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[2 * i] = bits_f(v[i] << 16);
            x[2 * i + 1] = bits_f(v[i] & 0xFFFF0000u);
        }
    }
    __device__ __forceinline__ static unsigned pack(float a, float b) {
        // round to nearest even, NaN stays NaN (v_cvt_pk_bf16_f32)
        return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
    }
    __device__ __forceinline__ static void store_vec(T* p, const float* y) {
        store16<NT>(reinterpret_cast<u32x4*>(p),
                    u32x4{pack(y[0], y[1]), pack(y[2], y[3]), pack(y[4], y[5]), pack(y[6], y[7])});
    }
    __device__ __forceinline__ static float load1(const T* p) {
        return bits_f(static_cast<unsigned>(*p) << 16);
    }
    __device__ __forceinline__ static void store1(T* p, float y) {
        *p = __builtin_bit_cast(uint16_t, static_cast<__bf16>(y));
    }
};

// The 16-byte vectors of one row of `cols` elements, dealt to STRIDE lanes: lane i holds vectors
// i, i + STRIDE, .. (slots 0, 1, ..; V of them at most, V > 1 only for rows of more than one
// slot).  An aligned row (SHIFT false: its start and length whole vectors) holds cols / EPV
// vectors from its start.  A shifted row (at least EPV elements, from any element boundary) has
// nv = ceil(cols / EPV): slot 0 from its start, the other slots up to its end, that is, moved
// back by the `sh` elements that the last vector would run past it.  Lane 0's vector of slot 1
// then starts with `sh` elements that the last vector of slot 0 holds as well.  (One slot: only
// the last vector moves.)  No access leaves the row, and nothing is loaded or stored element by
// element: both lanes that hold a duplicate compute the same value from it and store the same
// bits, and only one counts it in the row's sums (row_sum, row_dot; `mask` where a whole pass
// leaves duplicates out).  Which slot holds them is known when the code is compiled, and the
// slots past it lie at constant distances, so shifted rows need few registers that aligned ones
// do not (moving the last slot instead, known only for each row, spilled up to 53 registers more;
// moving only the last vector 124; so the shifted fp32 backward instances of classes 5 and 6 spill
// 63, 216 bytes per lane, and no other).  Before, shifted rows were read as the aligned vectors around them, with
// the outside elements masked and the first and last vectors stored element by element (GB/s,
// 30-400 MB, before -> now): forward bf16 77 2370 -> 3900, 333 3490 -> 4140, 4105 5170 -> 5210, 8193
// 2730 -> 4870; fp32 77 2380 -> 2750, 333 4470 -> 5440, 1001 5440 -> 5730, 4097 3820 -> 4940;
// backward fp32 77 4430 -> 5250, 1001 5570 -> 5770, 16383 3270 -> 4740, bf16 333 4520 -> 4560.
template <class E, bool SHIFT, int STRIDE, int V>
struct RowVecs {
    static constexpr int EPV = E::kEPV;
    int64_t start;  // element offset of the row
    int cols;
    int nv;         // vectors of the row
    __device__ __forceinline__ RowVecs(int64_t row_start, int c) : start(row_start), cols(c) {
        nv = SHIFT ? (c + EPV - 1) / EPV : c / EPV;
    }
    __device__ __forceinline__ bool in(int i, int s) const { return i + s * STRIDE < nv; }
    __device__ __forceinline__ int sh() const { return nv * EPV - cols; }
    // Elements that lane i's vector of slot s holds twice.
    __device__ __forceinline__ int dup(int i, int s) const {
        return SHIFT && (V > 1 ? s == 1 && i == 0 : i == nv - 1) ? sh() : 0;
    }
    __device__ __forceinline__ int64_t at(int i, int s) const {
        if constexpr (!SHIFT) return start + (i + s * STRIDE) * EPV;
        if constexpr (V == 1) return start + (i * EPV < cols - EPV ? i * EPV : cols - EPV);
        return (s > 0 ? start - sh() : start) + (i + s * STRIDE) * EPV;
    }
    __device__ __forceinline__ typename E::R load(const typename E::T* in, int i, int s) const {
        if constexpr (SHIFT) return E::load_any(in + at(i, s));
        return E::load_raw(in + at(i, s));
    }
    __device__ __forceinline__ void store(typename E::T* out, int i, int s, const float* y) const {
        if constexpr (SHIFT) E::store_any(out + at(i, s), y);
        else E::store_vec(out + at(i, s), y);
    }
    // Duplicates as `pad`, and a store without them, for passes that read the row again while
    // other lanes write it (in place, a duplicate may already hold its result).
    __device__ __forceinline__ void mask(int i, int s, float* x, float pad) const {
        if (SHIFT && (V == 1 || s == 1)) {
            const int d = dup(i, s);
#pragma unroll
            for (int e = 0; e < EPV; ++e) x[e] = e < d ? pad : x[e];
        }
    }
    __device__ __forceinline__ void store_own(typename E::T* out, int i, int s, const float* y) const {
        if constexpr (SHIFT) {
            const int d = dup(i, s);
            if (d > 0) {
#pragma unroll
                for (int e = 0; e < EPV; ++e)
                    if (e >= d) E::store1(out + at(i, s) + e, y[e]);
                return;
            }
        }
        store(out, i, s, y);
    }
};

// Sum of a lane's V vectors, each element of the row counted once: the tree of
// lane_reduce<V * EPV>, a vector at a time, with the duplicates left out.
template <class E, int V, bool SHIFT, int STRIDE>
__device__ __forceinline__ float row_sum(const RowVecs<E, SHIFT, STRIDE, V>& rv, int i, const float* x) {
    constexpr int EPV = E::kEPV;
    if constexpr (!SHIFT) {
        return lane_reduce<V * EPV, OpAdd>(x);
    } else {
        float sv[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (v == (V > 1 ? 1 : 0)) {
                const int d = rv.dup(i, v);
                float z[EPV];
#pragma unroll
                for (int e = 0; e < EPV; ++e) z[e] = e < d ? 0.0f : x[v * EPV + e];
                sv[v] = lane_reduce<EPV, OpAdd>(z);
            } else {
                sv[v] = lane_reduce<EPV, OpAdd>(x + v * EPV);
            }
        }
        return lane_reduce<V, OpAdd>(sv);
    }
}

// The same for the products a g (lane_dot's tree).  Both factors of a duplicate are left out: an
// infinite one times 0 would make the sum NaN.
template <class E, int V, bool SHIFT, int STRIDE>
__device__ __forceinline__ float row_dot(const RowVecs<E, SHIFT, STRIDE, V>& rv, int i, const float* a, const float* g) {
    constexpr int EPV = E::kEPV;
    if constexpr (!SHIFT) {
        return lane_dot<V * EPV>(a, g);
    } else {
        float sv[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (v == (V > 1 ? 1 : 0)) {
                const int d = rv.dup(i, v);
                float z[EPV], w[EPV];
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    z[e] = e < d ? 0.0f : a[v * EPV + e];
                    w[e] = e < d ? 0.0f : g[v * EPV + e];
                }
                sv[v] = lane_dot<EPV>(z, w);
            } else {
                sv[v] = lane_dot<EPV>(a + v * EPV, g + v * EPV);
            }
        }
        return lane_reduce<V, OpAdd>(sv);
    }
}

// Vectors of a row of `cols` elements (the last one partial, or shifted back).
template <class E>
__device__ __forceinline__ int span_vecs(int cols) {
    return (cols + E::kEPV - 1) / E::kEPV;
}

// Softmax of U rows per group, all loads first (U rows x V vectors in flight per lane).
//   row r of the item starts at element base + r * cols; rows r0, r0 + step, ...
// VEC false: element by element, for rows shorter than a vector (V = 1).
template <class E, int G, int V, int U, bool VEC, bool SHIFT = false>
__device__ __forceinline__ void rows_u(const typename E::T* in, typename E::T* out, int64_t base,
                                       int cols, int nrows, int r0, int step, int lane) {
    constexpr int EPV = E::kEPV;
    constexpr int K = V * EPV;
    float x[U][K];
    typename E::R raw[U][V];
    bool act[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = r0 + u * step;
        act[u] = r < nrows;
        const int64_t o = base + static_cast<int64_t>(r) * cols;
        if constexpr (VEC) {
            // the vectors as loaded (a lane's loads all issued before any use; unpacking
            // inside each conditional load would make every load wait for the previous one)
            const RowVecs<E, SHIFT, G, V> rv(o, cols);
#pragma unroll
            for (int v = 0; v < V; ++v)
                raw[u][v] = act[u] && rv.in(lane, v) ? rv.load(in, lane, v) : E::raw_fill(kNegInf);
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int j = lane + k * G;
                x[u][k] = (act[u] && j < cols) ? E::load1(in + o + j) : kNegInf;
            }
        }
    }
    if constexpr (VEC) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int v = 0; v < V; ++v) E::unpack(raw[u][v], &x[u][v * EPV]);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float m = group_reduce<G, OpMax>(lane_reduce<K, OpMax>(x[u]));
        const float ms = (m == kNegInf) ? 0.0f : m;  // fully masked row: every e is 0
#pragma unroll
        for (int k = 0; k < K; ++k) x[u][k] = __builtin_amdgcn_exp2f((x[u][k] - ms) * kLog2e);
        const int r = r0 + u * step;
        const int64_t o = base + static_cast<int64_t>(r) * cols;
        const RowVecs<E, SHIFT, G, V> rv(o, cols);
        const float s = group_reduce<G, OpAdd>(row_sum<E, V>(rv, lane, x[u]));
        const float inv = (s == 0.0f) ? 0.0f : __builtin_amdgcn_rcpf(s);
#pragma unroll
        for (int k = 0; k < K; ++k) x[u][k] *= inv;
        if constexpr (VEC) {
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (act[u] && rv.in(lane, v)) rv.store(out, lane, v, &x[u][v * EPV]);
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int j = lane + k * G;
                if (act[u] && j < cols) E::store1(out + o + j, x[u][k]);
            }
        }
    }
}

// The reductions of U rows held by lanes gb .. gb + n - 1 each (n <= 32, any n; i = lane - gb):
// a tree to the row's first lane (lane i < d takes lane i + d while i + d < n, d = 16, 8, 4, 2,
// 1), then one ds_bpermute from it, so every lane of a row ends with the same bits.  Each step
// is taken for all U rows before the next, so that their LDS round trips overlap.
template <class Op, int U>
__device__ __forceinline__ void seg_reduce(float (&a)[U], int i, int n, int gb) {
#pragma unroll
    for (int d = 16; d >= 1; d /= 2) {
        float o[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            o[u] = __builtin_bit_cast(
                float, __builtin_amdgcn_ds_bpermute((gb + i + d) << 2, __builtin_bit_cast(int, a[u])));
        const bool take = i < d && i + d < n;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (take) a[u] = Op::f(a[u], o[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        a[u] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(gb << 2, __builtin_bit_cast(int, a[u])));
}

// Packed tile (tile_for's G = n, not a power of two): aligned rows of n vectors, 64 / n rows side
// by side in a wave, row g on lanes [g n, g n + n), one vector per lane, U rows per group in
// flight.  A load instruction then moves 64 / n consecutive rows with almost every lane busy,
// where a power-of-two group would leave up to half of its lanes idle.
template <class E, int U>
__device__ __forceinline__ void rows_packed(const typename E::T* in, typename E::T* out,
                                            int64_t base, int n, int nrows, int r0, int step,
                                            int i, int gb, bool on) {
    constexpr int EPV = E::kEPV;
    const int cols = n * EPV;
    float x[U][EPV];
    typename E::R raw[U];
    bool act[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = r0 + u * step;
        act[u] = on && r < nrows;
        raw[u] = act[u] ? E::load_raw(in + base + static_cast<int64_t>(r) * cols + i * EPV)
                        : E::raw_fill(kNegInf);
    }
    float m[U], s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        E::unpack(raw[u], x[u]);
        m[u] = lane_reduce<EPV, OpMax>(x[u]);
    }
    seg_reduce<OpMax, U>(m, i, n, gb);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float ms = (m[u] == kNegInf) ? 0.0f : m[u];
#pragma unroll
        for (int k = 0; k < EPV; ++k) x[u][k] = __builtin_amdgcn_exp2f((x[u][k] - ms) * kLog2e);
        s[u] = lane_reduce<EPV, OpAdd>(x[u]);
    }
    seg_reduce<OpAdd, U>(s, i, n, gb);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float inv = (s[u] == 0.0f) ? 0.0f : __builtin_amdgcn_rcpf(s[u]);
#pragma unroll
        for (int k = 0; k < EPV; ++k) x[u][k] *= inv;
        if (act[u])
            E::store_vec(out + base + static_cast<int64_t>(r0 + u * step) * cols + i * EPV, x[u]);
    }
}

// One item in packed tiles, walked like run_item with 64 / n rows per wave.
template <class E, int U>
__device__ __forceinline__ uint32_t run_item_packed(const typename E::T* in, typename E::T* out,
                                                    int64_t base, int cols, int nrows, int reps,
                                                    int64_t stride, int wave, int nwaves,
                                                    int lane64) {
    const int n = cols / E::kEPV;
    const int rpw = 64 / n;
    const int sub = lane64 / n;
    const int i = lane64 - sub * n;
    const bool on = sub < rpw;
    const int gb = sub * n;
    const int step = nwaves * rpw;
    uint32_t done = 0;
    for (int k = 0; k < reps; ++k) {
        const int64_t b = base + k * stride;
        int r0 = wave * rpw;
        for (; r0 + (U - 1) * step < nrows; r0 += U * step) {
            rows_packed<E, U>(in, out, b, n, nrows, r0 + sub, step, i, gb, on);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int left = nrows - (r0 + u * step);
                done += left < rpw ? left : rpw;
            }
        }
        for (; r0 < nrows; r0 += step) {
            rows_packed<E, 1>(in, out, b, n, nrows, r0 + sub, step, i, gb, on);
            const int left = nrows - r0;
            done += left < rpw ? left : rpw;
        }
    }
    return done;
}

// One item with G lanes per row: `reps` ranges of `nrows` rows, range k starting at element
// base + k * stride.  Within a range the worker's rows are wave*RPW + sub + j*step, j = 0, 1,
// ... (RPW = 64/G rows per wave, step = rows covered by all the worker's waves at once); loop
// trip counts depend on the wave only, so lanes never diverge across iterations.
template <class E, int G, int V, int U, bool VEC, bool SHIFT>
__device__ __forceinline__ uint32_t run_item(const typename E::T* in, typename E::T* out,
                                             int64_t base, int cols, int nrows, int reps,
                                             int64_t stride, int wave, int nwaves, int lane64) {
    constexpr int RPW = 64 / G;
    const int sub = lane64 / G;
    const int lane = lane64 % G;
    const int step = nwaves * RPW;
    uint32_t done = 0;
    for (int k = 0; k < reps; ++k) {
        const int64_t b = base + k * stride;
        int r0 = wave * RPW;
        // U rows per group while the last of them still has a row; the rest one at a time, so a
        // short remainder does not pay for U rows
        for (; r0 + (U - 1) * step < nrows; r0 += U * step) {
            rows_u<E, G, V, U, VEC, SHIFT>(in, out, b, cols, nrows, r0 + sub, step, lane);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int left = nrows - (r0 + u * step);
                done += left < RPW ? left : RPW;
            }
        }
        if constexpr (U > 1) {
            for (; r0 < nrows; r0 += step) {
                rows_u<E, G, V, 1, VEC, SHIFT>(in, out, b, cols, nrows, r0 + sub, step, lane);
                const int left = nrows - r0;
                done += left < RPW ? left : RPW;
            }
        }
    }
    return done;
}

// ------------------------------------------------------------------------ workgroup rows
// Rows beyond the register tile, one row (or two) at a time per workgroup: all of its
// nt = 64 * nwaves lanes share the row, lane t holding vectors t, t + nt, ..., t + (L-1) nt (so
// each load instruction of a wave covers 1 KiB of consecutive bytes).  The row is read once
// into registers; max and sum are the in-lane tree, the wave's butterfly, then the waves'
// values combined in wave order through LDS (two barriers per row), so every lane of the
// workgroup ends with the same bits and a row's result depends on its values, its length and
// the workgroup size only.  Rows beyond L vectors per lane take two passes over HBM with a
// per-lane running max and rescaled sum, combined the same way.
constexpr int kTeamMaxRows = 2;  // rows a workgroup keeps in flight
__shared__ float team_slots[2][kTeamMaxRows][16];  // [max, sum][row][wave]: lane 0 of each wave

// Combine U values per wave (one per row) in wave order; slot set `which` is reused by the next
// rows only after the other set's barrier, which every wave reaches after reading this one.
template <class Op, int U>
__device__ __forceinline__ void team_combine(float (&v)[U], int which, int wave, int nwaves,
                                             int lane) {
    if (lane == 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) team_slots[which][u][wave] = v[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float r = team_slots[which][u][0];
        for (int i = 1; i < nwaves; ++i) r = Op::f(r, team_slots[which][u][i]);
        v[u] = r;
    }
}

// Lane t's vectors of slots s0 + c, c < L, of row rv (NT lanes to a slot); vectors past the row
// (or of an inactive row) read as `pad`.
template <class E, int L, bool SHIFT, int NT>
using TeamVecs = RowVecs<E, SHIFT, NT, (L > 1 ? L : 2)>;

template <class E, int L, bool SHIFT, int NT>
__device__ __forceinline__ void team_load(const typename E::T* in, const TeamVecs<E, L, SHIFT, NT>& rv,
                                          int t, int s0, bool act, typename E::R* raw,
                                          float pad = kNegInf) {
#pragma unroll
    for (int c = 0; c < L; ++c)
        raw[c] = (act && rv.in(t, s0 + c)) ? rv.load(in, t, s0 + c) : E::raw_fill(pad);
}

template <class E, int L>
__device__ __forceinline__ void team_unpack(const typename E::R* raw, float* x) {
#pragma unroll
    for (int c = 0; c < L; ++c) E::unpack(raw[c], x + c * E::kEPV);
}

// Duplicates of a shifted row as `pad` (passes over a row that is read twice).
template <class E, int L, bool SHIFT, int NT>
__device__ __forceinline__ void team_mask(const TeamVecs<E, L, SHIFT, NT>& rv, int t, int s0, float* x, float pad) {
#pragma unroll
    for (int c = 0; c < L; ++c) rv.mask(t, s0 + c, x + c * E::kEPV, pad);
}

template <class E, int L, bool SHIFT, int NT, bool OWN = false>
__device__ __forceinline__ void team_store(typename E::T* out, const TeamVecs<E, L, SHIFT, NT>& rv,
                                           int t, int s0, bool act, const float* y) {
#pragma unroll
    for (int c = 0; c < L; ++c) {
        if (act && rv.in(t, s0 + c)) {
            if constexpr (OWN) rv.store_own(out, t, s0 + c, y + c * E::kEPV);
            else rv.store(out, t, s0 + c, y + c * E::kEPV);
        }
    }
}

// Up to U rows (those with act[u], starting at elements off[u]) held in registers: L vectors
// per lane cover NT * L vectors of a row.  A row's arithmetic does not depend on U.
template <class E, int L, int U, bool SHIFT, int NT>
__device__ __forceinline__ void team_rows(const typename E::T* in, typename E::T* out,
                                          const int64_t (&off)[U], const bool (&act)[U], int cols,
                                          int t, int wave, int nwaves, int lane) {
    using RV = TeamVecs<E, L, SHIFT, NT>;
    constexpr int K = L * E::kEPV;
    float x[U][K];
    typename E::R raw[U][L];
#pragma unroll
    for (int u = 0; u < U; ++u)
        team_load<E, L, SHIFT, NT>(in, RV(off[u], cols), t, 0, act[u], raw[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) team_unpack<E, L>(raw[u], x[u]);
    float m[U];
#pragma unroll
    for (int u = 0; u < U; ++u) m[u] = group_reduce<64, OpMax>(lane_reduce<K, OpMax>(x[u]));
    team_combine<OpMax, U>(m, 0, wave, nwaves, lane);
    float s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float ms = (m[u] == kNegInf) ? 0.0f : m[u];
#pragma unroll
        for (int k = 0; k < K; ++k) x[u][k] = __builtin_amdgcn_exp2f((x[u][k] - ms) * kLog2e);
        s[u] = group_reduce<64, OpAdd>(row_sum<E, L>(RV(off[u], cols), t, x[u]));
    }
    team_combine<OpAdd, U>(s, 1, wave, nwaves, lane);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float inv = (s[u] == 0.0f) ? 0.0f : __builtin_amdgcn_rcpf(s[u]);
#pragma unroll
        for (int k = 0; k < K; ++k) x[u][k] *= inv;
        team_store<E, L, SHIFT, NT>(out, RV(off[u], cols), t, 0, act[u], x[u]);
    }
}

// The trace counts row j of an item's sequence for wave j mod nwaves.
__device__ __forceinline__ uint32_t team_rows_of_wave(int nrows, int reps, int wave, int nwaves) {
    const int64_t total = static_cast<int64_t>(nrows) * reps;
    return total > wave ? static_cast<uint32_t>((total - wave + nwaves - 1) / nwaves) : 0u;
}

template <int U>
struct RowWalk {
    int64_t base, stride, total, j = 0;
    int cols, nrows, k = 0, r = 0;
    __device__ RowWalk(int64_t b, int c, int n, int reps, int64_t st)
        : base(b), stride(st), total(static_cast<int64_t>(n) * reps), cols(c), nrows(n) {}
    __device__ bool more() const { return j < total; }
    __device__ void next(int64_t (&off)[U], bool (&act)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            act[u] = j < total;
            off[u] = base + k * stride + static_cast<int64_t>(r) * cols;
            if (act[u]) {
                ++j;
                if (++r == nrows) {
                    r = 0;
                    ++k;
                }
            }
        }
    }
};

// A row longer than NT * L vectors: chunks of L slots, read twice.
template <class E, int L, bool SHIFT, int NT>
__device__ __forceinline__ void team_row_two_pass(const typename E::T* in, typename E::T* out,
                                                  int64_t off, int cols, int t, int wave,
                                                  int nwaves, int lane) {
    constexpr int K = L * E::kEPV;
    const TeamVecs<E, L, SHIFT, NT> rv(off, cols);
    float m = kNegInf, s = 0.0f;
    for (int s0 = 0; s0 * NT < rv.nv; s0 += L) {
        float x[K];
        typename E::R raw[L];
        team_load<E, L, SHIFT, NT>(in, rv, t, s0, true, raw);
        team_unpack<E, L>(raw, x);
        team_mask<E, L, SHIFT, NT>(rv, t, s0, x, kNegInf);
        const float cm = lane_reduce<K, OpMax>(x);
        if (!(cm <= m)) {  // a larger maximum, or NaN, which the sum then keeps
            s *= __builtin_amdgcn_exp2f((m - cm) * kLog2e);
            m = cm;
        }
        if (m != kNegInf) {
#pragma unroll
            for (int k = 0; k < K; ++k) x[k] = __builtin_amdgcn_exp2f((x[k] - m) * kLog2e);
            s += lane_reduce<K, OpAdd>(x);
        }
    }
    float M[1] = {group_reduce<64, OpMax>(m)};
    team_combine<OpMax, 1>(M, 0, wave, nwaves, lane);
    const float Ms = (M[0] == kNegInf) ? 0.0f : M[0];
    const float scale = (m == kNegInf) ? 0.0f : __builtin_amdgcn_exp2f((m - Ms) * kLog2e);
    float S[1] = {group_reduce<64, OpAdd>(s * scale)};
    team_combine<OpAdd, 1>(S, 1, wave, nwaves, lane);
    const float inv = (S[0] == 0.0f) ? 0.0f : __builtin_amdgcn_rcpf(S[0]);
    for (int s0 = 0; s0 * NT < rv.nv; s0 += L) {
        float x[K];
        typename E::R raw[L];
        team_load<E, L, SHIFT, NT>(in, rv, t, s0, true, raw);
        team_unpack<E, L>(raw, x);
#pragma unroll
        for (int k = 0; k < K; ++k) x[k] = __builtin_amdgcn_exp2f((x[k] - Ms) * kLog2e) * inv;
        team_store<E, L, SHIFT, NT, true>(out, rv, t, s0, true, x);
    }
}

// Vectors per lane (and per input stream) of a register-held row: bsm::kTeamValues values per
// lane in kernel class 4, twice that in class 5.
template <class E, int KCLASS>
constexpr int kTeamMaxL = (KCLASS >= 5 ? 2 : 1) * bsm::kTeamValues / E::kEPV;  // 6 as 5

// Every row of an item, each by the whole workgroup.  The trace counts row r for wave
// r mod nwaves.
template <class E, int KCLASS, bool SHIFT>
__device__ __forceinline__ uint32_t team_item(const typename E::T* in, typename E::T* out,
                                              int64_t base, int cols, int nrows, int reps,
                                              int64_t stride, int wave, int nwaves, int lane) {
    constexpr int nt = bsm::team_threads(KCLASS);  // the workgroup: such plans run no other size
    const int t = wave * 64 + lane;
    const int per_lane = (span_vecs<E>(cols) + nt - 1) / nt;
    constexpr int kMaxL = kTeamMaxL<E, KCLASS>;  // 4 or 8 (class 4), 8 or 16 (class 5)
    if (per_lane <= 3) {
        // the shortest rows (at most 3 of the 4 vectors per lane): two in flight, so that a lane
        // keeps 5-6 loads outstanding (measured: 2500-element fp32 rows 5.7 TB/s against 4.9 one
        // at a time; rows filling 4 vectors per lane are 2% faster one at a time)
        RowWalk<2> w(base, cols, nrows, reps, stride);
        while (w.more()) {
            int64_t off[2];
            bool act[2];
            w.next(off, act);
            team_rows<E, 4, 2, SHIFT, nt>(in, out, off, act, cols, t, wave, nwaves, lane);
        }
    } else if (E::kBytes == 2 && kMaxL >= 6 && per_lane <= 6) {
        // bf16 rows of 5 or 6 vectors per lane (e.g. 8200 elements): two rows in flight, as for
        // the shortest rows (8200 bf16: 4.05 -> 4.3 TB/s against one row of 8 vectors per lane,
        // 5 of them used; fp32 rows lost 1.5-4% this way and keep one row of 8), in a tile of
        // exactly 5 slots where 5 suffice (8200 bf16: 4.76 -> 4.97 TB/s against 6; the
        // backward pass lost 5% with a 5-slot tile and keeps its 8)
        RowWalk<2> w(base, cols, nrows, reps, stride);
        while (w.more()) {
            int64_t off[2];
            bool act[2];
            w.next(off, act);
            if (per_lane <= 5)
                team_rows<E, (kMaxL >= 6 ? 5 : 4), 2, SHIFT, nt>(in, out, off, act, cols, t, wave,
                                                             nwaves, lane);
            else
                team_rows<E, (kMaxL >= 6 ? 6 : 4), 2, SHIFT, nt>(in, out, off, act, cols, t, wave,
                                                             nwaves, lane);
        }
    } else if (per_lane <= kMaxL) {
        RowWalk<1> w(base, cols, nrows, reps, stride);
        while (w.more()) {
            int64_t off[1];
            bool act[1];
            w.next(off, act);
            if (per_lane <= 4)
                team_rows<E, 4, 1, SHIFT, nt>(in, out, off, act, cols, t, wave, nwaves, lane);
            else if (kMaxL > 8 && per_lane <= 8)
                team_rows<E, (kMaxL > 8 ? 8 : kMaxL), 1, SHIFT, nt>(in, out, off, act, cols, t,
                                                                wave, nwaves, lane);
            else
                team_rows<E, kMaxL, 1, SHIFT, nt>(in, out, off, act, cols, t, wave, nwaves, lane);
        }
    } else {
        RowWalk<1> w(base, cols, nrows, reps, stride);
        while (w.more()) {
            int64_t off[1];
            bool act[1];
            w.next(off, act);
            team_row_two_pass<E, kMaxL, SHIFT, nt>(in, out, off[0], cols, t, wave, nwaves, lane);
        }
    }
    return team_rows_of_wave(nrows, reps, wave, nwaves);
}

// Register-tile choice per item (wave-uniform branch); the thresholds are bsm::tile_for's.
template <class E, int KCLASS, bool VEC, bool SHIFT>
__device__ __forceinline__ uint32_t dispatch_item(const typename E::T* in, typename E::T* out,
                                                  int64_t base, int cols, int nrows, int reps,
                                                  int64_t stride, int wave, int nwaves,
                                                  int lane64, bool team) {
    const int nvec = span_vecs<E>(cols);
#define BSM_RUN(G, V, U) run_item<E, G, V, U, VEC, SHIFT>(in, out, base, cols, nrows, reps, stride, wave, nwaves, lane64)
    if constexpr (VEC) {
        // the tile of bsm::tile_for: one wave-uniform branch per (G, V, U) the class can pick
        constexpr bool F = E::kBytes == 4;
        const bsm::Tile t = bsm::tile_for(nvec, KCLASS < 4 ? KCLASS : 4, E::kBytes, !SHIFT);
        if constexpr (!SHIFT && KCLASS == 0) {
            if (t.V == 1 && (t.G & (t.G - 1)) != 0)  // packed tile
                return run_item_packed<E, 4>(in, out, base, cols, nrows, reps, stride, wave,
                                             nwaves, lane64);
        }
#define BSM_TILE(g, v, u) if (t.G == g && t.V == v && t.U == u) return BSM_RUN(g, v, u)
        if constexpr (KCLASS == 0) BSM_TILE(8, 1, 4);
        BSM_TILE(16, 1, 4);
        if constexpr (F) BSM_TILE(32, 1, 8);
        BSM_TILE(32, 1, 4);
        if constexpr (KCLASS >= 1) {
            if constexpr (F) {
                BSM_TILE(32, 2, 4);
                BSM_TILE(16, 5, 1);
                BSM_TILE(64, 2, 3);
            }
            BSM_TILE(32, 2, 2);
            BSM_TILE(64, 2, 2);
        }
        if constexpr (KCLASS >= 2) {
            if constexpr (F) BSM_TILE(32, 5, 1);
            BSM_TILE(64, 4, 1);
        }
        if constexpr (KCLASS >= 3) {
            if constexpr (F) BSM_TILE(64, 5, 1);
            BSM_TILE(64, 8, 1);
        }
        if constexpr (KCLASS >= 4) {
            BSM_TILE(64, 10, 1);
            BSM_TILE(64, 12, 1);
        }
#undef BSM_TILE
    } else {
        return BSM_RUN(16, 1, 1);  // rows shorter than a vector
    }
#undef BSM_RUN
    if constexpr (VEC && KCLASS >= 4) {
        // the host gives long-row plans workgroup workers (team != 0): the waves share each row
        if (team)
            return team_item<E, KCLASS, SHIFT>(in, out, base, cols, nrows, reps, stride, wave,
                                               nwaves, lane64);
    }
    return 0;  // unreachable: the plan's class covers its longest row
}

// ------------------------------------------------------------------------------- backward
// Gradient of the row softmax (the backward pass of Section 1's batch algorithms): with y the
// forward output and dy the gradient with respect to y, dx = y * (dy - d), d = sum_j dy_j y_j.
// Same register tiles as the forward pass: d is an in-lane pairwise tree of the products, then
// the group's fixed butterfly, so the bits depend on the row's values and length only.  Two
// input streams: half as many rows per group in flight, and tiles up to 8 vectors per lane
// (longer rows are held by a workgroup).

template <class E, int G, int V, int U, bool VEC, bool SHIFT = false>
__device__ __forceinline__ void rows_u_bwd(const typename E::T* y, const typename E::T* dy,
                                           typename E::T* dx, int64_t base, int cols, int nrows,
                                           int r0, int step, int lane) {
    constexpr int EPV = E::kEPV;
    constexpr int K = V * EPV;
    if constexpr (E::kBytes == 2 && V == 8) {
        // bf16 rows of 257..512 vectors: y and dy stay packed as they were loaded (64 registers)
        // and are unpacked a vector at a time, once for d and once for dx; unpacked together
        // they take 128 registers.  Against two reads of the row (5/3 of the bytes): 64 slices of
        // 500 x 3328 179 -> 121 us, 500 x 3333 188 -> 128 us, 500 x 2056 118 -> 78 us.
        static_assert(U == 1, "one row per wave");
        const bool act = r0 < nrows;
        const RowVecs<E, SHIFT, G, V> rv(base + static_cast<int64_t>(r0) * cols, cols);
        typename E::R ra[V], rg[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const bool in = act && rv.in(lane, v);
            ra[v] = in ? rv.load(y, lane, v) : E::raw_fill(0.0f);
            rg[v] = in ? rv.load(dy, lane, v) : E::raw_fill(0.0f);
        }
        float sv[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            float a[EPV], g[EPV];
            E::unpack(ra[v], a);
            E::unpack(rg[v], g);
            if (SHIFT && v == 1) {
                const int d = rv.dup(lane, v);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    a[e] = e < d ? 0.0f : a[e];
                    g[e] = e < d ? 0.0f : g[e];
                }
            }
            sv[v] = lane_dot<EPV>(a, g);
        }
        const float d = group_reduce<G, OpAdd>(lane_reduce<V, OpAdd>(sv));
#pragma unroll
        for (int v = 0; v < V; ++v) {
            // opaque to the compiler, which would otherwise keep the values unpacked above
            asm volatile("" : "+v"(ra[v]), "+v"(rg[v]));
            float a[EPV], g[EPV];
            E::unpack(ra[v], a);
            E::unpack(rg[v], g);
#pragma unroll
            for (int e = 0; e < EPV; ++e) a[e] = a[e] * (g[e] - d);
            if (act && rv.in(lane, v)) rv.store(dx, lane, v, a);
        }
        return;
    }
    float a[U][K], g[U][K];
    typename E::R ra[U][V], rg[U][V];
    bool act[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = r0 + u * step;
        act[u] = r < nrows;
        const int64_t o = base + static_cast<int64_t>(r) * cols;
        if constexpr (VEC) {
            const RowVecs<E, SHIFT, G, V> rv(o, cols);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                if (act[u] && rv.in(lane, v)) {
                    ra[u][v] = rv.load(y, lane, v);
                    rg[u][v] = rv.load(dy, lane, v);
                } else {
                    ra[u][v] = rg[u][v] = E::raw_fill(0.0f);
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int j = lane + k * G;
                const bool in = act[u] && j < cols;
                a[u][k] = in ? E::load1(y + o + j) : 0.0f;
                g[u][k] = in ? E::load1(dy + o + j) : 0.0f;
            }
        }
    }
    if constexpr (VEC) {  // unpacked after every load is issued; vectors past the row are 0
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                E::unpack(ra[u][v], &a[u][v * EPV]);
                E::unpack(rg[u][v], &g[u][v * EPV]);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = r0 + u * step;
        const int64_t o = base + static_cast<int64_t>(r) * cols;
        const RowVecs<E, SHIFT, G, V> rv(o, cols);
        const float d = group_reduce<G, OpAdd>(row_dot<E, V>(rv, lane, a[u], g[u]));
#pragma unroll
        for (int k = 0; k < K; ++k) a[u][k] = a[u][k] * (g[u][k] - d);
        if constexpr (VEC) {
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (act[u] && rv.in(lane, v)) rv.store(dx, lane, v, &a[u][v * EPV]);
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int j = lane + k * G;
                if (act[u] && j < cols) E::store1(dx + o + j, a[u][k]);
            }
        }
    }
}

// The backward pass in packed tiles (rows of n vectors, n not a power of two, row j of a wave
// on lanes [j n, j n + n)): d = sum(dy * y) by the same tree as the forward pass's reductions,
// then dx = y (dy - d).
template <class E, int U>
__device__ __forceinline__ void rows_packed_bwd(const typename E::T* y, const typename E::T* dy,
                                                typename E::T* dx, int64_t base, int n, int nrows,
                                                int r0, int step, int i, int gb, bool on) {
    constexpr int EPV = E::kEPV;
    const int cols = n * EPV;
    float a[U][EPV], g[U][EPV];
    typename E::R ra[U], rg[U];
    bool act[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t o = base + static_cast<int64_t>(r0 + u * step) * cols + i * EPV;
        act[u] = on && r0 + u * step < nrows;
        ra[u] = act[u] ? E::load_raw(y + o) : E::raw_fill(0.0f);
        rg[u] = act[u] ? E::load_raw(dy + o) : E::raw_fill(0.0f);
    }
    float d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        E::unpack(ra[u], a[u]);
        E::unpack(rg[u], g[u]);
        d[u] = lane_dot<EPV>(a[u], g[u]);
    }
    seg_reduce<OpAdd, U>(d, i, n, gb);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int k = 0; k < EPV; ++k) a[u][k] = a[u][k] * (g[u][k] - d[u]);
        if (act[u])
            E::store_vec(dx + base + static_cast<int64_t>(r0 + u * step) * cols + i * EPV, a[u]);
    }
}

template <class E, int U>
__device__ __forceinline__ uint32_t run_item_packed_bwd(const typename E::T* y,
                                                        const typename E::T* dy,
                                                        typename E::T* dx, int64_t base, int cols,
                                                        int nrows, int reps, int64_t stride,
                                                        int wave, int nwaves, int lane64) {
    const int n = cols / E::kEPV;
    const int rpw = 64 / n;
    const int sub = lane64 / n;
    const int i = lane64 - sub * n;
    const bool on = sub < rpw;
    const int gb = sub * n;
    const int step = nwaves * rpw;
    uint32_t done = 0;
    for (int k = 0; k < reps; ++k) {
        const int64_t b = base + k * stride;
        int r0 = wave * rpw;
        for (; r0 + (U - 1) * step < nrows; r0 += U * step) {
            rows_packed_bwd<E, U>(y, dy, dx, b, n, nrows, r0 + sub, step, i, gb, on);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int left = nrows - (r0 + u * step);
                done += left < rpw ? left : rpw;
            }
        }
        for (; r0 < nrows; r0 += step) {
            rows_packed_bwd<E, 1>(y, dy, dx, b, n, nrows, r0 + sub, step, i, gb, on);
            const int left = nrows - r0;
            done += left < rpw ? left : rpw;
        }
    }
    return done;
}

template <class E, int G, int V, int U, bool VEC, bool SHIFT>
__device__ __forceinline__ uint32_t run_item_bwd(const typename E::T* y, const typename E::T* dy,
                                                 typename E::T* dx, int64_t base, int cols,
                                                 int nrows, int reps, int64_t stride, int wave,
                                                 int nwaves, int lane64) {
    constexpr int RPW = 64 / G;
    const int sub = lane64 / G;
    const int lane = lane64 % G;
    const int step = nwaves * RPW;
    uint32_t done = 0;
    for (int k = 0; k < reps; ++k) {
        const int64_t b = base + k * stride;
        int r0 = wave * RPW;
        // as run_item: U rows per group while the last of them has a row, then one at a time
        for (; r0 + (U - 1) * step < nrows; r0 += U * step) {
            rows_u_bwd<E, G, V, U, VEC, SHIFT>(y, dy, dx, b, cols, nrows, r0 + sub, step, lane);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int left = nrows - (r0 + u * step);
                done += left < RPW ? left : RPW;
            }
        }
        if constexpr (U > 1) {
            for (; r0 < nrows; r0 += step) {
                rows_u_bwd<E, G, V, 1, VEC, SHIFT>(y, dy, dx, b, cols, nrows, r0 + sub, step, lane);
                const int left = nrows - r0;
                done += left < RPW ? left : RPW;
            }
        }
    }
    return done;
}

// Backward rows beyond the register tile, one (or two) at a time per workgroup, laid out as
// in team_rows: y and dy held in registers, d = sum dy * y formed by the in-lane tree, the
// wave's butterfly and the waves' values in wave order; one barrier per rows, alternating the
// slot set (`which`), so a set is rewritten only after every wave has passed the next barrier.
template <class E, int L, int U, bool SHIFT, int NT>
__device__ __forceinline__ void team_rows_bwd(const typename E::T* y, const typename E::T* dy,
                                              typename E::T* dx, const int64_t (&off)[U],
                                              const bool (&act)[U], int cols, int t,
                                              int wave, int nwaves, int lane, int which) {
    using RV = TeamVecs<E, L, SHIFT, NT>;
    constexpr int K = L * E::kEPV;
    float a[U][K], g[U][K];
    typename E::R ra[U][L], rg[U][L];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const RV rv(off[u], cols);
        team_load<E, L, SHIFT, NT>(y, rv, t, 0, act[u], ra[u], 0.0f);  // padding: products 0
        team_load<E, L, SHIFT, NT>(dy, rv, t, 0, act[u], rg[u], 0.0f);
    }
    float d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const RV rv(off[u], cols);
        team_unpack<E, L>(ra[u], a[u]);
        team_unpack<E, L>(rg[u], g[u]);
        d[u] = group_reduce<64, OpAdd>(row_dot<E, L>(rv, t, a[u], g[u]));
    }
    team_combine<OpAdd, U>(d, which, wave, nwaves, lane);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int k = 0; k < K; ++k) a[u][k] = a[u][k] * (g[u][k] - d[u]);
        team_store<E, L, SHIFT, NT>(dx, RV(off[u], cols), t, 0, act[u], a[u]);
    }
}

// A backward row longer than NT * L vectors: d over chunks, then y and dy read again.
template <class E, int L, bool SHIFT, int NT>
__device__ __forceinline__ void team_row_bwd_two_pass(const typename E::T* y,
                                                      const typename E::T* dy, typename E::T* dx,
                                                      int64_t off, int cols, int t,
                                                      int wave, int nwaves, int lane, int which) {
    constexpr int K = L * E::kEPV;
    const TeamVecs<E, L, SHIFT, NT> rv(off, cols);
    float s = 0.0f;
    for (int s0 = 0; s0 * NT < rv.nv; s0 += L) {
        float a[K], g[K];
        typename E::R ra[L], rg[L];
        team_load<E, L, SHIFT, NT>(y, rv, t, s0, true, ra, 0.0f);
        team_load<E, L, SHIFT, NT>(dy, rv, t, s0, true, rg, 0.0f);
        team_unpack<E, L>(ra, a);
        team_unpack<E, L>(rg, g);
#pragma unroll
        for (int k = 0; k < K; ++k) g[k] *= a[k];
        team_mask<E, L, SHIFT, NT>(rv, t, s0, g, 0.0f);
        s += lane_reduce<K, OpAdd>(g);
    }
    float d[1] = {group_reduce<64, OpAdd>(s)};
    team_combine<OpAdd, 1>(d, which, wave, nwaves, lane);
    for (int s0 = 0; s0 * NT < rv.nv; s0 += L) {
        float a[K], g[K];
        typename E::R ra[L], rg[L];
        team_load<E, L, SHIFT, NT>(y, rv, t, s0, true, ra, 0.0f);
        team_load<E, L, SHIFT, NT>(dy, rv, t, s0, true, rg, 0.0f);
        team_unpack<E, L>(ra, a);
        team_unpack<E, L>(rg, g);
#pragma unroll
        for (int k = 0; k < K; ++k) a[k] = a[k] * (g[k] - d[0]);
        team_store<E, L, SHIFT, NT, true>(dx, rv, t, s0, true, a);
    }
}

template <class E, int KCLASS, bool SHIFT>
__device__ __forceinline__ uint32_t team_item_bwd(const typename E::T* y, const typename E::T* dy,
                                                  typename E::T* dx, int64_t base, int cols,
                                                  int nrows, int reps, int64_t stride, int wave,
                                                  int nwaves, int lane) {
    constexpr int nt = bsm::team_threads(KCLASS);
    const int t = wave * 64 + lane;
    const int per_lane = (span_vecs<E>(cols) + nt - 1) / nt;
    constexpr int kMaxL = kTeamMaxL<E, KCLASS>;  // vectors per lane and stream
    constexpr bool kPair = 2 * 4 * E::kEPV <= bsm::kTeamValues;  // as in team_item
    int which = 0;
    if (kPair && per_lane <= 4) {
        RowWalk<2> w(base, cols, nrows, reps, stride);
        while (w.more()) {
            int64_t off[2];
            bool act[2];
            w.next(off, act);
            team_rows_bwd<E, 4, 2, SHIFT, nt>(y, dy, dx, off, act, cols, t, wave, nwaves, lane,
                                          which);
            which ^= 1;
        }
    } else if (per_lane <= kMaxL) {
        RowWalk<1> w(base, cols, nrows, reps, stride);
        while (w.more()) {
            int64_t off[1];
            bool act[1];
            w.next(off, act);
            team_rows_bwd<E, kMaxL, 1, SHIFT, nt>(y, dy, dx, off, act, cols, t, wave, nwaves,
                                              lane, which);
            which ^= 1;
        }
    } else {
        RowWalk<1> w(base, cols, nrows, reps, stride);
        while (w.more()) {
            int64_t off[1];
            bool act[1];
            w.next(off, act);
            team_row_bwd_two_pass<E, kMaxL, SHIFT, nt>(y, dy, dx, off[0], cols, t, wave, nwaves,
                                                   lane, which);
            which ^= 1;
        }
    }
    // The next item starts again with slot set 0, which this item's last rows may have used:
    // every wave has read its slots before any wave goes on.
    __syncthreads();
    return team_rows_of_wave(nrows, reps, wave, nwaves);
}

template <class E, int KCLASS, bool VEC, bool SHIFT>
__device__ __forceinline__ uint32_t dispatch_item_bwd(const typename E::T* y,
                                                      const typename E::T* dy, typename E::T* dx,
                                                      int64_t base, int cols, int nrows, int reps,
                                                      int64_t stride, int wave, int nwaves,
                                                      int lane64, bool team) {
    const int nvec = span_vecs<E>(cols);
    if constexpr (VEC && KCLASS >= 4) {
        // rows beyond the register tile: the workgroup's waves share each row
        if (team && nvec > 512)
            return team_item_bwd<E, KCLASS, SHIFT>(y, dy, dx, base, cols, nrows, reps, stride,
                                                   wave, nwaves, lane64);
    }
#define BSM_RUN_BWD(G, V, U) run_item_bwd<E, G, V, U, VEC, SHIFT>(y, dy, dx, base, cols, nrows, reps, stride, wave, nwaves, lane64)
    if constexpr (VEC) {
        // the tile of bsm::tile_for_bwd (rows of 33..64 vectors keep 64 lanes x 1 vector: with
        // two input streams the forward pass's 32 x 2 tile measured 3% slower on 384 x 512 x
        // 512 bf16)
        constexpr bool F = E::kBytes == 4;
        const bsm::Tile t = bsm::tile_for_bwd(nvec, KCLASS < 3 ? KCLASS : 3, E::kBytes, !SHIFT);
        if constexpr (!SHIFT && KCLASS == 0) {
            if ((t.G & (t.G - 1)) != 0)  // packed tile
                return run_item_packed_bwd<E, 2>(y, dy, dx, base, cols, nrows, reps, stride, wave,
                                                 nwaves, lane64);
        }
#define BSM_TILE(g, v, u) if (t.G == g && t.V == v && t.U == u) return BSM_RUN_BWD(g, v, u)
        if constexpr (KCLASS == 0) BSM_TILE(8, 1, 2);
        BSM_TILE(16, 1, 2);
        if constexpr (F) BSM_TILE(32, 1, 4);
        BSM_TILE(32, 1, 2);
        if constexpr (KCLASS >= 1) {
            if constexpr (F) {
                BSM_TILE(64, 1, 4);
                BSM_TILE(64, 2, 2);
            }
            BSM_TILE(64, 1, 2);
            BSM_TILE(64, 2, 1);
        }
        if constexpr (KCLASS >= 2) BSM_TILE(64, 4, 1);
        if constexpr (KCLASS >= 3) BSM_TILE(64, 8, 1);
#undef BSM_TILE
    } else {
        return BSM_RUN_BWD(16, 1, 1);  // rows shorter than a vector
    }
#undef BSM_RUN_BWD
    return 0;  // unreachable: the plan's class covers its longest row
}

// Worker w of the table is workgroup w (all its waves share each item) or, when per_wave is
// set, wave (w * waves_per_workgroup + wave), which then runs its own items alone.  BWD selects
// the backward op (a = y, b = dy, out = dx); the forward op reads a only.
template <class E, int KCLASS, bool BWD, bool SHIFTED>
__device__ __forceinline__ void worker_loop(const typename E::T* a, const typename E::T* b,
                                            typename E::T* out, const int32_t* __restrict__ worker_ptr,
                                            const bsm_item* __restrict__ items, int base_aligned,
                                            int per_wave, bsm_trace_rec* __restrict__ trace) {
    const int w = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int nwaves = static_cast<int>(blockDim.x) >> 6;
    const int lane64 = static_cast<int>(threadIdx.x) & 63;
    const uint64_t t0 = trace ? __builtin_amdgcn_s_memrealtime() : 0;
    const int worker = per_wave ? w * nwaves + wave : w;
    const int my_wave = per_wave ? 0 : wave;
    const int my_nwaves = per_wave ? 1 : nwaves;
    uint32_t rows = 0;
    const int i0 = worker_ptr[worker];
    const int i1 = worker_ptr[worker + 1];
    for (int i = i0; i < i1; ++i) {
        const int64_t base = items[i].elem_offset;
        const int cols = items[i].cols;
        const int nrows = items[i].nrows;
        const int reps = items[i].reps;
        const int64_t stride = static_cast<int64_t>(items[i].rep_stride) * cols;
        // Access path: whole aligned 16-byte vectors when every row of the item starts and ends
        // on one; in the instances for plans with other rows, or launches on buffers that are
        // not 16-byte aligned (SHIFTED), vectors at element boundaries, and element by element
        // rows shorter than a vector.
        const bool whole = !SHIFTED ||
            (base_aligned && ((base | static_cast<int64_t>(cols)) & (E::kEPV - 1)) == 0);
#define BSM_ARGS cols, nrows, reps, stride, my_wave, my_nwaves, lane64
        if constexpr (BWD) {
            if (whole)
                rows += dispatch_item_bwd<E, KCLASS, true, false>(a, b, out, base, BSM_ARGS, !per_wave);
            else if (SHIFTED && cols >= E::kEPV)
                rows += dispatch_item_bwd<E, KCLASS, true, SHIFTED>(a, b, out, base, BSM_ARGS, !per_wave);
            else if constexpr (SHIFTED)
                rows += dispatch_item_bwd<E, KCLASS, false, false>(a, b, out, base, BSM_ARGS, !per_wave);
        } else {
            if (whole)
                rows += dispatch_item<E, KCLASS, true, false>(a, out, base, BSM_ARGS, !per_wave);
            else if (SHIFTED && cols >= E::kEPV)
                rows += dispatch_item<E, KCLASS, true, SHIFTED>(a, out, base, BSM_ARGS, !per_wave);
            else if constexpr (SHIFTED)
                rows += dispatch_item<E, KCLASS, false, false>(a, out, base, BSM_ARGS, !per_wave);
        }
#undef BSM_ARGS
    }
    if (trace && lane64 == 0) {
        bsm_trace_rec rec;
        rec.wg = static_cast<uint32_t>(w);
        // XCC_ID register (id 20), bits [3:0]; HW_ID register (id 4), all 32 bits
        rec.xcc_id = __builtin_amdgcn_s_getreg(20 | (0 << 6) | ((4 - 1) << 11)) & 0xF;
        rec.hw_id = __builtin_amdgcn_s_getreg(4 | (0 << 6) | ((32 - 1) << 11));
        rec.rows = rows;
        rec.t_start = t0;
        rec.t_end = __builtin_amdgcn_s_memrealtime();
        trace[static_cast<int64_t>(w) * nwaves + wave] = rec;
    }
}

// Launch bounds: any workgroup size up to 1024 threads (128 VGPRs per lane); long-row plans run
// workgroups of bsm::team_threads(class) threads (classes 4 and 5: 256, two or more per CU;
// class 6: 512, one per CU), so their rows may hold up to 256 VGPRs per lane.  bf16 plans of
// class 3 run workgroups of at most 256 threads: their 64 x 8 tile needs about 160 VGPRs (at
// 128 it spilled, 4.7-4.8 TB/s on 2304-4096-element rows; at 163 it runs three waves per SIMD,
// 5.0-5.2 TB/s).
template <class E, int KCLASS>
constexpr int kMaxThreads = KCLASS >= 4 ? bsm::team_threads(KCLASS)
                                        : (E::kBytes == 2 && KCLASS == 3 ? 256 : 1024);
template <class E, int KCLASS>
constexpr int kMinWavesPerSimd = (KCLASS >= 4 || (E::kBytes == 2 && KCLASS == 3)) ? 2 : 1;

// SHIFTED: the instance for plans with slices whose rows do not start and end on 16-byte
// vectors, and for buffers that are not 16-byte aligned (kept apart so that the other launches'
// instances carry none of its registers).
template <class E, int KCLASS, bool SHIFTED>
__global__ void __launch_bounds__((kMaxThreads<E, KCLASS>), (kMinWavesPerSimd<E, KCLASS>))
bsm_softmax_kernel(const typename E::T* in, typename E::T* out, const int32_t* __restrict__ worker_ptr,
                   const bsm_item* __restrict__ items, int base_aligned, int per_wave,
                   bsm_trace_rec* __restrict__ trace) {
    worker_loop<E, KCLASS, false, SHIFTED>(in, nullptr, out, worker_ptr, items, base_aligned,
                                           per_wave, trace);
}

// dx = softmax backward of (y, dy) under the same work table.
template <class E, int KCLASS, bool SHIFTED>
__global__ void __launch_bounds__((kMaxThreads<E, KCLASS>), (kMinWavesPerSimd<E, KCLASS>))
bsm_softmax_bwd_kernel(const typename E::T* y, const typename E::T* dy, typename E::T* dx,
                       const int32_t* __restrict__ worker_ptr, const bsm_item* __restrict__ items,
                       int base_aligned, int per_wave, bsm_trace_rec* __restrict__ trace) {
    worker_loop<E, KCLASS, true, SHIFTED>(y, dy, dx, worker_ptr, items, base_aligned, per_wave, trace);
}

}  // namespace bsm_dev
