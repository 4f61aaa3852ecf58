// Launch wrappers exported by bsm_kernels.hip to the C-ABI layer (internal).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "bsm.h"

namespace bsm {

// Kernel classes: the longest row decides how large a register tile the kernel instance
// carries (a bigger tile costs registers, hence occupancy, for every row).
//   0: rows of <= 32 16-byte vectors   (fp32 C <= 128,  bf16 C <= 256; tiles up to 64)
//   1: <= 128 vectors                  (fp32 C <= 512,  bf16 C <= 1024)
//   2: <= 256 vectors                  (fp32 C <= 1024, bf16 C <= 2048)
//   3: <= 512 vectors                  (fp32 C <= 2048, bf16 C <= 4096)
//   4: <= 8192 elements, held by a 256-thread workgroup (up to 32 values per lane)
//   5: <= 16384 elements, held by a 256-thread workgroup (up to 64 values per lane)
//   6: any length (a 512-thread workgroup holds up to 32768 elements, longer rows read twice)
// Kernel instance for a plan whose longest row is max_cols elements.
int kernel_class_for(int32_t max_cols, int elem_bytes);

// Launches the persistent kernel: n_wg workgroups of wg_threads threads.  Worker v owns items
// [d_worker_ptr[v], d_worker_ptr[v+1]); workers are workgroups, or waves when per_wave is 1.
// shifted (the plan has rows that do not start and end on 16-byte vectors), or buffers that are not 16-byte
// aligned, select the instance with 16-byte accesses at element boundaries; temporal selects ordinary (cache-resident) instead of nontemporal
// row accesses.
hipError_t launch_softmax(bsm_dtype dtype, int kernel_class, bool shifted, bool temporal,
                          const void* in, void* out, const int32_t* d_worker_ptr,
                          const bsm_item* d_items, int n_wg, int wg_threads, int per_wave,
                          void* trace, hipStream_t stream);

// The backward op under the same table: dx = y * (dy - sum(dy * y)) per row.
hipError_t launch_softmax_backward(bsm_dtype dtype, int kernel_class, bool shifted, bool temporal,
                                   const void* y, const void* dy, void* dx,
                                   const int32_t* d_worker_ptr, const bsm_item* d_items, int n_wg,
                                   int wg_threads, int per_wave, void* trace, hipStream_t stream);

// Batched matrix product under a table whose slices are the outputs C_b (m x n each, batch
// after batch): layout 0 (NT) C_b = alpha A_b B_b^T, layout 1 (NN) C_b = alpha A_b B_b; bf16
// A and B, fp32 or bf16 C.
// Matrix-product launches: threads per workgroup, LDS bytes per workgroup, the waves per SIMD
// the kernel is compiled for, and the output rows a workgroup takes per round; single_pass:
// the one-pass score softmax (layout 2, shapes for which gemm_single_pass_shape holds).
int gemm_wg_threads();
bool gemm_single_pass_shape(int n, int k);
int gemm_lds_bytes_per_wg(bool bf16_out, bool single_pass);
int gemm_wide_lds_bytes_per_wg(bool bf16_out);  // of the forms with a 128-wide B block
bool gemm_wide_pays(int layout, bool bf16_out, int64_t batch, int m, int n, int k, int n_cu, int wgs_per_cu);
int gemm_waves_per_simd(bool single_pass);
// Workgroups per CU when the topology does not say: as many as the form the shape takes is
// compiled for.
int gemm_default_wgs_per_cu(int layout, int64_t batch, int m, int n, int k, int n_cu, bool single_pass);
int gemm_rows_per_wg(bool single_pass);

// Worker w of the table is workgroup w (gemm_wg_threads() threads, gemm_rows_per_wg() rows
// per round).  temporal: ordinary instead of nontemporal stores of C and loads of A.
// single_pass (layout 2): the one-pass form where the shape and 16-byte operands allow it,
// else the two-pass form.  wide: the forms with a 128-wide B block pay (gemm_wide_pays), and the
// plan's workgroups per CU leave room for their LDS.
hipError_t launch_gemm(int layout, bool bf16_out, bool temporal, bool single_pass, bool wide, const void* a,
                       const void* b, void* c, int64_t batch, int m, int n, int k, float alpha,
                       const int32_t* d_worker_ptr, const bsm_item* d_items, int n_wg, void* trace,
                       hipStream_t stream);

// The score softmax by row-tile workgroups of q = 4 or 8 waves (64 q threads, 32 rows per round):
// gemm_row_softmax_waves says which q a shape takes, 0 for none.
int gemm_row_lds_bytes_per_wg(int q);
int gemm_row_softmax_waves(int64_t batch, int m, int n, int k);
hipError_t launch_gemm_row(int q, bool bf16_out, bool temporal, const void* a, const void* b, void* c, int64_t batch,
                           int m, int n, int k, float alpha, const int32_t* d_worker_ptr, const bsm_item* d_items,
                           int n_wg, void* trace, hipStream_t stream);

// NT and NN by row-tile workgroups (gemm_wg_threads() threads, 32 rows per round).  parts:
// workgroups that share a worker's rows, each with its own columns; gemm_row_parts says how many
// a shape takes, 0 for the general form.
int gemm_few_rows_lds_bytes_per_wg(int layout);
int gemm_few_rows_lds_bytes_two_per_cu(int layout);  // so many that a CU holds two
int gemm_few_rows_wgs_per_cu(int layout);  // that a CU holds at once
int gemm_row_parts(int layout, bool bf16_out, int64_t batch, int m, int n, int k, int n_cu);
hipError_t launch_gemm_few_rows(int layout, int parts, int lds_bytes, bool bf16_out, bool temporal, const void* a,
                                const void* b, void* c, int64_t batch, int m, int n, int k, float alpha, const int32_t* d_worker_ptr,
                                const bsm_item* d_items, int n_wg, void* trace, hipStream_t stream);

// Workgroups of the plan's forward instance that fit on one CU at once (registers and LDS).
hipError_t resident_wgs_per_cu(bsm_dtype dtype, int kernel_class, bool shifted, int wg_threads,
                               int* n);

hipError_t launch_copy(const void* src, void* dst, int64_t bytes, int n_cu, hipStream_t stream);

// Device address of `device`'s copy of the static scratch buffer of bsm_softmax_noalloc
// (BSM_NOALLOC_SCRATCH_BYTES bytes, 256-byte aligned), looked up once per device with
// hipGetSymbolAddress; `device` must be current.
hipError_t noalloc_scratch(int device, void** ptr);

}  // namespace bsm
