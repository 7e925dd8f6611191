// gemm_bf16_kernel.h -- what the bf16 MFMA GEMM kernels of the local matmul of
// an SBP linear layer share (CDNA4 / gfx950): arguments, work-item order,
// output stores. The kernels themselves are in gemm_bf16_dma.h.
//
// A launch computes C[i][j] = sum_k A(i,k) B(k,j) for an m x n output over a
// reduction of length k, with fp32 accumulation, where each operand is a
// strided view read in place:
//   A_KMAJ:  A(i,k) = A[i*lda + k]   else  A(i,k) = A[k*lda + i]
//   B_KMAJ:  B(k,j) = B[j*ldb + k]   else  B(k,j) = B[k*ldb + j]
// The three local products of an SBP linear (AutoDDL Sec. 4.2 local matmul
// and its backward) are the orientations
//   forward       Y  = X  W     A k-major,  B n-major
//   backward-data dX = dY W^T   A k-major,  B k-major
//   backward-wt   dW = X^T dY   A m-major,  B n-major.
//
//   * Split reduction (splits > 1): each workgroup reduces one k-range and
//     writes its fp32 partial tile to slice `split` of a workspace laid out
//     like the output; a second kernel (split_reduce_kernel) adds the slices
//     in split order -- deterministic -- and writes the output. Kernel
//     boundaries order the two, so no device-scope fences or atomics are
//     needed (on gfx950 such fences write back and invalidate the XCD's L2).
//   * Workgroup -> tile order is XCD-aware: consecutive workgroup ids go to
//     different XCDs, so ids are remapped to give each XCD a contiguous run
//     of tiles (shared A rows / B columns stay in that XCD's L2).
//   * Any m, n, k (including k = 0, which writes zeros).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm.h"

namespace sbpk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct GemmArgs {
    const uint16_t *A;
    const uint16_t *B;
    void *C;
    int64_t lda, ldb, ldc;
    int32_t m, n, k;
    int32_t tiles_m, tiles_n;
    int32_t splits;             // reduction splits (>= 1)
    int32_t kchunk;             // reduction elements per split (a multiple of 64)
    float *ws;                  // split partials: splits slices of m x n floats,
                                // row stride partial_ld(n)
    int32_t vec_c4, vec_c8;     // C's base and ldc allow aligned 16-byte stores of
                                // 4 fp32 / 8 bf16 elements
    int32_t accumulate;         // fp32 C: add the product to C's contents
    // Batched products (the attention core): nbatch = batches x heads
    // independent m x n x k products; product z = b * heads + h reads A at
    // A + b sa_b + h sa_h (elements), likewise B, and writes C at
    // C + b sc_b + h sc_h. nbatch = 1 for a single product. Batched launches
    // never split the reduction.
    int32_t nbatch, heads;
    int64_t sa_b, sa_h, sb_b, sb_h, sc_b, sc_h;
};

// Arguments of the pipelined kernel's shifted form, for operands that start
// inside a 16-byte block (a shard view at an element offset that is not a
// multiple of 8) or whose contiguous extent is not a multiple of 8: A and B
// point at the 16-byte boundary at or below the view, and the kernel works
// in an index space shifted by the view's offset within that block --
// output rows by sm (an m-major A), output columns by sn (an n-major B), the
// reduction by sk (both operands k-major, with the same offset). Kernel row
// i is output row i - sm, and so on; reduction index kk is valid for
// sk <= kk < sk + k. kmask: the first and last reduction chunks hold
// elements outside that range (an offset, or k not a multiple of 8), which
// the kernel zeroes in LDS before those steps. The unshifted kernels take
// plain GemmArgs, and the accessors below give them zero shifts.
struct GemmArgsShift : GemmArgs {
    int32_t sm, sn, sk, kmask;
};
__device__ __forceinline__ int shift_m(const GemmArgs &) { return 0; }
__device__ __forceinline__ int shift_n(const GemmArgs &) { return 0; }
__device__ __forceinline__ int shift_k(const GemmArgs &) { return 0; }
__device__ __forceinline__ int kmask_of(const GemmArgs &) { return 0; }
__device__ __forceinline__ int shift_m(const GemmArgsShift &g) { return g.sm; }
__device__ __forceinline__ int shift_n(const GemmArgsShift &g) { return g.sn; }
__device__ __forceinline__ int shift_k(const GemmArgsShift &g) { return g.sk; }
__device__ __forceinline__ int kmask_of(const GemmArgsShift &g) { return g.kmask; }

// Operand and output bases of batch item z (uniform per work item).
template <bool OUT_F32>
__device__ __forceinline__ void batch_bases(const GemmArgs &g, int z, const uint16_t **A,
                                            const uint16_t **B, void **C) {
    *A = g.A;
    *B = g.B;
    *C = g.C;
    if (g.nbatch > 1) {
        const int64_t zb = z / g.heads, zh = z % g.heads;
        *A += zb * g.sa_b + zh * g.sa_h;
        *B += zb * g.sb_b + zh * g.sb_h;
        *C = static_cast<char *>(g.C) + (zb * g.sc_b + zh * g.sc_h) * (OUT_F32 ? 4 : 2);
    }
}

// Logical tile index of this workgroup: XCD-contiguous runs, see header.
// Tile-rows per run of the grouped tile order (measured on the 24-layer
// step: 4 rows 4.64-4.74 ms, 2 rows +0.4 %, 8 rows +0.8 %, 1 or 16 rows
// +2 %).
#ifndef SBP_TILE_GROUP
#define SBP_TILE_GROUP 4
#endif
__device__ __forceinline__ int remap_xcd(int wg, int total) {
#ifdef SBP_NO_XCD_REMAP
    return wg;
#endif
    constexpr int NX = 8;
    int per = total / NX;
    int rem = total % NX;
    int x = wg % NX;
    int idx = wg / NX;
    return (x < rem) ? x * (per + 1) + idx : rem * (per + 1) + (x - rem) * per + idx;
}

// Store of a GEMM output that this launch does not read back: non-temporal,
// so the output stream does not displace the operand tiles that other
// workgroups still re-read from L2 (measured: the step's fp32 partial-sum
// outputs 10-13 % faster, the whole step 4 %). Split partials take other
// stores (st_part).
template <typename T>
__device__ __forceinline__ void st_nt(T *p, T v) {
    __builtin_nontemporal_store(v, p);
}

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
    __bf16 h = (__bf16)f;   // round to nearest even (v_cvt_pk_bf16_f32)
    return __builtin_bit_cast(uint16_t, h);
}


}  // namespace sbpk
