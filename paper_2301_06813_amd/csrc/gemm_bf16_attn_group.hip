// Grouped launch of the two products of the attention scores' backward pass,
// dQ = dS K and dK = dS^T Q, over all (batch, head) items (see
// gemm_bf16_dma_bwd_kernel): one launch in place of two, and dS, the largest
// operand of both, is read once from HBM and once from the caches.
#include "gemm_bf16_launch.h"

namespace sbpi {

// The instances that the plan model chooses among (plan.cpp kPipe).
#define SBP_ATTN_INSTANCES(X)                                       \
    X(256, 256, 64, 2, 2, 4, 1, sbpk::EPI_DIRECT)                   \
    X(256, 192, 64, 2, 4, 2, 1, sbpk::EPI_DIRECT)                   \
    X(128, 128, 64, 2, 2, 2, 1, sbpk::EPI_DIRECT)                   \
    X(128, 64, 64, 2, 2, 2, 1, sbpk::EPI_DIRECT)                    \
    X(64, 128, 64, 2, 2, 2, 1, sbpk::EPI_DIRECT)                    \
    X(64, 64, 64, SBP_NS_64x64, 2, 2, 1, sbpk::EPI_DIRECT)          \
    X(64, 64, 64, 2, 2, 2, 1, sbpk::EPI_DIRECT)                     \
    X(128, 128, 128, 2, 2, 2, 2, sbpk::EPI_STAGED)                  \
    X(128, 64, 128, 3, 2, 2, 2, sbpk::EPI_STAGED)                   \
    X(64, 128, 128, 3, 2, 2, 2, sbpk::EPI_STAGED)                   \
    X(64, 64, 128, 4, 2, 2, 2, sbpk::EPI_STAGED)

namespace {

template <bool F32>
hipError_t launch_attn_tile(const Plan &p, const sbpk::GemmArgs &d, const sbpk::GemmArgs &w,
                            int data_first, int grid, hipStream_t s) {
    char name[192];
    const char *tf = F32 ? "true" : "false";
#define SBP_ATTN_TILE(BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_)                              \
    if (p.bm == BM_ && p.bn == BN_ && p.bk == BKD_ && (p.ns == 0 || p.ns == NS_) &&             \
        p.kg == KG_ && p.epi == EPI_) {                                                        \
        if (profiling()) snprintf(name, sizeof(name),                                                           \
                 "gemm_bf16_dma_bwd_kernel<%d, %d, %d, %d, %d, %d, %d, %d, %s, %s, false, "    \
                 "false>",                                                                     \
                 BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_, tf, tf);                          \
        return launch_kernel(                                                                  \
            sbpk::gemm_bf16_dma_bwd_kernel<BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_, F32,    \
                                           F32, false, false>,                                 \
            name, dim3(grid), dim3(64 * WGM_ * WGN_ * KG_), s, d, w, data_first);              \
    }
    SBP_ATTN_INSTANCES(SBP_ATTN_TILE)
#undef SBP_ATTN_TILE
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_pair_fwd_weight(bool f32, const Plan &p, const sbpk::GemmArgs &d,
                                  const sbpk::GemmArgs &w, int data_first, int grid,
                                  hipStream_t s) {
    return f32 ? launch_attn_tile<true>(p, d, w, data_first, grid, s)
               : launch_attn_tile<false>(p, d, w, data_first, grid, s);
}

}  // namespace sbpi
