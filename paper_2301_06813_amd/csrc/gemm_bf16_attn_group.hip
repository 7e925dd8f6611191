// Grouped launch of the two products of the attention scores' backward pass,
// dQ = dS K and dK = dS^T Q, over all (batch, head) items (see
// gemm_bf16_dma_bwd_kernel): one launch in place of two, and dS, the largest
// operand of both, is read once from HBM and once from the caches.
#include "gemm_bf16_launch.h"

namespace sbpi {

namespace {

template <bool F32, int ACCUM>
hipError_t launch_attn_tile(const Plan &p, const sbpk::GemmArgs &d, const sbpk::GemmArgs &w,
                            int data_first, int grid, hipStream_t s) {
    char name[192];
    const char *tf = F32 ? "true" : "false";
#define SBP_ATTN_TILE(BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_)                              \
    if (p.bm == BM_ && p.bn == BN_ && p.bk == BKD_ && (p.ns == 0 || p.ns == NS_) &&             \
        p.kg == KG_ && p.epi == EPI_) {                                                        \
        if (profiling())                                                                       \
            snprintf(name, sizeof(name),                                                       \
                     "gemm_bf16_dma_bwd_kernel<%d, %d, %d, %d, %d, %d, %d, %d, %s, %s, false, " \
                     "false%s>",                                                               \
                     BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_, tf, tf, ACCUM ? ", 1" : "");  \
        return launch_kernel(                                                                  \
            sbpk::gemm_bf16_dma_bwd_kernel<BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_, F32,    \
                                           F32, false, false, ACCUM>,                          \
            name, dim3(grid), dim3(64 * WGM_ * WGN_ * KG_), s, d, w, data_first);              \
    }
    SBP_MODEL_INSTANCES(SBP_ATTN_TILE)
#undef SBP_ATTN_TILE
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_pair_fwd_weight(bool f32, bool acc, const Plan &p, const sbpk::GemmArgs &d,
                                  const sbpk::GemmArgs &w, int data_first, int grid,
                                  hipStream_t s) {
    if (acc) return launch_attn_tile<true, sbpk::ACC_SOME>(p, d, w, data_first, grid, s);
    return f32 ? launch_attn_tile<true, sbpk::ACC_NONE>(p, d, w, data_first, grid, s)
               : launch_attn_tile<false, sbpk::ACC_NONE>(p, d, w, data_first, grid, s);
}

}  // namespace sbpi
