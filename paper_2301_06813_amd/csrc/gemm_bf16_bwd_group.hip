// Grouped backward launch: the backward-data and backward-weight products of
// one linear in a single grid (see gemm_bf16_dma_bwd_kernel).
#include "gemm_bf16_launch.h"

namespace sbpi {

// Grouped launch of a forward-orientation and a backward-weight product
// (gemm_bf16_attn_group.hip), both with fp32 or both with bf16 outputs; acc: one
// of them (or both) is added to its output.
hipError_t launch_pair_fwd_weight(bool f32, bool acc, const Plan &p, const sbpk::GemmArgs &d,
                                  const sbpk::GemmArgs &w, int data_first, int grid,
                                  hipStream_t s);

namespace {

// ACCUM: ACC_NONE, or ACC_SOME where an unsplit product of the pair is added to its
// output (the instances of SBP_MODEL_INSTANCES and the shifted ones).
template <bool OD, bool OW, int ACCUM>
hipError_t launch_group_tile(const Plan &p, const sbpk::GemmArgsShift &ds,
                             const sbpk::GemmArgsShift &ws, int data_first, int grid,
                             hipStream_t s) {
    const sbpk::GemmArgs d = ds, w = ws;   // the unshifted kernels' arguments
    char name[192];
    const char *tf[2] = {"false", "true"};
    const char *const end[2] = {ACCUM ? ", false, true, 1>" : ">",
                                ACCUM ? ", true, true, 1>" : ", true>"};
#define SBP_BWD_CASE(BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_, SHIFT_, D_, W_)               \
    if (p.bm == BM_ && p.bn == BN_ && p.bk == BKD_ && (p.ns == 0 || p.ns == NS_) &&             \
        p.kg == KG_ && p.epi == EPI_) {                                                        \
        if (profiling())                                                                       \
            snprintf(name, sizeof(name),                                                       \
                     "gemm_bf16_dma_bwd_kernel<%d, %d, %d, %d, %d, %d, %d, %d, %s, %s%s", BM_, \
                     BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_, tf[OD], tf[OW], end[SHIFT_]);      \
        return launch_kernel(                                                                  \
            sbpk::gemm_bf16_dma_bwd_kernel<BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_, OD, OW, \
                                           SHIFT_, true, ACCUM>,                               \
            name, dim3(grid), dim3(64 * WGM_ * WGN_ * KG_), s, D_, W_, data_first);            \
    }
#define SBP_BWD_SHIFT_TILE(BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_) \
    SBP_BWD_CASE(BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_, true, ds, ws)
#define SBP_BWD_TILE(BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_) \
    SBP_BWD_CASE(BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_, false, d, w)
    if (p.shift) {
        SBP_DMA_SHIFT_INSTANCES(SBP_BWD_SHIFT_TILE)
    } else if constexpr (ACCUM == sbpk::ACC_NONE) {
        SBP_DMA_INSTANCES(SBP_BWD_TILE)
    } else {
        SBP_MODEL_INSTANCES(SBP_BWD_TILE)
    }
#undef SBP_BWD_TILE
#undef SBP_BWD_SHIFT_TILE
#undef SBP_BWD_CASE
    return hipErrorInvalidValue;
}

template <int ACCUM>
hipError_t launch_group(bool od, bool ow, const Plan &p, const sbpk::GemmArgsShift &d,
                        const sbpk::GemmArgsShift &w, int data_first, int grid, hipStream_t s) {
    if (od && ow) return launch_group_tile<true, true, ACCUM>(p, d, w, data_first, grid, s);
    if (od) return launch_group_tile<true, false, ACCUM>(p, d, w, data_first, grid, s);
    if (ow) return launch_group_tile<false, true, ACCUM>(p, d, w, data_first, grid, s);
    if constexpr (ACCUM == sbpk::ACC_NONE)
        return launch_group_tile<false, false, ACCUM>(p, d, w, data_first, grid, s);
    return hipErrorInvalidValue;   // accumulating outputs are fp32
}

}  // namespace

hipError_t launch_bf16_bwd_group(const Gemm &gd, const Plan &pd, const Gemm &gw,
                                 const Plan &pw, float *ws, hipStream_t s) {
    if (pd.bm != pw.bm || pd.bn != pw.bn || pd.bk != pw.bk || pd.ns != pw.ns || pd.kg != pw.kg ||
        pd.epi != pw.epi || pd.shift != pw.shift || !pd.dma || !pw.dma)
        return hipErrorInvalidValue;
    float *const ws_w = ws + plan_ws_floats(gd, pd);
    const sbpk::GemmArgsShift d = make_args(gd, pd, ws);
    const sbpk::GemmArgsShift w = make_args(gw, pw, ws_w);
    const int grid = d.tiles_m * d.tiles_n * d.splits * d.nbatch +
                     w.tiles_m * w.tiles_n * w.splits * w.nbatch;
    const int data_first = pd.kblk_per_split >= pw.kblk_per_split;
    const bool od = gd.out_dtype == DT_F32 || pd.splits > 1;
    const bool ow = gw.out_dtype == DT_F32 || pw.splits > 1;
    // a split product is added to its output by its reduction
    const bool acc = (gd.accumulate && pd.splits == 1) || (gw.accumulate && pw.splits == 1);
    if (gd.orient == OR_FWD) {   // batched (attention): never split, same output type
        if (od != ow || pd.splits > 1 || pw.splits > 1 || pd.shift) return hipErrorInvalidValue;
        return launch_pair_fwd_weight(od, acc, pd, d, w, data_first, grid, s);
    }
    hipError_t e = acc ? launch_group<sbpk::ACC_SOME>(od, ow, pd, d, w, data_first, grid, s)
                       : launch_group<sbpk::ACC_NONE>(od, ow, pd, d, w, data_first, grid, s);
    if (e != hipSuccess) return e;
    if (pd.splits > 1 && pw.splits > 1)
        return launch_split_reduce_pair(gd, pd.splits, ws, gw, pw.splits, ws_w, s);
    if (pd.splits > 1 && (e = launch_split_reduce(gd, pd.splits, ws, s)) != hipSuccess) return e;
    if (pw.splits > 1 && (e = launch_split_reduce(gw, pw.splits, ws_w, s)) != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace sbpi
