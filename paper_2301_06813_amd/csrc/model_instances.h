// model_instances.h -- epilogue codes, and the pipelined instances that the plan
// model chooses among (plan.cpp's kPipe, which the compiler checks against this
// list): tile, reduction step, stages, wave layout, reduction groups, epilogue.
// Only these exist as the grouped launch of an attention scores' backward pass
// and in the accumulating form.
#pragma once

namespace sbpk {

// Epilogue variants of the tile body.
enum : int {
    EPI_DIRECT = 0,   // each lane stores its MFMA elements (4-byte / 2-byte stores)
    EPI_STAGED = 1,   // tile staged in LDS, stored as 16-byte row chunks by all threads
    EPI_ROWQ = 2      // MFMA operands swapped so that each lane holds 4 consecutive
                      // outputs of one row: 16-byte (fp32) / 8-byte (bf16) stores
                      // straight from registers, no LDS and no wait
};

}  // namespace sbpk

// Stages of the four-stage tiles.
#ifndef SBP_NS_64x64
#define SBP_NS_64x64 4
#endif

#define SBP_MODEL_INSTANCES(X)                                      \
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
