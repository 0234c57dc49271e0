// Launch arguments of the direct CONV kernels (conv.hip, conv_tile.hip).
#pragma once

#include <cstdint>

#include "sa_device.h"
#include "structadmm.h"

namespace sa {

constexpr int kBK = 64;  // K slice per stage (= compacted row padding)

// One conv group of a launch (every group of a layer runs in one launch).
struct ConvGroup {
    const uint16_t *X;   // NHWC input, or the group's gathered Xcol rows
    const uint16_t *Wc;  // group base
    uint32_t x_bytes;
    int32_t Cx, M, K, ldk, run, run_base, o_off, mtiles, begin;
    FastDiv divRun, divMt;
};
struct ConvArgs {
    uint16_t *Y;
    float *part;          // split K: binary32 partial sums [ksplit][part_stride]
    int64_t part_stride;  // floats per chunk (N*P*Q*Cy rounded up to 4)
    int32_t ksplit, base_blocks;
    int32_t H, W, C, D, stride, pad, P, Q, NPQ, Cy;
    int32_t ldy;  // Y's row pitch (>= Cy)
    int32_t ngroups, nblocks, tiles;
    int32_t flat;  // 1x1, stride 1, no padding: output pixel = input pixel
    FastDiv divPQ, divQ, divD, divCy;
    ConvGroup g[SA_MAX_CONV_GROUPS];
};

}  // namespace sa
