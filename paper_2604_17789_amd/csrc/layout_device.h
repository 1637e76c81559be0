// Device code shared by the kernels that put a row-major MXFP4 operand into the tiled layout (layout.hip, rotq.hip).
#ifndef DUQPP_LAYOUT_DEVICE_H
#define DUQPP_LAYOUT_DEVICE_H

#include "duqpp_internal.h"

namespace duqpp {

// A unit of work is one row tile x 8 groups: 4 KiB of codes and 256 bytes of scales, moved by one wave; of scales alone 64 groups.
__host__ __device__ inline int64_t tile_units(const LayoutParams& p) {
    const int steps = p.GP / 8;
    return (int64_t)((p.rows + 31) / 32) * (p.scales_only ? (steps + 7) / 8 : steps);
}

// Scales: lane (row, h) has 32 bytes of its row's 64, which are four K steps.
__device__ __forceinline__ void tile_scales_unit(const LayoutParams& p, int64_t unit, int lane) {
    const uint32_t NI = p.GP / 8, across = (NI + 7) / 8, u = (uint32_t)unit;
    const int64_t rt = u / across;
    const int step0 = 8 * (int)(u % across) + 4 * (lane >> 5), r = lane & 31;
    const int64_t row = 32 * rt + r;
    const uint8_t* src = p.src_scales + (row < p.rows ? row : p.rows - 1) * p.G;
    uint2 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = *(const uint2*)(src + 8 * (step0 + i < (int)NI ? step0 + i : (int)NI - 1));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (step0 + i >= (int)NI) continue;
        uint32_t* dst = (uint32_t*)(p.dst_scales + (rt * NI + step0 + i) * 256 + r * 4);
        dst[0] = row < p.rows ? v[i].x : 0x7F7F7F7Fu;
        dst[32] = row < p.rows ? v[i].y : 0x7F7F7F7Fu;
    }
}

// Codes: lane (row % 8, group) of four loads reads 16 bytes, so that a row's 128 bytes are one run, and stores them at
// group * 512 + row * 16, where eight rows are a run of 128 bytes again: both sides move whole lines without LDS.  (With a
// thread per (group, row) in the order of the tiled layout the reads were 16 bytes out of every row's line.)  Rows and
// groups of the padding read a valid place and are replaced, so that no branch stands between the loads.
__device__ __forceinline__ void tile_unit(const LayoutParams& p, int64_t unit, int lane) {
    if (p.scales_only) return tile_scales_unit(p, unit, lane);
    const uint32_t NI = p.GP / 8, u = (uint32_t)unit;         // (2^32 units would be 17 TB)
    const int64_t rt = u / NI;
    const int q8 = (int)(u % NI);
    const int ch = lane & 7, r8 = lane >> 3;
    const int j = 8 * q8 + ch, jl = j < p.G ? j : p.G - 1;
    uint4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t row = 32 * rt + 8 * i + r8, rl = row < p.rows ? row : p.rows - 1;
        v[i] = *(const uint4*)(p.src_codes + (rl * p.G + jl) * 16);
    }
    const int r = lane & 31, h = lane >> 5, j0 = 8 * q8 + 4 * h;
    const int64_t srow = 32 * rt + r;
    const uint8_t* sr = p.src_scales + (srow < p.rows ? srow : p.rows - 1) * p.G;
    uint32_t s = 0;
    if ((p.G & 3) == 0 && ((uintptr_t)p.src_scales & 3) == 0) {            // the rows of scales are whole words
        s = *(const uint32_t*)(sr + (j0 < p.G ? j0 : 0));
        if (j0 >= p.G || srow >= p.rows) s = 0x7F7F7F7Fu;
    } else {
        uint32_t one[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) one[b] = sr[j0 + b < p.G ? j0 + b : 0];
        // used as loaded: or the compiler moves each load into the branch that needs it and waits there, four round trips
        // instead of one (1030 x 1056: 2.7 -> 2.2 us)
        asm("" : "+v"(one[0]), "+v"(one[1]), "+v"(one[2]), "+v"(one[3]));
#pragma unroll
        for (int b = 0; b < 4; ++b) s |= (j0 + b < p.G && srow < p.rows ? one[b] : 127u) << (8 * b);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool pad = 32 * rt + 8 * i + r8 >= p.rows || j >= p.G;
        if (pad) v[i] = make_uint4(0, 0, 0, 0);
        *(uint4*)(p.dst_codes + (rt * p.GP + j) * 512 + (8 * i + r8) * 16) = v[i];
    }
    *(uint32_t*)(p.dst_scales + unit * 256 + lane * 4) = s;
}

}  // namespace duqpp
#endif
