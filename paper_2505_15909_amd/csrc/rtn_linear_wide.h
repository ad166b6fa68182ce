// What the two kernels of path 3 share: the wide kernel (rtn_linear_wide.hip) and the block kernel (rtn_linear_block.h).
#pragma once
#include "rtn_device.h"
#include "rtn_internal.h"

namespace rtn {

// Kernel arguments of the block kernel, packed: a launch costs 0.3 us less per 2 KiB of them (6144 x 4096 at 64 rows 10.6 us with 4 KiB,
// 10.1 with less than 1).
struct BlockProblem {
    const half_t* A;
    const uint8_t* qw;
    const half_t* scales;
    const half_t* zeros;   // ZP only
    half_t* C;
    float* ws;
    int M, N, K;
    int G;                 // groups per row
    int XB;                // column tiles
    uint32_t u_share;      // workgroup sg covers the units (four packed tiles) sg*base + min(sg, rem), ...: base | rem << 16
    uint32_t groups;       // units per group (1 where a unit holds several) | K splits << 16 | wavefronts along K << 24
    uint32_t upg_inv;      // floor(2^32 / units per group) + 1 (0 when that is 1)
};
// Row tiles of a problem: workgroups from first on, blocks of them per K split; the first row; how many are as tall as the launch's tallest,
// the ones after them have 32 rows less; row tiles | sliced << 17 | problem << 20.  sliced: their order over the XCDs (xcd_wide_tile).
struct BlockPart {
    int first, blocks, row0, tall;
    uint32_t info;
};
constexpr int kMaxBlockParts = 2 * kMaxBlockGroup;
struct BlockGroup {
    int n;                 // parts; the first one is of the first problem
    BlockPart part[kMaxBlockParts];
    BlockProblem p[kMaxBlockGroup];
};

constexpr int kBlockThreads = 512;              // eight wavefronts
// Launch of a group of one precision (BITS), with (ZP) or without zero points; ng groups per unit, row tiles of up to mb blocks.
template <int BITS, bool ZP> hipError_t launch_block(const BlockGroup& g, int ng, int mb, unsigned grid, hipStream_t st);

namespace {

constexpr int kStepK = 128;                     // columns per k-step
constexpr uint32_t kOutOfRange = 0x7FFF0000u;   // beyond any resource size used here (< 2 GiB)
constexpr int kBufferFlags = 0x00020000;        // raw buffer, 32-bit data format

// Scales (or zero points) of one weight row: NG consecutive fp16 values, of a k-step or a unit.  A row holds a multiple of NG of
// them (K is a multiple of a unit's columns), so the loads are aligned.
template <int NG> struct RowScales { u32x4_t v[NG / 8]; };
template <> struct RowScales<1> { uint16_t v; };
template <> struct RowScales<2> { uint32_t v; };
template <> struct RowScales<4> { u32x2_t v; };

template <int NG>
__device__ __forceinline__ RowScales<NG> load_row_scales(__amdgpu_buffer_rsrc_t r, uint32_t off, int soff) {
    RowScales<NG> s;
    if constexpr (NG == 1) s.v = __builtin_amdgcn_raw_buffer_load_b16(r, off, soff, 0);
    else if constexpr (NG == 2) s.v = __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0);
    else if constexpr (NG == 4) s.v = __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0);
    else {
#pragma unroll
        for (int i = 0; i < NG / 8; ++i) s.v[i] = __builtin_amdgcn_raw_buffer_load_b128(r, off + i * 16, soff, 0);
    }
    return s;
}

template <int NG>
__device__ __forceinline__ half_t row_scale(const RowScales<NG>& s, int i) {
    if constexpr (NG == 1) return __builtin_bit_cast(half_t, s.v);
    else {
        uint32_t word;                                    // by value: bit_cast of a vector-element lvalue reads element 0
        if constexpr (NG == 2) word = s.v;
        else if constexpr (NG == 4) word = s.v[i >> 1];
        else word = s.v[i >> 3][(i >> 1) & 3];
        return __builtin_bit_cast(half2_t, word)[i & 1];
    }
}

}  // namespace

}  // namespace rtn
