// Fused dequantise-GEMM for larger batches (Section 5: the same weight-only quantised linear layer,
// C = A (q S)^T, when more than a few tokens are processed at once and the matrix cores, not the weight
// stream, start to bound the time).  Two kernels, both with exact integer codes in the MFMAs and the fp16 scale
// applied in fp32 to the partial sum of each group (or of the part of a group that lies in a share of K: scaling is
// linear, so groups may straddle splits).
//
// Block kernel.  A workgroup is 8 wavefronts, 8 / WK side by side along N times WK along K; a wavefront owns 32 output columns
// and all 32 MB rows of the row tile as v_mfma_f32_32x32x16_f16 blocks.
//   - Packed weights go from global memory straight into registers in operand order: lane -> row lane & 15 of tile-row
//     (lane >> 4) & 1, 16-byte chunk 2 q + lane / 32 of a tile, so that two 1 KiB loads hold a 128-column k-step (4 bit) and
//     8 consecutive columns are one operand half.  Four k-steps are in registers.
//   - The activations of a step go from global memory straight into LDS (four stages of 64 or 128 columns), swizzled by which
//     piece a lane fetches; the reads of a 16-column slice are issued a slice ahead of its MFMAs, and the one barrier of a stage
//     stands before its last slice, whose operands are in registers by then.  Wavefronts that share no activations (WK = 8)
//     take no barrier at all.
//   - Scales come once per unit of four packed tiles, two units ahead: per-step loads of two bytes a lane touch 32 cache lines
//     each, twice as many as the weights (57344 x 8192 int4 at 32 rows 65 us with them, 52 without).
//   - The WK partial tiles are summed through LDS in a fixed order.
// What bounds it: at 128 rows on a full chip, power: with zeros for data the same launch takes 47 us instead of 66.  At 32 to 64 rows
// the weight stream and the vector instructions (unpacking: 9 per 8 weights, for MB MFMAs of 32 cycles each) overlap only
// partly.  On small matrices the 5-6 us of launch, first data and last store, which is what WK is for: K shared by
// the wavefronts of a workgroup needs no second launch.  32 x 32 blocks rather than 16 x 16: an MFMA issues every 32 cycles
// instead of 16 and leaves twice the issue slots to the unpacking.  Measured against the wide kernel in the
// shapes it had for such sizes (16 x 16 blocks, register-staged activations, a barrier a step), graph replay over rotating weights:
// int4 group 128, 64 rows 6144 x 4096 14.0 -> 9.7, 106496 x 16384 315 -> 257; 96 rows 28672 x 4096 37.3 -> 29.2; 160 rows
// 61.6 -> 46.7; group 64 with zero points, 256 rows 28672 x 4096 112 -> 80.  Tried and not kept: eight k-steps of weights in
// registers (no faster at 32 rows, 2 % slower at 64), a different first k-step per workgroup (no change), loads without the
// streaming hint (8 % slower).
//
// Wide kernel (small problems: see block_or_wide_plan).  Eight wavefronts side by side along N share the staged activations; every
// wavefront owns one 16-row weight tile-row and all 16 MB activation rows of the workgroup's row block as v_mfma_f32_16x16x32_f16
// blocks:
//   - packed weights go from global memory straight into registers in MFMA operand order, three 128-column k-steps deep;
//   - the activations of a k-step are staged through registers and LDS by the whole workgroup, double buffered, in 16-byte pieces
//     whose position inside a row is XOR-swizzled with the row number.
// What bounds it where it runs is latency: a launch of 5 to 15 us is the start, a chain of a few k-steps of half a microsecond and the
// last store.  Half the columns per workgroup and steps a quarter as long as the block kernel's units give twice the
// workgroups and a shorter chain: 4448 x 512 int4 at 29 rows 4.6 us (block kernel 6.3), 14000 x 1536 at 32 rows 7.7 (10.0), 1008 x
// 1536 g32 at 1885 rows 13.6 (17.5); from 15 us on, with 8-bit weights at up to 64 rows from 30, the block kernel is level or ahead.
//
// Row tiles beyond the first are separate workgroups that re-read the weights; the workgroup index is decoded so that the
// workgroups sharing a weight range are dispatched back to back on the same XCD and the second reader hits that XCD's L2.
#include "rtn_device.h"
#include "rtn_internal.h"
#include <algorithm>
#include <type_traits>

namespace rtn {

namespace {

constexpr int kStepK = 128;                     // columns per k-step
constexpr uint32_t kOutOfRange = 0x7FFF0000u;   // beyond any resource size used here (< 2 GiB)
constexpr int kBufferFlags = 0x00020000;        // raw buffer, 32-bit data format
constexpr int kWideThreads = 512;               // wide kernel: eight wavefronts of one tile-row each

struct WideParams {
    const half_t* A;
    const uint8_t* qw;
    const half_t* scales;
    const half_t* zeros;   // ZP only
    half_t* C;
    float* ws;
    int M, N, K;
    int G;              // groups per row
    int spg;            // k-steps per group (1 for groups of up to a k-step)
    int gps;            // groups per k-step: 1, or 2 / 4 for groups of 64 / 32 columns
    int NT;             // N / 16
    int KL;             // tiles per weight row
    int XB;             // workgroups along N
    int sliced;         // order of the column tiles over the XCDs, see xcd_wide_tile
    int ZB;             // row blocks
    int split_k;
    int ks_base, ks_rem;   // workgroup sg covers k-steps [sg*ks_base + min(sg, ks_rem), ...)
    uint32_t spg_inv;      // floor(2^32 / spg) + 1 (0 when spg == 1): k-step -> group by multiply-high
    uint32_t qw_bytes, sc_bytes, a_bytes;
};

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

// The wide kernel.  GPS: groups per k-step -- 1 (group size 128), 2 (64), 4 (32), or 0: a group spans several k-steps.  From 1 up
// every group starts its partial sums from zero, which its first MFMA takes as a constant operand instead of a cleared register,
// and is scaled as soon as its last 32-column slice is done.  ZP: the integer zero point of the step's group goes into the unpack
// (operand = q + Z).  At least two wavefronts per SIMD (256 registers each): the MFMAs then keep their accumulators in ordinary
// vector registers, where the scale multiply-add can read them directly.
template <int BITS, int MB, int GPS, bool ZP>
__global__ __launch_bounds__(kWideThreads, 2) void wide_mfma_kernel(const WideParams p) {
    constexpr int MPT = Layout<BITS>::MFMA_PER_TILE;
    constexpr int TPS = kStepK / Layout<BITS>::TK;        // tiles per k-step: 1 / 2
    constexpr int NG = GPS > 1 ? GPS : 1;                 // scales per k-step
    constexpr int SPG = 4 / NG;                           // 32-column slices per group, of those in one k-step
    constexpr int ROWS = 16 * MB;
    constexpr int BUF_BYTES = ROWS * kStepK * 2;
    __shared__ __align__(16) uint8_t lds_a[2 * BUF_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nl = lane & 15, kq = lane >> 4;

    int xb, z;                                            // N block, row block (all row blocks of one N block on one XCD)
    if (!xcd_wide_tile(blockIdx.x, p.XB, p.ZB, p.sliced != 0, &xb, &z)) return;     // padding to a multiple of 8 (whole workgroup)
    const int m0 = z * ROWS;
    const int sg = blockIdx.y;
    const int ks0 = sg * p.ks_base + min(sg, p.ks_rem);
    const int T = p.ks_base + (sg < p.ks_rem ? 1 : 0);    // k-steps of this workgroup

    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.qw), 0, p.qw_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(p.scales), 0, p.sc_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(p.A), 0, p.a_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(ZP ? p.zeros : p.scales), 0, p.sc_bytes, kBufferFlags);
    (void)rz;
    const uint32_t magic = fp16_magic_vgpr();

    const int nt = xb * (kWideThreads / 64) + wave;       // tile-row of this wavefront
    const bool nt_ok = nt < p.NT;
    // Load addresses: the lane's part goes into the vector offset, fixed for the whole kernel (out of range once and
    // for all for tile-rows and activation rows that do not exist); the k-step's part is wave-uniform and goes into the
    // scalar offset, so a step's loads cost no vector instructions.  Prefetches past the workgroup's last step load
    // that last step again (in bounds, never used).
    const uint32_t w_lane = nt_ok ? (uint32_t)nt * (uint32_t)p.KL * 1024u + lane * 16 : kOutOfRange;
    const uint32_t s_lane = nt_ok ? ((uint32_t)nt * 16 + nl) * (uint32_t)p.G * 2u : kOutOfRange;

    // ---- activation staging: thread t moves the 16-byte piece st_p of rows st_row0, st_row0 + RP, ... ----
    constexpr int RP = kWideThreads / 16;                 // rows covered by one pass of the workgroup's threads
    constexpr int NP = (ROWS + RP - 1) / RP;              // passes
    const int st_p = tid & 15, st_row0 = tid >> 4;        // row & 15 == st_row0 & 15 in every pass
    u32x4_t areg[NP];
    uint32_t a_lane[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int row = st_row0 + RP * i;
        a_lane[i] = (row < ROWS && m0 + row < p.M) ? ((uint32_t)(m0 + row) * (uint32_t)p.K + st_p * 8) * 2u : kOutOfRange;
    }
    auto a_load = [&](int t) {                            // k-step t of this workgroup (rows that do not exist: zeros)
        const int so = (int)((uint32_t)(ks0 + min(t, T - 1)) * (kStepK * 2u));
#pragma unroll
        for (int i = 0; i < NP; ++i) areg[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, a_lane[i], so, 0);
    };
    auto a_store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int row = st_row0 + RP * i;
            if (ROWS % RP == 0 || row < ROWS)
                *reinterpret_cast<u32x4_t*>(lds_a + buf * BUF_BYTES + (row * 16 + (st_p ^ (row & 15))) * 16) = areg[i];
        }
    };

    // ---- weight / scale ring, three k-steps deep ----
    u32x4_t wbuf[3][TPS];
    RowScales<NG> sbuf[3], zbuf[ZP ? 3 : 1];
    (void)zbuf;
    auto w_load = [&](int slot, int t) {
        const uint32_t ks = (uint32_t)(ks0 + min(t, T - 1));
        const uint32_t j = GPS > 0 ? ks * NG : __umulhi(ks, p.spg_inv);
        sbuf[slot] = load_row_scales<NG>(rs, s_lane, (int)(j * 2u));
        if constexpr (ZP) zbuf[slot] = load_row_scales<NG>(rz, s_lane, (int)(j * 2u));
#pragma unroll
        for (int c = 0; c < TPS; ++c)
            wbuf[slot][c] = __builtin_amdgcn_raw_buffer_load_b128(rw, w_lane, (int)((ks * TPS + c) * 1024u), 2 /* nt */);
    };

    float4_t acc[MB], part[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        acc[b] = (float4_t){0.f, 0.f, 0.f, 0.f};
        part[b] = (float4_t){0.f, 0.f, 0.f, 0.f};
    }

    // steps left in the current group when this workgroup starts (groups of several k-steps)
    int left = GPS > 0 ? 1 : p.spg - (int)((uint32_t)ks0 - __umulhi((uint32_t)ks0, p.spg_inv) * (uint32_t)p.spg);

    auto step = [&](int slot, int t) {
        a_store((t + 1) & 1);                             // A(t+1), loaded during the previous step
        a_load(t + 2);
        __builtin_amdgcn_sched_barrier(0);                // the store goes first: behind the weights' requests it cost 12 % (14000 x 1536)
        w_load((slot + 2) % 3, t + 2);
        __builtin_amdgcn_sched_barrier(0);                // keep the prefetch ahead of this step's arithmetic
        const uint8_t* abase = lds_a + (t & 1) * BUF_BYTES + (nl * 16) * 16;
        // the group, or this workgroup's share of it, ends with this step
        const bool ends = GPS > 0 ? true : ((--left == 0) || (t == T - 1));
        // the activation operands of a 32-column slice are read one slice ahead of the MFMAs that use them
        half8_t a_next[MB];
#pragma unroll
        for (int b = 0; b < MB; ++b) a_next[b] = *reinterpret_cast<const half8_t*>(abase + (b * 256 + (kq ^ nl)) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            half8_t a[MB];
#pragma unroll
            for (int b = 0; b < MB; ++b) a[b] = a_next[b];
            if (i < 3) {
#pragma unroll
                for (int b = 0; b < MB; ++b)
                    a_next[b] = *reinterpret_cast<const half8_t*>(abase + (b * 256 + (((i + 1) * 4 + kq) ^ nl)) * 16);
            }
            half8_t bw;
            if constexpr (ZP) bw = unpack_operand_zp<BITS>(wbuf[slot][i / MPT], i % MPT, magic, (float)row_scale<NG>(zbuf[slot], i / SPG));
            else bw = unpack_operand<BITS>(wbuf[slot][i / MPT], i % MPT, magic);
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                const float4_t c_in = (GPS > 0 && i % SPG == 0) ? (float4_t){0.f, 0.f, 0.f, 0.f} : part[b];
                part[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[b], bw, c_in, 0, 0, 0);
            }
            if (i % SPG == SPG - 1 && ends) {
                const float sc = (float)row_scale<NG>(sbuf[slot], i / SPG);
#pragma unroll
                for (int b = 0; b < MB; ++b) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[b][e] = fmaf(sc, part[b][e], acc[b][e]);
                    if constexpr (GPS == 0) part[b] = (float4_t){0.f, 0.f, 0.f, 0.f};
                }
            }
            if constexpr (NG > 1) {
                // pins this group's sums here: left alone the compiler keeps the partial sums of several groups alive and
                // adds them up at the end of the step, which spills
#pragma unroll
                for (int b = 0; b < MB; ++b) {
                    if (i % SPG == SPG - 1) asm volatile("" : "+v"(acc[b]));
                    else asm volatile("" : "+v"(part[b]));
                }
            }
            if (i < 3) __builtin_amdgcn_sched_barrier(0);                // keeps the next slice's reads ahead of this slice's MFMAs
        }
        if (ends) left = p.spg;
        __syncthreads();
    };

    // ---- prologue: the same issue order as in the loop (activations of a step before its weights), so that
    // the loop's waits are counted waits and not waits for everything ----
    a_load(0);
    __builtin_amdgcn_sched_barrier(0);
    w_load(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    a_store(0);
    a_load(1);
    __builtin_amdgcn_sched_barrier(0);
    w_load(1, 1);
    __syncthreads();

    int t = 0;
    for (; t + 3 <= T; t += 3) {          // no control flow between steps: every wait inside is an exact count
        step(0, t);
        step(1, t + 1);
        step(2, t + 2);
    }
    if (t < T) {
        step(0, t);
        if (t + 1 < T) step(1, t + 1);
    }

    // ---- store: lane holds rows m = 16 b + 4 kq + e, column n = 16 nt + nl ----
    if (!nt_ok) return;
    const int n = nt * 16 + nl;
#pragma unroll
    for (int b = 0; b < MB; ++b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + b * 16 + kq * 4 + e;
            if (m < p.M) {
                if (p.split_k == 1) p.C[(int64_t)m * p.N + n] = (half_t)acc[b][e];
                else p.ws[((int64_t)sg * p.M + m) * p.N + n] = acc[b][e];
            }
        }
    }
}

// 16 bytes per lane from global memory into 1 KiB of LDS at a wave-uniform address.
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, uint8_t* lds, uint32_t lane_off, int off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, lane_off, off, 0, 0);
}

// Workgroup barrier behind all but the N newest loads.  __syncthreads() would wait for all loads into LDS, those of the
// stages to come included.
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// The same with a count that is a constant once everything is inlined.  A workgroup whose wavefronts share no activations
// needs no barrier.
template <bool BARRIER>
__device__ __forceinline__ void wait_stage_n(int n) {
    if constexpr (BARRIER) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(n) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(n) : "memory");
}

typedef float float16_t __attribute__((ext_vector_type(16)));

struct BlockParams {
    const half_t* A;
    const uint8_t* qw;
    const half_t* scales;
    const half_t* zeros;   // ZP only
    half_t* C;
    float* ws;
    int M, N, K;
    int G;                 // groups per row
    int NT;                // N / 16
    int KL;                // packed tiles per weight row
    int XB, ZB, sliced;    // column tiles, row tiles, their order over the XCDs (xcd_wide_tile)
    int split_k;
    int u_base, u_rem;     // workgroup sg covers the units (four packed tiles) sg*u_base + min(sg, u_rem), ...
    int upg;               // units per group (1 where a unit holds several)
    uint32_t upg_inv;      // floor(2^32 / upg) + 1 (0 when upg == 1)
    uint32_t qw_bytes, sc_bytes;
};

// The problems of one launch: problem i has the workgroups first[i] .. first[i + 1], blocks[i] of them per K split.
struct BlockGroup {
    int n;
    int first[kMaxBlockGroup + 1], blocks[kMaxBlockGroup];
    BlockParams p[kMaxBlockGroup];
};

// Stages and depths of a shape of the block kernel.
template <int BITS, int MB, int WN, int WK>
struct BlockShape {
    static constexpr int KA = WK >= 4 || MB * WK >= 6 ? 64 : kStepK;              // columns of an activation stage, per wavefront along K
    static constexpr int R = kStepK / KA;                           // stages per k-step
    static constexpr int ROWS = 32 * MB;
    static constexpr int SLICE_BYTES = ROWS * KA * 2;               // one stage of one share of K
    static constexpr int STAGE = WK * SLICE_BYTES;
    static constexpr int S = 4 * STAGE <= 150 * 1024 ? 4 : 2;       // activation stages
    static constexpr int D = BITS == 4 ? 4 : 2;     // k-steps of weights in registers
    static constexpr int SPU = BITS == 4 ? 4 : 2;                   // k-steps per unit
    static constexpr int UN = D > 2 * SPU ? D : 2 * SPU;            // k-steps per turn of the loop: every buffer index is a literal
    static_assert(UN % D == 0 && UN % (2 * SPU) == 0 && UN * R % S == 0 && S * STAGE <= 150 * 1024, "");
};

template <int BITS, int MB, int NG, int WN, int WK, bool ZP>
__global__ __launch_bounds__(64 * WN * WK, MB == 1 ? 4 : 2) void block_mfma_kernel(const BlockGroup group) {
    int gi = 0;
    while (gi + 1 < group.n && (int)blockIdx.x >= group.first[gi + 1]) ++gi;
    const BlockParams& p = group.p[gi];
    const int local = (int)blockIdx.x - group.first[gi];
    typedef BlockShape<BITS, MB, WN, WK> Shape;
    constexpr int TPS = kStepK / Layout<BITS>::TK;        // packed tiles per k-step: 1 / 2
    constexpr int SPU = Shape::SPU, UN = Shape::UN;
    constexpr int SPG = 8 * SPU / NG;                     // 16-column slices per group, of those in a unit (8 in a k-step)
    constexpr int ROWS = Shape::ROWS, KA = Shape::KA, R = Shape::R, S = Shape::S, D = Shape::D, STAGE = Shape::STAGE;
    constexpr int PIECES = KA / 8;                        // 16-byte pieces of a staged row
    constexpr int RPI = 64 / PIECES;                      // rows per load instruction
    constexpr int SWZ = 16 / PIECES;                      // rows that share 256 bytes of LDS
    constexpr int SPS = KA / 16;                          // slices per stage
    constexpr int PD = 1;                   // slices the operand reads run ahead
    constexpr int NA = ROWS / RPI / WN;                   // activation loads per wavefront and stage
    static_assert(ROWS % (RPI * WN) == 0 && PD < SPS, "");
    __shared__ __align__(16) uint8_t lds0[STAGE], lds1[STAGE], lds2[S > 2 ? STAGE : 16], lds3[S > 2 ? STAGE : 16];
    auto stage = [&](int i) { return i == 0 ? lds0 : i == 1 ? lds1 : i == 2 ? lds2 : lds3; };

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wk = wave / WN;
    const int row = lane & 31, h = lane >> 5;

    int xb, z;
    const int sg = local / group.blocks[gi];
    if (!xcd_wide_tile(local - sg * group.blocks[gi], p.XB, p.ZB, p.sliced != 0, &xb, &z)) return;
    const int m0 = z * ROWS;
    const int u_wg = sg * p.u_base + min(sg, p.u_rem);             // units of this workgroup: u_wg .. u_wg + n_wg
    const int n_wg = p.u_base + (sg < p.u_rem ? 1 : 0);
    const int TU = (n_wg + WK - 1) / WK;                           // units every wavefront runs; those beyond its share add zeros
    const int u0 = u_wg + wk * TU;
    const int own = max(0, min(TU, n_wg - wk * TU));

    const int a_rows = min(ROWS, p.M - m0);
    half_t* a0 = const_cast<half_t*>(p.A) + (int64_t)m0 * p.K;
    const uint32_t a_bytes = (uint32_t)a_rows * (uint32_t)p.K * 2u;
    const uint32_t magic = fp16_magic_vgpr();

    // weight row of this lane: row lane & 15 of tile-row nt
    const int nt = (xb * WN + wn) * 2 + ((lane >> 4) & 1);
    const bool nt_ok = nt < p.NT;
    const uint32_t w_lane = nt_ok ? (uint32_t)nt * (uint32_t)p.KL * 1024u + (h * 16 + (lane & 15)) * 16 : kOutOfRange;
    const uint32_t s_lane = nt_ok ? ((uint32_t)nt * 16 + (lane & 15)) * (uint32_t)p.G * 2u : kOutOfRange;

    // Rows past M are zeros, not copies of the last row: they are multiplied all the same, and zeros draw less power (8B layer at
    // 200 rows, 256 multiplied: 118.9 -> 113.6 us).
    uint32_t a_lane[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int r = (wn * NA + i) * RPI + lane / PIECES;
        a_lane[i] = r < a_rows ? (uint32_t)r * (uint32_t)p.K * 2u + (uint32_t)(((lane % PIECES) ^ ((r / SWZ) % PIECES)) * 16) : kOutOfRange;
    }
    // steps past the last one request nothing: their resource is empty (zeros arrive)
    auto a_load = [&](int st, int q) {                    // stage q of this wavefront's share
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(a0, 0, q < own * SPU * R ? a_bytes : 0u, kBufferFlags);
#pragma unroll
        for (int i = 0; i < NA; ++i)
            load_to_lds(r, stage(st) + wk * Shape::SLICE_BYTES + (wn * NA + i) * 1024, a_lane[i], (u0 * SPU * R + q) * (KA * 2));
    };
    u32x4_t wbuf[D][TPS][2];
    auto w_load = [&](int slot, int t) {                  // k-step t of this wavefront's share
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.qw), 0, t < own * SPU ? p.qw_bytes : 0u, kBufferFlags);
#pragma unroll
        for (int c = 0; c < TPS; ++c)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                wbuf[slot][c][q] = __builtin_amdgcn_raw_buffer_load_b128(rw, w_lane + q * 512, ((u0 * SPU + t) * TPS + c) * 1024, 2 /* nt */);
    };
    RowScales<NG> sbuf[2], zbuf[ZP ? 2 : 1];
    (void)zbuf;
    auto s_load = [&](int slot, int u) {                  // unit u of this wavefront's share
        const uint32_t unit = (uint32_t)(u0 + u);
        const uint32_t j = NG > 1 ? unit * NG : (p.upg_inv == 0 ? unit : __umulhi(unit, p.upg_inv));
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(p.scales), 0, u < own ? p.sc_bytes : 0u, kBufferFlags);
        sbuf[slot] = load_row_scales<NG>(rs, s_lane, (int)(j * 2u));
        if constexpr (ZP) {
            const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(p.zeros), 0, u < own ? p.sc_bytes : 0u, kBufferFlags);
            zbuf[slot] = load_row_scales<NG>(rz, s_lane, (int)(j * 2u));
        }
    };
    // weight operand of slice s of step v (mod UN)
    auto operand = [&](int v, int s) {
        const u32x4_t& chunk = wbuf[v % D][BITS == 4 ? 0 : s >> 2][s & 1];
        const int i = BITS == 4 ? s >> 1 : (s >> 1) & 1;
        if constexpr (ZP) return unpack_operand_zp<BITS>(chunk, i, magic, (float)row_scale<NG>(zbuf[v / SPU % 2], ((v % SPU) * 8 + s) / SPG));
        else return unpack_operand<BITS>(chunk, i, magic);
    };

    float16_t acc[MB], part[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) { acc[b][e] = 0.f; part[b][e] = 0.f; }

    half8_t aop[PD + 1][MB];
    // piece 2 s + h of a row stands at slot (2 s + h) ^ (row's swizzle): one exclusive-or per slice on the lane's own address
    const uint32_t rd = wk * Shape::SLICE_BYTES + row * (KA * 2) + ((h ^ ((row / SWZ) % PIECES)) * 16);
    auto a_read = [&](int st, int s) {                    // operands of slice s of a step
        uint32_t o = rd;
        if (s % SPS) asm volatile("v_xor_b32 %0, %1, %2" : "=v"(o) : "n"((s % SPS) * 32), "v"(rd));
#pragma unroll
        for (int b = 0; b < MB; ++b) aop[s % (PD + 1)][b] = *reinterpret_cast<const half8_t*>(stage(st) + o + b * (32 * KA * 2));
    };

    // Weight loads requested since the stage after stage rr of a step (those of older steps have been used).  Scales are not
    // counted: a unit's wait is for a load more than it need be.
    auto weights_since = [](int rr) {
        int n = 0;
        for (int j = rr + 1 - S > rr - D * R ? rr + 1 - S : rr - D * R; j < rr; ++j) n += (j + 64 * R) % R == R - 1 ? 2 * TPS : 0;
        return n;
    };
    auto wait_stage = [&](int n) { wait_stage_n<(WN > 1)>(n); };

    int left = p.upg - (int)((uint32_t)u0 - (p.upg_inv == 0 ? (uint32_t)u0 : __umulhi((uint32_t)u0, p.upg_inv)) * (uint32_t)p.upg);
    half8_t bw;

    // k-step t, v = t mod UN.  tail: no weights are requested any more
    auto step = [&](int v, int t, bool tail) {
        const bool unit_ends = NG > 1 || v % SPU != SPU - 1 ? false : ((--left == 0) || t == own * SPU - 1);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int r = s / SPS, us = (v % SPU) * 8 + s; // stage of the step, slice of the unit
            const bool turn = s % SPS == SPS - PD;        // the operands of the rest of the stage are in registers: it is free
            if (turn) {
                // the next stage has landed: only what was requested after it may be outstanding
                if (tail) wait_stage((S - 2) * NA);
                else wait_stage((S - 2) * NA + weights_since(r));
                __builtin_amdgcn_sched_barrier(0);
            }
            a_read((v * R + (s + PD) / SPS) % S, (s + PD) % 8);
            const half8_t b_now = bw;
            bw = s == 7 ? operand((v + 1) % UN, 0) : operand(v, s + 1);
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                float16_t c_in;
                if (NG > 1 && us % SPG == 0) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) c_in[e] = 0.f;
                } else c_in = part[b];
                part[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(aop[s % (PD + 1)][b], b_now, c_in, 0, 0, 0);
            }
            if (turn) {
                __builtin_amdgcn_sched_barrier(0);
                a_load((v * R + r) % S, t * R + r + S);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (us % SPG == SPG - 1) {
                if (NG > 1 || unit_ends) {
                    const float sc = (float)row_scale<NG>(sbuf[v / SPU % 2], us / SPG);
#pragma unroll
                    for (int b = 0; b < MB; ++b) {
#pragma unroll
                        for (int e = 0; e < 16; ++e) acc[b][e] = fmaf(sc, part[b][e], acc[b][e]);
                        if constexpr (NG == 1)
#pragma unroll
                            for (int e = 0; e < 16; ++e) part[b][e] = 0.f;
                    }
                }
                // pins the sums here, as in the wide kernel
#pragma unroll
                for (int b = 0; b < MB; ++b) asm volatile("" : "+v"(acc[b]));
            } else if constexpr (SPG < 8) {
#pragma unroll
                for (int b = 0; b < MB; ++b) asm volatile("" : "+v"(part[b]));
            }
            if (s == 7 && !tail) {
                __builtin_amdgcn_sched_barrier(0);
                w_load(v % D, t + D);
                if (v % SPU == SPU - 1) s_load(v / SPU % 2, t / SPU + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (NG == 1 && unit_ends) left = p.upg;
    };

    // ---- prologue: the requests of the steps before the first one, in the order of the loop (its waits are counts) ----
    s_load(0, 0);
    s_load(1, 1);
    constexpr int AHEAD = S > D * R ? S : D * R;
#pragma unroll
    for (int q = -AHEAD; q < 0; ++q) {
        __builtin_amdgcn_sched_barrier(0);
        if (q >= -S) a_load(q + S, q + S);
        __builtin_amdgcn_sched_barrier(0);
        if (q >= -D * R && (q + AHEAD * R) % R == R - 1) w_load((q + D * R) / R, (q + D * R) / R);
        __builtin_amdgcn_sched_barrier(0);
    }
    wait_stage((S - 1) * NA + weights_since(0));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < PD; ++s) a_read(0, s);
    bw = operand(0, 0);
    __builtin_amdgcn_sched_barrier(0);

    int t = 0;
    for (; t + UN <= TU * SPU; t += UN) {                 // no control flow between steps: every wait inside is an exact count
#pragma unroll
        for (int v = 0; v < UN; ++v) step(v, t + v, false);
    }
    if (t < TU * SPU) {                                   // an odd unit
#pragma unroll
        for (int v = 0; v < SPU; ++v) step(v, t + v, true);
    }
    wait_and_barrier<0>();                                // no load into LDS outlives the workgroup

    // Lane holds column 16 nt + (lane & 15), rows m0 + 32 b + 8 (e / 4) + 4 h + e % 4.  Rows past M and columns
    // past N are outside the resource and dropped by the hardware (a row tile of results is under 2 GiB, see the launch).
    auto finish = [&](auto partial) {
        constexpr uint32_t BYTES = partial.value ? 4 : 2;
        const uint32_t row_bytes = (uint32_t)p.N * BYTES;
        const __amdgpu_buffer_rsrc_t rc = partial.value
            ? __builtin_amdgcn_make_buffer_rsrc(p.ws + ((int64_t)sg * p.M + m0) * p.N, 0, (uint32_t)a_rows * row_bytes, kBufferFlags)
            : __builtin_amdgcn_make_buffer_rsrc(p.C + (int64_t)m0 * p.N, 0, (uint32_t)a_rows * row_bytes, kBufferFlags);
        const uint32_t c_lane = nt_ok ? h * 4 * row_bytes + (uint32_t)(nt * 16 + (lane & 15)) * BYTES : 0x80000000u;
        auto store = [&](int b, int e, float v) {
            const uint32_t off = c_lane + (uint32_t)(b * 32 + (e >> 2) * 8 + (e & 3)) * row_bytes;
            if constexpr (partial.value) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rc, off, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, (half_t)v), rc, off, 0, 0);
        };
        if constexpr (WK == 1) {
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e) store(b, e, acc[b][e]);
        } else {
            // the WK partial tiles through the first stage, EC elements a round, each wavefront summing its part of them in order
            constexpr int EC = STAGE >= WN * WK * 4096 ? 16 : STAGE >= WN * WK * 2048 ? 8 : 4;
            static_assert(EC % WK == 0 && EC * WN * WK * 256 <= STAGE, "");
            float* buf = reinterpret_cast<float*>(lds0);
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int e0 = 0; e0 < 16; e0 += EC) {
                    if (b + e0 > 0) __syncthreads();
#pragma unroll
                    for (int e = 0; e < EC; ++e) buf[(wave * EC + e) * 64 + lane] = acc[b][e0 + e];
                    __syncthreads();
                    float v[EC / WK][WK];
#pragma unroll
                    for (int e = 0; e < EC / WK; ++e)
#pragma unroll
                        for (int k = 0; k < WK; ++k) v[e][k] = buf[((k * WN + wn) * EC + wk * (EC / WK) + e) * 64 + lane];
#pragma unroll
                    for (int e = 0; e < EC / WK; ++e) {
                        float sum = v[e][0];
#pragma unroll
                        for (int k = 1; k < WK; ++k) sum += v[e][k];
                        store(b, e0 + wk * (EC / WK) + e, sum);
                    }
                }
        }
    };
    if (p.split_k == 1) finish(std::false_type{});
    else finish(std::true_type{});
}

template <int BITS, int MB, int WN, int WK, bool ZP>
hipError_t launch_block_ng(const BlockGroup& bp, int ng, unsigned grid, hipStream_t st) {
    dim3 block(64 * WN * WK);
    switch (ng) {
        case 1: hipLaunchKernelGGL((block_mfma_kernel<BITS, MB, 1, WN, WK, ZP>), dim3(grid), block, 0, st, bp); break;
        case 2: hipLaunchKernelGGL((block_mfma_kernel<BITS, MB, 2, WN, WK, ZP>), dim3(grid), block, 0, st, bp); break;
        case 4: hipLaunchKernelGGL((block_mfma_kernel<BITS, MB, 4, WN, WK, ZP>), dim3(grid), block, 0, st, bp); break;
        case 8: hipLaunchKernelGGL((block_mfma_kernel<BITS, MB, 8, WN, WK, ZP>), dim3(grid), block, 0, st, bp); break;
        case 16:
            if constexpr (BITS == 4) { hipLaunchKernelGGL((block_mfma_kernel<BITS, MB, 16, WN, WK, ZP>), dim3(grid), block, 0, st, bp); break; }
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int BITS, int MB, int WN, int WK>
hipError_t launch_block_zp(const BlockGroup& g, int ng, unsigned grid, hipStream_t st) {
    if (!g.p[0].zeros) return launch_block_ng<BITS, MB, WN, WK, false>(g, ng, grid, st);
    if constexpr (WK < 8) return launch_block_ng<BITS, MB, WN, WK, true>(g, ng, grid, st);
    return hipErrorInvalidValue;
}

template <int BITS>
hipError_t launch_block(const BlockGroup& bp, int ng, int mb, int wk, unsigned grid, hipStream_t st) {
    switch (mb * 10 + wk) {
        case 11: return launch_block_zp<BITS, 1, 8, 1>(bp, ng, grid, st);
        case 12: return launch_block_zp<BITS, 1, 4, 2>(bp, ng, grid, st);
        case 14: return launch_block_zp<BITS, 1, 2, 4>(bp, ng, grid, st);
        case 18: return launch_block_zp<BITS, 1, 1, 8>(bp, ng, grid, st);
        case 21: return launch_block_zp<BITS, 2, 8, 1>(bp, ng, grid, st);
        case 22: return launch_block_zp<BITS, 2, 4, 2>(bp, ng, grid, st);
        case 24: return launch_block_zp<BITS, 2, 2, 4>(bp, ng, grid, st);
        case 28: return launch_block_zp<BITS, 2, 1, 8>(bp, ng, grid, st);
        case 31: return launch_block_zp<BITS, 3, 8, 1>(bp, ng, grid, st);
        case 32: return launch_block_zp<BITS, 3, 4, 2>(bp, ng, grid, st);
        case 34: return launch_block_zp<BITS, 3, 2, 4>(bp, ng, grid, st);
        case 41: return launch_block_zp<BITS, 4, 8, 1>(bp, ng, grid, st);
        case 42: return launch_block_zp<BITS, 4, 4, 2>(bp, ng, grid, st);
        case 44: return launch_block_zp<BITS, 4, 2, 4>(bp, ng, grid, st);
    }
    return hipErrorInvalidValue;
}

template <int BITS, int MB, bool ZP>
hipError_t launch_wide_gps(const WideParams& wp, dim3 grid, hipStream_t st) {
    const dim3 block(kWideThreads);
    if (wp.gps == 4) hipLaunchKernelGGL((wide_mfma_kernel<BITS, MB, 4, ZP>), grid, block, 0, st, wp);
    else if (wp.gps == 2) hipLaunchKernelGGL((wide_mfma_kernel<BITS, MB, 2, ZP>), grid, block, 0, st, wp);
    else if (wp.spg == 1) hipLaunchKernelGGL((wide_mfma_kernel<BITS, MB, 1, ZP>), grid, block, 0, st, wp);
    else hipLaunchKernelGGL((wide_mfma_kernel<BITS, MB, 0, ZP>), grid, block, 0, st, wp);
    return hipGetLastError();
}

template <int BITS>
hipError_t launch_wide(const WideParams& wp, int mb, dim3 grid, hipStream_t st) {
    switch (mb) {
        case 2: return wp.zeros ? launch_wide_gps<BITS, 2, true>(wp, grid, st) : launch_wide_gps<BITS, 2, false>(wp, grid, st);
        case 3: return wp.zeros ? launch_wide_gps<BITS, 3, true>(wp, grid, st) : launch_wide_gps<BITS, 3, false>(wp, grid, st);
        case 4: return wp.zeros ? launch_wide_gps<BITS, 4, true>(wp, grid, st) : launch_wide_gps<BITS, 4, false>(wp, grid, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool wide_plan_valid(const LinearArgs& a, const LinearPlan& p) {
    if (a.g % kStepK != 0 && a.g != 64 && a.g != 32) return false;
    if (p.m_rows16 == 8) {                                // 128-row tiles
        return (a.zeros || a.g % kStepK == 0) && p.n_tiles16 == 2 && p.waves_n == 8 && p.split_k >= 1 && p.split_k <= a.K / kStepK;
    }
    if (p.m_rows16 < 2 || p.m_rows16 > 4) return false;
    if (p.n_tiles16 != 1 && p.n_tiles16 != 2 && p.n_tiles16 != 4) return false;
    if (p.m_rows16 * p.n_tiles16 > 8) return false;       // register tile: at most 8 accumulator blocks
    if (p.waves_n != 4 && p.waves_n != 8 && !(p.waves_n == 16 && p.n_tiles16 == 1)) return false;
    if (p.split_k < 1 || p.split_k > a.K / kStepK) return false;
    // the instantiations with zero points and with groups under 128 columns
    if ((a.zeros || a.g % kStepK != 0) && (p.waves_n != 8 || p.n_tiles16 > 2)) return false;
    return true;
}

// Row blocks of 32 rows per workgroup: row tiles of up to 16 m_rows16 rows, as many as that takes, of equal height.
static int block_rows32(int64_t M, int64_t N, int m_rows16) {
    const int64_t tiles = (M + 16 * m_rows16 - 1) / (16 * m_rows16);
    const int mb = (int)((M + 32 * tiles - 1) / (32 * tiles));
    return N >= (1 << 22) ? std::min(mb, 2) : mb;         // (N < 2^23: the packed matrix is under 2 GiB, K at least 256)
}

// Several problems of one precision and number of groups per unit, all with workgroups of one shape: mb row blocks, 8 / wk
// wavefronts along N, wk along K.
static hipError_t launch_blocks(const LinearArgs* args, const LinearPlan* plans, int n, int mb, int wk, hipStream_t st) {
    BlockGroup g;
    g.n = n;
    int64_t first = 0;
    const int unit = args[0].bits == 4 ? 512 : 256;       // columns of four packed tiles
    for (int i = 0; i < n; ++i) {
        const LinearArgs& a = args[i];
        BlockParams& bp = g.p[i];
        bp.A = static_cast<const half_t*>(a.A);
        bp.qw = static_cast<const uint8_t*>(a.qweight);
        bp.scales = static_cast<const half_t*>(a.scales);
        bp.zeros = static_cast<const half_t*>(a.zeros);
        bp.C = static_cast<half_t*>(a.C);
        bp.ws = a.workspace;
        bp.M = (int)a.M; bp.N = (int)a.N; bp.K = (int)a.K;
        bp.G = (int)(a.K / a.g);
        bp.NT = (int)(a.N / 16);
        bp.KL = (int)(a.K / (unit / 4));
        bp.upg = a.g >= unit ? (int)(a.g / unit) : 1;
        bp.upg_inv = bp.upg == 1 ? 0u : (uint32_t)(((uint64_t)1 << 32) / (uint32_t)bp.upg) + 1u;
        const int cols = 32 * 8 / wk;
        bp.XB = (int)((a.N + cols - 1) / cols);
        bp.ZB = (int)((a.M + 32 * mb - 1) / (32 * mb));
        bp.split_k = plans[i].split_k;
        bp.u_base = (int)(a.K / unit) / bp.split_k;
        bp.u_rem = (int)(a.K / unit) % bp.split_k;
        bp.qw_bytes = (uint32_t)((size_t)a.N * a.K * a.bits / 8);
        bp.sc_bytes = (uint32_t)((size_t)a.N * bp.G * 2);
        bp.sliced = xcd_slices_save_a_round(bp.XB, bp.ZB, bp.split_k) ? 1 : 0;
        g.blocks[i] = wide_blocks(bp.XB, bp.ZB, bp.sliced != 0);
        g.first[i] = (int)first;
        first += (int64_t)g.blocks[i] * bp.split_k;
    }
    if (first >= (int64_t)1 << 31) return hipErrorInvalidValue;
    g.first[n] = (int)first;
    const int ng = args[0].g >= unit ? 1 : (int)(unit / args[0].g);
    return args[0].bits == 4 ? launch_block<4>(g, ng, mb, wk, (unsigned)first, st) : launch_block<8>(g, ng, mb, wk, (unsigned)first, st);
}

static hipError_t launch_linear_block(const LinearArgs& a, const LinearPlan& p, int wk, hipStream_t st) {
    hipError_t e = launch_blocks(&a, &p, 1, block_rows32(a.M, a.N, p.m_rows16), wk, st);
    if (e != hipSuccess) return e;
    if (p.split_k > 1) e = launch_splitk_reduce(a.workspace, static_cast<half_t*>(a.C), a.M * a.N, p.split_k, st);
    return e;
}

hipError_t launch_linear_blocks(const LinearArgs* args, const LinearPlan* plans, int n, int mb, int wk, hipStream_t st) {
    // workgroups in order of length: the longest start first
    const int unit = args[0].bits == 4 ? 512 : 256;
    LinearArgs a[kMaxBlockGroup];
    LinearPlan p[kMaxBlockGroup];
    int order[kMaxBlockGroup];
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order, order + n, [&](int x, int y) { return args[x].K / unit / plans[x].split_k > args[y].K / unit / plans[y].split_k; });
    size_t used = 0;
    for (int i = 0; i < n; ++i) {
        a[i] = args[order[i]];
        p[i] = plans[order[i]];
        if (p[i].split_k == 1) continue;
        a[i].workspace = a[i].workspace + used / sizeof(float);
        used += ((size_t)a[i].M * a[i].N * sizeof(float) * p[i].split_k + 255) & ~(size_t)255;
    }
    hipError_t e = launch_blocks(a, p, n, mb, wk, st);
    for (int i = 0; i < n && e == hipSuccess; ++i)
        if (p[i].split_k > 1) e = launch_splitk_reduce(a[i].workspace, static_cast<half_t*>(a[i].C), a[i].M * a[i].N, p[i].split_k, st);
    return e;
}

// Path 3 is two kernels: eight wavefronts of one tile-row are the wide kernel; any other configuration means the block kernel's
// workgroup of as many columns -- 64, 128 or 256: 8 wavefronts, 4, 2 or 1 of them along K -- or, as eight wavefronts of two
// tile-rows, with waves_k of the eight along K.
hipError_t launch_linear_wide(const LinearArgs& a, const LinearPlan& p, hipStream_t st) {
    if (p.waves_n != 8 || p.n_tiles16 != 1) {
        const bool given = p.waves_n == 8 && p.n_tiles16 == 2 && (p.waves_k == 2 || p.waves_k == 4 || p.waves_k == 8);
        int wk = given ? p.waves_k : std::max(1, 256 / (16 * p.n_tiles16 * p.waves_n));
        if (wk == 8 && (a.zeros || block_rows32(a.M, a.N, p.m_rows16) > 2)) wk = 4;
        return launch_linear_block(a, p, wk, st);
    }
    constexpr int kCols = kWideThreads / 64 * 16;
    WideParams wp;
    wp.A = static_cast<const half_t*>(a.A);
    wp.qw = static_cast<const uint8_t*>(a.qweight);
    wp.scales = static_cast<const half_t*>(a.scales);
    wp.zeros = static_cast<const half_t*>(a.zeros);
    wp.C = static_cast<half_t*>(a.C);
    wp.ws = a.workspace;
    wp.M = (int)a.M; wp.N = (int)a.N; wp.K = (int)a.K;
    wp.G = (int)(a.K / a.g);
    wp.gps = a.g < kStepK ? (int)(kStepK / a.g) : 1;
    wp.spg = a.g < kStepK ? 1 : (int)(a.g / kStepK);
    wp.spg_inv = wp.spg == 1 ? 0u : (uint32_t)(((uint64_t)1 << 32) / (uint32_t)wp.spg) + 1u;
    wp.NT = (int)(a.N / 16);
    wp.KL = (int)(a.K / (a.bits == 4 ? Layout<4>::TK : Layout<8>::TK));
    wp.XB = (int)((a.N + kCols - 1) / kCols);
    wp.ZB = p.m_blocks;
    wp.split_k = p.split_k;
    wp.ks_base = (int)(a.K / kStepK) / p.split_k;
    wp.ks_rem = (int)(a.K / kStepK) % p.split_k;
    wp.qw_bytes = (uint32_t)((size_t)a.N * a.K * a.bits / 8);
    wp.sc_bytes = (uint32_t)((size_t)a.N * wp.G * 2);
    wp.a_bytes = (uint32_t)((size_t)a.M * a.K * 2);
    wp.sliced = xcd_slices_save_a_round(wp.XB, wp.ZB, p.split_k) ? 1 : 0;
    dim3 grid((unsigned)wide_blocks(wp.XB, wp.ZB, wp.sliced != 0), (unsigned)p.split_k, 1);
    hipError_t e = a.bits == 4 ? launch_wide<4>(wp, p.m_rows16, grid, st) : launch_wide<8>(wp, p.m_rows16, grid, st);
    if (e != hipSuccess) return e;
    if (p.split_k > 1) e = launch_splitk_reduce(a.workspace, static_cast<half_t*>(a.C), a.M * a.N, p.split_k, st);
    return e;
}

}  // namespace rtn
