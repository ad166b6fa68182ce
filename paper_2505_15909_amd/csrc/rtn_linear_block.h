// Fused dequantise-GEMM from 17 rows (shared launches of a layer from 5, of a grouped call from one): the block kernel, one translation unit per precision and variant
// (rtn_linear_block4.hip, ...).  Exact integer codes in the MFMAs, the fp16 scale applied in fp32 to the partial sum of each group (or of
// the part of a group that lies in a share of K: scaling is linear, so groups may straddle splits).
//
// Block kernel.  A workgroup is 8 wavefronts, 8 / WK side by side along N times WK along K; a wavefront owns 32 output columns
// and all 32 MB rows of the row tile as v_mfma_f32_32x32x16_f16 blocks.
//   - Packed weights go from global memory straight into registers in operand order: lane -> row lane & 15 of tile-row
//     (lane >> 4) & 1, 16-byte chunk 2 q + lane / 32 of a tile, so that two 1 KiB loads hold a 128-column k-step (4 bit) and
//     8 consecutive columns are one operand half.  Four k-steps are in registers.
//   - The activations of a step go from global memory straight into LDS (four stages of 32 to 128 columns, see BlockShape), swizzled by which
//     piece a lane fetches; the reads of a 16-column slice are issued a slice ahead of its MFMAs, and the one barrier of a stage
//     stands before its last slice, whose operands are in registers by then.  Wavefronts that share no activations (WK = 8)
//     take no barrier at all.
//   - Scales come once per unit of four packed tiles, two units ahead: per-step loads of two bytes a lane touch 32 cache lines
//     each, twice as many as the weights (57344 x 8192 int4 at 32 rows 65 us with them, 52 without).
//   - The WK partial tiles are summed through LDS in a fixed order.
// Loads return in order: a wavefront that waits for its activations has waited for the weights requested before them, so no more
// weights are in flight than the staged rows lead by.  Up to 16 rows only those are staged, which with several wavefronts along K doubles
// the lead, and the MFMAs' other 16 rows read zeros (eight modules of 2048 x 7168 at one row 15.8 -> 14.7 us; with copies of the rows, which
// draw more power, 8 % slower at 16 rows than 32 staged ones).
// A launch of more than a round consists of parts, a problem's row tiles of one height, longest workgroups first: 200 rows are 128 + 96, and
// the short tiles fill the last round (8B layer int4 112 -> 100 us; inside one part, tall and short in turn, it stayed at 107).  Within
// one round all are tall and the tiles of a column next to one another: in step they read its weights once (4096 x 14336 int8 at 140 rows
// 33 us, with two heights 37, and 43 in two parts).
// Every problem has its own number of wavefronts along K.
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
#pragma once
#include "rtn_linear_wide.h"
#include <type_traits>

namespace rtn {

namespace {

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

// Stages and depths of a shape of the block kernel: row tiles of up to MB blocks of 32 rows.  Four activation stages of up to 32 KiB (16
// with one block): one kernel has all shapes that fit, and a launch may give every problem its own.  The others have a kernel of their
// own: most wavefronts along K on two blocks and more, with two stages of 64 columns (four of 32: 4 % slower at 128 rows), and eight on 8-bit
// weights, with four of 64 columns (of 32: 6144 x 4096 at 32 rows 11.1 us instead of 10.3).  4-bit weights have both: of 32 columns where
// a wavefront has one unit (4096 columns and less: 6144 x 4096 7.5 us instead of 8.1), of 64 from two, where the weights are asked for as far
// ahead as the rows are (4096 x 7168 at 32 rows 14.6 us with 32, 13.0 with 64; 4096 x 14336 at 28 rows 25.3 and 21.0).
// FIT: stages no larger than the shape needs, for a kernel that has no other shape.
template <int BITS, int MB, int WN, int WK, bool HALF = false, bool FIT = false>
struct BlockShape {
    static constexpr bool ALONE = !HALF && block_shape_alone(BITS, MB, WK);
    static constexpr int KA = WK == 1 || (WK == 2 && MB <= 2) || (HALF && WK == 4) ? kStepK : WK == 8 && !ALONE && !HALF && !FIT ? 32 : 64;   // columns of an activation stage, per wavefront along K
    static constexpr int R = kStepK / KA;                           // stages per k-step
    static constexpr int S = ALONE && MB > 1 ? 2 : 4;               // activation stages
    static constexpr int D = BITS == 4 ? 4 : 2;     // k-steps of weights in registers
    static constexpr int SPU = BITS == 4 ? 4 : 2;                   // k-steps per unit
    static constexpr int UN = D > 2 * SPU ? D : 2 * SPU;            // k-steps per turn of the loop: every buffer index is a literal
    static constexpr int STAGE = ALONE || FIT ? WK * 32 * MB * KA * 2 : MB == 1 ? 16384 : MB == 3 ? 24576 : 32768;
    static_assert(UN % D == 0 && UN % (2 * SPU) == 0 && UN * R % S == 0 && WK * (HALF ? 16 : 32 * MB) * KA * 2 <= STAGE && S * STAGE <= 150 * 1024, "");
};

constexpr int kZeroRow = 256;

// One row tile of MB blocks: column tile xb, rows from m0, part sg of K.  TALL: blocks of the launch's tallest tiles, which give the shape
// of the stages.  args: where p came from, for what is needed at the end.  HALF: at most 16 rows; the MFMAs' other 16 read a row of zeros.
template <int BITS, int MB, int TALL, int NG, int WN, int WK, bool ZP, bool HALF = false, bool FIT = false>
__device__ __forceinline__ void block_tile(const BlockProblem& p, const BlockProblem& args, int xb, int m0, int sg, uint8_t* lds0, uint8_t* lds1, uint8_t* lds2, uint8_t* lds3) {
    typedef BlockShape<BITS, TALL, WN, WK, HALF, FIT> Shape;
    constexpr int TPS = kStepK / Layout<BITS>::TK;        // packed tiles per k-step: 1 / 2
    constexpr int SPU = Shape::SPU, UN = Shape::UN;
    constexpr int SPG = 8 * SPU / NG;                     // 16-column slices per group, of those in a unit (8 in a k-step)
    constexpr int ROWS = HALF ? 16 : 32 * MB, KA = Shape::KA, R = Shape::R, S = Shape::S, D = Shape::D, STAGE = Shape::STAGE;
    constexpr int SLICE_BYTES = ROWS * KA * 2;            // one stage of one share of K
    constexpr int PIECES = KA / 8;                        // 16-byte pieces of a staged row
    constexpr int RPI = 64 / PIECES;                      // rows per load instruction
    constexpr int SWZ = 16 / PIECES;                      // rows that share 256 bytes of LDS
    constexpr int SPS = KA / 16;                          // slices per stage
    constexpr int PD = 1;                   // slices the operand reads run ahead
    constexpr int NA = ROWS / RPI / WN;                   // activation loads per wavefront and stage
    static_assert(ROWS % (RPI * WN) == 0 && PD < SPS, "");
    auto stage = [&](int i) { return i == 0 ? lds0 : i == 1 ? lds1 : i == 2 ? lds2 : lds3; };

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wk = wave / WN;
    const int row = lane & 31, h = lane >> 5;

    const int u_base = (int)(p.u_share & 0xFFFFu), u_rem = (int)(p.u_share >> 16), upg = (int)(p.groups & 0xFFFFu);
    const int u_wg = sg * u_base + min(sg, u_rem);                 // units of this workgroup: u_wg .. u_wg + n_wg
    const int n_wg = u_base + (sg < u_rem ? 1 : 0);
    // (what several shapes of a kernel have in common the compiler may put into vector registers, and loop over the lanes at each load)
    const uint32_t qw_bytes = __builtin_amdgcn_readfirstlane((uint32_t)p.N * ((uint32_t)p.K / 8u) * BITS);
    const uint32_t sc_bytes = __builtin_amdgcn_readfirstlane((uint32_t)p.N * (uint32_t)p.G * 2u);
    const int TU = (n_wg + WK - 1) / WK;                           // units every wavefront runs; those beyond its share add zeros
    const int u0 = u_wg + wk * TU;
    const int own = max(0, min(TU, n_wg - wk * TU));

    const int a_rows = __builtin_amdgcn_readfirstlane(min(ROWS, p.M - m0));
    half_t* a0 = const_cast<half_t*>(p.A) + (int64_t)m0 * p.K;
    // held in scalar registers: left alone the compiler reads the pointers again after each barrier, and waits for them with every LDS read
    uint8_t* qw = const_cast<uint8_t*>(p.qw);
    half_t* scales = const_cast<half_t*>(p.scales);
    half_t* zeros = const_cast<half_t*>(p.zeros);
    asm volatile("" : "+s"(a0), "+s"(qw), "+s"(scales));
    if constexpr (ZP) asm volatile("" : "+s"(zeros));
    const uint32_t a_bytes = (uint32_t)a_rows * (uint32_t)p.K * 2u;
    const uint32_t magic = fp16_magic_vgpr();

    // weight row of this lane: row lane & 15 of tile-row nt
    const int nt = (xb * WN + wn) * 2 + ((lane >> 4) & 1);
    const bool nt_ok = nt < p.N / 16;
    const uint32_t w_lane = nt_ok ? (uint32_t)nt * (uint32_t)(p.K / Layout<BITS>::TK) * 1024u + (h * 16 + (lane & 15)) * 16 : kOutOfRange;
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
            load_to_lds(r, stage(st) + wk * SLICE_BYTES + (wn * NA + i) * 1024, a_lane[i], (u0 * SPU * R + q) * (KA * 2));
    };
    u32x4_t wbuf[D][TPS][2];
    auto w_load = [&](int slot, int t) {                  // k-step t of this wavefront's share
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(qw, 0, t < own * SPU ? qw_bytes : 0u, kBufferFlags);
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
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(scales, 0, u < own ? sc_bytes : 0u, kBufferFlags);
        sbuf[slot] = load_row_scales<NG>(rs, s_lane, (int)(j * 2u));
        if constexpr (ZP) {
            const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(zeros, 0, u < own ? sc_bytes : 0u, kBufferFlags);
            zbuf[slot] = load_row_scales<NG>(rz, s_lane, (int)(j * 2u));
        }
    };
    // Two scales in a register are taken apart in a copy made when their unit starts: from the register itself the compiler takes the
    // halves where it is loaded and waits for it there (10 % slower), and opaque at every use it converts a zero point again for
    // every operand (18192 x 2560 int8 group 128 with zero points at 64 rows 18.6 us, 18.0 this way).
    RowScales<NG> s_copy, z_copy;
    (void)s_copy; (void)z_copy;
    auto take = [](RowScales<NG>& to, const RowScales<NG>& from) {
        if constexpr (NG == 2) asm volatile("v_mov_b32 %0, %1" : "=v"(to.v) : "v"(from.v));
    };
    auto unit_scale = [&](const RowScales<NG>& copy, const RowScales<NG>& loaded, int i) { return (float)row_scale<NG>(NG == 2 ? copy : loaded, i); };
    // weight operand of slice s of step v (mod UN)
    auto operand = [&](int v, int s) {
        const u32x4_t& chunk = wbuf[v % D][BITS == 4 ? 0 : s >> 2][s & 1];
        const int i = BITS == 4 ? s >> 1 : (s >> 1) & 1;
        if constexpr (ZP) return unpack_operand_zp<BITS>(chunk, i, magic, unit_scale(z_copy, zbuf[v / SPU % 2], ((v % SPU) * 8 + s) / SPG));
        else return unpack_operand<BITS>(chunk, i, magic);
    };

    float16_t acc[MB], part[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) { acc[b][e] = 0.f; part[b][e] = 0.f; }

    half8_t aop[PD + 1][MB];
    // piece 2 s + h of a row stands at slot (2 s + h) ^ (row's swizzle): one exclusive-or per slice on the lane's own address
    uint32_t rd = wk * SLICE_BYTES + row * (KA * 2) + ((h ^ ((row / SWZ) % PIECES)) * 16);
    if constexpr (HALF) {                                 // both addresses first: with a branch the compiler has values of its sides in vector registers
        uint32_t zero = STAGE + h * 16;
        asm volatile("" : "+v"(rd), "+v"(zero));
        rd = row >= 16 ? zero : rd;
    }
    if constexpr (HALF) {                                 // a row of zeros behind each stage; every wavefront writes it for itself
#pragma unroll
        for (int i = 0; i < S; ++i) *reinterpret_cast<uint32_t*>(stage(i) + STAGE + lane * 4) = 0;
    }
    auto a_read = [&](int st, int s) {                    // operands of slice s of a step
        uint32_t o = rd;
        if (s % SPS) asm volatile("v_xor_b32 %0, %1, %2" : "=v"(o) : "n"((s % SPS) * 32), "v"(rd));
#pragma unroll
        for (int b = 0; b < MB; ++b) aop[s % (PD + 1)][b] = *reinterpret_cast<const half8_t*>(stage(st) + o + b * (32 * KA * 2));
    };

    // 8-bit weights, of which two steps are in registers, are requested before the next step's first ones are unpacked, which has to wait for
    // them: 67 rows of 8128 x 3072 group 128 14.2 -> 13.7 us, 9216 x 5632 at 91 rows 26.0 -> 25.5.  (4-bit weights, four steps of
    // them, do not mind.)
    constexpr bool LATE = BITS == 8;
    // Weight loads requested since the stage after stage rr of a step (those of older steps have been used).  Scales are not
    // counted: a unit's wait is for a load more than it need be.
    auto weights_since = [](int rr) {
        int n = 0;
        const int from = rr + 1 - S;
        for (int j = from > rr - D * R ? from : rr - D * R; j < rr; ++j) n += (j + 64 * R) % R == R - 1 ? 2 * TPS : 0;
        return n;
    };
    auto wait_stage = [&](int n) { wait_stage_n<(WN > 1)>(n); };

    int left = upg - (int)((uint32_t)u0 - (p.upg_inv == 0 ? (uint32_t)u0 : __umulhi((uint32_t)u0, p.upg_inv)) * (uint32_t)upg);
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
            if (us == 0) take(s_copy, sbuf[v / SPU % 2]);
            if (ZP && !LATE && us == 8 * SPU - 1) take(z_copy, zbuf[(v + 1) / SPU % 2]);
            const half8_t b_now = bw;
            if (!LATE || s < 7) bw = s == 7 ? operand((v + 1) % UN, 0) : operand(v, s + 1);
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
                    const float sc = unit_scale(s_copy, sbuf[v / SPU % 2], us / SPG);
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
            if (LATE && s == 7) {
                if (ZP && us == 8 * SPU - 1) take(z_copy, zbuf[(v + 1) / SPU % 2]);
                bw = operand((v + 1) % UN, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (NG == 1 && unit_ends) left = upg;
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
    if (ZP) take(z_copy, zbuf[0]);
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
    // The scales requested past the last unit are not used: without this their registers are free while the loads are under way, and an odd
    // unit, which takes them for something else, waits for every load of the wavefront (18192 x 2560 int8 group 128 at 64 rows 18.9 us, 17.8 this way; 6144 x 2560 int4 at 60 rows 9.4 and 9.1).
    auto keep = [](const RowScales<NG>& s) {
        if constexpr (NG <= 4) asm volatile("" :: "v"(s.v));
        else
#pragma unroll
            for (int i = 0; i < NG / 8; ++i) asm volatile("" :: "v"(s.v[i]));
    };
    keep(sbuf[0]); keep(sbuf[1]);
    if constexpr (ZP) { keep(zbuf[0]); keep(zbuf[1]); }

    // Lane holds column 16 nt + (lane & 15), rows m0 + 32 b + 8 (e / 4) + 4 h + e % 4.  Rows past M and columns
    // past N are outside the resource and dropped by the hardware (a row tile of results is under 2 GiB, see the launch).
    auto finish = [&](auto partial) {
        constexpr uint32_t BYTES = partial.value ? 4 : 2;
        const uint32_t row_bytes = (uint32_t)args.N * BYTES;
        const __amdgpu_buffer_rsrc_t rc = partial.value
            ? __builtin_amdgcn_make_buffer_rsrc(args.ws + ((int64_t)sg * args.M + m0) * args.N, 0, (uint32_t)a_rows * row_bytes, kBufferFlags)
            : __builtin_amdgcn_make_buffer_rsrc(args.C + (int64_t)m0 * args.N, 0, (uint32_t)a_rows * row_bytes, kBufferFlags);
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
    if (((args.groups >> 16) & 0xFFu) == 1) finish(std::false_type{});
    else finish(std::true_type{});
}

// The part that workgroup blockIdx.x belongs to, its problem and its tile; false for the padding.  The first part and its problem, which is
// the first one, are read before it is known whether they are the right ones: the arguments come from memory, and to read the number of
// parts, then the part, then the problem, each after the other has arrived, put 0.2-0.4 us before the first request for data (int8,
// 18192 x 2560 at 64 rows 18.5 us, 18.1 this way; 67 rows of 8128 x 3072 13.8 and 13.4).
__device__ __forceinline__ bool block_part(const BlockGroup& group, BlockPart* part, int* problem, BlockProblem* p, int* xb, int* z, int* sg) {
    *part = group.part[0];
    *p = group.p[0];
    *problem = 0;
    // values from here on: left alone the compiler picks the address first and reads once, after it
    asm volatile("" : "+s"(part->first), "+s"(part->blocks), "+s"(part->row0), "+s"(part->tall), "+s"(part->info));
    asm volatile("" : "+s"(p->A), "+s"(p->qw), "+s"(p->scales), "+s"(p->zeros));
    asm volatile("" : "+s"(p->M), "+s"(p->N), "+s"(p->K), "+s"(p->G), "+s"(p->XB), "+s"(p->u_share), "+s"(p->groups), "+s"(p->upg_inv));
    if (group.n > 1 && (int)blockIdx.x >= group.part[1].first) {
        int gi = 1;
        while (gi + 1 < group.n && (int)blockIdx.x >= group.part[gi + 1].first) ++gi;
        *part = group.part[gi];
        *problem = (int)(part->info >> 20);
        *p = group.p[*problem];
    }
    const int local = (int)blockIdx.x - part->first;
    *sg = local / part->blocks;
    return xcd_wide_tile(local - *sg * part->blocks, p->XB, (int)(part->info & 0xFFFFu), (part->info >> 17 & 1) != 0, xb, z);
}

// Row tiles of two heights, MB blocks and one less, as many of each as M takes: 200 rows are 128 + 96, not twice 128.
template <int BITS, int MB, int NG>
__global__ __launch_bounds__(kBlockThreads, MB == 1 ? 4 : 2) void block_mfma_kernel(const BlockGroup group) {
    constexpr int STAGE = BlockShape<BITS, MB, 8, 1>::STAGE;
    constexpr int BYTES = STAGE + (MB == 1 ? kZeroRow : 0);
    __shared__ __align__(256) uint8_t lds0[BYTES], lds1[BYTES], lds2[BYTES], lds3[BYTES];
    int problem, xb, z, sg;
    BlockPart part;
    BlockProblem p;
    if (!block_part(group, &part, &problem, &p, &xb, &z, &sg)) return;
    const int wk = (int)(p.groups >> 24);
    auto run = [&](auto height, int m0) {
        constexpr int H = decltype(height)::value;
        if constexpr (MB == 1) {
            if (p.M <= 16 && wk > 1) {
                if (wk == 2) block_tile<BITS, 1, 1, NG, 4, 2, false, true>(p, group.p[problem], xb, m0, sg, lds0, lds1, lds2, lds3);
                else if (wk == 4) block_tile<BITS, 1, 1, NG, 2, 4, false, true>(p, group.p[problem], xb, m0, sg, lds0, lds1, lds2, lds3);
                else block_tile<BITS, 1, 1, NG, 1, 8, false, true>(p, group.p[problem], xb, m0, sg, lds0, lds1, lds2, lds3);
                return;
            }
        }
        if (wk == 1) block_tile<BITS, H, MB, NG, 8, 1, false>(p, group.p[problem], xb, m0, sg, lds0, lds1, lds2, lds3);
        else if (MB > 2 || wk == 2) block_tile<BITS, H, MB, NG, 4, 2, false>(p, group.p[problem], xb, m0, sg, lds0, lds1, lds2, lds3);
        if constexpr (MB <= 2) {
            if (wk == 4) block_tile<BITS, H, MB, NG, 2, 4, false>(p, group.p[problem], xb, m0, sg, lds0, lds1, lds2, lds3);
            if constexpr (MB == 1 && !block_shape_alone(BITS, 1, 8))
                if (wk == 8) block_tile<BITS, H, MB, NG, 1, 8, false>(p, group.p[problem], xb, m0, sg, lds0, lds1, lds2, lds3);
        }
    };
    if constexpr (MB > 1) {
        if (z >= part.tall) {
            run(std::integral_constant<int, MB - 1>{}, part.row0 + part.tall * 32 + z * (32 * (MB - 1)));
            return;
        }
    }
    run(std::integral_constant<int, MB>{}, part.row0 + z * (32 * MB));
}

// One shape, which every part of the launch has: those whose stages do not fit the kernel above or are not its own, 64-row tiles without
// wavefronts along K, and all with zero points.  A launch with
// zero points is one problem, so there is nothing to share, and the common kernel cost it: with groups of 32 columns on 32-row tiles eight
// registers went to scratch memory (6144 x 4096 at 24 rows 11.8 us, 11.3 here), and with stages of 32 KiB where 16 do, half of them lie
// beyond the offset that an LDS read holds and every read takes an addition (4096 x 14336 group 64 at 256 rows 43.9 us, 43.1; without
// zero points 28672 x 4096 group 128 at 117 rows 38.1 and 37.3, group 64 at 256 rows 73.9 and 71.8).
template <int BITS, int MB, int NG, int WK, bool ZP>
__global__ __launch_bounds__(kBlockThreads, MB == 1 && WK < 8 ? 4 : 2) void block_mfma_alone_kernel(const BlockGroup group) {
    typedef BlockShape<BITS, MB, 8 / WK, WK, false, true> Shape;
    static_assert(ZP || Shape::ALONE || (MB == 2 && WK == 1) || (MB == 1 && WK == 8), "");
    constexpr int LAST = Shape::S > 2 ? Shape::STAGE : 16;
    __shared__ __align__(16) uint8_t lds0[Shape::STAGE], lds1[Shape::STAGE], lds2[LAST], lds3[LAST];
    int problem, xb, z, sg;
    BlockPart part;
    BlockProblem p;
    if (!block_part(group, &part, &problem, &p, &xb, &z, &sg)) return;
    if constexpr (MB > 1) {
        if (z >= part.tall) {
            block_tile<BITS, MB - 1, MB, NG, 8 / WK, WK, ZP, false, true>(p, group.p[problem], xb, part.row0 + part.tall * 32 + z * (32 * (MB - 1)), sg, lds0, lds1, lds2, lds3);
            return;
        }
    }
    block_tile<BITS, MB, MB, NG, 8 / WK, WK, ZP, false, true>(p, group.p[problem], xb, part.row0 + z * (32 * MB), sg, lds0, lds1, lds2, lds3);
}

}  // namespace

template <int BITS, bool ZP>
hipError_t launch_block(const BlockGroup& g, int ng, int mb, unsigned grid, hipStream_t st) {
    auto with_groups = [&](auto blocks, auto groups) {
        constexpr int MB = decltype(blocks)::value, NG = decltype(groups)::value, DEEP = MB <= 2 ? 8 : 4;
        const int wk = (int)(g.p[0].groups >> 24);
        auto alone_kernel = [&](auto waves) {
            hipLaunchKernelGGL((block_mfma_alone_kernel<BITS, MB, NG, decltype(waves)::value, ZP>), dim3(grid), dim3(kBlockThreads), 0, st, g);
            return hipGetLastError();
        };
        if constexpr (ZP) {                               // no shape with eight wavefronts along K
            switch (wk) {
                case 1: return alone_kernel(std::integral_constant<int, 1>{});
                case 2: return alone_kernel(std::integral_constant<int, 2>{});
                case 4: return alone_kernel(std::integral_constant<int, 4>{});
            }
        } else {
            if constexpr (MB == 2) {
                bool one = true;
                for (int i = 0; i < g.n; ++i) one = one && g.p[g.part[i].info >> 20].groups >> 24 == 1;
                if (one) return alone_kernel(std::integral_constant<int, 1>{});
            }
            bool alone = block_shape_alone(BITS, mb, wk);
            if (MB == 1 && wk == 8)                       // several units for a wavefront (BlockShape)
                for (int i = 0; i < g.n; ++i) alone = alone || (g.p[g.part[i].info >> 20].u_share & 0xFFFFu) + (g.p[g.part[i].info >> 20].u_share >> 16 ? 1 : 0) > 8;
            if (MB == 1 && alone) {                       // 16 rows and less are staged as such by the common kernel
                alone = false;
                for (int i = 0; i < g.n; ++i) alone = alone || g.p[g.part[i].info >> 20].M > 16;
            }
            if (!alone) {
                hipLaunchKernelGGL((block_mfma_kernel<BITS, MB, NG>), dim3(grid), dim3(kBlockThreads), 0, st, g);
                return hipGetLastError();
            }
            if constexpr (block_shape_alone(BITS, MB, DEEP) || MB == 1)
                if (wk == DEEP) return alone_kernel(std::integral_constant<int, DEEP>{});
        }
        return hipErrorInvalidValue;
    };
    auto with_blocks = [&](auto blocks) {
        switch (ng) {
            case 1: return with_groups(blocks, std::integral_constant<int, 1>{});
            case 2: return with_groups(blocks, std::integral_constant<int, 2>{});
            case 4: return with_groups(blocks, std::integral_constant<int, 4>{});
            case 8: return with_groups(blocks, std::integral_constant<int, 8>{});
            case 16: if constexpr (BITS == 4) return with_groups(blocks, std::integral_constant<int, 16>{});
        }
        return hipErrorInvalidValue;
    };
    switch (mb) {
        case 1: return with_blocks(std::integral_constant<int, 1>{});
        case 2: return with_blocks(std::integral_constant<int, 2>{});
        case 3: return with_blocks(std::integral_constant<int, 3>{});
        case 4: return with_blocks(std::integral_constant<int, 4>{});
    }
    return hipErrorInvalidValue;
}

}  // namespace rtn
