// Matrix-core-bound GEMM of the quantised linear layer for large batches (Section 5: with many input tokens
// the layer is a dense matrix product; the paper then dequantises the weights to 16 bit and calls a dense GEMM,
// and measures where that overtakes the fused kernel).  One kernel core, three weight sources:
//   - packed 4-bit / 8-bit codes: dequantised on the way into LDS (fused path for a hundred rows and more),
//   - dense fp16 weights [N, K]: the 16-bit GEMM of the dequantise-then-GEMM path.
//
// A workgroup of 8 wavefronts (2 along M x 4 along N) computes a TM x 256 tile of C, TM = 128 or 256; a
// wavefront owns (TM / 2) x 64 of it as MBW x 4 v_mfma_f32_16x16x32_f16 blocks (MBW = 4 or 8: 64 or 128 fp32
// accumulator registers).  K advances in steps of 64 columns; a row of a staged tile is 128 bytes = eight 16-byte
// pieces, piece p stored at slot p ^ (row & 7): conflict-free for the b128 operand reads (lane -> row nl, piece
// 4 i + kq) and for the stores of dequantised weights, which have the operand pattern.
//
// What bounds it: with the whole chip busy, power.  The clock falls from 2.4 to about 1.55 GHz under this kernel (1.33
// under the vendor library's GEMM, whose matrix cores are busier per cycle, at the same time per product); on a quarter
// of the chip a step is 20 % faster.  So the design spends as little as it can per MFMA:
//   - fp16 tiles (activations, dense weights) go from global memory straight into LDS, no registers and no LDS store
//     instructions (the swizzle is in which piece a lane fetches);
//   - a step runs in phases of 16 MFMAs; each phase reads the operands of the next one, so no MFMA waits for the LDS;
//   - the one barrier of a step stands before its last phase, whose operands are in registers by then.  From there on
//     the step's stage is free: the last phase reads the next step's first operands, and it and the phases behind it
//     request a later step's tiles into the freed stage, so a request has a step (two, where the stages are short) to
//     arrive and the matrix cores work across the barrier;
//   - the two slices of a step go into an accumulator one right after the other, but for the 128-row 8-bit tile (see the step below);
//   - the MFMAs take the weights as their first operand: a lane then holds four consecutive columns of a row and the
//     results leave as whole 128-byte runs (as 2-byte stores in 32-byte runs the epilogue took 10 % of a K = 4096 tile).
// Measured against staging through registers with the barrier at the end of each step (28672 x 4096 at 2048 rows: int4
// 440 -> 395 us; 8192 x 28672 at 4096: int4 1556 -> 1445, dense 1490 -> 1376; 8192 x 8192 x 8192 dense 905 -> 770 us; by
// now, with what is said below, 364, 1345, 1304 and 726 = 1.51 PFLOP/s, the vendor library's time to 1 %).
// v_mfma_f32_32x32x16_f16 is 6 % faster on a quarter of the chip and 5 % slower on all of it (twice the accumulator traffic
// per flop); a raised wavefront priority around the MFMAs is 5-8 % slower.
//
// A launch takes several independent problems: its workgroups find theirs by a scan over first[], whose order (longest first)
// lets the short ones fill the last round.  A launch of one problem takes the time it took without the table.
//
// Fused dequantisation: a packed tile is unpacked once per workgroup (not once per wavefront), multiplied by
// its group's scale in fp16 (one rounding per weight, relative error 2^-11, far inside the layer's tolerance)
// and written to LDS as ordinary fp16, so the inner loop is that of the dense GEMM and carries no
// per-accumulator scale arithmetic.
#include "rtn_device.h"
#include "rtn_internal.h"
#include <algorithm>

namespace rtn {

namespace {

constexpr int kTN = 256;                        // columns of C per workgroup
constexpr int kBK = 64;                         // columns of K per step
constexpr int kChunkK = 128;                    // packed weights are fetched in 128-column chunks (two steps)
constexpr int kThreads = 512;
constexpr int kBufferFlags = 0x00020000;
constexpr uint32_t kNoRow = 0x80000000u;        // beyond a resource of 2 GiB; in a larger one, data of rows that are never stored
constexpr int kZGroup = 4;                      // row tiles in a group (1, 2, 8: within 1 %; 16: 1-2 % slower)

struct TileParams {
    const half_t* A;
    const void* B;          // packed codes or fp16 [N, K]
    const half_t* scales;
    half_t* C;
    float* ws;
    int M, N, K;
    int G;                  // groups per row (packed sources)
    int cpg;                // 128-column chunks per group
    uint32_t cpg_inv;       // floor(2^32 / cpg) + 1 (0 when cpg == 1)
    uint32_t cpg_one;       // all ones when cpg == 1, else 0: chunk -> group is umulhi(c, cpg_inv) + (c & cpg_one)
    int KL;                 // packed tiles per weight row
    int XB, ZB;             // tiles along N, along M
    int split_k;
    int kc_base, kc_rem;    // workgroup sg covers 128-column chunks [sg*kc_base + min(sg, kc_rem), ...)
    uint32_t b_bytes, sc_bytes;   // packed sources only
};

// The problems of one launch: problem i has the workgroups first[i] .. first[i + 1], blocks[i] of them (a multiple of the XCDs)
// per K split.
struct TileGroup {
    int n;
    int first[kMaxTileGroup + 1], blocks[kMaxTileGroup];
    TileParams p[kMaxTileGroup];
};

__device__ __forceinline__ uint32_t swizzled(int row, int piece) {      // byte offset inside a staged tile
    return (uint32_t)(row * 128 + ((piece ^ (row & 7)) * 16));
}

// 16 bytes per lane from global memory into 1 KiB of LDS at a wave-uniform address
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, uint8_t* lds, uint32_t lane_off, int off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, lane_off, off, 0, 0);
}

// Workgroup barrier behind the loads older than the N newest ones and every LDS access.  __syncthreads() would wait for
// all loads into LDS, those of the stages to come included.
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// BSRC: 0 = dense fp16 weights, 4 / 8 = packed codes.  MBW: 16-row blocks per wavefront along M (4 or 8).
template <int BSRC, int MBW>
__global__ __launch_bounds__(kThreads, 2) void tile_gemm_kernel(const TileGroup group) {
    int gi = 0;
    while (gi + 1 < group.n && (int)blockIdx.x >= group.first[gi + 1]) ++gi;
    const TileParams p = group.p[gi];                        // by value: read once, not again after each barrier
    const int local = (int)blockIdx.x - group.first[gi];
    const int sg = local / group.blocks[gi];                 // K split
    constexpr int TM = 32 * MBW;
    constexpr int A_BYTES = TM * 128, B_BYTES = kTN * 128;
    constexpr int PH = MBW / 2;                              // phases per step (two row blocks, 64 columns each)
    // Stages in LDS (a request has SA or SB steps less a phase to arrive), at most 160 KiB in all.  Dense weights stream
    // from HBM and get three; three for the short dense tile's activations, whose steps are half as long (4096 x 14336 at
    // 2048 rows: 223 -> 190 us).  Four for the short packed tile gained nothing.
    constexpr int SA = BSRC == 0 && MBW == 4 ? 3 : 2, SB = BSRC == 0 ? 3 : 2;
    // The requests of a step, up to 64 KiB a compute unit, kept the wavefronts from issuing their MFMAs when they all stood in the one
    // phase behind the barrier.  The activations' go out in AP phases from the barrier on, the dense weights', which have a
    // stage more, from phase BP behind it: dense 8192 x 8192 x 8192 788 -> 761 us, 8192 x 28672 at 4096 rows 1411 -> 1360, 28672 x
    // 4096 at 1024 203 -> 194; int8 8192 x 8192 at 8192 862 -> 848; int4 there 818 -> 803.  The 128-row packed tiles have few.
    constexpr int AP = BSRC == 0 || MBW == 8 ? 2 : 1, BP = BSRC == 0 && PH == 4 ? 2 : 0;
    // The activation operands of the next phase take the place of this one's, row block by row block, but for the last phase of a step:
    // with two sets the 256-row packed tiles, which unpack as well, spill (int4 8192 x 8192 at 8192 rows 803 us, 800 this way; int8 811 and
    // 806).  Dense tiles have the registers, and are 1 % faster with two sets.
    constexpr bool IN_PLACE = BSRC != 0 && MBW == 8;
    // The 128-row 8-bit tile takes one slice after the other: a last phase that also replaces both slices' weights waits for its LDS reads
    // (4096 x 14336 at 200 rows 237 us, 221 this way; 8192 x 28672 472 and 440, in three splits 177 and 167; 4 bit and dense the other
    // way, 3 and 1.5 %).
    constexpr bool BY_SLICE = BSRC == 8 && MBW == 4;
    constexpr int U = BSRC == 0 ? 6 : 4;                     // steps per turn of the loop: every stage index is a literal
    // one object per stage: the compiler then knows that a load into one stage cannot touch reads of the other
    __shared__ __align__(16) uint8_t lds_a0[A_BYTES], lds_a1[A_BYTES], lds_a2[SA > 2 ? A_BYTES : 16];
    __shared__ __align__(16) uint8_t lds_b0[B_BYTES], lds_b1[B_BYTES], lds_b2[SB > 2 ? B_BYTES : 16];
    auto stage_a = [&](int i) { return i == 0 ? lds_a0 : i == 1 ? lds_a1 : lds_a2; };
    auto stage_b = [&](int i) { return i == 0 ? lds_b0 : i == 1 ? lds_b1 : lds_b2; };

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int nl = lane & 15, kq = lane >> 4;

    int xb, zb;                                              // tile along N, along M
    if (!xcd_tile(local - sg * group.blocks[gi], p.XB, p.ZB, kZGroup, &xb, &zb)) return;
    const int m0 = zb * TM, n0 = xb * kTN;
    const int kc0 = sg * p.kc_base + min(sg, p.kc_rem);      // first 128-column chunk
    const int T = 2 * (p.kc_base + (sg < p.kc_rem ? 1 : 0)); // 64-column steps of this workgroup
    const int ks0 = 2 * kc0;

    // Row-major fp16 operands are addressed through a resource that starts at this workgroup's first row (no 32-bit
    // limit on the whole matrix).  Rows past M or N read zeros (an offset beyond the resource; they are multiplied like the others and
    // draw less power than copies of a row), steps past the last one the last step; those rows are never stored, those
    // steps never used.
    const int a_rows = min(TM, p.M - m0), b_rows = min(kTN, p.N - n0);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<half_t*>(p.A) + (int64_t)m0 * p.K, 0, (uint32_t)a_rows * (uint32_t)p.K * 2u, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rb = BSRC == 0
        ? __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(static_cast<const half_t*>(p.B)) + (int64_t)n0 * p.K, 0,
                                            (uint32_t)b_rows * (uint32_t)p.K * 2u, kBufferFlags)
        : __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.B), 0, p.b_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(p.scales), 0, p.sc_bytes, kBufferFlags);
    const uint32_t magic = fp16_magic_vgpr();

    // ---- staging of row-major fp16 tiles (A always, B when dense): straight into LDS, 1 KiB (8 rows) per instruction;
    // lane l fills slot l & 7 of row l >> 3, so it fetches the piece that the swizzle puts there ----
    constexpr int NA = TM / 64, NB = kTN / 64;               // instructions per wavefront and step
    uint32_t a_lane[NA], b_lane[NB];
    const int st_row = lane >> 3, st_piece = (lane & 7) ^ (lane >> 3);
#pragma unroll
    for (int i = 0; i < NA; ++i)
        a_lane[i] = (wave * NA + i) * 8 + st_row < a_rows ? ((uint32_t)((wave * NA + i) * 8 + st_row) * (uint32_t)p.K + st_piece * 8) * 2u : kNoRow;
#pragma unroll
    for (int i = 0; i < NB; ++i)
        b_lane[i] = (wave * NB + i) * 8 + st_row < b_rows ? ((uint32_t)((wave * NB + i) * 8 + st_row) * (uint32_t)p.K + st_piece * 8) * 2u : kNoRow;
    // Where registers are short two of the four addresses are the other two plus a row group: with four the 4-bit tall tile spills as many
    // registers, at the same speed to 1 % (28672 x 4096 at 2048 rows 380 us, 383 spilling; 8192 x 8192 at 8192 796 and 789).  Rows past M
    // are beyond the resource by themselves there; K < 2^23 keeps the offsets of 256 rows in 32 bits.
    const uint32_t a_first = ((uint32_t)(wave * NA * 8 + st_row) * (uint32_t)p.K + st_piece * 8) * 2u;
    auto a_off = [&](int i) {
        if constexpr (BSRC == 4 && IN_PLACE) {
            uint32_t next, o = i < 2 ? a_first : a_lane[2];
            if (i & 1) asm volatile("v_add_u32 %0, %1, %2" : "=v"(next) : "s"(16u * (uint32_t)p.K), "v"(o));
            return i & 1 ? next : o;
        } else {
            return a_lane[i];
        }
    };
    auto a_dma = [&](int stage, int t, int i) {
        load_to_lds(ra, stage_a(stage) + (wave * NA + i) * 1024, a_off(i), (ks0 + min(t, T - 1)) * (kBK * 2));
    };
    auto b_dma = [&](int stage, int t, int i) {
        load_to_lds(rb, stage_b(stage) + (wave * NB + i) * 1024, b_lane[i], (ks0 + min(t, T - 1)) * (kBK * 2));
    };

    // ---- packed weights: wavefront w dequantises tile-rows 2w and 2w+1 of the 16 in the weight tile.  A unit is one
    // packed tile per tile-row -- two steps at 4 bit, one at 8 bit -- and its scales; two units are in registers ----
    constexpr int SPU = BSRC == 4 ? 2 : 1;                   // steps per unit
    u32x4_t breg[2][2];
    uint16_t sreg[2][2];                                     // (8 bit)
    uint32_t s_next[2], s_pair[2];                           // (4 bit) scales of two units
    uint32_t w_lane[2], s_lane[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int nt = min(n0 / 16 + 2 * wave + q, p.N / 16 - 1);
        w_lane[q] = (uint32_t)nt * (uint32_t)p.KL * 1024u + lane * 16;
        s_lane[q] = (uint32_t)(nt * 16 + nl) * (uint32_t)p.G * 2u;
    }
    // Marked as read once (2) but for 4-bit weights in tall tiles, which other row tiles come back to: without the mark 28672 x 4096 at 512
    // rows 94.0 -> 91.5 us, at 2048 371 -> 369, 8192 x 28672 at 512 in four splits 197 -> 189, 10240 x 8192 at 1024 156 -> 152.  8-bit
    // weights take twice the room (4096 x 14336 at 1024 rows 144 -> 151 without it), and few row tiles are short (8192 x 28672 at 257
    // rows int4 126 -> 131).
    constexpr int STREAM = BSRC == 4 && MBW == 8 ? 0 : 2;
    auto group_of = [&](uint32_t kc) { return __umulhi(kc, p.cpg_inv) + (kc & p.cpg_one); };      // branch-free
    // Scales of 4-bit weights come for two units at once, the second one's in the lanes of odd kq: a load of two bytes a lane touches 16 cache
    // lines (8192 x 28672 at 4096 rows 1381 -> 1362 us, 28672 x 4096 at 2048 381 -> 375, 8192 x 8192 at 8192 with half of them left out
    // 772 -> 766).
    auto b_load_packed = [&](int set, int t) {               // the unit of step t; returns how many loads that takes
        const uint32_t ks = (uint32_t)(ks0 + min(t, T - 1));
        const uint32_t kc = ks >> 1;
        const uint32_t tile = SPU == 2 ? kc : ks;
        if (BSRC == 4 && set == 0) {
            const uint32_t a = group_of(kc), b = group_of((uint32_t)(ks0 + min(t + 2, T - 1)) >> 1);
#pragma unroll
            for (int q = 0; q < 2; ++q) s_next[q] = __builtin_amdgcn_raw_buffer_load_b16(rs, s_lane[q] + (kq & 1 ? b : a) * 2u, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if constexpr (BSRC == 8) sreg[set][q] = __builtin_amdgcn_raw_buffer_load_b16(rs, s_lane[q], (int)(group_of(kc) * 2u), 0);
            breg[set][q] = __builtin_amdgcn_raw_buffer_load_b128(rb, w_lane[q], (int)(tile * 1024u), STREAM);
        }
        return BSRC == 4 && set == 1 ? 2 : 4;
    };
    auto s_take = [&]() {                                    // rows of 16 lanes: the even ones' scales and the odd ones', each in all lanes
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const auto r = __builtin_amdgcn_permlane16_swap(s_next[q], s_next[q], false, false);
            s_pair[q] = r[0] | r[1] << 16;
        }
    };
    // word w of the step: tile-row w >> 1, 32-column operand w & 1
    auto b_store_packed = [&](int set, int half, int stage, int w) {
        const int q = w >> 1, o = w & 1;
        const half_t s = BSRC == 4 ? __builtin_bit_cast(half2_t, s_pair[q])[set] : __builtin_bit_cast(half_t, sreg[set][q]);
        const half2_t s2 = {s, s};
        Half8Words h;
        if constexpr (BSRC == 4) h.v = unpack_word4(breg[set][q][2 * half + o], magic);
        else h.v = unpack_words8(breg[set][q][2 * o], breg[set][q][2 * o + 1]);
#pragma unroll
        for (int e = 0; e < 4; ++e) h.h2[e] = h.h2[e] * s2;             // fp16(q * S)
        *reinterpret_cast<half8_t*>(stage_b(stage) + swizzled((2 * wave + q) * 16 + nl, o * 4 + kq)) = h.v;
    };
    // piece w of four of the weights of step u (mod 4)
    auto b_fill = [&](int u, int w) {
        if constexpr (BSRC == 4) b_store_packed((u >> 1) & 1, u & 1, u & 1, w);
        else if constexpr (BSRC == 8) b_store_packed(u & 1, 0, u & 1, w);
    };

    float4_t acc[MBW][4];
#pragma unroll
    for (int b = 0; b < MBW; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[b][r] = (float4_t){0.f, 0.f, 0.f, 0.f};

    // operand rows of this lane: A rows wm*TM/2 + 16 b + nl, B rows wn*64 + 16 r + nl; (row & 7) == (nl & 7)
    const uint32_t a_rd = (uint32_t)((wm * (TM / 2) + nl) * 128);
    const uint32_t b_rd = (uint32_t)((wn * 64 + nl) * 128);
    const uint32_t po0 = (uint32_t)((kq ^ (nl & 7)) * 16), po1 = (uint32_t)(((4 + kq) ^ (nl & 7)) * 16);
    half8_t aop[2][2][2], bop[2][4];                         // operands: of two phases, row block, slice (slice, row block); of a step, slice
    auto set = [](int u, int ph) { return IN_PLACE ? u & 1 : ph & 1; };
    auto read_a = [&](int u, int ph, int b) {                // row block b of phase ph of step u (mod U)
#pragma unroll
        for (int i = 0; i < 2; ++i)
            aop[set(u, ph)][b][i] = *reinterpret_cast<const half8_t*>(stage_a(u % SA) + a_rd + (ph * 2 + b) * 2048 + (i ? po1 : po0));
    };
    auto read_slice = [&](int u, int i) {                    // all operands of a slice
#pragma unroll
        for (int r = 0; r < 4; ++r) bop[i][r] = *reinterpret_cast<const half8_t*>(stage_b(u % SB) + b_rd + r * 2048 + (i ? po1 : po0));
#pragma unroll
        for (int b = 0; b < 4; ++b) aop[i][b >> 1][b & 1] = *reinterpret_cast<const half8_t*>(stage_a(u % SA) + a_rd + b * 2048 + (i ? po1 : po0));
    };
    auto read_b = [&](int u, int r) {
#pragma unroll
        for (int i = 0; i < 2; ++i) bop[i][r] = *reinterpret_cast<const half8_t*>(stage_b(u % SB) + b_rd + r * 2048 + (i ? po1 : po0));
    };

    // One step = PH phases of 16 MFMAs; every phase reads the operands of the next one.  The last phase's operands are in
    // registers when the barrier before it is passed, so from there on this step's stage is free: the last phase reads
    // the next step's first operands, and from it on the tiles of a later step are requested into the stage just freed.
    // The two slices of a step go into an accumulator one right after the other: that draws less power than to come back for it later
    // (from registers alone, on the whole chip, 2.05 PFLOP/s against 1.95), and power is what bounds a full chip.  It takes all of a step's
    // weight operands in registers; the last phase replaces them as it goes.  Against a slice after the other: dense 8192 x 8192 x 8192
    // 768 -> 746 us, 4096 x 14336 at 2048 rows 188 -> 181; int4 830 -> 800, 8192 x 28672 at 4096 rows 1451 -> 1392; int8 832 -> 806, 1472
    // -> 1402; 128-row tiles int4 3 % and dense 1.5 % faster over 40 and 10 shapes, int8 4.3 % slower (BY_SLICE).
    auto step = [&](int u, int t) {
#pragma unroll
        for (int ph = 0; ph < PH; ++ph) {
            if (ph == PH - 1) {
                // the next step's tiles have landed: only what was requested after them may be outstanding
                if constexpr (BSRC == 0) wait_and_barrier<(SA - 2) * NA + (SB - 2) * NB>();
                else if (BSRC == 8 || u == 1) wait_and_barrier<4>();         // the packed unit requested in the last step
                else if (u == 3) wait_and_barrier<2>();                      // (without scales)
                else wait_and_barrier<0>();
                __builtin_amdgcn_sched_barrier(0);
            }
            auto mfma = [&](int b, int r) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[ph * 2 + b][r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bop[i][r], aop[set(u, ph)][b][i], acc[ph * 2 + b][r], 0, 0, 0);
            };
            if constexpr (BY_SLICE) {
                read_slice(ph == PH - 1 ? u + 1 : u, PH - 1 - ph);
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[b][r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bop[ph][r], aop[ph][b >> 1][b & 1], acc[b][r], 0, 0, 0);
            } else if (IN_PLACE && ph < PH - 1) {
#pragma unroll
                for (int b = 0; b < 2; ++b) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) mfma(b, r);
                    read_a(u, ph + 1, b);
                }
            } else {
                for (int b = 0; b < 2; ++b) read_a(ph == PH - 1 ? u + 1 : u, ph == PH - 1 ? 0 : ph + 1, b);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    mfma(r & 1, r);
                    mfma(~r & 1, r);
                    if (ph == PH - 1) read_b(u + 1, r);
                }
            }
            // weights on their way into LDS: not in the phase before the barrier, which would wait for the stores; in the last one, which
            // has most operands, only where there are two phases (they belong to the step after the next then, into the stage just freed)
            int words = 0;
            if (BSRC != 0 && (PH == 2 || ph < 2)) {
                words = 2;
                if (BSRC == 4 && u == (PH == 2 ? 2 : 3) && ph == (PH == 2 ? 1 : 0)) s_take();      // from here on the next two units
                const int w = PH == 2 ? 2 - 2 * ph : 2 * ph;
                b_fill((u + (PH == 2 && ph == 1 ? 2 : 1)) & 3, w);
                b_fill((u + (PH == 2 && ph == 1 ? 2 : 1)) & 3, w + 1);
            }
            const int pa = (ph + 1) % PH;                     // phases since the barrier
            int vm = 0;
            const int fu = pa == 0 ? u : u + U - 1, ft = pa == 0 ? t : t - 1;    // the step whose stage that barrier freed
            if (pa < AP) {
#pragma unroll
                for (int k = pa * NA / AP; k < (pa + 1) * NA / AP; ++k) a_dma(fu % SA, ft + SA, k);
                vm += NA / AP;
                __builtin_amdgcn_sched_barrier(0x78F);       // everything but memory loads may cross: the counted waits rely on their order
            }
            if constexpr (BSRC == 0) {
                if (BP == 0 ? pa == 0 : pa >= BP) {
                    constexpr int EACH = BP == 0 ? NB : NB / (PH - BP);
#pragma unroll
                    for (int k = (pa - BP) * EACH; k < (pa - BP + 1) * EACH; ++k) b_dma(fu % SB, ft + SB, k);
                    vm += EACH;
                }
            } else if (pa == AP - 1) {
                if constexpr (BSRC == 4) {
                    if ((fu & 1) == 0) vm += b_load_packed((fu >> 1) & 1, ft + 4);       // chunk ft / 2 has just been used up
                } else {
                    vm += b_load_packed((fu + 1) & 1, ft + 3);
                }
            }
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                if (BY_SLICE) {
                    if (g < 4) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                } else if (ph == PH - 1) {
                    if (g < 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    if (g & 1) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                } else if (IN_PLACE ? g % 4 == 3 : g < 4) __builtin_amdgcn_sched_group_barrier(0x100, IN_PLACE ? 2 : 1, 0);
                if (words) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                if (g < vm) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
            if (words) __builtin_amdgcn_sched_group_barrier(0x200, 4, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- prologue: the requests of the steps before the first one, in the order of the loop (its waits are counts);
    // step 0 in LDS, its first operands in registers ----
    if constexpr (BSRC != 0) {
        b_load_packed(0, 0);
        b_load_packed(1, SPU);
    } else if constexpr (SB > SA) {
#pragma unroll
        for (int k = 0; k < NB; ++k) b_dma(0, 0, k);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < SA; ++v) {
#pragma unroll
        for (int k = 0; k < (v == SA - 1 ? NA / AP : NA); ++k) a_dma(v, v, k);       // (the rest, in the first step)
        if constexpr (BSRC == 0) {
            __builtin_amdgcn_sched_barrier(0);
            if (v < SA - 1 || BP == 0)
#pragma unroll
                for (int k = 0; k < NB; ++k) b_dma(v + SB - SA, v + SB - SA, k);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (BSRC != 0) {
        if constexpr (BSRC == 4) s_take();
#pragma unroll
        for (int w = 0; w < 4; ++w) b_fill(0, w);
#pragma unroll
        for (int w = 0; w < (PH == 2 ? 2 : 0); ++w) b_fill(1, w);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (BSRC == 8 && AP == 1) b_load_packed(0, 2);
    wait_and_barrier<(SA - 2) * NA + NA / AP + (BSRC == 0 ? (SB - (BP == 0 ? 1 : 2)) * NB : BSRC == 8 && AP == 1 ? 4 : 0)>();
    if constexpr (BY_SLICE) {
        read_slice(0, 0);
    } else {
        for (int b = 0; b < 2; ++b) read_a(0, 0, b);
#pragma unroll
        for (int r = 0; r < 4; ++r) read_b(0, r);
    }
    __builtin_amdgcn_sched_barrier(0);

    for (int t = 0;; t += U) {            // T is even; leaving between two steps keeps every wait inside an exact count
        bool done = false;
#pragma unroll
        for (int u = 0; u < U; u += 2) {
            step(u, t + u);
            step(u + 1, t + u + 1);
            if (t + u + 2 >= T) {
                done = true;
                break;
            }
        }
        if (done) break;
    }
    wait_and_barrier<0>();                // no load into LDS outlives the workgroup

    // ---- store: the MFMAs take the weights as the first operand, so a lane holds row 16 b + nl and the four columns
    // 16 r + 4 kq + e.  Partial sums go out as they are (16 bytes per lane); fp16 results change lanes through the
    // wavefront's own part of LDS, 16 rows x 128 bytes at a time, so that a store writes whole 128-byte runs ----
    if (p.split_k > 1) {
#pragma unroll
        for (int b = 0; b < MBW; ++b) {
            const int m = m0 + wm * (TM / 2) + b * 16 + nl;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int n = n0 + wn * 64 + r * 16 + kq * 4;
                if (m < p.M && n < p.N) *reinterpret_cast<float4_t*>(p.ws + ((int64_t)sg * p.M + m) * p.N + n) = acc[b][r];
            }
        }
        return;
    }
    typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
    uint8_t* mine = lds_b0 + wave * 2048;
#pragma unroll
    for (int b = 0; b < MBW; ++b) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            half4_t h = {(half_t)acc[b][r][0], (half_t)acc[b][r][1], (half_t)acc[b][r][2], (half_t)acc[b][r][3]};
            *reinterpret_cast<half4_t*>(mine + nl * 128 + (((r * 2 + (kq >> 1)) ^ (nl & 7)) * 16) + (kq & 1) * 8) = h;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = h * 8 + (lane >> 3), piece = lane & 7;
            const u32x4_t v = *reinterpret_cast<const u32x4_t*>(mine + row * 128 + ((piece ^ (row & 7)) * 16));
            const int m = m0 + wm * (TM / 2) + b * 16 + row, n = n0 + wn * 64 + piece * 8;
            if (m >= p.M || n >= p.N) continue;
            // Marked as streaming with dense weights: results that stay in the caches push the operands out (28672 x 4096 at 2048 rows
            // 365 -> 340 us, where the vendor library takes 342; 8192 x 8192 x 8192 736 -> 726; dequantise + GEMM 28672 x 4096 at 2048
            // rows 417 -> 394, 4096 x 4096 at 8192 208 -> 194, with a kernel that reads the results behind it 457 -> 432, 227 -> 224).
            // With packed weights nothing is gained, and such a reader is 0.5 % slower (28672 x 4096 at 2048 rows 407 -> 409).
            u32x4_t* c = reinterpret_cast<u32x4_t*>(p.C + (int64_t)m * p.N + n);
            if constexpr (BSRC == 0) __builtin_nontemporal_store(v, c);
            else *c = v;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

template <int BSRC, int MBW>
hipError_t launch_tile_inst(const TileGroup& group, hipStream_t st) {
    hipLaunchKernelGGL((tile_gemm_kernel<BSRC, MBW>), dim3((unsigned)group.first[group.n]), dim3(kThreads), 0, st, group);
    return hipGetLastError();
}

// All problems of a launch in tiles of 128 or (tall) 256 rows.
hipError_t launch_tiles(TileGroup& group, int bsrc, bool tall, hipStream_t st) {
    const int tm = tall ? 256 : 128;
    group.first[0] = 0;
    for (int i = 0; i < group.n; ++i) {
        TileParams& tp = group.p[i];
        tp.XB = (tp.N + kTN - 1) / kTN;
        tp.ZB = (tp.M + tm - 1) / tm;
        group.blocks[i] = (tp.XB * tp.ZB + kXcds - 1) / kXcds * kXcds;
        group.first[i + 1] = group.first[i] + group.blocks[i] * tp.split_k;
    }
    if (bsrc == 0) return tall ? launch_tile_inst<0, 8>(group, st) : launch_tile_inst<0, 4>(group, st);
    if (bsrc == 4) return tall ? launch_tile_inst<4, 8>(group, st) : launch_tile_inst<4, 4>(group, st);
    return tall ? launch_tile_inst<8, 8>(group, st) : launch_tile_inst<8, 4>(group, st);
}

// rows16: 16-row blocks per wavefront (4 or 8), 0 = choose.
hipError_t launch_tile(const TileParams& tp, int bsrc, int64_t M, int rows16, hipStream_t st) {
    const bool tall = rows16 ? rows16 == 8
                             : M > 128 && tile_model_us(bsrc == 0, 8, M, tp.N, tp.K, tp.split_k) < tile_model_us(bsrc == 0, 4, M, tp.N, tp.K, tp.split_k);
    TileGroup group;
    group.n = 1;
    group.p[0] = tp;
    return launch_tiles(group, bsrc, tall, st);
}

void fill_common(TileParams& tp, const void* A, void* C, float* ws, int64_t M, int64_t N, int64_t K, int split_k) {
    tp.A = static_cast<const half_t*>(A);
    tp.C = static_cast<half_t*>(C);
    tp.ws = ws;
    tp.M = (int)M; tp.N = (int)N; tp.K = (int)K;
    tp.split_k = split_k;
    const int KC = (int)(K / kChunkK);
    tp.kc_base = KC / split_k;
    tp.kc_rem = KC % split_k;
}

}  // namespace

// One workgroup runs per compute unit, so a launch takes rounds of 32 workgroups on each of the eight XCDs; the one with most
// of the tiles (xcd_tile) counts for all (245 rows of 8208 x 9728: 33 tall tiles in seven splits are 231 workgroups, but 35
// of them on one XCD: 88 us, against 63 for 66 short tiles in three).  A 64-column step of a full round takes
// 1.58 us with a 256-row tile and 1.00 with a 128-row one (packed weights; 1.54 and 0.87 dense), of a round that fills half
// the chip or less 1.26 and 0.82 (1.12 and 0.87): the clock depends on how much of the chip is busy.  A round costs 6 us
// besides; a split adds the reduce launch and the partial sums' trip through the workspace, mostly cache.  Fitted to 480
// measured launches of this kernel when all requests of a step went out behind its barrier and each slice came back to its accumulators.
// Against 2888 launches as it is -- thirteen shapes of 3072 to 28672 columns at 128 to 3072 rows, both heights, one to eight splits -- the
// times are too long by 9 and 8 % at 4 bit (128- and 256-row tiles), by -4 and 3 % at 8 bit, 5-7 % rms, and dense ones by some 10 % (8192 x
// 8192 x 8192 812 us here, 726 measured); alike enough for the pick, which is 0.1 % behind the best measured pair on the mean at 4 bit and
// 0.5 % at 8 (4 and 9 % at most).
double tile_model_us(bool dense, int rows16, int64_t M, int64_t N, int64_t K, int split_k) {
    const bool tall = rows16 == 8;
    const double half = tall ? (dense ? 1.12 : 1.26) : (dense ? 0.87 : 0.82);
    const double full = tall ? (dense ? 1.54 : 1.58) : (dense ? 0.87 : 1.00);
    const int64_t per_xcd = (((N + kTN - 1) / kTN) * ((M + 32 * rows16 - 1) / (32 * rows16)) + kXcds - 1) / kXcds;
    const int64_t tiles = per_xcd * kXcds * split_k;
    const double steps = (double)((K / kBK + split_k - 1) / split_k), part = (double)(tiles % 256) / 256.0;
    double t = (double)(tiles / 256) * (steps * full + 6.0);
    if (part > 0.0) t += steps * (half + (full - half) * (part > 0.5 ? 2.0 * part - 1.0 : 0.0)) + 6.0;
    if (split_k > 1) t += 5.3 + (2.0 * split_k * M * N * 4.0 + 2.0 * M * N) / 8.0e6;
    return t;
}

bool tile_plan_valid(const LinearArgs& a, const LinearPlan& p) {
    if (a.g % kChunkK != 0 || a.K % kChunkK != 0) return false;
    return p.split_k >= 1 && p.split_k <= a.K / kChunkK;
}

static TileParams packed_params(const LinearArgs& a, float* workspace, int split_k) {
    TileParams tp;
    fill_common(tp, a.A, a.C, workspace, a.M, a.N, a.K, split_k);
    tp.B = a.qweight;
    tp.scales = static_cast<const half_t*>(a.scales);
    tp.G = (int)(a.K / a.g);
    tp.cpg = (int)(a.g / kChunkK);
    tp.cpg_inv = tp.cpg == 1 ? 0u : (uint32_t)(((uint64_t)1 << 32) / (uint32_t)tp.cpg) + 1u;
    tp.cpg_one = tp.cpg == 1 ? 0xFFFFFFFFu : 0u;
    tp.KL = (int)(a.K / (a.bits == 4 ? 128 : 64));
    tp.b_bytes = (uint32_t)((size_t)a.N * a.K * a.bits / 8);
    tp.sc_bytes = (uint32_t)((size_t)a.N * tp.G * 2);
    return tp;
}

hipError_t launch_linear_tile(const LinearArgs& a, const LinearPlan& p, hipStream_t st) {
    hipError_t e = launch_tile(packed_params(a, a.workspace, p.split_k), a.bits, a.M, p.m_rows16 == 4 || p.m_rows16 == 8 ? p.m_rows16 : 0, st);
    if (e != hipSuccess) return e;
    if (p.split_k > 1) e = launch_splitk_reduce(a.workspace, a.C, a.M * a.N, p.split_k, st);
    return e;
}

hipError_t launch_linear_tiles(const LinearArgs* args, const int* split, int n, int rows16, hipStream_t st) {
    if (n < 1 || n > kMaxTileGroup) return hipErrorInvalidValue;
    int order[kMaxTileGroup];
    for (int i = 0; i < n; ++i) order[i] = i;
    std::sort(order, order + n, [&](int x, int y) { return args[x].K / split[x] > args[y].K / split[y]; });   // longest first
    float* partials[kMaxTileGroup];
    size_t used = 0;
    for (int i = 0; i < n; ++i) {
        partials[i] = split[i] > 1 ? args[i].workspace + used / sizeof(float) : nullptr;
        if (split[i] > 1) used += ((size_t)args[i].M * args[i].N * sizeof(float) * split[i] + 255) & ~(size_t)255;
    }
    TileGroup group;
    group.n = n;
    for (int k = 0; k < n; ++k) group.p[k] = packed_params(args[order[k]], partials[order[k]], split[order[k]]);
    hipError_t e = launch_tiles(group, args[0].bits, rows16 == 8, st);
    for (int i = 0; i < n && e == hipSuccess; ++i)
        if (split[i] > 1) e = launch_splitk_reduce(partials[i], args[i].C, args[i].M * args[i].N, split[i], st);
    return e;
}

hipError_t launch_gemm_fp16(const void* A, const void* W, void* C, float* workspace, int64_t M, int64_t N, int64_t K,
                            int rows16, int split_k, hipStream_t st) {
    TileParams tp;
    fill_common(tp, A, C, workspace, M, N, K, split_k);
    tp.B = W;
    tp.scales = static_cast<const half_t*>(W);           // unused by the dense source; any valid pointer
    tp.G = 1; tp.cpg = 1; tp.cpg_inv = 0; tp.cpg_one = 0xFFFFFFFFu; tp.KL = 0;
    tp.b_bytes = 0;
    tp.sc_bytes = 16;
    hipError_t e = launch_tile(tp, 0, M, rows16, st);
    if (e != hipSuccess) return e;
    if (split_k > 1) e = launch_splitk_reduce(workspace, C, M * N, split_k, st);
    return e;
}

}  // namespace rtn
