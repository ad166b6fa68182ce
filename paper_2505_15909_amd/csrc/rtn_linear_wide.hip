// Fused dequantise-GEMM for larger batches (Section 5: the same weight-only quantised linear layer,
// C = A (q S)^T, when more than a few tokens are processed at once and the matrix cores, not the weight
// stream, start to bound the time).  Two kernels (the other one: rtn_linear_block.h), both with exact integer codes in the MFMAs and the fp16 scale
// applied in fp32 to the partial sum of each group (or of the part of a group that lies in a share of K: scaling is
// linear, so groups may straddle splits).
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
#include "rtn_linear_wide.h"
#include <algorithm>
#include <type_traits>

namespace rtn {

namespace {

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

// Row blocks of 32 rows of the tallest row tile: as many tiles as up to 16 m_rows16 rows each take, of this height or one block less
// (tall_row_tiles), of one height within a round (block_parts).
static int block_rows32(int64_t M, int64_t N, int m_rows16) {
    const int64_t tiles = (M + 16 * m_rows16 - 1) / (16 * m_rows16);
    const int mb = (int)((M + 32 * tiles - 1) / (32 * tiles));
    return N >= (1 << 22) ? std::min(mb, 2) : mb;         // (N < 2^23: the packed matrix is under 2 GiB, K at least 256)
}

// Several problems of one precision and number of groups per unit: row tiles of up to mb blocks, wk wavefronts along K
// for each, 8 / wk along N.  The longest workgroups start first: by units of K and by height.
static hipError_t launch_blocks(const LinearArgs* args, const LinearPlan* plans, int n, int mb, const int* wk, hipStream_t st) {
    const int unit = args[0].bits == 4 ? 512 : 256;       // columns of four packed tiles
    struct Part { int problem, row0, rows, tall, blocks; bool sliced; int64_t length; };
    Part parts[kMaxBlockParts];
    BlockTiles tiles[kMaxBlockGroup];
    int count = 0;
    int64_t workgroups = 0;
    for (int i = 0; i < n; ++i) {
        tiles[i] = block_tiles(args[i].M, args[i].N, mb, wk[i], plans[i].split_k);
        workgroups += tiles[i].workgroups();
    }
    for (int i = 0; i < n; ++i) {
        const BlockParts p = block_parts(tiles[i], mb, workgroups <= 256);
        const int64_t units = (args[i].K / unit + plans[i].split_k * wk[i] - 1) / (plans[i].split_k * wk[i]);
        for (int k = 0; k < p.n; ++k)
            parts[count++] = {i, p.part[k].row0, p.part[k].rows, p.part[k].tall, wide_blocks((int)tiles[i].columns, p.part[k].rows, p.sliced),
                              p.sliced, units * (p.part[k].tall > 0 ? mb : mb - 1)};
    }
    std::stable_sort(parts, parts + count, [](const Part& x, const Part& y) { return x.length > y.length; });
    BlockGroup g = {};
    g.n = count;
    int slot[kMaxBlockGroup], filled = 0;                 // problems in the order of their first parts (block_part)
    std::fill(slot, slot + n, -1);
    for (int part = 0; part < count; ++part) {
        const int i = parts[part].problem;
        if (slot[i] >= 0) continue;
        slot[i] = filled;
        const LinearArgs& a = args[i];
        BlockProblem& bp = g.p[filled++];
        bp.A = static_cast<const half_t*>(a.A);
        bp.qw = static_cast<const uint8_t*>(a.qweight);
        bp.scales = static_cast<const half_t*>(a.scales);
        bp.zeros = static_cast<const half_t*>(a.zeros);
        bp.C = static_cast<half_t*>(a.C);
        bp.ws = a.workspace;
        bp.M = (int)a.M; bp.N = (int)a.N; bp.K = (int)a.K;
        bp.G = (int)(a.K / a.g);
        bp.XB = (int)tiles[i].columns;
        const uint32_t units = (uint32_t)(a.K / unit), split = (uint32_t)plans[i].split_k, upg = a.g >= unit ? (uint32_t)(a.g / unit) : 1u;
        bp.u_share = units / split | (units % split) << 16;      // (K < 2^23: both under 2^15)
        bp.groups = upg | split << 16 | (uint32_t)wk[i] << 24;
        bp.upg_inv = upg == 1 ? 0u : (uint32_t)(((uint64_t)1 << 32) / upg) + 1u;
    }
    int64_t first = 0;
    for (int i = 0; i < count; ++i) {
        BlockPart& part = g.part[i];
        part.first = (int)first;
        part.blocks = parts[i].blocks;
        part.row0 = parts[i].row0;
        part.tall = parts[i].tall;
        part.info = (uint32_t)parts[i].rows | (parts[i].sliced ? 1u << 17 : 0u) | (uint32_t)slot[parts[i].problem] << 20;   // (M <= 2^20: at most 2^15 tiles)
        first += (int64_t)part.blocks * plans[parts[i].problem].split_k;
    }
    if (first >= (int64_t)1 << 31) return hipErrorInvalidValue;
    const int ng = args[0].g >= unit ? 1 : (int)(unit / args[0].g);
    if (args[0].zeros) return args[0].bits == 4 ? launch_block<4, true>(g, ng, mb, (unsigned)first, st) : launch_block<8, true>(g, ng, mb, (unsigned)first, st);
    return args[0].bits == 4 ? launch_block<4, false>(g, ng, mb, (unsigned)first, st) : launch_block<8, false>(g, ng, mb, (unsigned)first, st);
}

static hipError_t launch_linear_block(const LinearArgs& a, const LinearPlan& p, int wk, hipStream_t st) {
    hipError_t e = launch_blocks(&a, &p, 1, block_rows32(a.M, a.N, p.m_rows16), &wk, st);
    if (e != hipSuccess) return e;
    if (p.split_k > 1) e = launch_splitk_reduce(a.workspace, static_cast<half_t*>(a.C), a.M * a.N, p.split_k, st);
    return e;
}

hipError_t launch_linear_blocks(const LinearArgs* args, const LinearPlan* plans, int n, int mb, hipStream_t st) {
    int wk[kMaxBlockGroup];
    LinearArgs a[kMaxBlockGroup];
    size_t used = 0;
    for (int i = 0; i < n; ++i) {
        a[i] = args[i];
        wk[i] = plans[i].waves_k;
        if (plans[i].split_k == 1) continue;
        a[i].workspace = a[i].workspace + used / sizeof(float);
        used += ((size_t)a[i].M * a[i].N * sizeof(float) * plans[i].split_k + 255) & ~(size_t)255;
    }
    hipError_t e = launch_blocks(a, plans, n, mb, wk, st);
    for (int i = 0; i < n && e == hipSuccess; ++i)
        if (plans[i].split_k > 1) e = launch_splitk_reduce(a[i].workspace, static_cast<half_t*>(a[i].C), a[i].M * a[i].N, plans[i].split_k, st);
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
