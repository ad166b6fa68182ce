// Host-side interfaces between the C-ABI translation unit and the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <vector>

namespace rtn {

constexpr size_t kMaxLdsBytes = 160 * 1024;   // LDS of one gfx950 compute unit, usable by one workgroup

// Resolved launch configuration of the fused dequantise-GEMM.
struct LinearPlan {
    int path;       // 1 = MFMA skinny kernel, 2 = vector-ALU dot kernel, 3 = wide and block kernels (larger batches),
                    // 4 = tile kernel, 128 or 256 rows x 256 columns per workgroup (matrix-core bound batches)
    int prefetch;   // k-chunks in flight per wavefront (register buffers): 1, 2 or 4
    int waves_n;    // wavefronts along N per workgroup
    int waves_k;    // wavefronts along K per workgroup
    int split_k;    // workgroups along K
    int m_rows16;   // 16-row activation blocks per wavefront: 1, 2 or 4 (prefetch must be 1 above 1)
    int m_blocks;   // activation blocks of 16 * m_rows16 rows (grid.z)
    int n_tiles16;  // path 3: 16-column weight tile-rows per wavefront: 1, 2 or 4
};

struct LinearArgs {
    const void* A;
    const void* qweight;
    const void* scales;
    void* C;
    float* workspace;
    int64_t M, N, K, g;
    int bits;
    const void* zeros = nullptr;   // fp16 [N, K/g] integer zero points (asymmetric variant; skinny and wide kernels) or null
};

// How a skinny-kernel workgroup gets its activations: k-chunks per wavefront, stages, bytes of its whole slice, LDS it takes.
struct StagePlan { int per, nstage; size_t slice, lds; };
StagePlan linear_stages(const LinearArgs& a, const LinearPlan& p);

hipError_t launch_quantize(const void* W, int64_t N, int64_t K, int bits, int64_t g, float divisor,
                           void* qweight, void* scales, hipStream_t st);
// Asymmetric variant: codes, fp16 scales and fp16 integer zero points Z, dequantised weight S (q + Z).
hipError_t launch_quantize_asym(const void* W, int64_t N, int64_t K, int bits, int64_t g, void* qweight, void* scales,
                                void* zeros, hipStream_t st);
// zeros: null for the symmetric variant.
hipError_t launch_unpack(const void* qweight, const void* scales, int64_t N, int64_t K, int bits, int64_t g,
                         bool dequant, void* out, hipStream_t st, const void* zeros = nullptr);
hipError_t launch_linear(const LinearArgs& a, const LinearPlan& p, hipStream_t st);
// n independent problems with resolved plans: compatible skinny-kernel launches are merged into grouped launches.  common_plan:
// the plans were made for one launch.
hipError_t launch_linear_grouped(const LinearArgs* args, const LinearPlan* plans, int n, bool common_plan, hipStream_t st);
// The launch (0, 1, ...) that each of them goes out with.
std::vector<int> grouped_launches(const LinearArgs* args, const LinearPlan* plans, int n, bool common_plan);
// Wide kernel: whether column tiles go to the XCDs in contiguous slices, none more than one tile longer than another,
// instead of dealt in turn.  Only where that saves a round of workgroups on the XCD with most of them (32 compute units):
// then it pays (816 rows of 384 x 10240: 62 us -> 22, 143 of 20912 x 14848: 230 -> 126); otherwise the cuts, which may
// part the row tiles that share a column tile's weights, only cost (int8, 71 rows of 3072 x 8192: 16.4 us dealt, 18.0
// sliced; 221 rows of 5984 x 12288: 59 and 66).  118 shapes measured, none on the wrong side.
inline bool xcd_slices_save_a_round(int64_t XB, int64_t ZB, int64_t split_k) {
    const int64_t dealt = (XB + 7) / 8 * ZB * split_k, sliced = (XB * ZB + 7) / 8 * split_k;
    return (sliced + 31) / 32 < (dealt + 31) / 32;
}
inline int wide_blocks(int XB, int ZB, bool sliced) { return 8 * (sliced ? (XB * ZB + 7) / 8 : (XB + 7) / 8 * ZB); }
// Path 3: plan check (group size 32, 64 or a multiple of 128; m_rows16 x n_tiles16 as the file's header lists them) and launch, on the
// wide kernel (eight wavefronts of one tile-row) or the block kernel (everything else, by the columns of a workgroup).
bool wide_plan_valid(const LinearArgs& a, const LinearPlan& p);
hipError_t launch_linear_wide(const LinearArgs& a, const LinearPlan& p, hipStream_t st);
// The block kernel of path 3 on several independent problems at once: one precision and number of groups per unit of four packed
// tiles, row tiles of up to mb blocks of 32 rows, waves_k of each problem's plan of eight wavefronts along K; partial sums of K
// splits go to the workspace one problem after another.
constexpr int kMaxBlockGroup = 8;
// Whether a shape (mb row blocks, wk wavefronts along K) has a kernel of its own: such a launch has it for all its problems.
constexpr bool block_shape_alone(int bits, int mb, int wk) { return mb * wk > 8 || (bits == 8 && wk == 8); }
// Row tiles of the block kernel: ceil(M / 32 mb) of them, the first tall_row_tiles(M, mb) of 32 mb rows, the others of 32 rows less.
inline int tall_row_tiles(int64_t M, int mb) {
    const int64_t tiles = (M + 32 * mb - 1) / (32 * mb), tall = (M + 31) / 32 - tiles * (mb - 1);
    return (int)(mb == 1 ? tiles : tall > 0 ? tall : 0);
}
// The workgroups of a problem in a launch of the block kernel: column tiles (256 / wavefronts along K columns), row tiles, K splits.
struct BlockTiles {
    int64_t columns;
    int rows, tall, split;
    int64_t workgroups() const { return columns * rows * split; }
};
inline BlockTiles block_tiles(int64_t M, int64_t N, int mb, int wk, int split) {
    return {(N + 256 / wk - 1) / (256 / wk), (int)((M + 32 * mb - 1) / (32 * mb)), tall_row_tiles(M, mb), split};
}
// Its parts: a launch of at most a round of workgroups (256, of all its problems) has tiles of one height, which keeps those of a column in
// step on its weights; a larger one has the tall tiles and the low ones apart.  sliced: the order over the XCDs, as above, one
// for both parts -- each by itself may save no round where both together do (3232 x 3584 int4 group 64 at 605 rows 38 us, 30
// this way; 25856 x 4608 int8 at 278 rows 110 and 92).
struct BlockParts {
    int n;
    bool sliced;
    struct { int row0, rows, tall; int64_t on_xcd; } part[2];      // first row, row tiles, tall ones of them; workgroups on the fullest XCD
};
inline BlockParts block_parts(const BlockTiles& t, int mb, bool one_round) {
    BlockParts p = {};
    if (one_round || t.tall == 0 || t.tall == t.rows) {
        p.n = 1;
        p.part[0] = {0, t.rows, t.tall > 0 ? t.rows : 0, 0};
    } else {
        p.n = 2;
        p.part[0] = {0, t.tall, t.tall, 0};
        p.part[1] = {t.tall * 32 * mb, t.rows - t.tall, 0, 0};
    }
    int64_t dealt[2] = {}, sliced[2] = {};
    for (int i = 0; i < p.n; ++i) {
        dealt[i] = (t.columns + 7) / 8 * p.part[i].rows * t.split;
        sliced[i] = (t.columns * p.part[i].rows + 7) / 8 * t.split;
    }
    p.sliced = (sliced[0] + sliced[1] + 31) / 32 < (dealt[0] + dealt[1] + 31) / 32;
    for (int i = 0; i < p.n; ++i) p.part[i].on_xcd = p.sliced ? sliced[i] : dealt[i];
    return p;
}
hipError_t launch_linear_blocks(const LinearArgs* args, const LinearPlan* plans, int n, int mb, hipStream_t st);
// Path 4 (tile kernel, weights dequantised into LDS): plan check (group size a multiple of 128) and launch.
bool tile_plan_valid(const LinearArgs& a, const LinearPlan& p);
hipError_t launch_linear_tile(const LinearArgs& a, const LinearPlan& p, hipStream_t st);
// The tile kernel on several independent problems of one precision at once, in tiles of 16 rows16 x 2 rows (rows16 = 4 or 8); partial
// sums of K splits go to the workspace one problem after another.
constexpr int kMaxTileGroup = kMaxBlockGroup;
hipError_t launch_linear_tiles(const LinearArgs* args, const int* split, int n, int rows16, hipStream_t st);
// Dense fp16 GEMM C[M,N] = A[M,K] W[N,K]^T with the same tile kernel (K a multiple of 128; rows16 = 4 or 8); split_k > 1 goes
// through the fp32 workspace [split_k][M][N].
hipError_t launch_gemm_fp16(const void* A, const void* W, void* C, float* workspace, int64_t M, int64_t N, int64_t K,
                            int rows16, int split_k, hipStream_t st);
// Modelled time of a tile-kernel launch (rows16 = 4 or 8: 128- or 256-row tiles), the reduce pass of a K split included.
double tile_model_us(bool dense, int rows16, int64_t M, int64_t N, int64_t K, int split_k);
// Sums split_k fp32 partial outputs [split_k][MN] in a fixed order into fp16 C (MN a multiple of 16).
hipError_t launch_splitk_reduce(const float* workspace, void* C_fp16, int64_t MN, int split_k, hipStream_t st);

// LDS bytes the skinny kernel needs for a plan (staged activation slice incl. the zero row, or the
// in-workgroup split-K reduction buffer, whichever is larger).
size_t linear_lds_bytes(const LinearArgs& a, const LinearPlan& p);
// Whether the plan's activation staging fits the LDS limit and the per-thread staging registers.
bool linear_plan_fits(const LinearArgs& a, const LinearPlan& p, size_t lds_limit);

}  // namespace rtn
