// Host-only report of the launches behind a call: reads problems from standard input, prints the launches with their
// plans.  The library's C-ABI translation unit is part of this one, so that its planning functions can be called; no GPU
// work, nothing is launched.  Built and read by tests/test_host_plans.py.
#include "../../paper_2505_15909_amd/csrc/rtn_api.hip"
#include "../../paper_2505_15909_amd/csrc/rtn_device.h"
#include <stdio.h>
#include <new>

static long heap_calls = 0;
void* operator new(size_t n) {
    ++heap_calls;
    if (void* p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

static char stand_in[64];                                      // addresses only, nothing is read or written

static LinearArgs problem(int64_t M, int64_t N, int64_t K, int bits, int64_t g, bool workspace) {
    LinearArgs a;
    a.A = a.qweight = a.scales = stand_in;
    a.C = stand_in;
    a.workspace = workspace ? reinterpret_cast<float*>(stand_in) : nullptr;
    a.M = M; a.N = N; a.K = K; a.bits = bits; a.g = g;
    return a;
}

static void print_plan(const LinearArgs& a, const LinearPlan& p) {
    printf(" [%ld %d %d %d %d %d %d %d %d]", (long)a.M, p.path, p.prefetch, p.waves_n, p.waves_k, p.split_k, p.m_rows16, p.m_blocks, p.n_tiles16);
}

int main() {
    char what[16];
    while (scanf("%15s", what) == 1) {
        if (!strcmp(what, "linear")) {                         // M N K bits g workspace -> status, cut and launches
            long M, N, K, g, ws;
            int bits;
            if (scanf("%ld %ld %ld %d %ld %ld", &M, &N, &K, &bits, &g, &ws) != 6) return 1;
            LinearArgs part[2];
            LinearPlan plan[2];
            int n = 0;
            const rtn_status st = linear_launches(problem(M, N, K, bits, g > 0 ? g : K, ws > 0), nullptr, (size_t)ws, part, plan, &n);
            printf("%d", (int)st);
            for (int i = 0; st == RTN_OK && i < n; ++i) print_plan(part[i], plan[i]);
        } else if (!strcmp(what, "asym")) {                    // the same with zero points: status and plan
            long M, N, K, g, ws;
            int bits;
            if (scanf("%ld %ld %ld %d %ld %ld", &M, &N, &K, &bits, &g, &ws) != 6) return 1;
            LinearArgs a = problem(M, N, K, bits, g > 0 ? g : K, ws > 0);
            a.zeros = stand_in;
            LinearPlan plan;
            const rtn_status st = resolve_plan_zp(a, (size_t)ws, &plan);
            printf("%d", (int)st);
            if (st == RTN_OK) print_plan(a, plan);
        } else if (!strcmp(what, "tile")) {                    // M N K rows16 split -> modelled time of a tile-kernel launch
            long M, N, K;
            int rows16, split;
            if (scanf("%ld %ld %ld %d %d", &M, &N, &K, &rows16, &split) != 5) return 1;
            printf("%.6f", rtn::tile_model_us(false, rows16, M, N, K, split));
        } else if (!strcmp(what, "wide")) {                    // XB ZB split -> 1 if sliced, then [xb zb xcd ...] of the launch
            int XB, ZB, split;
            if (scanf("%d %d %d", &XB, &ZB, &split) != 3) return 1;
            const bool sliced = rtn::xcd_slices_save_a_round(XB, ZB, split);
            const int blocks = rtn::wide_blocks(XB, ZB, sliced);
            printf("%d [", sliced ? 1 : 0);
            for (int b = 0; b < blocks; ++b) {
                int xb, zb;
                if (rtn::xcd_wide_tile(b, XB, ZB, sliced, &xb, &zb)) printf("%d %d %d ", xb, zb, b % rtn::kXcds);
            }
            printf("]");
        } else if (!strcmp(what, "parts")) {                   // mb n, then M N wk split each -> 1 if one round, then a launch's [problem row0 rows tall on_xcd]
            int mb, n;                                         // and of each part [columns, then xb zb xcd of its workgroups]
            if (scanf("%d %d", &mb, &n) != 2 || n < 1 || n > rtn::kMaxBlockGroup) return 1;
            rtn::BlockTiles t[rtn::kMaxBlockGroup];
            int64_t workgroups = 0;
            for (int i = 0; i < n; ++i) {
                long M, N;
                int wk, split;
                if (scanf("%ld %ld %d %d", &M, &N, &wk, &split) != 4) return 1;
                t[i] = rtn::block_tiles(M, N, mb, wk, split);
                workgroups += t[i].workgroups();
            }
            printf("%d", workgroups <= 256 ? 1 : 0);
            for (int i = 0; i < n; ++i) {
                const rtn::BlockParts p = rtn::block_parts(t[i], mb, workgroups <= 256);
                for (int k = 0; k < p.n; ++k) {
                    printf(" [%d %d %d %d %ld] [%ld", i, p.part[k].row0, p.part[k].rows, p.part[k].tall, (long)p.part[k].on_xcd, (long)t[i].columns);
                    const int blocks = rtn::wide_blocks((int)t[i].columns, p.part[k].rows, p.sliced);
                    for (int b = 0; b < blocks; ++b) {
                        int xb, zb;
                        if (rtn::xcd_wide_tile(b, (int)t[i].columns, p.part[k].rows, p.sliced, &xb, &zb)) printf(" %d %d %d", xb, zb, b % rtn::kXcds);
                    }
                    printf("]");
                }
            }
        } else if (!strcmp(what, "merged")) {                  // mb n, then M N K bits g wk split each -> modelled time of that shared launch
            MergedPlan m = {};
            int n, longest;
            LinearArgs a[rtn::kMaxBlockGroup];
            if (scanf("%d %d", &m.mb, &n) != 2 || n < 1 || n > rtn::kMaxBlockGroup) return 1;
            for (int i = 0; i < n; ++i) {
                long M, N, K, g;
                int bits;
                if (scanf("%ld %ld %ld %d %ld %d %d", &M, &N, &K, &bits, &g, &m.waves[i], &m.split[i]) != 7) return 1;
                a[i] = problem(M, N, K, bits, g > 0 ? g : K, true);
            }
            printf("%.6f", merged_blocks_us(a, n, m, (size_t)1 << 40, &longest));
        } else if (!strcmp(what, "heap")) {                    // n, then M N K bits g each -> heap allocations of planning a shared launch
            int n;
            LinearArgs a[rtn::kMaxBlockGroup];
            if (scanf("%d", &n) != 1 || n < 1 || n > rtn::kMaxBlockGroup) return 1;
            for (int i = 0; i < n; ++i) {
                long M, N, K, g;
                int bits;
                if (scanf("%ld %ld %ld %d %ld", &M, &N, &K, &bits, &g) != 5) return 1;
                a[i] = problem(M, N, K, bits, g > 0 ? g : K, true);
            }
            const long before = heap_calls;
            const MergedPlan blocks = remembered_merge(a, n, (size_t)256 << 20), tiles = remembered_merge(a, n, (size_t)256 << 20, true);
            printf("%ld %d", heap_calls - before, blocks.us > 0.0 && tiles.us > 0.0 ? 1 : 0);
        } else if (!strcmp(what, "issued") || !strcmp(what, "issued_grouped")) {   // workspace n, then M N K bits g each
            // the launches of rtn_layer_forward (status 0; 1 = the small-batch kernel's merged launch, -1 = one by one in order) or of the block
            // kernel in rtn_grouped_forward (those of one module go on): [kernel mb wk, then module and split each]
            long ws;
            int n;
            if (scanf("%ld %d", &ws, &n) != 2 || n < 1 || n > 32) return 1;
            LinearArgs a[32];
            LinearPlan plan[32];
            SharedLaunch l[32];
            for (int i = 0; i < n; ++i) {
                long M, N, K, g;
                int bits;
                if (scanf("%ld %ld %ld %d %ld", &M, &N, &K, &bits, &g) != 5) return 1;
                a[i] = problem(M, N, K, bits, g > 0 ? g : K, ws > 0);
            }
            bool tiles = false;
            int status = 0, count = 0;
            if (strlen(what) > 6) {
                GroupedCall call;
                if (plan_grouped_call(a, n, (size_t)ws, &call) != RTN_OK) return 1;
                for (const SharedLaunch& b : call.blocks) l[count++] = b;
                for (int i : call.left) {
                    l[count].count = 1;
                    l[count++].member[0] = i;
                }
            } else if (n > 1 && n <= 16 && merged_layer_plans(a, n, (size_t)ws, plan)) {
                status = 1;
            } else {
                count = layer_launches(a, n, (size_t)ws, l, &tiles);
                if (count < 0) status = -1;
            }
            printf("%d", status);
            for (int i = 0; i < count; ++i) {
                const bool alone = l[i].count == 1;
                printf(" [%d %d %d", alone ? 0 : tiles ? 4 : 3, alone ? 0 : l[i].plan.mb, alone ? 0 : l[i].plan.wk);
                for (int k = 0; k < l[i].count; ++k) printf(" %d %d", l[i].member[k], alone ? 0 : l[i].plan.split[k]);
                printf("]");
            }
        } else if (!strcmp(what, "sets")) {                    // workspace n, then M N K bits g each -> status, then plan and [share, 1 if the plan can run] of each module
            long ws;                                           // share: of the modelled time of its set, in picoseconds, 0 in none
            int n;
            if (scanf("%ld %d", &ws, &n) != 2 || n < 1 || n > 64) return 1;
            LinearArgs a[64];
            LinearPlan plan[64];
            SetShare share[64];
            for (int i = 0; i < n; ++i) {
                long M, N, K, g;
                int bits;
                if (scanf("%ld %ld %ld %d %ld", &M, &N, &K, &bits, &g) != 5) return 1;
                a[i] = problem(M, N, K, bits, g > 0 ? g : K, ws > 0);
            }
            const rtn_status st = grouped_plans(a, n, (size_t)ws, plan, share);
            printf("%d", (int)st);
            for (int i = 0; st == RTN_OK && i < n; ++i) {
                print_plan(a[i], plan[i]);
                printf(" [%ld %d]", (long)(share[i].us * 1e6), rtn::linear_plan_fits(a[i], plan[i], (size_t)device_max_lds()) ? 1 : 0);
            }
        } else if (!strcmp(what, "set_rows")) {                // N K bits g n, then M each -> [modules of 1, 2, .. 16 rows] that such a set is planned for
            long N, K, g;
            int bits, n, member[kModuleSet], rows[kSetRows + 1] = {};
            if (scanf("%ld %ld %d %ld %d", &N, &K, &bits, &g, &n) != 5 || n < 2 || n > kModuleSet) return 1;
            LinearArgs a[kModuleSet];
            for (int i = 0; i < n; ++i) {
                long M;
                if (scanf("%ld", &M) != 1 || M < 1 || M > kSetRows) return 1;
                a[i] = problem(M, N, K, bits, g > 0 ? g : K, true);
                member[i] = i;
            }
            module_set_rows(a, member, n, rows);
            printf("0 [");
            for (int m = 1; m <= kSetRows; ++m) printf("%d ", rows[m]);
            printf("]");
        } else if (!strcmp(what, "layer") || !strcmp(what, "grouped")) {   // bits g workspace n, then M N K each
            // layer -> 1 if one launch, plans; grouped -> status, [launch of each module that no launch of the block kernel has]
            long g, ws;
            int bits, n;
            if (scanf("%d %ld %ld %d", &bits, &g, &ws, &n) != 4 || n < 1 || n > 16) return 1;
            LinearArgs a[16];
            LinearPlan plan[16];
            for (int i = 0; i < n; ++i) {
                long M, N, K;
                if (scanf("%ld %ld %ld", &M, &N, &K) != 3) return 1;
                a[i] = problem(M, N, K, bits, g > 0 ? g : K, ws > 0);
            }
            if (what[0] == 'g') {
                GroupedCall call;
                const rtn_status st = plan_grouped_call(a, n, (size_t)ws, &call);
                printf("%d [", (int)st);
                for (size_t k = 0; k < call.left.size(); ++k) a[k] = a[call.left[k]];
                if (st == RTN_OK)
                    for (int l : rtn::grouped_launches(a, call.plans.data(), (int)call.left.size(), false)) printf("%d ", l);
                printf("]\n");
                continue;
            }
            const bool one = merged_layer_plans(a, n, (size_t)ws, plan);
            printf("%d", one ? 1 : 0);
            for (int i = 0; one && i < n; ++i) print_plan(a[i], plan[i]);
        } else {
            return 1;
        }
        printf("\n");
    }
    return 0;
}
