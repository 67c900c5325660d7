// SVIP hot path for MI355X (gfx950): launch code and the C ABI declared in include/svip.h; the kernels
// live in draft_kernels.h, loop_kernels.h, verify_kernels.h, greedy_kernels.h, pair_kernels.h and warp_kernels.h.
//
// svip_draft_step  =  k_draft_stats    grid (rows * records / 4) one wave per record: (m, S, t) of a tile of a row
//                     k_draft_finish_* grid (rows)               merge of the records: entropy, stop test, inverse
//                                      CDF inside the one record that holds the draw (greedy: the first maximum)
//                     k_draft_step     both in one launch, for small steps: the row's last workgroup merges
// svip_verify      =  k_verify_stats   grid (stat rows * slices) per-slice (reference, sum) of every needed row
//                     k_accept         grid (sequences), 1 wave  p/q tests, ballot scan for the first rejection (small calls: in k_resid)
//                     k_resid          grid (sequences * slices) slice masses of the residual / bonus row; the workgroup
//                                      that finishes a sequence last draws the token
// svip_verify_greedy = k_argmax        grid (target rows * slices) first maximum per slice, no exponentials
//                     k_accept_greedy  grid (sequences), 1 wave  argmax p == x test, ballot, correction = argmax p
//
// svip_pair_stats  =  k_verify_stats   (rows j < draft_len of both models), k_pair_L (logsumexps),
//                     k_pair_sums      grid (slices, positions)  sum min(p,q), sum q log(q/p), sum q log q
//                     k_pair_finish    one thread per position   beta, KL, cross entropy, the bounds
//
// svip_loop_run   =  k_group_stats, k_group_finish   several draft positions per pair of launches (sampling)
//                     k_stream_rows, k_stream_advance   the same with the greedy verification of the round
//
// svip_warp_logits =  k_warp           grid (rows), 1024 threads  top-k / top-p thresholds by radix select, masked copy
//
// The passes are bound by HBM reads of the logits; there is no dense contraction, hence no MFMA.
// Nothing spins or waits on the device: kernels of one call are ordered by the stream; inside the
// residual pass the "last workgroup" hand-over of exchange.h lets a sequence's draw follow its slices
// without a second launch.  Each finishing step issues all of its independent loads before the first
// dependent one, because at small batches a step is bound by round trips to memory, not by bandwidth.
// Workgroups are handed to the chip's 8 XCDs in turn and each XCD has its own L2: k_draft_stats and k_resid
// map workgroups to (row, records) so that everything of row b runs on XCD b % 8, where the workgroup that
// finishes the row reads records and a tile again.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>

#include <type_traits>

#include "../../include/svip.h"
#include "../../include/svip_bench.h"
#include "row_math.h"
#include "svip_internal.h"

#include "kernel_args.h"
#include "sample_weights.h"
#include "draft_kernels.h"
#include "greedy_kernels.h"
#include "loop_kernels.h"
#include "verify_kernels.h"
#include "pair_kernels.h"
#include "warp_kernels.h"

namespace svip {

// svip_workspace_reset: the flag word and the ticket counters at the end of the workspace.
struct ZeroArgs {
    unsigned *flags;
    uint4 *tail;
    size_t n16;
};
__global__ void k_zero(ZeroArgs z)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *z.flags = 0u;
    const uint4 zero = {0u, 0u, 0u, 0u};
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < z.n16; i += (size_t)gridDim.x * blockDim.x)
        z.tail[i] = zero;
}

// Reference kernels of the benchmark hooks: an empty launch, and a read-only stream with the access
// pattern of the statistics passes (256-thread workgroups, NV 16-byte non-temporal loads per thread, a
// wave reads 1 KiB contiguous per load) that only folds what it read into one word per wave.
__global__ __launch_bounds__(64) void k_empty(int) {}

struct StreamArgs {
    const u32x4 *buf;
    size_t nvec;
    unsigned *sink;
};
template <int NV>
__global__ __launch_bounds__(WG) void k_stream_read(StreamArgs a)
{
    const size_t base = (size_t)blockIdx.x * (WG * NV) + threadIdx.x;
    u32x4 v[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const size_t i = base + (size_t)u * WG;
        const u32x4 zero = {0u, 0u, 0u, 0u};
        v[u] = i < a.nvec ? __builtin_nontemporal_load(a.buf + i) : zero;
    }
    unsigned x = 0u;
#pragma unroll
    for (int u = 0; u < NV; ++u) x ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    x = (unsigned)wave_reduce((int)x, OpMax{});
    if ((threadIdx.x & 63) == 0) a.sink[(size_t)blockIdx.x * NWAVE + (threadIdx.x >> 6)] = x;
}

// Scratch of svip_draft_step_static: the workspace of a draft step for callers that cannot allocate one.
// One copy per GPU the library runs on, held until the process ends.  Host code never uses this name as an
// address: static_scratch() asks the runtime for the array's device address, once per device.
static __device__ __align__(256) unsigned char scratch[SVIP_STATIC_SCRATCH_BYTES];

// ---- host side -------------------------------------------------------------------------------

// Launch-shape overrides for experiments (svip_bench_set_tuning; all zero = the library's own choice).
// Workspace sizes are always computed for the library's own choice; a forced shape that needs more than
// the workspace holds is rejected by the call.
static svip_bench_tuning g_tune = {0, 0, 0, 0, 0, 0, 0};
static int *g_warp_routes = nullptr;             // svip_bench_warp_routes

// Slices per row of the passes that give a slice to a workgroup: enough workgroups to fill 256 CUs several
// times over, at most MAX_SLICES; want_one_batch (the residual pass): slices of min_tiles tiles, which the
// sampler scans as one batch and whose tiles each get a mass of their own.
static Geo make_geo(int V, int vec, long long rows, bool want_one_batch, int forced_ns, int min_tiles = 4, bool fine = false)
{
    Geo g;
    g.V = V;
    const int nvec = (V + vec - 1) / vec;
    g.ntiles = (nvec + WG - 1) / WG;
    long long ns;
    if (want_one_batch) {
        // slices of min_tiles tiles (4: 32 logits per thread, and few enough tiles for tile masses)
        long long cap = g.ntiles / min_tiles;
        if (cap < 1) cap = 1;
        ns = cap;
        const long long need = (g.ntiles + LOCATE_UNROLL - 1) / LOCATE_UNROLL;
        if (ns < need) ns = need;
        // large batches are bound by bandwidth, not by latency: longer slices of an odd number of
        // tiles (7) stream better than one-batch slices of 4, at the price of a two-batch search
        if (rows >= 512 && g.ntiles >= 14) ns = (g.ntiles + 6) / 7;
    } else {
        // streaming passes: about 8192 workgroups of at least 8 tiles each.  fine: rows of 8 to 23 tiles, of one or two such slices, two to
        // four (as many as the acceptance test requests together) of at least 4 tiles, while that makes few workgroups: us, coarse / finer,
        // of svip_verify (see finer_stats), svip_verify_greedy, svip_pair_stats and, the logsumexps recomputed, svip_verify:
        //   workgroups  10 tiles                           14 tiles                          20 tiles                          23 tiles
        //     160..300  13.4 12.6,  7.2 6.2, 17.3 14.5     13.8 11.9, 7.2 5.6, 17.5 13.6     18.0 16.5, 7.6 6.4, 19.9 16.1     14.3 13.2, 7.5 6.7, 18.8 15.4
        //     640..700  14.8 13.8,  8.3 7.1, 20.6 17.9     15.6 14.2, 8.1 7.1, 19.2 16.8     16.1 15.2, 7.7 6.9, 18.9 16.7     17.8 17.8, 8.4 7.7, 19.7 18.3
        //   1050..1250  20.6 20.0,  9.0 8.3, 25.3 23.4     15.7 14.9, 8.6 7.6, 23.4 21.0     18.9 17.4, 8.5 7.5, 24.5 23.4     20.2 19.7, 9.3 9.0, 27.8 25.9
        //    ... recomp. 17.2 16.1                         16.7 15.5                         17.5 16.6                         21.4 21.0
        //   1970..2020  18.1 18.2 (recomputed)             17.9 17.8                         22.0 21.9                         22.9 23.6, 24.1 24.6
        //   2800                                                                             24.9 26.0                         28.0 29.0, 26.7 28.1
        // Four in place of three, 24 to 31 tiles: up to 400 workgroups 0 to 9 % less, at 650 to 720 from 4 % less to 5 % more (30 tiles
        // of bf16, 648: 14.9 15.8, 8.5 8.3, 22.0 23.3), beyond up to 6 % more: not taken.  Errors against 64 bits are smaller with finer
        // slices (rms of acceptance probabilities 5.6e-8 / 5.0e-8, of the four divergences 0.94 to 0.99 times what it is).
        ns = (8192 + rows - 1) / rows;
        long long most = g.ntiles / 8;
        if (fine && g.ntiles < 24) {
            const long long finer = g.ntiles >= 16 ? 4 : g.ntiles / 4;
            if (rows * finer <= 1250) most = finer;
        }
        if (ns > most) ns = most;
    }
    if (forced_ns > 0) ns = forced_ns;
    if (ns > MAX_SLICES) ns = MAX_SLICES;
    if (ns > g.ntiles) ns = g.ntiles;
    if (ns < 1) ns = 1;
    g.tps = (g.ntiles + (int)ns - 1) / (int)ns;
    // an odd number of tiles per slice staggers the slices' start addresses over the memory
    // channels; slices that start a power of two apart measured up to 15 % slower
    if (!want_one_batch && g.tps > 1 && (g.tps & 1) == 0 && !g_tune.even_tiles_per_slice) g.tps += 1;
    g.ns = (g.ntiles + g.tps - 1) / g.tps;
    return g;
}

static Scale make_scale(float temperature)
{
    Scale s;
    s.inv_T = 1.0 / (double)temperature;
    s.c = 1.4426950408889634 * s.inv_T;
    s.c_hi = (float)s.c;
    s.c_lo = (float)(s.c - (double)s.c_hi);
    s.c_dn = s.c_hi;
    while ((double)s.c_dn >= s.c) s.c_dn = nextafterf(s.c_dn, 0.f);      // strictly below c: the remainder is > 0
    s.c_up = (float)(s.c - (double)s.c_dn);
    return s;
}

// The highest logit whose product with the scale's c_dn is below fp32's range; -inf if there is none.
static float beyond_range(const Scale &s)
{
    if (!(s.c_dn > 1.f)) return -INFINITY;
    float m = (float)(-(double)FLT_MAX / (double)s.c_dn);
    while (!isinf(m * s.c_dn)) m = nextafterf(m, -INFINITY);
    return m;
}

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

static bool dtype_ok(int d) { return d == SVIP_F32 || d == SVIP_BF16 || d == SVIP_F16; }
static int vec_of(int d) { return d == SVIP_F32 ? 4 : 8; }       // logits per 16-byte vector

// Calls f with a value of the storage type that d names (f is a generic lambda).
template <typename F>
static void by_dtype(int d, F f)
{
    if (d == SVIP_BF16) f(bf16{});
    else if (d == SVIP_F16) f(f16{});
    else f(float{});
}

// Benchmark timing hook (svip_bench_time_kernels): caller-owned HIP events, attached pair by pair to
// the launches of one kernel class.
struct KernelTimer {
    void *const *start = nullptr, *const *stop = nullptr;
    int n = 0, used = 0;
};
static KernelTimer g_timer[SVIP_BENCH_KERNEL_CLASSES];

// One kernel launch on the stream; the launch's own status is returned (an error some earlier,
// unrelated HIP call left behind is neither consumed nor reported).  `cls` names the kernel class for
// the timing hook.
template <typename A>
static bool launch(void (*kernel)(A), unsigned grid, unsigned block, hipStream_t st, const A &args, int cls = -1)
{
    A copy = args;
    void *argv[] = {&copy};
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (cls >= 0 && g_timer[cls].used < g_timer[cls].n) {
        e0 = static_cast<hipEvent_t>(g_timer[cls].start[g_timer[cls].used]);
        e1 = static_cast<hipEvent_t>(g_timer[cls].stop[g_timer[cls].used]);
        ++g_timer[cls].used;
    }
    if (!e0)        // the plain launch is the one stream capture records
        return hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(grid), dim3(block), argv, 0, st) == hipSuccess;
    return hipExtLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(grid), dim3(block), argv, 0, st, e0, e1, 0) ==
           hipSuccess;
}

// Whether the sampling draft step keeps the masses of its records' chunks (see draft_kernels.h).
constexpr long long DRAFT_QUARTER_WAVES = 8100;
static bool quarter_records(int B, const Geo &g) { return g.tps == 1 && (long long)B * g.ns <= DRAFT_QUARTER_WAVES; }

// ---- workspace each call needs (its own geometry; svip_workspace_bytes bounds them all) -------

// flag word + ticket counters + slice masses of the residual pass (mass_slices per sequence)
static size_t ws_fixed_bytes(int B, int mass_slices)
{
    return HEADER_BYTES + ws_rec_bytes(B) + ws_mass_bytes(B, mass_slices) + ws_ticket_bytes(B);
}

static size_t need_draft(int B, const Geo &g, bool greedy)
{
    const size_t rec = !greedy && quarter_records(B, g) ? sizeof(QuarterRec) : sizeof(WaveRec);
    return ws_fixed_bytes(B, 0) + align256((size_t)B * g.ns * rec);
}
static size_t need_verify_greedy(int B, int k, const Geo &g)
{
    return ws_fixed_bytes(B, 0) + align256((size_t)B * (k + 1) * g.ns * sizeof(unsigned long long));
}
static size_t need_verify(int B, int k, bool recompute_lse, const Geo &g, const Geo &gs)
{
    const size_t stat_rows = (size_t)B * ((recompute_lse ? k : 0) + k + 1);
    return ws_fixed_bytes(B, gs.ns) + align256(stat_rows * g.ns * sizeof(Partial));
}
static size_t need_pair(int B, int k, bool recompute_lse, const Geo &g, const Geo &g2, size_t *part_bytes,
                        size_t *L_bytes)
{
    const size_t stat_rows = (size_t)B * ((recompute_lse ? k : 0) + k + 1), pos = (size_t)B * k;
    const size_t lb = align256(pos * 2 * sizeof(double));
    if (part_bytes) *part_bytes = align256(stat_rows * g.ns * sizeof(LsePart));      // (less than counted: the front ends earlier)
    if (L_bytes) *L_bytes = lb;
    return ws_fixed_bytes(B, 0) + align256(stat_rows * g.ns * sizeof(Partial)) + lb + align256(pos * g2.ns * 3 * sizeof(double));
}

// The slicing each pass uses (forced = an experiment's override, 0 = the library's choice).
// The draft step: one record (= one wave of the statistics launch) per tile of 32 logits per thread, so the
// search reads little again; up to 128 records per row (two per lane of the finish: 64 rows of 151936 bf16 logits, 75
// tiles, 10.7 us per step instead of 11.4 with 38 records of two tiles, 16 rows of 128256 fp32 logits 7.6 / 8.65).
// Rows of more tiles put more of them into a record, and so do batches that would otherwise launch more than 8100
// waves (eight per SIMD): about a quarter of a one-tile wave's instructions are per-record overhead, which then
// outweighs the finer grain and the shorter search (rows of 128256 logits, us per step with 63 and with 32 records: 64
// rows 9.6 / 10.1, 128 rows 12.6 / 12.75, 144 rows 13.8 / 13.9, 192 rows 16.3 / 15.4, 256 rows 19.5 / 18.6).
static Geo geo_draft(int B, int V, int vec, int forced)
{
    Geo g;
    g.V = V;
    const int nvec = (V + vec - 1) / vec;
    g.ntiles = (nvec + WG - 1) / WG;
    int ns = g.ntiles < MAX_SLICES ? g.ntiles : MAX_SLICES;
    if (g.ntiles > MAX_SLICES && g.ntiles <= 2 * MAX_SLICES && (long long)B * g.ntiles <= DRAFT_QUARTER_WAVES) ns = g.ntiles;
    if ((long long)B * ns > DRAFT_QUARTER_WAVES && ns == g.ntiles && ns > 1) ns = (ns + 1) / 2;
    if (forced > 0) ns = forced < MAX_SLICES ? forced : MAX_SLICES;
    if (ns > g.ntiles) ns = g.ntiles;
    if (ns < 1) ns = 1;
    g.tps = (g.ntiles + ns - 1) / ns;
    g.ns = (g.ntiles + g.tps - 1) / g.tps;
    return g;
}
static Geo geo_stats(long long stat_rows, int V, int vec, int forced, bool fine = false)
{
    return make_geo(V, vec, stat_rows, false, forced, 4, fine);
}
// A call needs a workspace for slices of at least 8 tiles.  It takes finer ones in every workspace of at least svip_workspace_bytes, and in
// no smaller one: its results are the same bits in all of the former, and in all of the latter.
static bool room_for_finer(size_t have, int B, int k, int V) { return (have & ~(size_t)255) >= svip_workspace_bytes(B, k, V); }
// The same for logsumexps, whose slices of a.geo are there already.  A logit of +inf or NaN has to cost a row the same tiles as before: a
// row of one slice all of them, and two slices are halved.  Returns how many slices stand for one (see RowStats).
static int finer_stats(VerifyArgs &a, long long stat_rows, int vec, int forced, bool fine)
{
    const Geo g = geo_stats(stat_rows, a.geo.V, vec, forced, fine);
    a.first_half = 0;
    if (g.ns <= a.geo.ns) return 1;
    if (a.geo.ns == 1) {
        a.geo = g;
        return 4;
    }
    a.first_half = (a.geo.tps + 1) / 2;
    a.geo.ns *= 2;
    return 2;
}
// f with that number as a constant.
template <typename F>
static bool by_parts(int parts, F f)
{
    if (parts == 4) return f(std::integral_constant<int, 4>{});
    if (parts == 2) return f(std::integral_constant<int, 2>{});
    return f(std::integral_constant<int, 1>{});
}
// the residual pass: slices of four tiles like the draft step (at 64 sequences of 128K logits, 16 slices of
// 4 tiles take 13 us, 32 slices of 2 tiles 16 us, 8 slices 20 us, one tile per slice 26 us)
static Geo geo_resid(int B, int V, int vec, int forced) { return make_geo(V, vec, B, true, forced, 4); }

// ---- the calls behind the entry points ---------------------------------------------------------

static bool workspace_ok(const void *ws, size_t have, size_t need)
{
    return ws && (reinterpret_cast<uintptr_t>(ws) & 255u) == 0 && (have & ~(size_t)255) >= need;
}

static svip_status check_draft(const DraftCall &c)
{
    if (!c.logits || (!c.greedy && !c.u_sample) || !c.token_out || !c.lse_out || !c.stop_out) return SVIP_ERR_NULL;
    if (c.pos && !c.cap) return SVIP_ERR_NULL;
    if (!dtype_ok(c.dtype)) return SVIP_ERR_DTYPE;
    if (c.B <= 0 || c.B > MAX_BATCH || c.V <= 0 || c.k_max < 1 || c.k_max > SVIP_MAX_K || c.step_j < 0 ||
        c.step_j >= c.k_max || c.io_stride < 1 || c.row_stride < c.V || (c.pos && c.pos_stride < c.V))
        return SVIP_ERR_SHAPE;
    const int vec = vec_of(c.dtype);
    if (!aligned16(c.logits) || c.row_stride % vec != 0 || (c.pos && c.pos_stride % vec != 0)) return SVIP_ERR_ALIGN;
    if (!(c.temperature > 0.f) || !isfinite(c.temperature) || !(c.h >= 0.f)) return SVIP_ERR_PARAM;
    return SVIP_OK;
}

// floor(n / d) = umulhi(n, magic_of(d)) for d > 1 while n * d < 2^32
static unsigned magic_of(unsigned d) { return d > 1u ? (unsigned)(0x100000000ull / d) + 1u : 0u; }

// The arguments of the draft kernels but for the launch's shape.
static DraftArgs draft_args(const DraftCall &c, const Geo &geo, void *records)
{
    DraftArgs a;
    a.geo = geo;
    a.logits = c.logits;
    a.row_stride = c.row_stride;
    a.pos = c.pos;
    a.pos_stride = c.pos_stride;
    a.cap = c.cap;
    a.B = c.B;
    a.sc = make_scale(c.temperature);
    a.common_range = a.sc.c < 1e30;           // both parts of the constant are finite
    a.h = c.h;
    a.step_j = c.step_j;
    a.k_max = c.k_max;
    a.u = c.u_sample;
    a.stop_in = c.stop_in;
    a.token = c.token_out;
    a.entropy = c.entropy_out;
    a.q_tok = c.q_tok_out;
    a.lse = c.lse_out;
    a.stop = c.stop_out;
    a.draft_len = c.draft_len_out;
    a.io_stride = c.io_stride;
    a.part = records;
    a.tickets = nullptr;
    return a;
}

// Whether a step is one launch (k_draft_step) or two.  One saves a launch (1.8 us in a graph, 2.5 us of the caller's time) and
// pays with an exchange through memory, which takes longer the more rows are at it: their records are stored past the L2 and
// fetched from behind it, sampling twice as many words as greedy, by two waves.  us per step in a graph, two launches / one:
//   sampling, 16-bit  1 row of 128256 5.88 / 5.79, 8 6.56 / 6.17, 32 (512 workgroups) 8.13 / 7.53, 48 (768) 8.88 / 8.38, 64 (1024)
//                     9.70 / 9.31, 80 (1280) 10.53 / 10.39, 88 (1408) 10.91 / 11.10, 104 (1664) 11.68 / 12.11; 192 of 32000 (768) 8.92 / 8.41,
//                     256 (1024) 9.72 / 9.44, 320 (1280) 10.58 / 10.43; 768 of 2000 8.15 / 7.03, 1536 10.13 / 8.56, 2048 10.30 / 10.87
//     over 64 records 16 rows of 151936 (304) 7.92 / 7.48, 32 (608) 8.98 / 9.07, 56 10.43 / 11.21
//   sampling, fp32    1 row of 32000 4.83 / 4.60, 16 6.15 / 5.89, 64 (512) 7.26 / 7.00, 88 (704) 7.74 / 7.54, 96 (768) 7.88 / 7.77,
//                     112 (896) 8.43 / 8.37, 128 (1024) 8.50 / 8.64; 48 of 65536 (768) 7.93 / 8.03, 64 (1024) 8.62 / 8.86
//     over 64 records 8 rows of 128256 (256) 6.73 / 7.39
//   greedy            1 row of 32000 fp32 4.50 / 4.38, 8 of 128256 bf16 6.05 / 5.49, 64 (1024) 8.98 / 8.40, 112 (1792) 11.02 / 10.98;
//                     32 of 128256 fp32 (1024) 8.08 / 8.03, 40 8.65 / 8.93, 56 of 151936 bf16 (1064) 9.41 / 9.14, 4096 of 2000 11.6 / 12.9
// Sampling has one line for all types, where fp32 rows cross over.  16-bit rows would gain 1 to 4 % more on a line of their own at 1280
// workgroups.  A forced shape (an experiment's override) takes two, and so does a workspace of less than svip_workspace_bytes: two
// launches need no counters, and in one that only holds what some call needs, calls of other sizes may have overwritten them.  So does the
// fixed scratch: calls that overlap there leave nothing behind that a later call would read, and nothing could clear it.
static unsigned row_workgroups(const Geo &g) { return ((unsigned)g.ns + NWAVE - 1) / NWAVE; }
static bool one_launch_step(const DraftCall &c, const Geo &g)
{
    if (g.tps != 1 || g_tune.draft_slices) return false;
    if (!c.counters || (c.workspace_bytes & ~(size_t)255) < svip_workspace_bytes(c.B, c.k_max, c.V)) return false;
    const long long workgroups = ((long long)c.B + 7) / 8 * 8 * row_workgroups(g);
    if (c.greedy) return workgroups <= 1024;
    if (!quarter_records(c.B, g)) return false;
    if (g.ns > 64) return vec_of(c.dtype) == 8 && workgroups <= 512;
    return workgroups <= 768;
}

// The shape of the statistics launch over `rows` rows; returns its workgroups.
static unsigned shape_draft_stats(DraftArgs &a, unsigned rows)
{
    const unsigned waves = (unsigned)a.geo.ns * rows;
    // Rows pinned to XCDs (see k_draft_stats) while the launch has at most 8100 waves: measured, rows of 128K bf16
    // logits, us per step without / with: 16 rows 8.15 / 8.07, 32 rows 9.2 / 8.9, 64 rows 11.2 / 10.8, 72 rows
    // (4536 one-tile waves) 11.5 / 10.85, 88 rows 12.3 / 11.5, 192 rows (6144 two-tile waves) 16.8 / 16.4; 64 and
    // 256 rows of 32000 logits 8.4 / 8.0 and 13.0 / 12.6; but 256 rows of 128K (8192 two-tile waves) 20.65 / 20.8.
    // Rows of fewer than four records would leave most of a workgroup's waves without one.
    a.rows_by_xcd = waves <= 8100u && a.geo.ns >= NWAVE;
    const unsigned grid = a.rows_by_xcd ? ((rows + 7u) / 8u) * 8u * (((unsigned)a.geo.ns + NWAVE - 1) / NWAVE)
                                        : (waves + NWAVE - 1) / NWAVE;
    // the kernel's division: n < 2^26 waves with d <= 64, or n <= 8100 with d <= 128 (grouped positions: n < 2^18, d <= 192)
    a.div = a.rows_by_xcd ? ((unsigned)a.geo.ns + NWAVE - 1) / NWAVE : (unsigned)a.geo.ns;
    a.div_magic = magic_of(a.div);
    return grid;
}

svip_status draft_step_call(const DraftCall &c)
{
    const svip_status s = check_draft(c);
    if (s != SVIP_OK) return s;
    const Geo geo = geo_draft(c.B, c.V, vec_of(c.dtype), g_tune.draft_slices);
    if (!workspace_ok(c.workspace, c.workspace_bytes, need_draft(c.B, geo, c.greedy))) return SVIP_ERR_WORKSPACE;
    const unsigned rows = (unsigned)c.B;
    const Workspace w = carve(c.workspace, c.workspace_bytes, c.B, 0);
    DraftArgs a = draft_args(c, geo, w.part);
    hipStream_t st = static_cast<hipStream_t>(c.stream);
    bool ok = false;
    if (one_launch_step(c, geo)) {
        a.tickets = w.tickets;
        a.div = row_workgroups(geo);
        a.div_magic = magic_of(a.div);
        by_dtype(c.dtype, [&](auto tag) {
            using DT = decltype(tag);
            const auto kernel = c.greedy ? (geo.ns <= 64 ? k_draft_step<DT, GREEDY, 1> : k_draft_step<DT, GREEDY, 2>)
                                         : (geo.ns <= 64 ? k_draft_step<DT, QUARTERS, 1> : k_draft_step<DT, QUARTERS, 2>);
            ok = launch(kernel, (rows + 7u) / 8u * 8u * a.div, WG, st, a, SVIP_BENCH_K_DRAFT_STATS);
        });
        return ok ? SVIP_OK : SVIP_ERR_HIP;
    }
    const unsigned grid = shape_draft_stats(a, rows);
    by_dtype(c.dtype, [&](auto tag) {
        using DT = decltype(tag);
        const int tps = a.geo.tps;
        const auto stats = [&](auto kind) {
            constexpr RecordKind K = decltype(kind)::value;
            return launch(tps == 1 ? k_draft_stats<DT, K, 1> : (tps == 2 ? k_draft_stats<DT, K, 2> : k_draft_stats<DT, K, 0>), grid,
                          WG, st, a, SVIP_BENCH_K_DRAFT_STATS);
        };
        if (c.greedy)
            ok = stats(std::integral_constant<RecordKind, GREEDY>{}) &&
                 launch(a.geo.ns <= 64 ? k_draft_finish_greedy<1> : k_draft_finish_greedy<2>, rows, 64, st, a, SVIP_BENCH_K_DRAFT_FINISH);
        else if (quarter_records(c.B, a.geo))
            ok = launch(k_draft_stats<DT, QUARTERS, 1>, grid, WG, st, a, SVIP_BENCH_K_DRAFT_STATS) &&
                 launch(a.geo.ns <= 64 ? k_draft_finish_quarters<DT, 1> : k_draft_finish_quarters<DT, 2>, rows, QUARTER_FINISH_THREADS,
                        st, a, SVIP_BENCH_K_DRAFT_FINISH);
        else
            ok = stats(std::integral_constant<RecordKind, TOTAL>{}) &&
                 launch(k_draft_finish_total<DT>, rows, TOTAL_FINISH_THREADS, st, a, SVIP_BENCH_K_DRAFT_FINISH);
    });
    return ok ? SVIP_OK : SVIP_ERR_HIP;
}

// Grouped positions: records of one tile, at most three per lane of the finish, for every position of a launch.  Rows per
// position are rounded up to whole rounds of the XCDs where there are that many, so that a row's records are on XCD b % 8,
// where the workgroup of its sequence reads them.
static Geo geo_group(int V, int vec)
{
    Geo g;
    g.V = V;
    g.ntiles = ((V + vec - 1) / vec + WG - 1) / WG;
    g.ns = g.ntiles;
    g.tps = 1;
    return g;
}
constexpr int GROUP_MAX_RECORDS = 3 * 64;
static int group_lane_rows(int B) { return B < 8 ? B : (B + 7) / 8 * 8; }

int group_waves(int B, int V, int dtype)
{
    const Geo g = geo_group(V, vec_of(dtype));
    return g.ns <= GROUP_MAX_RECORDS && B <= (1 << 16) ? B * g.ns : 0;
}
bool draft_shape_forced() { return g_tune.draft_slices != 0; }
static size_t group_record_bytes(int B, const Geo &g, int group, bool greedy)
{
    return align256((size_t)group_lane_rows(B) * group * g.ns * (greedy ? sizeof(WaveRec) : sizeof(QuarterRec)));
}
size_t group_bytes(int B, int V, int dtype, int group, bool greedy)
{
    const Geo g = geo_group(V, vec_of(dtype));
    return group_record_bytes(B, g, group, greedy) +
           (greedy ? align256((size_t)group_lane_rows(B) * (group + 1) * g.ns * sizeof(unsigned long long)) : 0);
}

static svip_status group_args(const DraftCall &c, int group, void *buffer, size_t bytes, GroupArgs *a)
{
    const svip_status s = check_draft(c);
    if (s != SVIP_OK) return s;
    if (!c.pos || !c.cap || !c.stop_in || !c.draft_len_out) return SVIP_ERR_NULL;
    if (group_waves(c.B, c.V, c.dtype) == 0 || group < 1 || group > (c.greedy ? STREAM_MAX_GROUP : c.k_max)) return SVIP_ERR_SHAPE;
    if (bytes < group_bytes(c.B, c.V, c.dtype, group, c.greedy)) return SVIP_ERR_WORKSPACE;
    a->d = draft_args(c, geo_group(c.V, vec_of(c.dtype)), buffer);
    a->group = group;
    a->lane_rows = group_lane_rows(c.B);
    a->lane_magic = magic_of((unsigned)a->lane_rows);
    return SVIP_OK;
}
// A kernel's instance for one, two or three records per lane.
template <typename K>
static K by_records(int ns, K k1, K k2, K k3) { return ns <= 64 ? k1 : (ns <= 128 ? k2 : k3); }

svip_status draft_group_call(const DraftCall &c, int group, void *buffer, size_t bytes)
{
    GroupArgs a;
    const svip_status s = group_args(c, group, buffer, bytes, &a);
    if (s != SVIP_OK) return s;
    if (c.greedy || c.step_j + group > c.k_max) return SVIP_ERR_SHAPE;
    const unsigned grid = shape_draft_stats(a.d, (unsigned)(a.lane_rows * group));
    const unsigned threads = 64u * (unsigned)(group < GROUP_FINISH_WAVES ? group : GROUP_FINISH_WAVES);
    hipStream_t st = static_cast<hipStream_t>(c.stream);
    bool ok = false;
    by_dtype(c.dtype, [&](auto tag) {
        using DT = decltype(tag);
        ok = launch(k_group_stats<DT>, grid, WG, st, a, SVIP_BENCH_K_DRAFT_STATS) &&
             launch(by_records(a.d.geo.ns, k_group_finish<DT, 1>, k_group_finish<DT, 2>, k_group_finish<DT, 3>), (unsigned)c.B, threads,
                    st, a, SVIP_BENCH_K_DRAFT_FINISH);
    });
    return ok ? SVIP_OK : SVIP_ERR_HIP;
}

svip_status greedy_stream_call(const DraftCall &c, const void *target, int group, int ahead, const LoopArgs &l, int last_round,
                               Mail active, Mail running, Mail rounds)
{
    GroupArgs a;
    const svip_status s = group_args(c, group, l.rb.group, l.rb.group_bytes, &a);
    if (s != SVIP_OK) return s;
    if (!c.greedy || ahead < 1 || !target) return SVIP_ERR_SHAPE;
    if (!aligned16(target)) return SVIP_ERR_ALIGN;
    a.target = target;
    a.keys = reinterpret_cast<unsigned long long *>(l.rb.group + group_record_bytes(c.B, a.d.geo, group, true));
    a.flags = static_cast<unsigned *>(c.workspace);
    a.ahead = ahead;
    a.last_round = last_round;
    a.active = active;
    a.running = running;
    a.rounds = rounds;
    a.l = l;
    const int per_seq = 2 * group + 1;
    const unsigned grid = shape_draft_stats(a.d, (unsigned)(a.lane_rows * per_seq));
    const unsigned threads = 64u * (unsigned)(per_seq < GROUP_FINISH_WAVES ? per_seq : GROUP_FINISH_WAVES);
    hipStream_t st = static_cast<hipStream_t>(c.stream);
    bool ok = false;
    by_dtype(c.dtype, [&](auto tag) { ok = launch(k_stream_rows<decltype(tag)>, grid, WG, st, a, SVIP_BENCH_K_DRAFT_STATS); });
    ok = ok && launch(by_records(a.d.geo.ns, k_stream_advance<1>, k_stream_advance<2>, k_stream_advance<3>), (unsigned)c.B, threads, st, a,
                      SVIP_BENCH_K_DRAFT_FINISH);
    return ok ? SVIP_OK : SVIP_ERR_HIP;
}

// Device address of `scratch` on the current device, or nullptr.  The first call on a device looks the
// symbol up (hipGetSymbolAddress with that device current); every GPU holds its own copy of the array at
// its own address.  Nothing in it has to start at zero: a draft step in two launches writes every record before it reads it.
static void *static_scratch()
{
    constexpr int MAX_DEVICES = 64;
    static void *ptr[MAX_DEVICES] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
    if (!ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        ptr[dev] = p;
    }
    return ptr[dev];
}

static svip_status verify_greedy_call(const VerifyCall &c)
{
    if (!c.target || !c.draft_tokens || !c.draft_len || !c.n_accepted_out || !c.next_token_out) return SVIP_ERR_NULL;
    if (!dtype_ok(c.dtype)) return SVIP_ERR_DTYPE;
    if (c.B <= 0 || c.B > MAX_BATCH || c.V <= 0 || c.k_max < 1 || c.k_max > SVIP_MAX_K || c.row_stride < c.V ||
        c.seq_stride_t < (long long)c.k_max * c.row_stride + c.V)
        return SVIP_ERR_SHAPE;
    const long long rows = (long long)c.B * (c.k_max + 1);
    if (rows * MAX_SLICES > 0x7FFFFFFFLL) return SVIP_ERR_SHAPE;
    const int vec = vec_of(c.dtype);
    if (!aligned16(c.target) || c.row_stride % vec != 0 || c.seq_stride_t % vec != 0) return SVIP_ERR_ALIGN;
    GreedyArgs a;
    a.geo = geo_stats(rows, c.V, vec, g_tune.stats_slices);
    if (!workspace_ok(c.workspace, c.workspace_bytes, need_verify_greedy(c.B, c.k_max, a.geo))) return SVIP_ERR_WORKSPACE;
    a.geo = geo_stats(rows, c.V, vec, g_tune.stats_slices, room_for_finer(c.workspace_bytes, c.B, c.k_max, c.V));
    const Workspace w = carve(c.workspace, c.workspace_bytes, c.B, 0);
    a.target = c.target;
    a.seq_t = c.seq_stride_t;
    a.row_stride = c.row_stride;
    a.pos = c.pos;
    a.B = c.B;
    a.k = c.k_max;
    a.tokens = c.draft_tokens;
    a.draft_len = c.draft_len;
    a.n_accepted = c.n_accepted_out;
    a.next_token = c.next_token_out;
    a.skip = c.skip;
    a.keys = static_cast<unsigned long long *>(w.part);
    a.flags = w.flags;
    hipStream_t st = static_cast<hipStream_t>(c.stream);
    bool ok = false;
    by_dtype(c.dtype, [&](auto tag) {
        ok = launch(k_argmax<decltype(tag)>, (unsigned)(rows * a.geo.ns), WG, st, a, SVIP_BENCH_K_VERIFY_STATS);
    });
    ok = ok && launch(k_accept_greedy, (unsigned)c.B, 64, st, a, SVIP_BENCH_K_ACCEPT);
    return ok ? SVIP_OK : SVIP_ERR_HIP;
}

// Whether the acceptance test runs inside the residual pass, where every workgroup of a sequence repeats it, or in a launch of its
// own.
//   - Drafts of more positions than a wave has lanes have their own launch: the passes are a serial chain, those behind the first
//     rejection are needed only once, and what they read may lie under next_token_out.
//   - 1536 workgroups of the residual pass are resident at a time (1280 and fewer of the form for slices of more than TILE_MASSES
//     tiles); those behind them wait for the test's chain of loads once more, and the more slices a sequence has the more often
//     the test is repeated.  us per call of 4 positions, in the pass / own launch:
//       workgroups   128256 bf16, 16 slices   50257 fp16, 7   32000 fp32, 8   32000 bf16, 4   8000 bf16, 1
//         1024           29.8 / 31.1                                           31.6 / 32.9     31.6 / 33.9
//         1536           36.0 / 37.9           36.5 / 38.6     34.6 / 36.2     38.3 / 41.8     39.8 / 44.3
//        ~1670           39.7 / 39.8           39.6 / 39.2     38.1 / 37.9     42.9 / 43.4
//        ~2048           44.8 / 44.6           45.4 / 44.7     42.2 / 42.4     48.7 / 48.9     50.8 / 52.3
//         2560           51.2 / 50.1                           49.4 / 49.5                     59.8 / 61.0
//         4096           73.7 / 70.3                                                           86.9 / 87.5
//       (with draft logsumexps recomputed the second number is 1 to 4 % better from 1670 on: 16 slices, 2048: 58.7 / 57.3).
//       Longer slices, 1024 workgroups: 28672 bf16 48.8 / 50.6, 14336 fp32 43.2 / 45.2; 1280: 59.1 / 57.9, 49.9 / 51.8;
//       1536: 67.1 / 65.5, 58.9 / 58.6; 4608: 128256 bf16 144.6 / 135.2.
static bool accept_in_resid(int k_max, const Geo &slices, unsigned workgroups)
{
    const unsigned most = slices.tps > TILE_MASSES ? 1024u : (slices.ns > 4 ? 1536u : 2560u);
    return k_max <= LANE_POSITIONS && workgroups <= most;
}

svip_status verify_call(const VerifyCall &c)
{
    if (c.greedy) return verify_greedy_call(c);
    if (!c.target || !c.draft || !c.draft_tokens || !c.draft_len || !c.u_accept || !c.u_resample ||
        !c.n_accepted_out || !c.next_token_out)
        return SVIP_ERR_NULL;
    if (!dtype_ok(c.dtype)) return SVIP_ERR_DTYPE;
    if (c.B <= 0 || c.B > MAX_BATCH || c.V <= 0 || c.k_max < 1 || c.k_max > SVIP_MAX_K || c.row_stride < c.V ||
        c.seq_stride_t < (long long)c.k_max * c.row_stride + c.V ||
        c.seq_stride_d < (long long)(c.k_max - 1) * c.row_stride + c.V)
        return SVIP_ERR_SHAPE;
    const int kd = c.draft_lse ? 0 : c.k_max;
    const long long stat_rows = (long long)c.B * (kd + c.k_max + 1);
    if (stat_rows * MAX_SLICES > 0x7FFFFFFFLL) return SVIP_ERR_SHAPE;          // workgroups of the statistics pass
    const int vec = vec_of(c.dtype);
    if (!aligned16(c.target) || !aligned16(c.draft) || c.row_stride % vec != 0 || c.seq_stride_t % vec != 0 ||
        c.seq_stride_d % vec != 0)
        return SVIP_ERR_ALIGN;
    if (!(c.temperature > 0.f) || !isfinite(c.temperature)) return SVIP_ERR_PARAM;

    VerifyArgs a;
    a.geo = geo_stats(stat_rows, c.V, vec, g_tune.stats_slices);
    a.geo_s = geo_resid(c.B, c.V, vec, g_tune.resid_slices);
    if (!workspace_ok(c.workspace, c.workspace_bytes, need_verify(c.B, c.k_max, kd != 0, a.geo, a.geo_s)))
        return SVIP_ERR_WORKSPACE;
    // (rows this short have short slices in the residual pass too, unless an experiment forces others)
    const int parts = finer_stats(a, stat_rows, vec, g_tune.stats_slices,
                                  a.geo_s.tps <= TILE_MASSES && room_for_finer(c.workspace_bytes, c.B, c.k_max, c.V));
    a.target = c.target;
    a.draft = c.draft;
    a.seq_t = c.seq_stride_t;
    a.seq_d = c.seq_stride_d;
    a.row_stride = c.row_stride;
    a.pos = c.pos;
    a.skip = c.skip;
    a.B = c.B;
    a.k = c.k_max;
    a.kd = kd;
    a.bonus = 1;
    a.sc = make_scale(c.temperature);
    a.m0 = beyond_range(a.sc);
    a.tokens = c.draft_tokens;
    a.draft_len = c.draft_len;
    a.draft_lse = c.draft_lse;
    a.u_accept = c.u_accept;
    a.u_resample = c.u_resample;
    a.n_accepted = c.n_accepted_out;
    a.next_token = c.next_token_out;
    a.accept_prob = c.accept_prob_out;
    a.ws = carve(c.workspace, c.workspace_bytes, c.B, a.geo_s.ns);
    hipStream_t st = static_cast<hipStream_t>(c.stream);
    a.stat_items = stat_rows * a.geo.ns;
    unsigned g_stats = (unsigned)a.stat_items;
    if (g_tune.stats_workgroups > 0 && (unsigned)g_tune.stats_workgroups < g_stats) g_stats = (unsigned)g_tune.stats_workgroups;
    const unsigned g_resid = (unsigned)a.geo_s.ns * (((unsigned)c.B + 7u) / 8u) * 8u;   // sequences by XCD, see k_resid
    const bool test = accept_in_resid(c.k_max, a.geo_s, g_resid);
    bool ok = false;
    by_dtype(c.dtype, [&](auto tag) {
        using DT = decltype(tag);
        ok = launch(k_verify_stats<DT>, g_stats, WG, st, a, SVIP_BENCH_K_VERIFY_STATS) && by_parts(parts, [&](auto of) {
                 constexpr int P = decltype(of)::value;
                 return (test || launch(k_accept<DT, P>, (unsigned)c.B, 64, st, a, SVIP_BENCH_K_ACCEPT)) &&
                        launch(a.geo_s.tps <= TILE_MASSES ? (test ? k_resid<DT, true, true, P> : k_resid<DT, true, false, 1>)
                                                          : (test ? k_resid<DT, false, true, 1> : k_resid<DT, false, false, 1>),
                               g_resid, WG, st, a, SVIP_BENCH_K_RESID);
             });
    });
    return ok ? SVIP_OK : SVIP_ERR_HIP;
}

}  // namespace svip

using namespace svip;

extern "C" {

const char *svip_status_string(int status)
{
    switch (status) {
        case SVIP_OK: return "SVIP_OK";
        case SVIP_ERR_NULL: return "SVIP_ERR_NULL: a required pointer is NULL";
        case SVIP_ERR_SHAPE: return "SVIP_ERR_SHAPE: size, position or stride out of range";
        case SVIP_ERR_DTYPE: return "SVIP_ERR_DTYPE: unknown logits dtype";
        case SVIP_ERR_ALIGN: return "SVIP_ERR_ALIGN: pointer or stride not 16-byte aligned";
        case SVIP_ERR_WORKSPACE: return "SVIP_ERR_WORKSPACE: workspace missing, misaligned or too small";
        case SVIP_ERR_PARAM: return "SVIP_ERR_PARAM: temperature, threshold or constant out of range";
        case SVIP_ERR_HIP: return "SVIP_ERR_HIP: HIP runtime error";
        default: return "SVIP: unknown status";
    }
}

size_t svip_workspace_bytes(int B, int k_max, int V)
{
    if (B <= 0 || B > MAX_BATCH || k_max < 1 || k_max > SVIP_MAX_K || V <= 0) return 0;
    // slice statistics: the draft step slices its B rows finely (at most MAX_SLICES each); the
    // streaming passes (statistics of verify, argmax, diagnostics) have up to B (2 k + 1) rows, of
    // which make_geo cuts at most ceil(8192 / rows) slices each: rows + 8192 slices at most
    const size_t vrows = (size_t)B * (2 * (size_t)k_max + 1);
    // a row has at most `tiles` slices (fp32 rows have the most vectors)
    const size_t tiles = ((size_t)V + 4 * WG - 1) / (4 * WG);
    const size_t ns_max = tiles < MAX_SLICES ? tiles : MAX_SLICES;
    size_t part_bytes = (size_t)B * ns_max * sizeof(WaveRec);
    const size_t q_recs = (size_t)B * (tiles < 2 * MAX_SLICES ? tiles : 2 * MAX_SLICES);      // draft records with chunk masses
    const size_t q_bytes = (q_recs < DRAFT_QUARTER_WAVES ? q_recs : DRAFT_QUARTER_WAVES) * sizeof(QuarterRec);
    if (q_bytes > part_bytes) part_bytes = q_bytes;
    if ((vrows + 8192) * sizeof(Partial) > part_bytes) part_bytes = (vrows + 8192) * sizeof(Partial);
    // diagnostics: two logsumexps per position and three sums per slice of its second pass
    const size_t pos = (size_t)B * (size_t)k_max;
    return ws_fixed_bytes(B, (int)ns_max) + align256(part_bytes) + align256(pos * 2 * sizeof(double)) +
           align256((pos + 8192) * 3 * sizeof(double));
}

size_t svip_workspace_needed(int call, int dtype, int B, int k_max, int V)
{
    if (!dtype_ok(dtype) || B <= 0 || B > MAX_BATCH || k_max < 1 || k_max > SVIP_MAX_K || V <= 0) return 0;
    const int vec = vec_of(dtype);
    const long long rows_t = (long long)B * (k_max + 1), rows_all = (long long)B * (2 * k_max + 1);
    switch (call) {
        case SVIP_CALL_DRAFT_STEP: return need_draft(B, geo_draft(B, V, vec, 0), false);      // greedy records are no larger
        case SVIP_CALL_VERIFY: return need_verify(B, k_max, false, geo_stats(rows_t, V, vec, 0), geo_resid(B, V, vec, 0));
        case SVIP_CALL_VERIFY_RECOMPUTE:
            return need_verify(B, k_max, true, geo_stats(rows_all, V, vec, 0), geo_resid(B, V, vec, 0));
        case SVIP_CALL_VERIFY_GREEDY: return need_verify_greedy(B, k_max, geo_stats(rows_t, V, vec, 0));
        case SVIP_CALL_PAIR_STATS:
            return need_pair(B, k_max, false, geo_stats(rows_t, V, vec, 0), geo_stats((long long)B * k_max, V, vec, 0),
                             nullptr, nullptr);
        case SVIP_CALL_PAIR_STATS_RECOMPUTE:
            return need_pair(B, k_max, true, geo_stats(rows_all, V, vec, 0), geo_stats((long long)B * k_max, V, vec, 0),
                             nullptr, nullptr);
        default: return 0;
    }
}

svip_status svip_workspace_reset(void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!workspace || workspace_bytes < 2 * HEADER_BYTES || (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return SVIP_ERR_WORKSPACE;
    // the flag word, and the ticket counters at the end of the workspace (for any batch size up to MAX_BATCH
    // that this workspace may later be used with): a fill kernel, so that the call can be captured in a graph
    const size_t end = workspace_bytes & ~(size_t)255;
    size_t tail = ws_ticket_bytes(MAX_BATCH);
    if (tail > end - HEADER_BYTES) tail = end - HEADER_BYTES;
    ZeroArgs z;
    z.flags = static_cast<unsigned *>(workspace);
    z.tail = reinterpret_cast<uint4 *>(static_cast<char *>(workspace) + end - tail);
    z.n16 = tail / 16;
    const unsigned grid = (unsigned)((z.n16 + 255) / 256 < 1024 ? (z.n16 + 255) / 256 : 1024);
    return launch(k_zero, grid ? grid : 1u, 256, static_cast<hipStream_t>(hip_stream), z) ? SVIP_OK : SVIP_ERR_HIP;
}

svip_status svip_workspace_flags(const void *workspace, void *hip_stream, unsigned *flags_host)
{
    if (!workspace) return SVIP_ERR_WORKSPACE;
    if (!flags_host) return SVIP_ERR_NULL;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (hipMemcpyAsync(flags_host, workspace, sizeof(unsigned), hipMemcpyDeviceToHost, st) != hipSuccess)
        return SVIP_ERR_HIP;
    return hipStreamSynchronize(st) == hipSuccess ? SVIP_OK : SVIP_ERR_HIP;
}

svip_status svip_draft_step(const void *draft_logits, int dtype, int B, int V, long long row_stride,
                            float temperature, float h, int step_j, int k_max, const float *u_sample,
                            const unsigned char *stop_in, int *token_out, float *entropy_out,
                            float *q_tok_out, double *lse_out, unsigned char *stop_out,
                            int *draft_len_out, long long io_stride, void *workspace,
                            size_t workspace_bytes, void *hip_stream)
{
    const DraftCall c{false, draft_logits, dtype, B, V, row_stride, nullptr, 0, nullptr, temperature, h, step_j,
                      k_max, u_sample, stop_in, token_out, entropy_out, q_tok_out, lse_out, stop_out,
                      draft_len_out, io_stride, workspace, workspace_bytes, hip_stream, true};
    return draft_step_call(c);
}

svip_status svip_draft_step_static(const void *draft_logits, int dtype, int B, int V, long long row_stride,
                                   float temperature, float h, int step_j, int k_max, const float *u_sample,
                                   const unsigned char *stop_in, int *token_out, float *entropy_out,
                                   float *q_tok_out, double *lse_out, unsigned char *stop_out,
                                   int *draft_len_out, long long io_stride, void *hip_stream)
{
    // sizes first: a batch whose slice records do not fit the fixed scratch is refused before anything else
    if (!dtype_ok(dtype)) return SVIP_ERR_DTYPE;
    if (B <= 0 || B > MAX_BATCH || V <= 0) return SVIP_ERR_SHAPE;
    if (need_draft(B, geo_draft(B, V, vec_of(dtype), g_tune.draft_slices), false) > (size_t)SVIP_STATIC_SCRATCH_BYTES)
        return SVIP_ERR_WORKSPACE;
    void *ws = static_scratch();
    if (!ws) return SVIP_ERR_HIP;
    const DraftCall c{false, draft_logits, dtype, B, V, row_stride, nullptr, 0, nullptr, temperature, h, step_j,
                      k_max, u_sample, stop_in, token_out, entropy_out, q_tok_out, lse_out, stop_out,
                      draft_len_out, io_stride, ws, (size_t)SVIP_STATIC_SCRATCH_BYTES, hip_stream, false};
    return draft_step_call(c);
}

svip_status svip_draft_step_greedy(const void *draft_logits, int dtype, int B, int V, long long row_stride,
                                   float temperature, float h, int step_j, int k_max,
                                   const unsigned char *stop_in, int *token_out, float *entropy_out,
                                   float *q_tok_out, double *lse_out, unsigned char *stop_out,
                                   int *draft_len_out, long long io_stride, void *workspace,
                                   size_t workspace_bytes, void *hip_stream)
{
    const DraftCall c{true, draft_logits, dtype, B, V, row_stride, nullptr, 0, nullptr, temperature, h, step_j,
                      k_max, nullptr, stop_in, token_out, entropy_out, q_tok_out, lse_out, stop_out,
                      draft_len_out, io_stride, workspace, workspace_bytes, hip_stream, true};
    return draft_step_call(c);
}

svip_status svip_verify_greedy(const void *target_logits, int dtype, int B, int k_max, int V,
                               long long seq_stride_t, long long row_stride, const int *draft_tokens,
                               const int *draft_len, int *n_accepted_out, int *next_token_out,
                               void *workspace, size_t workspace_bytes, void *hip_stream)
{
    const VerifyCall c{true, target_logits, nullptr, dtype, B, k_max, V, seq_stride_t, 0, row_stride, nullptr, nullptr, 1.f,
                       draft_tokens, draft_len, nullptr, nullptr, nullptr, n_accepted_out, next_token_out,
                       nullptr, workspace, workspace_bytes, hip_stream};
    return verify_call(c);
}

svip_status svip_verify(const void *target_logits, const void *draft_logits, int dtype, int B,
                        int k_max, int V, long long seq_stride_t, long long seq_stride_d,
                        long long row_stride, float temperature, const int *draft_tokens,
                        const int *draft_len, const double *draft_lse, const float *u_accept,
                        const float *u_resample, int *n_accepted_out, int *next_token_out,
                        float *accept_prob_out, void *workspace, size_t workspace_bytes,
                        void *hip_stream)
{
    const VerifyCall c{false, target_logits, draft_logits, dtype, B, k_max, V, seq_stride_t, seq_stride_d,
                       row_stride, nullptr, nullptr, temperature, draft_tokens, draft_len, draft_lse, u_accept,
                       u_resample, n_accepted_out, next_token_out, accept_prob_out, workspace,
                       workspace_bytes, hip_stream};
    return verify_call(c);
}

svip_status svip_warp_logits(const void *logits_in, void *logits_out, int dtype, int B, int k_max, int V,
                             long long seq_stride, long long row_stride, float temperature, int top_k,
                             double top_p, int *kept_out, void *hip_stream)
{
    if (!logits_in || !logits_out) return SVIP_ERR_NULL;
    if (!dtype_ok(dtype)) return SVIP_ERR_DTYPE;
    if (B <= 0 || B > MAX_BATCH || V <= 0 || k_max < 1 || (long long)B * k_max > 0x7FFFFFFFLL || row_stride < V ||
        seq_stride < (long long)(k_max - 1) * row_stride + V)
        return SVIP_ERR_SHAPE;
    const int vec = vec_of(dtype);
    if (!aligned16(logits_in) || !aligned16(logits_out) || row_stride % vec != 0 || seq_stride % vec != 0)
        return SVIP_ERR_ALIGN;
    if (!(temperature > 0.f) || !isfinite(temperature) || top_k < 0 || !(top_p > 0.0)) return SVIP_ERR_PARAM;

    WarpArgs a;
    a.in = logits_in;
    a.out = logits_out;
    a.seq_stride = seq_stride;
    a.row_stride = row_stride;
    a.k = k_max;
    a.V = V;
    a.sc = make_scale(temperature);
    a.top_k = top_k;
    a.top_p = top_p;
    // weights <= 1 in units of 2^-shift: V of them must stay below 2^62
    int lg = 0;
    while ((1ll << lg) < (long long)V) ++lg;
    const int shift = 62 - lg < 44 ? 62 - lg : 44;
    a.fix_scale = ldexpf(1.f, shift);
    a.stream = 2.0 * B * k_max * V * (dtype == SVIP_F32 ? 4 : 2) > 288e6;        // (the cache: 256 MiB)
    a.kept = kept_out;
    a.no_shortcut = g_tune.warp_no_shortcut;
    a.routes = g_warp_routes;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    bool ok = false;
    by_dtype(dtype, [&](auto tag) {
        using DT = decltype(tag);
        const bool nucleus = !(top_k > 0 && top_k < V) && a.top_p < 1.0, shortcut = V >= NUCLEUS_MIN_V && !a.no_shortcut;
        ok = launch(!nucleus ? k_warp<DT, GENERAL> : (shortcut ? k_warp<DT, NUCLEUS> : k_warp<DT, HISTOGRAMS>),
                    (unsigned)((long long)B * k_max), WARP_WG, st, a);
    });
    return ok ? SVIP_OK : SVIP_ERR_HIP;
}

svip_status svip_pair_stats(const void *target_logits, const void *draft_logits, int dtype, int B,
                            int k_max, int V, long long seq_stride_t, long long seq_stride_d,
                            long long row_stride, float temperature, const int *draft_len,
                            const double *draft_lse, float c, float *stats_out, void *workspace,
                            size_t workspace_bytes, void *hip_stream)
{
    if (!target_logits || !draft_logits || !draft_len || !stats_out) return SVIP_ERR_NULL;
    if (!dtype_ok(dtype)) return SVIP_ERR_DTYPE;
    if (B <= 0 || B > MAX_BATCH || V <= 0 || k_max < 1 || k_max > SVIP_MAX_K || row_stride < V ||
        seq_stride_t < (long long)(k_max - 1) * row_stride + V || seq_stride_d < (long long)(k_max - 1) * row_stride + V)
        return SVIP_ERR_SHAPE;
    const int kd = draft_lse ? 0 : k_max;
    const long long stat_rows = (long long)B * (kd + k_max + 1), pos = (long long)B * k_max;
    if (stat_rows * MAX_SLICES > 0x7FFFFFFFLL) return SVIP_ERR_SHAPE;
    const int vec = vec_of(dtype);
    if (!aligned16(target_logits) || !aligned16(draft_logits) || row_stride % vec != 0 ||
        seq_stride_t % vec != 0 || seq_stride_d % vec != 0)
        return SVIP_ERR_ALIGN;
    if (!(temperature > 0.f) || !isfinite(temperature) || !(c >= 0.f) || !isfinite(c)) return SVIP_ERR_PARAM;

    PairArgs a;
    a.v.geo = geo_stats(stat_rows, V, vec, g_tune.stats_slices);
    a.geo2 = geo_stats(pos, V, vec, g_tune.pair_slices);
    if (!workspace_ok(workspace, workspace_bytes, need_pair(B, k_max, kd != 0, a.v.geo, a.geo2, nullptr, nullptr)))
        return SVIP_ERR_WORKSPACE;
    const bool fine = room_for_finer(workspace_bytes, B, k_max, V);
    const int parts = finer_stats(a.v, stat_rows, vec, g_tune.stats_slices, fine);
    a.geo2 = geo_stats(pos, V, vec, g_tune.pair_slices, fine);
    size_t part_bytes, L_bytes;
    need_pair(B, k_max, kd != 0, a.v.geo, a.geo2, &part_bytes, &L_bytes);
    a.v.geo_s = a.v.geo;
    a.v.target = target_logits;
    a.v.draft = draft_logits;
    a.v.seq_t = seq_stride_t;
    a.v.seq_d = seq_stride_d;
    a.v.row_stride = row_stride;
    a.v.pos = nullptr;
    a.v.skip = nullptr;
    a.v.B = B;
    a.v.k = k_max;
    a.v.kd = kd;
    a.v.bonus = 0;
    a.v.sc = make_scale(temperature);
    a.v.m0 = beyond_range(a.v.sc);
    a.v.tokens = nullptr;
    a.v.draft_len = draft_len;
    a.v.draft_lse = draft_lse;
    a.v.u_accept = nullptr;
    a.v.u_resample = nullptr;
    a.v.n_accepted = nullptr;
    a.v.next_token = nullptr;
    a.v.accept_prob = nullptr;
    a.v.ws = carve(workspace, workspace_bytes, B, 0);
    char *after = static_cast<char *>(a.v.ws.part) + part_bytes;
    a.L = reinterpret_cast<double *>(after);
    a.sums = reinterpret_cast<double *>(after + L_bytes);
    a.c = c;
    a.out = stats_out;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    a.v.stat_items = stat_rows * a.v.geo.ns;
    const unsigned g_stats = (unsigned)a.v.stat_items, g_pos = (unsigned)((pos + 63) / 64),
                   g_sums = (unsigned)(pos * a.geo2.ns);
    bool ok = false;
    by_dtype(dtype, [&](auto tag) { ok = launch(k_verify_stats<decltype(tag)>, g_stats, WG, st, a.v); });
    ok = ok && by_parts(parts, [&](auto of) { return launch(k_pair_L<decltype(of)::value>, g_pos, 64, st, a); });
    if (ok) by_dtype(dtype, [&](auto tag) { ok = launch(k_pair_sums<decltype(tag)>, g_sums, WG, st, a); });
    ok = ok && launch(k_pair_finish, g_pos, 64, st, a);
    return ok ? SVIP_OK : SVIP_ERR_HIP;
}

// ---- benchmark and experiment hooks (include/svip_bench.h) -------------------------------------------

svip_status svip_bench_time_kernels(int kernel_class, void *const *start_events, void *const *stop_events, int n_pairs)
{
    if (kernel_class < 0 || kernel_class >= SVIP_BENCH_KERNEL_CLASSES || n_pairs < 0) return SVIP_ERR_PARAM;
    if (n_pairs > 0 && (!start_events || !stop_events)) return SVIP_ERR_NULL;
    KernelTimer &t = g_timer[kernel_class];
    t.start = n_pairs ? start_events : nullptr;
    t.stop = n_pairs ? stop_events : nullptr;
    t.n = n_pairs;
    t.used = 0;
    return SVIP_OK;
}

int svip_bench_events_used(int kernel_class)
{
    return kernel_class >= 0 && kernel_class < SVIP_BENCH_KERNEL_CLASSES ? g_timer[kernel_class].used : -1;
}

svip_status svip_bench_empty_kernel(void *hip_stream)
{
    return launch(k_empty, 1u, 64u, static_cast<hipStream_t>(hip_stream), 0) ? SVIP_OK : SVIP_ERR_HIP;
}

size_t svip_bench_stream_sink_words(size_t bytes, int vectors_per_thread)
{
    if (vectors_per_thread != 4 && vectors_per_thread != 8 && vectors_per_thread != 16) return 0;
    const size_t nvec = bytes / 16, per_wg = (size_t)WG * vectors_per_thread;
    return ((nvec + per_wg - 1) / per_wg) * NWAVE;
}

svip_status svip_bench_stream_read(const void *buf, size_t bytes, int vectors_per_thread, unsigned *sink,
                                   void *hip_stream)
{
    if (!buf || !sink) return SVIP_ERR_NULL;
    if (!aligned16(buf)) return SVIP_ERR_ALIGN;
    const size_t words = svip_bench_stream_sink_words(bytes, vectors_per_thread);
    if (words == 0 || words / NWAVE > 0x7FFFFFFFull) return SVIP_ERR_SHAPE;
    StreamArgs a;
    a.buf = static_cast<const u32x4 *>(buf);
    a.nvec = bytes / 16;
    a.sink = sink;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const unsigned grid = (unsigned)(words / NWAVE);
    bool ok;
    if (vectors_per_thread == 4) ok = launch(k_stream_read<4>, grid, WG, st, a);
    else if (vectors_per_thread == 8) ok = launch(k_stream_read<8>, grid, WG, st, a);
    else ok = launch(k_stream_read<16>, grid, WG, st, a);
    return ok ? SVIP_OK : SVIP_ERR_HIP;
}

svip_status svip_bench_set_tuning(const svip_bench_tuning *tuning)
{
    const svip_bench_tuning zero = {0, 0, 0, 0, 0, 0, 0};
    const svip_bench_tuning t = tuning ? *tuning : zero;
    if (t.draft_slices < 0 || t.stats_slices < 0 || t.resid_slices < 0 || t.pair_slices < 0 ||
        t.stats_workgroups < 0)
        return SVIP_ERR_PARAM;
    g_tune = t;
    return SVIP_OK;
}

svip_status svip_bench_warp_routes(int *routes)
{
    g_warp_routes = routes;
    return SVIP_OK;
}

}  // extern "C"
