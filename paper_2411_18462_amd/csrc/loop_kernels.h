// Kernels of the decoding loop that take several draft positions of every sequence at once.  The rows of a trace do not
// depend on the tokens chosen before them, so positions need not wait for one another: at the loop's batch sizes a
// launch of one position is all latency (8 rows of 152K bf16 logits, 2.4 MB: 7 us for its two launches), and one of
// four costs hardly more.
#pragma once
#include "draft_kernels.h"
#include "greedy_kernels.h"
#include "loop_round.h"

namespace svip {

struct GroupArgs {
    DraftArgs d;               // records of one tile; the launch's rows in the order of `lane_rows`
    int group;                 // draft positions a launch covers
    int lane_rows;             // launch row y is position y / lane_rows of sequence y % lane_rows; at least B
    unsigned lane_magic;       // that division, as DraftArgs::div_magic
    // greedy loop only
    const void *target;        // traces laid out as the draft's
    unsigned long long *keys;  // [(group + 1) * lane_rows][ns] first-maximum keys of the target rows
    unsigned *flags;           // sticky device-data flags
    int last_round;            // a sequence pauses where its next round would be this one
    Mail active, running, rounds;      // counter[1], counter[0], counter[2] as the launch finds them
    LoopArgs l;
};

// Which record wave `wv` of this workgroup takes: row *b of `rows`, record *r of that row, as in k_draft_stats; false: none.
__device__ __forceinline__ bool wave_to_record(const DraftArgs &a, unsigned rows, int *b, int *r)
{
    const int nrec = a.geo.ns;
    const unsigned wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (a.rows_by_xcd) {
        const unsigned xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3;
        const unsigned q = a.div == 1u ? slot : __umulhi(slot, a.div_magic);
        *b = (int)(q * 8u + xcd);
        *r = (int)((slot - q * a.div) * NWAVE + wv);
        return *b < (int)rows && *r < nrec;
    }
    const unsigned gw = blockIdx.x * NWAVE + wv;
    if (gw >= rows * (unsigned)nrec) return false;
    *b = (int)(a.div == 1u ? gw : __umulhi(gw, a.div_magic));
    *r = (int)(gw - (unsigned)*b * (unsigned)nrec);
    return true;
}

// Row y of a launch as (position, sequence).
__device__ __forceinline__ bool group_row(const GroupArgs &a, int y, int *jj, int *b)
{
    *jj = (int)(a.lane_rows == 1 ? (unsigned)y : __umulhi((unsigned)y, a.lane_magic));
    *b = y - *jj * a.lane_rows;
    return *b < a.d.B;
}

// The record of tile r of a row, stored at index `at`: what k_draft_stats does for records of one tile, without its flag.
template <typename DT, RecordKind KIND>
__device__ __forceinline__ void tile_record(const DraftArgs &a, const DT *row, int r, size_t at)
{
    constexpr int N = VecOf<DT>::N, CPT = WG / 64;
    typename RawOf<DT>::type raw[CPT];
    float mw = neg_inf(), td = 0.f;
    LaneSums<KIND> sums;
    int first = -1;
    unsigned lowest = 0u;
    if (r < a.geo.V / (WG * N)) wave_load<DT, CPT, false>(row, a.geo.V, r * CPT, raw);
    else wave_load<DT, CPT, true>(row, a.geo.V, r * CPT, raw);
    bool ok = a.common_range && wave_tile<DT, CPT, KIND>(raw, r * CPT, mw, sums, td, first, lowest, a.sc);
    ok = ok && __ballot(!(td > neg_inf())) == 0ull;       // (a NaN among the logits, see k_draft_stats)
    finish_record<DT, KIND>(a, row, r, r + 1, at, ok, mw, sums, td, first, lowest);
}

// The draft records of positions step_j .. step_j + group - 1, one wave per record as in k_draft_stats.  Rows past a
// sequence's limit may lie past the end of its trace: nothing of them is touched.
template <typename DT>
__global__ __launch_bounds__(WG, 8) void k_group_stats(GroupArgs a)
{
    int y, r, jj, b;
    if (!wave_to_record(a.d, (unsigned)(a.group * a.lane_rows), &y, &r) || !group_row(a, y, &jj, &b)) return;
    const int cap = min(a.d.cap[b], a.d.k_max), stopped = a.d.stop_in[b], j = a.d.step_j + jj;
    if (stopped || j >= cap) return;
    tile_record<DT, QUARTERS>(a.d, static_cast<const DT *>(a.d.logits) + draft_row_offset(a.d, b, j), r, (size_t)y * a.d.geo.ns + r);
}

// ... and what follows from them: grid (sequences), a wave per position (positions in turn where there are more of them
// than waves).  Every position up to the sequence's limit gets its token and logsumexp; the draft ends with the first
// one whose entropy is above the threshold, or at the limit, and what stands behind that is read by nobody.
constexpr int GROUP_FINISH_WAVES = 16;
template <typename DT, int RPL>
__global__ __launch_bounds__(GROUP_FINISH_WAVES * 64) void k_group_finish(GroupArgs a)
{
    __shared__ int first_stop;
    const int b = blockIdx.x, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const int cap = min(a.d.cap[b], a.d.k_max);
    if (a.d.stop_in[b]) return;                           // (the flag is only stored behind the last barrier)
    const int n = min(a.group, cap - a.d.step_j);         // at least 1: a sequence at its limit has stopped
    if (threadIdx.x == 0) first_stop = n;
    __syncthreads();
    for (int jj = wave; jj < n; jj += nwaves) {
        const long long o = (long long)b * a.d.io_stride + jj;
        QuarterRow<RPL> r;
        r.load(a.d, ((size_t)jj * a.lane_rows + b) * a.d.geo.ns);
        const float u = a.d.u[o];
        r.merge(a.d);
        r.template find_token<DT>(a.d, static_cast<const DT *>(a.d.logits) + draft_row_offset(a.d, b, a.d.step_j + jj), u, o);
        const double tt = r.entropy_sum(), S = wave_sum(r.M);
        if (lane == 0 && write_entropy(a.d, o, r.mrow, S, tt)) atomicMin(&first_stop, jj);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int len = a.d.step_j + min(first_stop + 1, n);
        a.d.draft_len[b] = len;
        a.d.stop[b] = first_stop < n || len >= cap ? 1 : 0;   // otherwise the next group goes on
    }
}

// ---- greedy loop ----------------------------------------------------------------------------------
//
// Greedy verification of a position needs nothing but the argmax of its target row, which does not depend on the draft
// either.  So the sequences need not keep step: a pair of launches takes every running sequence forward by up to `group`
// draft positions of its own round, reads the target rows beside them, and where the draft ends there also verifies it, does
// the round's bookkeeping and sets up the sequence's next round.  No launch waits for the longest draft of the batch, and
// a round takes two launches for most sequences.
//   k_stream_rows     one wave per tile of 256 vectors: draft rows as in k_draft_stats, target rows as their first maximum
//   k_stream_advance  one workgroup per sequence, a wave per row of it
// state of a sequence between launches: rb.drafted, rb.tokens and rb.argmax of its round so far.
// First-maximum key (argmax_key) of one tile of a row by one wave.
template <typename DT>
__device__ __forceinline__ unsigned long long tile_argmax(const DT *row, int V, int tile)
{
    constexpr int N = VecOf<DT>::N, CPT = WG / 64;
    const int lane = threadIdx.x & 63;
    typename RawOf<DT>::type raw[CPT];
    if (tile < V / (WG * N)) wave_load<DT, CPT, false>(row, V, tile * CPT, raw);
    else wave_load<DT, CPT, true>(row, V, tile * CPT, raw);
    float z[CPT][N];
#pragma unroll
    for (int u = 0; u < CPT; ++u) unpack<DT>(raw[u], z[u]);
    float m = tree_max<N>(z[0]);
#pragma unroll
    for (int u = 1; u < CPT; ++u) m = vmax(m, tree_max<N>(z[u]));
    int at = -1;
#pragma unroll
    for (int u = CPT - 1; u >= 0; --u) {
#pragma unroll
        for (int e = N - 1; e >= 0; --e)
            if (z[u][e] == m) at = ((tile * CPT + u) * 64 + lane) * N + e;
    }
    const unsigned long long key = at >= 0 && at < V ? argmax_key(m, at) : 0ull;       // (past the end of the row: -inf)
    return wave_reduce(key, OpMax{});
}

template <typename DT>
__global__ __launch_bounds__(WG, 8) void k_stream_rows(GroupArgs a)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {            // what the launches before this one left
        post(a.running, a.l.rb.counter[0]);
        post(a.rounds, a.l.rb.counter[2]);
        post(a.active, a.l.rb.counter[1]);
    }
    int y, r, jj, b;
    if (!wave_to_record(a.d, (unsigned)((2 * a.group + 1) * a.lane_rows), &y, &r) || !group_row(a, y, &jj, &b)) return;
    const int cap = min(a.d.cap[b], a.d.k_max), stopped = a.d.stop_in[b], drafted = a.l.rb.drafted[b];
    const bool of_target = jj >= a.group;
    const int j = drafted + (of_target ? jj - a.group : jj);
    // the target row behind the last group's positions is known from there
    if (stopped || j >= cap + (of_target ? 1 : 0) || (of_target && j > 0 && j == drafted)) return;
    const long long off = draft_row_offset(a.d, b, j);
    if (of_target) {
        const unsigned long long key = tile_argmax<DT>(static_cast<const DT *>(a.target) + off, a.d.geo.V, r);
        if ((threadIdx.x & 63) == 0) a.keys[(size_t)(y - a.group * a.lane_rows) * a.d.geo.ns + r] = key;
    } else {
        tile_record<DT, GREEDY>(a.d, static_cast<const DT *>(a.d.logits) + off, r, (size_t)y * a.d.geo.ns + r);
    }
}

template <int RPL>
__global__ __launch_bounds__(GROUP_FINISH_WAVES * 64) void k_stream_advance(GroupArgs a)
{
    __shared__ int first_stop, token[STREAM_MAX_GROUP], amax[STREAM_MAX_GROUP + 1];
    const int b = blockIdx.x, lane = threadIdx.x & 63, ns = a.d.geo.ns;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const RoundBuffers &rb = a.l.rb;
    const int cap = min(a.d.cap[b], a.d.k_max), drafted = rb.drafted[b];
    if (a.d.stop_in[b]) return;                           // (the flag is only stored behind the last barrier)
    const int n = min(a.group, cap - drafted);            // at least 1: a sequence at its limit has ended its round
    if (threadIdx.x == 0) first_stop = n;
    __syncthreads();
    for (int i = wave; i < 2 * n + 1; i += nwaves) {
        if (i < n) {
            GreedyRow<RPL> r;
            r.load(a.d, ((size_t)i * a.lane_rows + b) * ns);
            r.merge(a.d);
            if (lane == 0) {
                token[i] = r.tok;
                if (above_threshold(a.d, entropy_of(log(r.S), r.S, r.tt))) atomicMin(&first_stop, i);
            }
        } else {
            const unsigned long long *keys = a.keys + ((size_t)(i - n) * a.lane_rows + b) * ns;
            unsigned long long best = 0ull;
            if (i > n || drafted == 0) {
                unsigned long long k[RPL];
#pragma unroll
                for (int v = 0; v < RPL; ++v) k[v] = lane + 64 * v < ns ? keys[lane + 64 * v] : 0ull;
#pragma unroll
                for (int v = 0; v < RPL; ++v) best = k[v] > best ? k[v] : best;
                best = wave_reduce(best, OpMax{});
                if (lane == 0) amax[i - n] = argmax_index(best);
            } else if (lane == 0) {
                amax[0] = rb.argmax[(size_t)b * (a.d.k_max + 1) + drafted];
            }
        }
    }
    __syncthreads();
    if (wave != 0) return;
    const int f = first_stop, here = min(f + 1, n), len = drafted + here;
    int *tokens = rb.tokens + (size_t)b * a.l.gamma_max, *am = rb.argmax + (size_t)b * (a.d.k_max + 1);
    if (f == n && len < cap) {                            // the draft goes on
        if (lane < n) tokens[drafted + lane] = token[lane];
        if (lane < n + 1) am[drafted + lane] = amax[lane];
        if (n == 64 && lane == 0) am[drafted + 64] = amax[64];
        if (lane == 0) rb.drafted[b] = len;
        return;
    }
    // verification as in accept_greedy_sequence
    int r = -1, next = -1;
    for (int j0 = 0; j0 <= len && r < 0; j0 += 64) {
        const int j = j0 + lane;
        int m = -1;
        bool reject = false;
        if (j <= len) {
            m = j < drafted ? am[j] : amax[j - drafted];
            if (j < len) {
                const int x = j < drafted ? tokens[j] : token[j - drafted];
                if (x < 0 || x >= a.d.geo.V) atomicOr(a.flags, (unsigned)SVIP_FLAG_BAD_TOKEN);
                reject = m != x;
            }
        }
        const unsigned long long rej = __ballot(reject);
        if (rej) {
            const int first = __ffsll((long long)rej) - 1;
            r = j0 + first;
            next = read_lane(m, first);
        } else if (len - j0 < 64) {
            r = len;
            next = read_lane(m, len - j0);
        }
    }
    const int round = rb.round[b];
    const bool goes_on = end_sequence(a.l, b, round, len, r, next, lane, 64,
                                      [&](int j) { return j < drafted ? tokens[j] : token[j - drafted]; });
    if (lane == 0) {
        rb.drafted[b] = 0;
        rb.round[b] = round + 1;
        const bool pause = round + 1 == a.last_round;
        if (pause) rb.stop[b] = 1;
        if (!goes_on) atomicSub(&rb.counter[0], 1);
        if (!goes_on || pause) {
            atomicMax(&rb.counter[2], round + 1);
            atomicSub(&rb.counter[1], 1);
        }
    }
}

}  // namespace svip
