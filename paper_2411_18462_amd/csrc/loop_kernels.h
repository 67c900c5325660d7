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
    int ahead;                 // rows to read past the last token's, see trace_rows.h
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
// Greedy verification of a position needs nothing but the argmax of its target row, and neither that nor the draft row's
// statistics depend on where the rounds begin and end: rows are read once each, in order, many at a time, and the rounds are
// then gone through on what is known of the rows.  A pair of launches reads up to `group` further draft rows of every
// running sequence and the target rows beside them, and takes the sequence through as many rounds as these decide.
//   k_stream_rows     one wave per tile of 256 vectors: draft rows as in k_draft_stats, target rows as their first maximum
//   k_stream_advance  one workgroup per sequence: a wave per row, then one wave for the rounds
// State of a sequence between launches: rb.drafted, rb.tokens and rb.argmax, what is known of its unfinished round.
// What bounds it: reading the rows.  8 sequences of 151936 bf16 logits, 48 tokens in drafts of 1.3: k_stream_rows takes 46 us for 243
// MB (5.3 TB/s) and k_stream_advance 19 us for 101 rows and 33 rounds (records 8, logarithms 1, rounds 6), the whole generation
// 144 us with what the host does before and after; a pair of launches per round, all of them latency, 482.

// Draft rows that a launch reads of a sequence, see trace_rows.h.
__device__ __forceinline__ int rows_to_read(const GroupArgs &a, int pos, int drafted, int cap, int start)
{
    return stream_rows(pos, drafted, cap, start, a.l.L, a.l.gamma_max, a.l.max_new, a.ahead, a.group);
}

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
    const RoundBuffers &rb = a.l.rb;
    if (blockIdx.x == 0 && threadIdx.x == 0) {            // what the launches before this one left
        post(a.running, rb.counter[0]);
        post(a.rounds, rb.counter[2]);
        post(a.active, rb.counter[1]);
    }
    if (a.l.round_log && rb.counter[1] == 0) {            // all is done: the log of sequences that ended before the last one
        const int b = (int)(blockIdx.x * WG + threadIdx.x), rounds = rb.counter[2];
        if (b < a.l.B && rb.done[b])
            for (int r = rb.round[b]; r < rounds; ++r) log_idle(a.l, b, r);
        return;
    }
    int y, r, jj, b;
    if (!wave_to_record(a.d, (unsigned)((2 * a.group + 1) * a.lane_rows), &y, &r) || !group_row(a, y, &jj, &b)) return;
    const int cap = min(a.d.cap[b], a.d.k_max), stopped = a.d.stop_in[b], drafted = rb.drafted[b], pos = a.d.pos[b];
    const int start = a.l.state[(size_t)b * SVIP_LOOP_NSTATE + 7];
    if (stopped) return;
    const int n = rows_to_read(a, pos, drafted, cap, start);
    const bool of_target = jj >= a.group;
    const int i = of_target ? jj - a.group : jj;
    // (the target row behind the rows of the launch before is known)
    if (of_target ? i > n || (i == 0 && drafted >= 0) : i >= n) return;
    const long long off = draft_row_offset(a.d, b, (drafted > 0 ? drafted : 0) + i);
    if (of_target) {
        const unsigned long long key = tile_argmax<DT>(static_cast<const DT *>(a.target) + off, a.d.geo.V, r);
        if ((threadIdx.x & 63) == 0) a.keys[(size_t)(y - a.group * a.lane_rows) * a.d.geo.ns + r] = key;
    } else {
        tile_record<DT, GREEDY>(a.d, static_cast<const DT *>(a.d.logits) + off, r, (size_t)y * a.d.geo.ns + r);
    }
}

// The first member at or behind j of a set of rows, bit j % 64 of word j / 64; `rows` if there is none.
constexpr int STREAM_WORDS = (SVIP_MAX_K + STREAM_MAX_GROUP) / 64 + 1;
__device__ __forceinline__ int next_in(const unsigned long long *set, int j, int rows)
{
    for (int w = j >> 6; w * 64 < rows; ++w) {
        const unsigned long long m = w == j >> 6 ? set[w] & (~0ull << (j & 63)) : set[w];
        if (m) return w * 64 + __ffsll((long long)m) - 1;
    }
    return rows;
}

template <int RPL>
__global__ __launch_bounds__(GROUP_FINISH_WAVES * 64) void k_stream_advance(GroupArgs a)
{
    // of the new rows: draft token, sum of the weights and of the weighted exponents; argmax of the target rows
    __shared__ int token[STREAM_MAX_GROUP], amax[STREAM_MAX_GROUP + 1];
    __shared__ double S[STREAM_MAX_GROUP], tt[STREAM_MAX_GROUP];
    __shared__ unsigned long long sets[3][STREAM_WORDS];
    __shared__ int2 next[STREAM_WORDS * 64];              // the first row from j on that ends a draft; whose token differs
    __shared__ int any_bad;
    constexpr int GROUP = RPL < 3 ? 4 : 2;                // rows of a wave whose records and keys are requested together
    const int b = blockIdx.x, lane = threadIdx.x & 63, ns = a.d.geo.ns;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const RoundBuffers &rb = a.l.rb;
    if (a.d.stop_in[b]) return;                           // (the flag is only stored behind the last barrier)
    int *st = a.l.state + (size_t)b * SVIP_LOOP_NSTATE;
    const int pos0 = __builtin_amdgcn_readfirstlane(rb.pos[b]), start = __builtin_amdgcn_readfirstlane(st[7]);
    int limit = __builtin_amdgcn_readfirstlane(a.d.cap[b]), cap = min(limit, a.d.k_max);   // (apart where the state says more than gamma_max)
    const int drafted = __builtin_amdgcn_readfirstlane(rb.drafted[b]), known = drafted > 0 ? drafted : 0;
    const int n = rows_to_read(a, pos0, drafted, cap, start);
    int *tokens = rb.tokens + (size_t)b * a.l.gamma_max, *am = rb.argmax + (size_t)b * (a.d.k_max + 1);
    for (int i0 = wave; i0 <= n; i0 += GROUP * nwaves) {
        unsigned long long k[GROUP][RPL];
        GreedyRow<RPL> r[GROUP];
#pragma unroll
        for (int q = 0; q < GROUP; ++q) {
            const size_t at = ((size_t)min(i0 + q * nwaves, n) * a.lane_rows + b) * ns;
#pragma unroll
            for (int v = 0; v < RPL; ++v) k[q][v] = lane + 64 * v < ns ? a.keys[at + lane + 64 * v] : 0ull;
        }
#pragma unroll
        for (int q = 0; q < GROUP; ++q) r[q].load(a.d, ((size_t)min(i0 + q * nwaves, n - 1) * a.lane_rows + b) * ns);
        asm volatile("" : : : "memory");                  // all of it is requested before any of it is waited for
#pragma unroll
        for (int q = 0; q < GROUP; ++q) {
            const int i = i0 + q * nwaves;
            if (i > n) break;
            unsigned long long best = 0ull;
#pragma unroll
            for (int v = 0; v < RPL; ++v) best = k[q][v] > best ? k[q][v] : best;
            best = wave_reduce(best, OpMax{});
            if (lane == 0) amax[i] = i > 0 || drafted < 0 ? argmax_index(best) : am[known];
            if (i == n) break;
            r[q].merge(a.d);
            if (lane == 0) {
                token[i] = r[q].tok;
                S[i] = r[q].S;
                tt[i] = r[q].tt;
            }
        }
    }
    if (threadIdx.x == 0) any_bad = 0;
    __syncthreads();
    // Rows from here on relative to pos0: draft rows 0 .. rows - 1 and target rows 0 .. rows are known, the first `known` of them
    // from the launches before.
    const int rows = known + n;
    const auto argmax_of = [&](int j) { return j < known ? am[j] : amax[j - known]; };
    const auto token_of = [&](int j) { return j < known ? tokens[j] : token[j - known]; };
    for (int w = wave; w * 64 < rows; w += nwaves) {
        const int j = w * 64 + lane;
        bool ends = false, differs = false, bad = false;
        if (j < rows) {
            const int x = token_of(j);
            ends = j >= known && above_threshold(a.d, entropy_of(log(S[j - known]), S[j - known], tt[j - known]));
            differs = argmax_of(j) != x;
            bad = x < 0 || x >= a.d.geo.V;
        }
        const unsigned long long e = __ballot(ends), d = __ballot(differs), x = __ballot(bad);
        if (lane == 0) {
            sets[0][w] = e;
            sets[1][w] = d;
            sets[2][w] = x;
            if (x) any_bad = 1;
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < rows; j += blockDim.x) next[j] = make_int2(next_in(sets[0], j, rows), next_in(sets[1], j, rows));
    __syncthreads();
    if (wave != 0) return;
    // The rounds that these rows decide, the first from p = 0.  Verification: position j is accepted iff the target row's argmax
    // is the draft token, and the first that is not gives its argmax in its place.  This is one thread's chain, so what it
    // looks up has been worked out for every row.
    const int first_round = __builtin_amdgcn_readfirstlane(rb.round[b]);
    int round = first_round, p = 0, all_drafted = 0, accepted = 0;
    bool done = false, pause = false, bad_token = false;
    const bool look = __builtin_amdgcn_readfirstlane(any_bad) != 0;
    while (!done && !pause && p < rows) {
        const int2 at = next[p];
        const int end = min(p + cap, rows), ends = __builtin_amdgcn_readfirstlane(at.x), differs = __builtin_amdgcn_readfirstlane(at.y);
        if (ends >= end && end < p + cap) break;                   // its draft goes on
        const int g = min(ends + 1, end) - p, na = min(differs - p, g);
        if (look) {                                                // verification looks at 64 positions at a time
            const int seen = p + min(g, (na / 64 + 1) * 64);
            bad_token = bad_token || next_in(sets[2], p, rows) < seen;
        }
        if (lane == 0) log_round(a.l, b, round, pos0 + p, limit, g, na);
        limit = cap = next_cap(a.l, limit, na == g);
        p += na + 1;
        ++round;
        all_drafted += g;
        accepted += na;
        done = finished(pos0 + p, start, cap, a.l.L, a.l.max_new);
        pause = round == a.last_round;
    }
    // Every token put out is the argmax of its target row.
    const int made = __builtin_amdgcn_readfirstlane(st[6]);
    int *o = a.l.out_tokens + (size_t)b * a.l.out_stride + made;
    for (int j = lane; j < p; j += 64) o[j] = argmax_of(j);
    // What is known of the next round moves to the front: each pass has read its values before it stores them, at or below
    // where it found them.
    const int left = p > rows ? -1 : rows - p;
    if (!done && !pause) {
        for (int j0 = p == 0 ? known : 0; j0 <= left; j0 += 64) {
            const int j = j0 + lane, m = j <= left ? argmax_of(p + j) : 0, x = j < left ? token_of(p + j) : 0;
            if (j <= left) am[j] = m;
            if (j < left) tokens[j] = x;
        }
    }
    if (lane != 0) return;
    if (bad_token) atomicOr(a.flags, (unsigned)SVIP_FLAG_BAD_TOKEN);
    rb.drafted[b] = left;
    if (round == first_round) return;
    st[0] = pos0 + p;
    st[1] = cap;
    st[2] = done ? 1 : 0;
    st[3] += round - first_round;
    st[4] += all_drafted;
    st[5] += accepted;
    st[6] = made + p;
    begin_sequence(rb, b, pos0 + p, cap, done);
    rb.round[b] = round;
    if (pause) rb.stop[b] = 1;
    if (done) atomicSub(&rb.counter[0], 1);
    if (done || pause) {
        atomicMax(&rb.counter[2], round);
        atomicSub(&rb.counter[1], 1);
    }
}

}  // namespace svip
