// Kernels of svip_draft_step and svip_draft_step_greedy.
#pragma once
#include "exchange.h"
#include "kernel_args.h"
#include "sample_weights.h"
#include "trace_rows.h"

namespace svip {

// ---- draft step -------------------------------------------------------------------------------

__device__ __forceinline__ long long draft_row_offset(const DraftArgs &a, int b, int j)
{
    return (long long)b * a.row_stride + (a.pos ? (long long)(__builtin_amdgcn_readfirstlane(a.pos[b]) + j) * a.pos_stride : 0ll);
}
// The row that a step's statistics request before the stop flag is looked at (behind it the row is that of step_j).
__device__ __forceinline__ long long step_row_offset(const DraftArgs &a, int b)
{
    long long row = 0;
    if (a.pos) row = __builtin_amdgcn_readfirstlane(a.pos[b]) + step_row(a.step_j, __builtin_amdgcn_readfirstlane(a.cap[b]));
    return (long long)b * a.row_stride + row * a.pos_stride;
}
__device__ __forceinline__ bool at_cap(const DraftArgs &a, int b)
{
    const int cap = a.cap ? min(a.cap[b], a.k_max) : a.k_max;
    return a.step_j + 1 >= cap;
}

// Entropy of weights e_i = exp2(x_i) with sum S and tt = sum e_i x_i:  H = ln S - ln2 tt / S, and whether it is above the
// threshold of the stop test (Section 2.2, Eq. stop_condition).
__device__ __forceinline__ double entropy_of(double lnS, double S, double tt)
{
    const double H = lnS - 0.6931471805599453 * tt / S;
    return H > 0.0 ? H : 0.0;
}
__device__ __forceinline__ bool above_threshold(const DraftArgs &a, double H) { return sqrt(H) > (double)a.h; }
// The row's outputs that follow from it; returns whether it is above the threshold.
__device__ __forceinline__ bool write_entropy(const DraftArgs &a, long long o, float m, double S, double tt)
{
    const double lnS = log(S), H = entropy_of(lnS, S, tt);
    if (a.entropy) a.entropy[o] = (float)H;
    a.lse[o] = (double)m * a.sc.inv_T + lnS;
    return above_threshold(a, H);
}
// The same with the stop test and draft length of a single step.
__device__ __forceinline__ void write_row_outputs(const DraftArgs &a, int b, long long o, float m, double S, double tt)
{
    const bool stop = write_entropy(a, o, m, S, tt) || at_cap(a, b);
    a.stop[b] = stop ? 1 : 0;
    if (a.draft_len) a.draft_len[b] = a.step_j + 1;
}

// The draft step is two launches ordered by the stream, or for small ones (one_launch_step in svip_kernels.hip) the same work in one.
//
// k_draft_stats: the statistics of a row as one record per WAVE.  Record r of a row covers tiles
// [r * tps, (r + 1) * tps), and a wave reads a tile (256 consecutive vectors) as four chunks of 64
// consecutive vectors, one load each.  Nothing is shared between the waves of a workgroup -- no LDS, no
// barrier, so no wave waits for data that another wave's loads are still bringing in.
// k_draft_finish_*: merges a row's records (one or two per lane), writes entropy, logsumexp and stop flag, and finds
// the token.  What a record holds besides the statistics decides how:
//   QUARTERS  (records of one tile, launches of at most DRAFT_QUARTER_WAVES waves) the mass of each of its four
//             chunks: record and chunk are picked from the records alone, and one wave reads that chunk again,
//             one vector per lane, one scan over the lanes -- no LDS, no barrier;
//   TOTAL     (beyond) one sum: the chosen record's tiles are read and searched by a workgroup.  The statistics of a
//             launch this large are bound by vector-ALU issue, and the quarters' sums cost them more than the
//             shorter search gives back: us per step of 128256 bf16 logits, quarters / totals: 1 row 5.9 / 6.2, 8 rows
//             6.6 / 7.0, 64 rows 9.7 / 9.8, 128 rows 12.6 / 12.4, 192 rows 16.3 / 15.4, 256 rows 19.5 / 18.6 (the last two
//             with records of two tiles for the totals);
//   GREEDY    one sum and the first index of the maximum, which is the token: nothing is read again.
//
// k_draft_step: both, where the row's last workgroup finishes it.
enum RecordKind { QUARTERS, TOTAL, GREEDY };

// A row's stop flag, requested without looking at it: with no flag array the load goes to the start of the
// records (any valid address) and the value is ignored.  flag_after_loads() is where the value is first looked
// at: no access to memory moves across it, and the flag cannot be consumed earlier.  Together they keep the flag
// and the loads issued between them in flight at the same time; written as `stop_in && stop_in[b]` followed by
// an early return, the compiler waits for the flag first and only then issues the other loads (it sinks them
// below the return, or moves the flag to a scalar register at once), one more trip to memory per kernel.
__device__ __forceinline__ unsigned request_stop_flag(const DraftArgs &a, int b)
{
    const unsigned char *p = a.stop_in ? a.stop_in + b : reinterpret_cast<const unsigned char *>(a.part);
    return *p;
}
__device__ __forceinline__ bool flag_after_loads(const DraftArgs &a, unsigned flag)
{
    asm volatile("" : "+v"(flag) : : "memory");
    return a.stop_in && flag;
}

// Per lane, what a wave has summed so far.  QUARTERS: the sum of the weights of each chunk of its one tile.  Otherwise:
// the sum of the weights, and beside it the number of weights that are exactly 1 in the vectors that hold the maximum.
// Those have to stay out of the fp32 sum (next to a 1 the tail of a confident row, 1e-4 and less, would lose its low bits).
template <RecordKind KIND> struct LaneSums {
    float S = 0.f, ones = 0.f;
    __device__ __forceinline__ void add(int, float below) { S += below; }
    __device__ __forceinline__ void add(int, float below, float exact_ones)
    {
        S += below;
        ones += exact_ones;
    }
    __device__ __forceinline__ void rescale(float f, float d, float &td)
    {
        if (f < 1.0f) {                     // the old maximum becomes an ordinary term
            const float all = S + ones;
            td = f > 0.f ? f * fmaf(d, all, td) : 0.f;       // (d may be beyond what fp32 holds then)
            S = f * all;
            ones = 0.f;
        }
    }
    __device__ __forceinline__ double total() const { return (double)ones + (double)S; }
};
template <> struct LaneSums<QUARTERS> {
    double S[4] = {};
    __device__ __forceinline__ void add(int, float) {}
    __device__ __forceinline__ void add(int chunk, float below, float exact_ones) { S[chunk] = (double)below + (double)exact_ones; }
    __device__ __forceinline__ void rescale(float, float, float &) {}         // one tile: nothing before it
};

// One tile of a wave relative to the WAVE's running maximum mw (the same in every lane): the sums of the weights and
// td = sum w (z - mw), per lane.  One reference for the whole wave instead of one per lane saves per logit
//  - the count of weights that are exactly 1 in most vectors: the maximum and its ties are found by one comparison per
//    vector (its own maximum is there anyway) and a branch the whole wave takes, for about one vector in four.  There
//    sum fract(w) (fract(1) = 0) is what goes into the fp32 sum.  A logit below the maximum by less than 2^-25 / c also
//    rounds to a weight of 1; in another vector it goes into the lane's fp32 sum, whose roundings are then 2^-24 of a
//    sum of at least 1 -- next to an entropy of at least ln 2, as the row has two tokens of equal weight;
//  - the floor of the exponent: masked (-inf) logits are lowered to the most negative finite number while still
//    packed (half an instruction per logit), so z - mw stays finite and 0 * (z - mw) is 0;
//  - a product per term of the entropy sum: w (z - mw) is accumulated by fused multiply-adds, and the scale is
//    applied once per record in fp64,
// and per wave the rescaling of its lanes to one another.  What that is worth grows with how far issue rather than
// latency bounds the launch; us per draft step in a graph, before / after: 8 rows of 128256 bf16 logits 7.74 / 7.63, 64 rows
// 10.19 / 10.06 (greedy 9.75 / 9.26), 128 rows 13.6 / 12.8, 256 rows 20.1 / 18.5.  Together with the records' chunk masses,
// the shorter searches and the tails' loads (below), the same step: 1 row 6.5 / 5.9, 8 rows 7.5 / 6.6, 64 rows 10.2 / 9.65
// (greedy 9.8 / 8.75), 128 rows 13.6 / 12.9, 256 rows 20.2 / 18.9 (greedy 21.0 / 18.1), 16 rows of 32000 fp32 6.64 / 6.1.
// A tile without any logit above the most negative finite number only counts, in `lowest` (see count_lowest), those that
// are that number: they have weights if the wave never sees anything higher, and none otherwise.  Rows that were filtered
// or masked consist mostly of such tiles, and all is decided from the registers that hold them (us per step, read again
// as uncommon_record does / so: 256 rows of 151936 bf16 logits after top-k 50 38.9 / 21.2, 64 rows of 128256 fp32
// 13.7 / 11.3).
// Returns false where this form does not do: where the wave's maximum stays so close to that number that a lowered logit
// would not weigh exactly 0 (fp16 logits around -65504, or at temperatures in the hundreds), where a vector holds that
// number beside -inf and nothing higher, or for a maximum beyond 1e30.
template <typename DT, int NU, RecordKind KIND>
__device__ __forceinline__ bool wave_tile(const typename RawOf<DT>::type (&raw)[NU], int c0, float &mw, LaneSums<KIND> &sums,
                                          float &td, int &idx, unsigned &lowest, const Scale &sc)
{
    constexpr int N = VecOf<DT>::N;
    float z[NU][N], gm[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        unpack_finite<DT>(raw[u], z[u]);
        gm[u] = tree_max<N>(z[u]);
    }
    float mt = gm[0];
#pragma unroll
    for (int u = 1; u < NU; ++u) mt = vmax(mt, gm[u]);
    mt = wave_max(mt);
    const float mn = mt > mw ? mt : mw;
    if (!((mn - FiniteLow<DT>::value()) * sc.c_dn > -X_FLOOR && mn < 1e30f)) {
        unsigned n;
        if (!(mt == FiniteLow<DT>::value() && count_lowest<DT, NU>(raw, &n))) return false;
        if (KIND == GREEDY && idx < 0) {
#pragma unroll
            for (int u = NU - 1; u >= 0; --u) {
                const unsigned long long hit = __ballot((n >> (8 * u)) & 0xFFu);
                if (hit) idx = ((c0 + u) * 64 + __ffsll((long long)hit) - 1) * N;
            }
        }
        lowest += n;
        return true;
    }
    const bool higher = mt > mw;
    if (higher) {
        if (mw != neg_inf()) sums.rescale(exp2_raw(scaled_below_floored(mw - mt, sc)), mw - mt, td);
        mw = mt;
        idx = -1;
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        float w[N], d[N];
#pragma unroll
        for (int e = 0; e < N; ++e) {
            d[e] = z[u][e] - mw;
            w[e] = exp2_raw(scaled_below(d[e], sc));
        }
        // two chains of N / 2 terms: no more roundings in a row than the tree of products had
        float ta = w[0] * d[0], tb = w[N / 2] * d[N / 2];
#pragma unroll
        for (int e = 1; e < N / 2; ++e) {
            ta = fmaf(w[e], d[e], ta);
            tb = fmaf(w[N / 2 + e], d[N / 2 + e], tb);
        }
        td += ta + tb;
        const unsigned long long hit = __ballot(gm[u] == mw);
        float Sb = tree_sum<N>(w), ones = 0.f;
        if (hit) {
            float fr[N];
#pragma unroll
            for (int e = 0; e < N; ++e) fr[e] = __builtin_amdgcn_fractf(w[e]);
            const float below = tree_sum<N>(fr);
            ones = rintf(Sb - below);
            Sb = below;
            if (KIND != QUARTERS) sums.add(u, Sb, ones);
            if (KIND == GREEDY && higher && idx < 0) {     // vectors come in index order: the first lane of the first one
                int at = 0;
#pragma unroll
                for (int e = N - 1; e >= 0; --e) at = z[u][e] == mw ? e : at;
                const int first = __ffsll((long long)hit) - 1;
                idx = ((c0 + u) * 64 + first) * N + read_lane(at, first);
            }
        } else if (KIND != QUARTERS) {
            sums.add(u, Sb);
        }
        if (KIND == QUARTERS) sums.add(u, Sb, ones);
        // the sums are formed here: the compiler would otherwise move all of them behind the last branch and keep
        // every weight of the tile in registers until then
        if constexpr (KIND == QUARTERS) asm volatile("" : "+v"(td), "+v"(sums.S[u]));
        else asm volatile("" : "+v"(td), "+v"(sums.S), "+v"(sums.ones));
    }
    return true;
}

// A record outside wave_tile's range, from memory again: tile by tile with a floor under every exponent, one chunk at a
// time in registers.  S[q]: this lane's sum over the record's chunks q, q + 4, ..; td in units of log2 here.
template <typename DT, RecordKind KIND>
__device__ __forceinline__ void uncommon_record(const DraftArgs &a, const DT *row, int tb, int te, float &mw, double (&S)[4],
                                                double &td, int &idx)
{
    constexpr int N = VecOf<DT>::N, CPT = WG / 64;
    mw = neg_inf();
    idx = -1;
    td = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) S[q] = 0.0;
#pragma unroll 1
    for (int t0 = tb; t0 < te; ++t0) {
        typename RawOf<DT>::type tile[CPT];
        if (t0 < a.geo.V / (WG * N)) wave_load<DT, CPT, false>(row, a.geo.V, t0 * CPT, tile);
        else wave_load<DT, CPT, true>(row, a.geo.V, t0 * CPT, tile);
        float z[N], m = neg_inf();
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            unpack<DT>(tile[u], z);
            m = vmax(m, tree_max<N>(z));
            asm volatile("" : "+v"(tile[u]));       // unpacked again below, not kept
        }
        m = wave_max(m);
        if (m == neg_inf()) continue;
        const bool higher = m > mw;
        if (higher) {
            const float x = scaled_below_floored(mw - m, a.sc);       // (the floor, and so 0, for the first tile)
            const double f = (double)exp2_raw(x);
            td = f * (td + (double)x * ((S[0] + S[1]) + (S[2] + S[3])));
#pragma unroll
            for (int q = 0; q < 4; ++q) S[q] *= f;
            mw = m;
            idx = -1;
        }
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            unpack<DT>(tile[u], z);
            float all = 0.f, below = 0.f, tx = 0.f;
#pragma unroll
            for (int h = 0; h < N; h += 4) {
                float w[4], fr[4], wx[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = scaled_below_floored(z[h + e] - mw, a.sc);
                    w[e] = exp2_raw(x);
                    fr[e] = __builtin_amdgcn_fractf(w[e]);
                    wx[e] = w[e] * x;
                }
                all += tree_sum<4>(w);
                below += tree_sum<4>(fr);
                tx += tree_sum<4>(wx);
                asm volatile("" : "+v"(all), "+v"(below), "+v"(tx));
            }
            S[u] += (double)below + (double)rintf(all - below);
            td += (double)tx;
            asm volatile("" : "+v"(td), "+v"(S[u]));
            if (KIND == GREEDY && higher && idx < 0) {
                const unsigned long long hit = __ballot(tree_max<N>(z) == mw);
                if (hit) {
                    int at = 0;
#pragma unroll
                    for (int e = N - 1; e >= 0; --e) at = z[e] == mw ? e : at;
                    const int first = __ffsll((long long)hit) - 1;
                    idx = ((t0 * CPT + u) * 64 + first) * N + read_lane(at, first);
                }
            }
        }
    }
}

// The wave's record from its lanes' sums.  PUBLISH: for a workgroup of the same launch (exchange.h).
template <bool PUBLISH>
__device__ __forceinline__ void store_record(const DraftArgs &a, size_t at, float mw, int first, double lane_sum, double t)
{
    const double S = wave_sum(lane_sum);
    WaveRec *to = static_cast<WaveRec *>(a.part) + at;
    if ((threadIdx.x & 63) == 0) {
        if (PUBLISH) {
            publish_f64(&to->S, S);
            publish_f64(&to->t, t);
            publish_f64(reinterpret_cast<double *>(&to->m), __hiloint2double(first, __float_as_int(mw)));
        } else {
            WaveRec p;
            p.m = mw;
            p.idx = first;
            p.S = S;
            p.t = t;
            *to = p;
        }
    }
}
template <bool PUBLISH>
__device__ __forceinline__ void store_record(const DraftArgs &a, size_t at, float mw, const double (&S)[4], double t)
{
    // one store of six lanes: the chunks' sums (lane q holds that of chunk q), t, and the maximum
    const int lane = threadIdx.x & 63;
    double x = wave_sum4(S);
    x = lane == 4 ? t : x;
    x = lane == 5 ? __hiloint2double(0, __float_as_int(mw)) : x;
    double *to = reinterpret_cast<double *>(static_cast<QuarterRec *>(a.part) + at) + lane;
    if (lane < 6) {
        if (PUBLISH) publish_f64(to, x);
        else *to = x;
    }
}

// What a wave stores of the tiles [tb, te) it has summed (ok: within wave_tile's range throughout).
template <typename DT, RecordKind KIND, bool PUBLISH = false>
__device__ __forceinline__ void finish_record(const DraftArgs &a, const DT *row, int tb, int te, size_t at, bool ok, float mw,
                                              LaneSums<KIND> &sums, float td, int first, unsigned lowest)
{
    constexpr int CPT = WG / 64;
    if (ok && mw == neg_inf() && __ballot(lowest != 0u)) {                 // nothing but the lowest number: all ties
        mw = FiniteLow<DT>::value();
#pragma unroll
        for (int u = 0; u < CPT; ++u) sums.add(u, 0.f, (float)((lowest >> (8 * u)) & 0xFFu));
    }
    if (ok) {
        const double t = wave_sum((double)td) * a.sc.c;
        if constexpr (KIND == QUARTERS) store_record<PUBLISH>(a, at, mw, sums.S, t);
        else store_record<PUBLISH>(a, at, mw, first, sums.total(), t);
    } else {
        double S[4], t2;
        uncommon_record<DT, KIND>(a, row, tb, te, mw, S, t2, first);
        const double t = wave_sum(t2);
        if constexpr (KIND == QUARTERS) store_record<PUBLISH>(a, at, mw, S, t);
        else store_record<PUBLISH>(a, at, mw, first, (S[0] + S[1]) + (S[2] + S[3]), t);
    }
}

// grid (ceil(rows * records / 4)), one wave per record.  TPS: tiles per record, 1, 2 or 0 for more.  A record of two
// whole tiles requests both before it works on the first (the arithmetic of the first runs while the second is
// still on its way), which takes more registers; launches with one tile per record keep the other form.
template <typename DT, RecordKind KIND, int TPS>
__global__ __launch_bounds__(WG, TPS == 1 ? 8 : 6) void k_draft_stats(DraftArgs a)
{
    constexpr int N = VecOf<DT>::N, CPT = WG / 64;       // chunks of 64 vectors per tile
    static_assert(KIND != QUARTERS || TPS == 1, "a quarter is a chunk");
    const int nrec = a.geo.ns;
    // All arguments are requested at once: left to itself the compiler loads those behind the first branch only there,
    // a second trip to the scalar cache before the first load of a logit.
    asm volatile("" : : "s"(a.logits), "s"(a.row_stride), "s"(a.pos), "s"(a.cap), "s"(a.stop_in), "s"(a.geo.V), "s"(a.part),
                 "s"(a.sc.c_dn), "s"(a.sc.c_up), "s"(a.sc.c), "s"(a.common_range), "s"(a.step_j));
    // Which record this wave takes is the same in all its lanes: worked out in scalar registers, with the one
    // division done by a multiplication the host prepared, so that none of it takes vector-ALU slots.  (This and the
    // reading of the tiles are written out here: shared with the loop's kernels as functions they compile to 8 vector
    // instructions more and, in fp32, 44 registers instead of 55; 16 steps of 16 rows of 32000 fp32 logits take 1 % longer.)
    const unsigned wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int b, r;
    if (a.rows_by_xcd) {
        // Workgroups go to the chip's 8 XCDs in turn, and so do the rows' workgroups of the finish: keeping row b on
        // XCD b % 8 lets that kernel find the row's records (and what it reads again) in the L2 of its own XCD, and
        // the lines of the records are written by one L2 each.  The grid is ceil(B / 8) * 8 * ceil(nrec / 4)
        // workgroups; those of rows past B exit.
        const unsigned xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3;           // div = workgroups per row
        const unsigned q = a.div == 1u ? slot : __umulhi(slot, a.div_magic);
        b = (int)(q * 8u + xcd);
        r = (int)((slot - q * a.div) * NWAVE + wv);
        if (b >= a.B || r >= nrec) return;
    } else {
        const unsigned gw = blockIdx.x * NWAVE + wv;                            // div = records per row
        if (gw >= (unsigned)a.B * (unsigned)nrec) return;
        b = (int)(a.div == 1u ? gw : __umulhi(gw, a.div_magic));
        r = (int)(gw - (unsigned)b * (unsigned)nrec);
    }
    const DT *row = static_cast<const DT *>(a.logits) + step_row_offset(a, b);
    const int tps = TPS ? TPS : a.geo.tps;
    const int tb = r * tps, te = min(tb + tps, a.geo.ntiles);
    const int fe = min(te, a.geo.V / (WG * N));           // end of the tiles wholly inside the row
    // The record's first tile is requested before the row's stop flag is looked at, so that the two travel
    // together (a step is bound by round trips to memory); a stopped row costs those loads and nothing else.
    const unsigned flag = request_stop_flag(a, b);
    typename RawOf<DT>::type raw[CPT];
    float mw = neg_inf(), td = 0.f;
    LaneSums<KIND> sums;
    int first = -1;
    unsigned lowest = 0u;
    bool ok = a.common_range;
    if (TPS == 2 && te - tb == 2 && te <= fe) {
        typename RawOf<DT>::type raw2[CPT];
        wave_load<DT, CPT, false>(row, a.geo.V, tb * CPT, raw);
        wave_load<DT, CPT, false>(row, a.geo.V, (tb + 1) * CPT, raw2);
        if (flag_after_loads(a, flag)) return;
        ok = ok && wave_tile<DT, CPT, KIND>(raw, tb * CPT, mw, sums, td, first, lowest, a.sc) &&
             wave_tile<DT, CPT, KIND>(raw2, (tb + 1) * CPT, mw, sums, td, first, lowest, a.sc);
    } else {
        if (tb < fe) wave_load<DT, CPT, false>(row, a.geo.V, tb * CPT, raw);
        else wave_load<DT, CPT, true>(row, a.geo.V, tb * CPT, raw);
        if (flag_after_loads(a, flag)) return;
        ok = ok && wave_tile<DT, CPT, KIND>(raw, tb * CPT, mw, sums, td, first, lowest, a.sc);
        if (TPS != 1) {
            for (int t0 = tb + 1; t0 < te && ok; ++t0) {
                if (t0 < fe) wave_load<DT, CPT, false>(row, a.geo.V, t0 * CPT, raw);
                else wave_load<DT, CPT, true>(row, a.geo.V, t0 * CPT, raw);
                ok = wave_tile<DT, CPT, KIND>(raw, t0 * CPT, mw, sums, td, first, lowest, a.sc) &&
                     __ballot(lowest & 0x80808080u) == 0ull;      // (the counts of 16 tiles or more leave their bytes)
            }
        }
    }
    // A NaN among the logits (only the 16-bit types get one past unpack_finite) shows in td, whose terms are all finite and
    // at most 0 otherwise; like a masked logit it weighs nothing, by the floor of uncommon_record's exponents.
    ok = ok && __ballot(!(td > neg_inf())) == 0ull;
    finish_record<DT, KIND>(a, row, tb, te, (size_t)b * nrec + r, ok, mw, sums, td, first, lowest);
}

// The record of tile r of a row, stored at index `at`: what k_draft_stats does for records of one tile.  stopped() is asked while
// the tile is on its way; returns what it said (true: no record).
struct NeverStopped {
    __device__ __forceinline__ bool operator()() const { return false; }
};
template <typename DT, RecordKind KIND, bool PUBLISH = false, typename Stopped = NeverStopped>
__device__ __forceinline__ bool tile_record(const DraftArgs &a, const DT *row, int r, size_t at, Stopped stopped = Stopped())
{
    constexpr int N = VecOf<DT>::N, CPT = WG / 64;
    typename RawOf<DT>::type raw[CPT];
    float mw = neg_inf(), td = 0.f;
    LaneSums<KIND> sums;
    int first = -1;
    unsigned lowest = 0u;
    if (r < a.geo.V / (WG * N)) wave_load<DT, CPT, false>(row, a.geo.V, r * CPT, raw);
    else wave_load<DT, CPT, true>(row, a.geo.V, r * CPT, raw);
    if (stopped()) return true;
    bool ok = a.common_range && wave_tile<DT, CPT, KIND>(raw, r * CPT, mw, sums, td, first, lowest, a.sc);
    ok = ok && __ballot(!(td > neg_inf())) == 0ull;       // (a NaN among the logits, see k_draft_stats)
    finish_record<DT, KIND, PUBLISH>(a, row, r, r + 1, at, ok, mw, sums, td, first, lowest);
    return false;
}

// The inverse CDF inside one chunk of a row by one wave: the smallest index whose inclusive prefix of weights
// exp2((z - m) c), counted from the start of the chunk, exceeds `target`.  A lane holds one vector; fp32 sums per
// vector, fp64 over the lanes.  The lane that holds the token reports it (see locate_batch).  If rounding leaves no
// crossing, it is the last index with positive weight (-1 if there is none).  (search_chunks of row_math.h with one chunk does
// the same in a step of 16 rows of 32000 fp32 logits that is 0.05 us longer.)
template <typename DT, typename Report>
__device__ __forceinline__ void search_chunk(const DT *row, int V, int chunk, float m, const Scale &sc, double target, Report report)
{
    constexpr int N = VecOf<DT>::N;
    const int lane = threadIdx.x & 63;
    float z[N], w[N];
    typename RawOf<DT>::type raw[1];
    wave_load<DT, 1, true>(row, V, chunk, raw);
    unpack<DT>(raw[0], z);
#pragma unroll
    for (int e = 0; e < N; ++e) w[e] = exp2_raw(scaled_below_floored(z[e] - m, sc));
    const double g = (double)tree_sum<N>(w);
    const double incl = wave_inclusive_sum(g);
    const unsigned long long hit = __ballot(g > 0.0 && incl > target), mass = __ballot(g > 0.0);
    double C = incl - g;
    int pick = -1, lastpos = -1;
    float wp = 0.f, wl = 0.f;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        C += (double)w[e];
        if (w[e] > 0.f) {
            lastpos = e;
            wl = w[e];
            if (pick < 0 && C > target) {
                pick = e;
                wp = w[e];
            }
        }
    }
    const int base = (chunk * 64 + lane) * N;
    if (hit) {
        if (lane == __ffsll((long long)hit) - 1) {
            if (pick < 0) report(base + lastpos, wl);
            else report(base + pick, wp);
        }
    } else if (mass) {
        if (lane == 63 - __clzll((long long)mass)) report(base + lastpos, wl);
    } else if (lane == 0) {
        report(-1, 0.f);
    }
}

// What the thread that finds the draft token does with it (see locate_batch's `report`); unit: the weight of 1 of the
// search in units of the row's sum S.
struct StoreDraftToken {
    static constexpr bool active = true;
    const DraftArgs &a;
    long long o;
    double unit, S;
    __device__ __forceinline__ void operator()(int tok, float w) const
    {
        a.token[o] = tok;
        if (a.q_tok) a.q_tok[o] = (float)((double)w * unit / S);
    }
};

// The flag as every wave of the row's workgroup sees it.  stop_out may be stop_in (a chain of steps uses one array), so no
// wave may store the row's new flag before all have read the old one: a wave that came late would take a row that stops
// at this step for one that had stopped before.  The barrier stands behind loads that all waves wait for anyway (us
// per step of bf16 logits in a graph, without / with: 8 rows of 128256 6.98 / 7.04, 64 rows 9.80 / 9.87, 256 rows of 151936
// 21.49 / 21.52).
__device__ __forceinline__ bool flag_for_all_waves(const DraftArgs &a, unsigned flag)
{
    const bool stopped = flag_after_loads(a, flag);
    __syncthreads();
    return stopped;
}

// A row already marked stopped: the two outputs every such row gets.
__device__ __forceinline__ void stopped_row(const DraftArgs &a, int b, long long o)
{
    if (threadIdx.x == 0) {
        a.token[o] = -1;
        a.stop[b] = 1;
    }
}

// Factor that brings a record with maximum m and sum S to the row maximum, and its log2 (0, 0 for an empty record).  Formed for
// empty records too and then dropped: with a branch around it the exponential waits for the sum and cannot run beside the
// merge's other chains.
__device__ __forceinline__ double record_factor(float m, double S, float mrow, const Scale &sc, double *xd)
{
    const double x = ((double)m - (double)mrow) * sc.c, f = exp2(x);
    const bool any = m != neg_inf() && S > 0.0;
    *xd = any ? x : 0.0;
    return any ? f : 0.0;
}

// A row's QUARTERS records, RPL consecutive ones per lane; `at` is the index of its first record.
template <int RPL>
struct QuarterRow {
    float m[RPL];
    double t[RPL], S4[RPL][4];
    float mrow;                          // after merge(): row maximum, factors and masses relative to it
    double f[RPL], xd[RPL], rS[RPL], M;
    // PUBLISHED: by workgroups of this launch
    template <bool PUBLISHED = false>
    __device__ __forceinline__ void load(const DraftArgs &a, size_t at)
    {
        const int lane = threadIdx.x & 63, nrec = a.geo.ns;
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            m[i] = neg_inf();
            t[i] = 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) S4[i][q] = 0.0;
            if (lane * RPL + i < nrec) {
                const QuarterRec *p = static_cast<const QuarterRec *>(a.part) + at + lane * RPL + i;
                if (PUBLISHED) {
                    const double *w = reinterpret_cast<const double *>(p);
#pragma unroll
                    for (int q = 0; q < 4; ++q) S4[i][q] = fetch_f64(w + q);
                    t[i] = fetch_f64(w + 4);
                    m[i] = __int_as_float(__double2loint(fetch_f64(w + 5)));
                } else {
                    m[i] = p->m;
                    t[i] = p->t;
#pragma unroll
                    for (int q = 0; q < 4; ++q) S4[i][q] = p->S[q];
                }
            }
        }
    }
    __device__ __forceinline__ void merge(const DraftArgs &a)
    {
        mrow = m[0];
#pragma unroll
        for (int i = 1; i < RPL; ++i) mrow = vmax(mrow, m[i]);
        mrow = wave_max(mrow);
        M = 0.0;
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            rS[i] = (S4[i][0] + S4[i][1]) + (S4[i][2] + S4[i][3]);
            f[i] = record_factor(m[i], rS[i], mrow, a.sc, &xd[i]);
            M += f[i] * rS[i];
        }
    }
    __device__ __forceinline__ double entropy_sum() const
    {
        double tt = 0.0;
#pragma unroll
        for (int i = 0; i < RPL; ++i) tt += f[i] * (t[i] + xd[i] * rS[i]);
        return wave_sum(tt);
    }
    // The token for the uniform u: lane, record and chunk from the masses (all in units of the row maximum), then the
    // search inside the chunk.
    template <typename DT>
    __device__ __forceinline__ void find_token(const DraftArgs &a, const DT *row, float u, long long o) const
    {
        const double incl = wave_inclusive_sum(M);
        const double S = read_lane(incl, 63);
        double target;
        const int at = pick_slice(M, (double)u * S, incl, &target);
        double G[4], frec = read_lane(f[0], at), Mrec = read_lane(f[0] * rS[0], at);
        float mrec = read_lane(m[0], at);
        int rec = at * RPL;
#pragma unroll
        for (int q = 0; q < 4; ++q) G[q] = read_lane(f[0] * S4[0][q], at);
#pragma unroll
        for (int i = 1; i < RPL; ++i) {               // a later one of the lane's records
            const double Mi = read_lane(f[i] * rS[i], at);
            if (Mi > 0.0 && !(Mrec > target)) {
                target -= Mrec;
                Mrec = Mi;
                frec = read_lane(f[i], at);
                mrec = read_lane(m[i], at);
                rec = at * RPL + i;
#pragma unroll
                for (int q = 0; q < 4; ++q) G[q] = read_lane(f[i] * S4[i][q], at);
            }
        }
        double in_chunk;
        const int chunk = rec * 4 + pick_piece(G, target, &in_chunk);
        // inside the chunk in units of the record's own maximum, as k_draft_stats formed the weights; the division runs
        // while the chunk is on its way
        in_chunk = frec > 0.0 ? in_chunk / frec : 0.0;
        // a record without mass is only picked where the row has none (a logit of +inf): nothing there has a weight then
        mrec = frec > 0.0 ? mrec : -neg_inf();
        search_chunk<DT>(row, a.geo.V, chunk, mrec, a.sc, in_chunk, StoreDraftToken{a, o, frec, S});
    }
};

// QUARTERS, grid (rows): two waves that share nothing but the flag's barrier; each loads and merges the records for
// itself, RPL consecutive records per lane.  Wave 1 writes entropy, logsumexp and stop flag (an fp64 logarithm and a square
// root), wave 0 finds the token.
constexpr int QUARTER_FINISH_THREADS = 128;
template <typename DT, int RPL>
__global__ __launch_bounds__(QUARTER_FINISH_THREADS) void k_draft_finish_quarters(DraftArgs a)
{
    const int b = blockIdx.x, lane = threadIdx.x & 63;
    const long long o = (long long)b * a.io_stride;
    asm volatile("" : : "s"(a.logits), "s"(a.row_stride), "s"(a.pos), "s"(a.stop_in), "s"(a.geo.V), "s"(a.part), "s"(a.sc.c),
                 "s"(a.sc.c_dn), "s"(a.sc.c_up), "s"(a.u), "s"(a.token), "s"(a.q_tok));       // requested at once
    // independent loads first: the row's flag, its uniform and its records travel together
    const unsigned flag = request_stop_flag(a, b);
    QuarterRow<RPL> r;
    r.load(a, (size_t)b * a.geo.ns);
    const float u = a.u[o];
    if (flag_for_all_waves(a, flag)) return stopped_row(a, b, o);
    r.merge(a);
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 1) {
        const double tt = r.entropy_sum(), S = wave_sum(r.M);
        if (lane == 0) write_row_outputs(a, b, o, r.mrow, S, tt);
        return;
    }
    r.template find_token<DT>(a, static_cast<const DT *>(a.logits) + draft_row_offset(a, b, a.step_j), u, o);
}

// A row's GREEDY records, RPL consecutive ones per lane; `at` is the index of its first record.
template <int RPL>
struct GreedyRow {
    WaveRec p[RPL];
    float mrow;                          // after merge(): row maximum, sums, token (uniform)
    double S, tt;
    int tok;
    template <bool PUBLISHED = false>
    __device__ __forceinline__ void load(const DraftArgs &a, size_t at)
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            p[i].m = neg_inf();
            p[i].idx = -1;
            p[i].S = 0.0;
            p[i].t = 0.0;
            if (lane * RPL + i < a.geo.ns) {
                const WaveRec *from = static_cast<const WaveRec *>(a.part) + at + lane * RPL + i;
                if (PUBLISHED) {
                    p[i].S = fetch_f64(&from->S);
                    p[i].t = fetch_f64(&from->t);
                    const double mi = fetch_f64(reinterpret_cast<const double *>(&from->m));
                    p[i].m = __int_as_float(__double2loint(mi));
                    p[i].idx = __double2hiint(mi);
                } else {
                    p[i] = *from;
                }
            }
        }
    }
    __device__ __forceinline__ void merge(const DraftArgs &a)
    {
        mrow = p[0].m;
#pragma unroll
        for (int i = 1; i < RPL; ++i) mrow = vmax(mrow, p[i].m);
        mrow = wave_max(mrow);
        S = tt = 0.0;
        int mine = -1;                                        // records are in index order: the first at the row maximum
#pragma unroll
        for (int i = RPL - 1; i >= 0; --i) {
            double xd;
            const double f = record_factor(p[i].m, p[i].S, mrow, a.sc, &xd);
            S += f * p[i].S;
            tt += f * (p[i].t + xd * p[i].S);
            if (p[i].m == mrow && p[i].idx >= 0) mine = p[i].idx;
        }
        S = wave_sum(S);
        tt = wave_sum(tt);
        const unsigned long long at_max = __ballot(mine >= 0);
        tok = at_max ? read_lane(mine, __ffsll((long long)at_max) - 1) : -1;
    }
};

// GREEDY, grid (rows), one wave, RPL consecutive records per lane.
template <int RPL>
__global__ __launch_bounds__(64) void k_draft_finish_greedy(DraftArgs a)
{
    const int b = blockIdx.x;
    const long long o = (long long)b * a.io_stride;
    const unsigned flag = request_stop_flag(a, b);        // travels together with the records
    GreedyRow<RPL> r;
    r.load(a, (size_t)b * a.geo.ns);
    if (flag_after_loads(a, flag)) return stopped_row(a, b, o);
    r.merge(a);
    if (threadIdx.x == 0) {
        a.token[o] = r.tok;
        if (a.q_tok) a.q_tok[o] = (float)(1.0 / r.S);     // the maximum has weight exp2(0) = 1
        write_row_outputs(a, b, o, r.mrow, r.S, r.tt);
    }
}

// The whole step in one launch: grid (rows rounded up to whole rounds of the XCDs * workgroups per row), one wave per record of one
// tile; the workgroup that is last to publish its records (exchange.h) merges them.  What bounds it is one chain: of a
// step of 16 rows of 32000 fp32 logits, 10600 cycles in all, the tile and its statistics take 4200, the stores 700, the ticket 1000, the
// fetch of the records 2000, merge and chunk 1400, the search 1200.  Entropy, logsumexp and stop test (1400) are a second wave's,
// beside the search: behind the chunk's request in the same wave they lengthened the step by 0.5 us.  (The records fetched as they lie,
// 64 words at a time, and dealt out through LDS: no faster, 5.95 us for 5.86.)
template <typename DT, RecordKind KIND, int RPL>
__global__ __launch_bounds__(WG, 4) void k_draft_step(DraftArgs a)
{
    static_assert(KIND != TOTAL, "records of one tile");
    asm volatile("" : : "s"(a.logits), "s"(a.row_stride), "s"(a.pos), "s"(a.cap), "s"(a.stop_in), "s"(a.geo.V), "s"(a.part),
                 "s"(a.sc.c_dn), "s"(a.sc.c_up), "s"(a.sc.c), "s"(a.common_range), "s"(a.step_j));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, nrec = a.geo.ns;
    const unsigned xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3;           // div = workgroups per row
    const unsigned q = a.div == 1u ? slot : __umulhi(slot, a.div_magic), s = slot - q * a.div;
    const int b = (int)(q * 8u + xcd), r = (int)s * NWAVE + wave;
    if (b >= a.B) return;
    const long long o = (long long)b * a.io_stride;
    const DT *row = static_cast<const DT *>(a.logits) + step_row_offset(a, b);
    const unsigned flag = request_stop_flag(a, b);
    const float u = KIND == QUARTERS ? a.u[o] : 0.f;
    const size_t first = (size_t)b * nrec;
    bool stopped;
    if (r < nrec) stopped = tile_record<DT, KIND, true>(a, row, r, first + r, [&] { return flag_after_loads(a, flag); });
    else stopped = flag_after_loads(a, flag);
    if (stopped) {
        if (s == 0) stopped_row(a, b, o);
        return;
    }
    stores_done();
    __syncthreads();
    if (wave > (KIND == QUARTERS ? 1 : 0)) return;
    // Waves 0 and 1 draw their tickets from counters of their own: they need not hear from one another, and the row's last
    // ones may be of different workgroups.
    unsigned *counter = ticket(a.tickets, b, TICKET_DRAFT + wave), t = 0u;
    if (lane == 0) t = take_ticket(counter);
    if ((unsigned)__builtin_amdgcn_readfirstlane((int)t) != a.div - 1u) return;
    // all of the row's waves have read its flag, and stored their records
    if (lane == 0) reset_tickets(counter);
    if constexpr (KIND == QUARTERS) {
        QuarterRow<RPL> rec;
        rec.template load<true>(a, first);
        rec.merge(a);
        if (wave == 1) {
            const double tt = rec.entropy_sum(), S = wave_sum(rec.M);
            if (lane == 0) write_row_outputs(a, b, o, rec.mrow, S, tt);
        } else {
            rec.template find_token<DT>(a, row, u, o);
        }
    } else {
        GreedyRow<RPL> rec;
        rec.template load<true>(a, first);
        rec.merge(a);
        if (lane == 0) {
            a.token[o] = rec.tok;
            if (a.q_tok) a.q_tok[o] = (float)(1.0 / rec.S);
            write_row_outputs(a, b, o, rec.mrow, rec.S, rec.tt);
        }
    }
}

// TOTAL, grid (rows), a record per lane.  Every wave loads and merges the records for itself: the waves then agree on
// the record to search without passing anything through LDS or waiting for one another.
// Waves 0 .. 3 search for the token; the extra wave writes entropy, logsumexp and stop flag and ends, so that
// work (an fp64 logarithm and a square root, 0.3 us) neither sits in front of the search nor holds up its barriers.
constexpr int TOTAL_FINISH_THREADS = WG + 64;
template <typename DT>
__global__ __launch_bounds__(TOTAL_FINISH_THREADS, 4) void k_draft_finish_total(DraftArgs a)
{
    constexpr int N = VecOf<DT>::N;
    __shared__ LocateLds loc;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, nrec = a.geo.ns;
    const long long o = (long long)b * a.io_stride;
    // independent loads first: the row's flag, its uniform and its records travel together
    const unsigned flag = request_stop_flag(a, b);
    WaveRec p;
    p.m = neg_inf();
    p.S = 0.0;
    p.t = 0.0;
    if (lane < nrec) p = static_cast<const WaveRec *>(a.part)[(size_t)b * nrec + lane];
    const float u = a.u[o];
    if (flag_for_all_waves(a, flag)) return stopped_row(a, b, o);
    const DT *row = static_cast<const DT *>(a.logits) + draft_row_offset(a, b, a.step_j);
    // everything relative to the row maximum: this lane's record by the factor f
    const float mrow = wave_max(p.m);
    double xd;
    const double f = record_factor(p.m, p.S, mrow, a.sc, &xd);
    const double M = f * p.S;
    const double incl = wave_inclusive_sum(M);
    const double S = read_lane(incl, 63);
    const double tt = wave_sum(f * (p.t + xd * p.S));
    // the extra wave: the outputs that do not depend on the token.  The test is on a scalar register, so the wave
    // branches to the end of the program and is gone before the search's first barrier.
    if (__builtin_amdgcn_readfirstlane(tid >> 6) == NWAVE) {
        if (lane == 0) write_row_outputs(a, b, o, mrow, S, tt);
        return;
    }
    double target;
    const int rec = pick_slice(M, (double)u * S, incl, &target);
    SoftmaxWeights<DT> wf{row, a.geo.V, make_exp_ref(a.sc, (double)mrow * a.sc.c)};
    // the thread that finds the token stores it; nothing else in this kernel has used the search's LDS
    const StoreDraftToken store{a, o, 1.0, S};
    float wtok;
    const int tb = rec * a.geo.tps, te = min(tb + a.geo.tps, a.geo.ntiles);
    // a record of one tile is searched as one batch of one tile, longer records two tiles at a time
    if (a.geo.tps == 1) locate_in_slice<N, 1>(wf, tb, te, target, loc, &wtok, NoHook(), true, store);
    else locate_in_slice<N, 2>(wf, tb, te, target, loc, &wtok, NoHook(), true, store);
}

}  // namespace svip
