// Kernels of svip_verify (Algorithm 2 Verify, Algorithm 4 Correct, the bonus sample of Algorithm 1).
#pragma once
#include <type_traits>

#include "exchange.h"
#include "kernel_args.h"
#include "sample_weights.h"

namespace svip {

// ---- verify: statistics ------------------------------------------------------------------------

// Statistics rows of sequence b are numbered jj = 0 .. kd + k: first the kd draft rows (only
// when the draft logsumexps are recomputed), then the k + 1 target rows.  Slice s of row jj is at stat_at: a sequence's
// rows lie side by side, as the lanes of the wave that merges them do.
__device__ __forceinline__ size_t stat_at(const VerifyArgs &a, int b, int jj, int s)
{
    return ((size_t)b * a.geo.ns + s) * (a.kd + a.k + 1) + jj;
}

// grid (sequences * rows per sequence * slices).  Draft rows are needed for j < draft_len[b],
// target rows for j <= draft_len[b]; workgroups of other rows exit at once.  (Handing the acceptance
// test to the workgroup that finishes a sequence last was measured and dropped here: the wait for the
// acknowledged stores and the ticket adds about 1 us to every workgroup of a kernel whose workgroups
// live about 5 us, and the pass went from 47 us to 63 us.)
template <typename DT>
__global__ __launch_bounds__(WG, 8) void k_verify_stats(VerifyArgs a)
{
    __shared__ CombineLds lds;
    const int rps = a.kd + a.k + 1;
    // one item = one slice of one statistics row; a workgroup takes items blockIdx, blockIdx + grid, ...
    // (the grid covers all items unless the launch asks for fewer, longer-lived workgroups)
    for (long long item = blockIdx.x; item < a.stat_items; item += gridDim.x) {
        const int y = (int)(item / a.geo.ns), s = (int)(item - (long long)y * a.geo.ns);
        const int b = y / rps, jj = y - b * rps;
        if (a.skip && a.skip[b]) continue;
        const int g = clamp_len(a.draft_len[b], a.k);
        const DT *row;
        if (jj < a.kd) {
            if (jj >= g) continue;
            row = static_cast<const DT *>(a.draft) + row_offset(a, a.seq_d, b, jj);
        } else {
            const int j = jj - a.kd;
            if (j >= g + a.bonus) continue;
            row = static_cast<const DT *>(a.target) + row_offset(a, a.seq_t, b, j);
        }
        int tb = s * a.geo.tps, n = a.geo.tps;
        if (a.first_half) {                          // halves of longer slices
            const int half = s & 1;
            tb = (s >> 1) * a.geo.tps + half * a.first_half;
            n = half ? a.geo.tps - a.first_half : a.first_half;
        }
        const int te = min(tb + n, a.geo.ntiles);
        // the LDS block can be reused at once: every wave has read the maxima before the second barrier of
        // slice_lse, and thread 0 has read the sums before its wave reaches the next item's first barrier
        const LsePart p = slice_lse<DT>(row, a.geo.V, tb, te, a.sc, a.m0, lds);
        if (threadIdx.x == 0) static_cast<LsePart *>(a.ws.part)[stat_at(a, b, jj, s)] = p;
    }
}

// ---- verify: acceptance test and first rejection -------------------------------------------

// The logsumexp of statistics row jj of sequence b from its slices: the sums are brought to the largest
// reference with single-precision exp2 of the (small, exactly formed) reference differences and added in fp64.  CH slices
// are requested together, the first of them (request) before the caller's other loads are waited for.  A slice with a logit of +inf or
// NaN has no sum and does not count.  PARTS: where a row of its length has longer slices (finer_stats in svip_kernels.hip), consecutive
// slices that such a logit takes with it: 2, or 4 for all of a row of at most four.  (Instances of their own: the tests cost
// other calls 0.1 to 0.2 us.)
template <int CH, int PARTS>
struct RowStats {
    float r = neg_inf();
    double S = 0.0;
    LsePart p[CH];
    __device__ __forceinline__ void request(const VerifyArgs &a, int b, int jj, int s0 = 0)
    {
#pragma unroll
        for (int u = 0; u < CH; ++u)
            p[u] = static_cast<const LsePart *>(a.ws.part)[stat_at(a, b, jj, s0 + u < a.geo.ns ? s0 + u : s0)];
    }
    __device__ __forceinline__ void add(int n)
    {
        if (PARTS == 2) {
#pragma unroll
            for (int u = 0; u + 1 < CH; u += 2)
                if (!(p[u].S + p[u + 1].S > 0.0)) p[u].S = p[u + 1].S = 0.0;         // (either may be no number)
        }
        if constexpr (PARTS == 4) {
            static_assert(CH == 4, "all of the row");
            if (!((p[0].S + p[1].S) + (p[2].S + p[3].S) > 0.0)) p[0].S = p[1].S = p[2].S = p[3].S = 0.0;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u)            // after all of the loads (else each is waited for in turn)
            if (!(u < n) || !(p[u].S > 0.0)) {
                p[u].m = neg_inf();
                p[u].S = 0.0;
            }
        float rc = p[0].m;
#pragma unroll
        for (int u = 1; u < CH; ++u) rc = vmax(rc, p[u].m);
        if (rc == neg_inf()) return;
        if (rc > r) {
            if (r != neg_inf()) S *= (double)exp2_raw((float)((double)r - (double)rc));
            r = rc;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u)
            if (p[u].m != neg_inf()) S += p[u].S * (double)exp2_raw((float)((double)p[u].m - (double)r));
    }
    // what request() fetched, then the rest of the row
    __device__ __forceinline__ void merge(const VerifyArgs &a, int b, int jj)
    {
        add(a.geo.ns);
        for (int s0 = CH; s0 < a.geo.ns; s0 += CH) {
            request(a, b, jj, s0);
            add(a.geo.ns - s0);
        }
    }
    __device__ __forceinline__ double L() const { return (double)r + log2(S); }      // logsumexp * log2(e)
};
// What the acceptance test of a sequence gives: what the draw needs (uniform over the wave), and what the call reports.
struct Accepted {
    double Lp, Lq;      // logsumexp * log2(e) of target row r, and of draft row r if that was rejected
    int r;              // target row to draw from: the first rejection, or the draft length for a bonus
    bool resid;         // residual of row r, or the bonus row
    float prob;         // not PASSES: accept probability of position `lane`, -1 from the draft length on
    unsigned flags;     // bad device data met on the way (per lane)
};

// Slices of a row requested together.  us per call, 4 / 8 / 10 of them: 64 sequences of 16 positions and 128256 bf16 logits (7
// slices) 58.8 / 59.6 / 60.0, 32 of 8 and 50257 fp16 (3 slices) 24.2 / 24.9 / 25.6.
constexpr int ACCEPT_SLICES = 4;

// Drafts of at most this many positions have a lane for each (and one more pass for the bonus row behind 64 accepted ones).
constexpr int LANE_POSITIONS = 64;

// The acceptance test of sequence b by one wave: lane = position, 64 positions per pass.  Lanes j <= draft_len merge the
// statistics of target row j; lanes j < draft_len run the acceptance test; a ballot finds the first rejection.
// PASSES: drafts of any length; goes on behind the pass of the first rejection only if the accept probabilities are wanted, and
// writes them.  Otherwise (k <= LANE_POSITIONS) nothing is written.
template <typename DT, bool PASSES, int PARTS>
__device__ __forceinline__ Accepted accept_sequence(const VerifyArgs &a, int b, int lane)
{
    // One wave, a chain of trips to memory: the draft length, then tokens / uniforms / logsumexps / slice
    // statistics, then the two gathered logits.  The first pass's loads that need no draft length (everything
    // indexed by position j < k) are requested together with it, and the gathers before the slice statistics
    // are merged, so a sequence takes three trips instead of five.
    int graw = a.draft_len[b];
    int x0 = 0;
    float u0 = 0.f;
    double lse0 = 0.0;
    if (lane < a.k) {
        x0 = a.tokens[(size_t)b * a.k + lane];
        u0 = a.u_accept[(size_t)b * a.k + lane];
        if (a.draft_lse) lse0 = a.draft_lse[(size_t)b * a.k + lane];
    }
    asm volatile("" : "+v"(graw) : : "memory");     // the draft length is first looked at here
    const int g = clamp_len(graw, a.k);
    const DT *tgt = static_cast<const DT *>(a.target) + row_offset(a, a.seq_t, b, 0);
    const DT *drf = static_cast<const DT *>(a.draft) + row_offset(a, a.seq_d, b, 0);
    constexpr double LOG2E = 1.4426950408889634;
    Accepted res;
    res.r = -1;                 // first rejection, once known
    res.Lp = res.Lq = 0.0;
    res.prob = 0.f;
    res.flags = graw != g ? (unsigned)SVIP_FLAG_BAD_DRAFT_LEN : 0u;
    for (int j0 = 0; j0 <= g && (res.r < 0 || (PASSES && a.accept_prob)); j0 += 64) {
        const int j = j0 + lane;
        bool reject = false;
        double Lp = 0.0, Lq = 0.0;
        if (j <= g) {
            int x = x0;
            double u = (double)u0, lse_q = lse0;
            if (PASSES && j0 > 0 && j < g) {
                x = a.tokens[(size_t)b * a.k + j];
                u = (double)a.u_accept[(size_t)b * a.k + j];
                if (a.draft_lse) lse_q = a.draft_lse[(size_t)b * a.k + j];
            }
            DT zp_stored = DT(), zq_stored = DT();          // requested here, widened after the statistics are merged
            if (j < g) {
                if (x < 0 || x >= a.geo.V) {
                    res.flags |= (unsigned)SVIP_FLAG_BAD_TOKEN;
                    x = x < 0 ? 0 : a.geo.V - 1;
                }
                zp_stored = (tgt + (long long)j * a.row_stride)[x];
                zq_stored = (drf + (long long)j * a.row_stride)[x];
            }
            RowStats<ACCEPT_SLICES, PARTS> target, draft;
            target.request(a, b, a.kd + j);
            if (a.kd && j < g) draft.request(a, b, j);
            target.merge(a, b, a.kd + j);
            Lp = target.L();
            if (j < g) {
                if (a.kd) {
                    draft.merge(a, b, j);
                    Lq = draft.L();
                } else {
                    Lq = lse_q * LOG2E;
                }
                const double zp = (double)widen(not_before_here(zp_stored)), zq = (double)widen(not_before_here(zq_stored));
                const double p = exp2(zp * a.sc.c - Lp);
                const double q = exp2(zq * a.sc.c - Lq);
                reject = !(u * q < p);
                const double ratio = q > 0.0 ? p / q : (p > 0.0 ? 1.0 : 0.0);
                const float prob = (float)(ratio < 1.0 ? ratio : 1.0);
                if (!PASSES) res.prob = prob;
                else if (a.accept_prob) a.accept_prob[(size_t)b * a.k + j] = prob;
            }
        }
        if (res.r < 0) {
            const unsigned long long rej = __ballot(reject);
            if (rej) {
                const int first = __ffsll((long long)rej) - 1;
                res.r = j0 + first;
                res.Lp = read_lane(Lp, first);
                res.Lq = read_lane(Lq, first);
            } else if (g - j0 < 64) {      // row g (the bonus row) was merged in this pass
                res.r = g;
                res.Lp = read_lane(Lp, g - j0);
            }
        }
    }
    res.resid = res.r < g;
    if (lane >= g) res.prob = -1.f;          // nothing to report there
    return res;
}

// grid (sequences), one wave: the acceptance test in a launch of its own (see accept_in_resid in svip_kernels.hip).
template <typename DT, int PARTS>
__global__ __launch_bounds__(64) void k_accept(VerifyArgs a)
{
    const int b = blockIdx.x, lane = threadIdx.x;
    if (a.skip && a.skip[b]) return;
    const Accepted acc = accept_sequence<DT, true, PARTS>(a, b, lane);
    if (acc.flags) atomicOr(a.ws.flags, acc.flags);
    if (lane == 0) {
        SeqRec rec;
        rec.Lp = acc.Lp;
        rec.Lq = acc.Lq;
        rec.r = acc.r;
        rec.resid = acc.resid ? 1 : 0;
        a.ws.rec[b] = rec;
        a.n_accepted[b] = acc.r;
    }
}

// ---- verify: residual / bonus sampling ------------------------------------------------------

// What a slice's workgroup hands to the sequence's last workgroup: the mass of each half of its tiles (two chunks; slices
// longer than TILE_MASSES tiles fold the rest into the last entries and are searched as a whole).
constexpr int SLICE_MASSES = 2 * TILE_MASSES;

// What the thread that finds the correction or bonus token does with it (see locate_batch's `report`).
struct StoreNextToken {
    static constexpr bool active = true;
    int *next_token;
    int b;
    __device__ __forceinline__ void operator()(int tok, float) const { next_token[b] = tok; }
};

// Weights of chunks [chunk, chunk + NU) of a row, one vector of each per lane: residual max(0, p - q), or p alone.
template <typename DT, int NU, bool RESID>
__device__ __forceinline__ void chunk_weights(const DT *prow, const DT *qrow, int V, int chunk, const ExpRef &ep, const ExpRef &eq,
                                              float (&w)[NU][VecOf<DT>::N])
{
    constexpr int N = VecOf<DT>::N;
    typename RawOf<DT>::type rp[NU], rq[NU];
    wave_load<DT, NU, true>(prow, V, chunk, rp);
    if (RESID) wave_load<DT, NU, true>(qrow, V, chunk, rq);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        float z[N];
        unpack<DT>(rp[u], z);
#pragma unroll
        for (int e = 0; e < N; ++e) w[u][e] = ep(z[e]);
        if (RESID) {
            unpack<DT>(rq[u], z);
#pragma unroll
            for (int e = 0; e < N; ++e) w[u][e] = fmaxf(w[u][e] - eq(z[e]), 0.f);
        }
    }
}

// Sum of the target weights p of chunks [chunk, chunk + NU) of a row, per lane.
template <typename DT, int NU>
__device__ __forceinline__ double target_mass(const DT *prow, int V, int chunk, const ExpRef &ep)
{
    constexpr int N = VecOf<DT>::N;
    double mass = 0.0;
    const auto add = [&](const typename RawOf<DT>::type &raw) {
        float w[N];
        unpack<DT>(raw, w);
#pragma unroll
        for (int e = 0; e < N; ++e) w[e] = ep(w[e]);
        mass += (double)tree_sum<N>(w);
        if constexpr (N == 8) asm volatile("" : "+v"(mass));        // one vector after the other, behind all of the loads
    };
    if ((chunk + NU) * 64 <= V / N) {
        typename RawOf<DT>::type raw[NU];
        wave_load<DT, NU, false>(prow, V, chunk, raw);         // all in flight together
#pragma unroll
        for (int u = 0; u < NU; ++u) add(raw[u]);
    } else {
#pragma unroll 1
        for (int u = 0; u < NU && (long long)(chunk + u) * 64 * N < V; ++u) {
            typename RawOf<DT>::type one[1];
            wave_load<DT, 1, true>(prow, V, chunk + u, one);
            add(one[0]);
        }
    }
    return mass;
}

// No residual mass (p <= q everywhere, up to rounding): the token is drawn from p instead, by one wave that walks the row in
// groups of chunks -- once for the masses, of which lane l keeps that of its share of the row, then through the share that holds
// the crossing.  It takes a rejection where p and q agree to the last bits, or draft logsumexps that are not the rows', so
// it may not cost the usual call anything: target masses summed beside the residual's, as a second number per slice, take
// 0.3 to 0.8 us of every call of 20 to 60.  us per call, 8 sequences of 151936 bf16 logits, one chunk / four / eight in flight:
// 244 / 78 / 66 (with mass 20); 8 of 32000 fp32 98 / 34 / 30; 64 of 128256 fp16, one / eight 358 / 87 (with mass 36).
template <typename DT, typename Report>
__device__ __forceinline__ void draw_from_target(const DT *prow, const Geo &geo, const ExpRef &ep, float u, Report report)
{
    constexpr int N = VecOf<DT>::N, GROUP = 8;
    const int lane = threadIdx.x & 63;
    const int groups = (geo.ntiles * (WG / 64) + GROUP - 1) / GROUP, share = (groups + 63) / 64;
    double mine = 0.0;
#pragma unroll 1
    for (int g = 0; g < groups; ++g) {
        const double mass = wave_sum(target_mass<DT, GROUP>(prow, geo.V, g * GROUP, ep));
        if (g / share == lane) mine += mass;
    }
    const double incl = wave_inclusive_sum(mine), total = read_lane(incl, 63);
    double target, before = 0.0, run = 0.0;
    const int first = pick_slice(mine, (double)u * total, incl, &target) * share * GROUP;
    int at = first;                              // the chunk that holds the crossing, else the last one with mass
#pragma unroll 1
    for (int c = first; c < first + share * GROUP && !(run > target); ++c) {
        const double mass = wave_sum(target_mass<DT, 1>(prow, geo.V, c, ep));
        if (mass > 0.0) {
            at = c;
            before = run;
        }
        run += mass;
    }
    float w[1][N];
    chunk_weights<DT, 1, false>(prow, prow, geo.V, at, ep, ep, w);
    search_chunks<N, 1>(w, at, target - before, report);
}

// Waves per SIMD the residual pass is compiled for: 6 where its registers allow (draw_from_target would otherwise take the
// common path's sixth wave with it); the bf16 draw without the test, and the forms for longer slices, need more than 80.
template <typename DT>
constexpr int resid_waves(bool tiles, bool test) { return tiles && (test || !std::is_same<DT, bf16>::value) ? 6 : 4; }

// grid (sequences * slices): the residual / bonus draw, and (TEST; k <= LANE_POSITIONS) the acceptance test before it.  One wave of
// every workgroup works out the first rejection from the statistics of the sequence's rows (a few kilobytes), or reads what
// k_accept has left; then the workgroup sums the weights of its slice by half tiles -- residual max(0, p - q) of the rejected
// position, or target p of the bonus row -- and publishes them; the workgroup that draws the sequence's final ticket picks the
// half tile that holds u * total, and one wave finds the token there by the inverse CDF and reports the test.  All workgroups
// of the sequence have read its inputs by then, so a sequence's outputs may lie on its own inputs (not on another sequence's).
// What bounds it is the chain of trips to memory (statistics, two rows, publish, ticket, masses, half tile).  us per call with
// the test in a launch of its own (one wave per sequence) and the search in a workgroup / so: 64 sequences of 16 positions and
// 128256 bf16 logits 61.0 / 58.9 (this kernel alone 13.3 + 4.7 / 14.6), 8 of 64 and 151936 28.7 / 27.3, 32 of 8 and 50257 fp16
// 26.5 / 24.6.  With every wave testing for itself instead of one for its workgroup: 60.5, 27.3, 25.8 -- the loads of the
// statistics are many and small.  TILES: slices have at most TILE_MASSES tiles; otherwise the search walks the chosen slice.
template <typename DT, bool TILES, bool TEST, int PARTS>
__global__ __launch_bounds__(WG, resid_waves<DT>(TILES, TEST)) void k_resid(VerifyArgs a)
{
    constexpr int N = VecOf<DT>::N;
    __shared__ double sums[NWAVE][TILE_MASSES];
    const int ns = a.geo_s.ns;
    // Workgroups go to the chip's 8 XCDs in turn: all slices of sequence b are kept on XCD b % 8, so the
    // workgroup that finishes the sequence reads the chosen tile again from the L2 that already streamed it
    // (13.2 -> 12.9 us at 64 sequences of 128K logits, 35 -> 33 us at 256).  The grid is ceil(B / 8) * 8 * ns.
    const unsigned xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3;
    const int b = (int)((slot / (unsigned)ns) * 8u + xcd), s = (int)(slot % (unsigned)ns), tid = threadIdx.x;
    if (b >= a.B) return;
    if (a.skip && a.skip[b]) return;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    Accepted acc;
    if constexpr (TEST) {
        __shared__ Accepted shared_acc;
        if (wave == 0) {
            acc = accept_sequence<DT, false, PARTS>(a, b, lane);
            if (lane == 0) shared_acc = acc;
        }
        __syncthreads();
        if (wave != 0) acc = shared_acc;
        acc.r = __builtin_amdgcn_readfirstlane(acc.r);
        acc.resid = __builtin_amdgcn_readfirstlane(acc.resid);
    } else {
        const SeqRec rec = a.ws.rec[b];
        acc.Lp = rec.Lp;
        acc.Lq = rec.Lq;
        acc.r = rec.r;
        acc.resid = rec.resid != 0;
    }
    const DT *prow = static_cast<const DT *>(a.target) + row_offset(a, a.seq_t, b, acc.r);
    const DT *qrow = static_cast<const DT *>(a.draft) + row_offset(a, a.seq_d, b, acc.r);
    const ExpRef ep = make_exp_ref(a.sc, acc.Lp), eq = make_exp_ref(a.sc, acc.Lq);
    double *slots = a.ws.mass + (size_t)b * ns * SLICE_MASSES;
    const int tb = s * a.geo_s.tps, te = min(tb + a.geo_s.tps, a.geo_s.ntiles);
    float M[TILE_MASSES] = {};
    if (acc.resid) slice_mass<DT, true>(prow, qrow, a.geo_s.V, tb, te, ep, eq, M);
    else slice_mass<DT, false>(prow, qrow, a.geo_s.V, tb, te, ep, eq, M);
    const double Md[TILE_MASSES] = {(double)M[0], (double)M[1], (double)M[2], (double)M[3]};
    const double mine = wave_sum4(Md);                     // lane v: that of tile v
    if (lane < TILE_MASSES) sums[wave][lane] = mine;
    __syncthreads();
    if (TILES && wave != 0) return;
    bool last = false;
    if (wave == 0) {
        const int tile = lane >> 1, half = lane & 1;       // entry `lane` of the slice
        if (lane < SLICE_MASSES) publish_f64(slots + s * SLICE_MASSES + lane, sums[2 * half][tile] + sums[2 * half + 1][tile]);
        stores_done();
        unsigned t = 0u;
        if (lane == 0) t = take_ticket(ticket(a.ws.tickets, b, TICKET_RESID));
        last = (unsigned)__builtin_amdgcn_readfirstlane((int)t) == (unsigned)ns - 1u;
        if (TILES && !last) return;
    }

    // ---- the sequence's last workgroup; lane = slice ----
    const StoreNextToken store{a.next_token, b};
    int slice = -1;
    double target = 0.0;
    if (last) {
        const float u = a.u_resample[b];
        unsigned long long x[SLICE_MASSES] = {};
        if (lane < ns) {
#pragma unroll
            for (int v = 0; v < SLICE_MASSES; ++v) x[v] = fetch_u64(slots + lane * SLICE_MASSES + v);     // all in flight together
        }
        if (lane == 0) reset_tickets(ticket(a.ws.tickets, b, TICKET_RESID));
        double G[SLICE_MASSES], mass = 0.0;
#pragma unroll
        for (int v = 0; v < SLICE_MASSES; ++v) {
            G[v] = __longlong_as_double((long long)x[v]);
            mass += G[v];
        }
        const double incl = wave_inclusive_sum(mass), total = read_lane(incl, 63);
        if (acc.resid && !(total > 0.0)) {
            draw_from_target<DT>(prow, a.geo_s, ep, u, store);
        } else {
            slice = pick_slice(mass, (double)u * total, incl, &target);
            if (TILES) {
                double Gs[SLICE_MASSES], in_half;
#pragma unroll
                for (int v = 0; v < SLICE_MASSES; ++v) Gs[v] = read_lane(G[v], slice);
                const int chunk = (slice * a.geo_s.tps * 2 + pick_piece(Gs, target, &in_half)) * (WG / 128);
                float w[2][N];
                if (acc.resid) chunk_weights<DT, 2, true>(prow, qrow, a.geo_s.V, chunk, ep, eq, w);
                else chunk_weights<DT, 2, false>(prow, qrow, a.geo_s.V, chunk, ep, eq, w);
                search_chunks<N, 2>(w, chunk, in_half, store);
            }
        }
        if constexpr (TEST) {
            if (acc.flags) atomicOr(a.ws.flags, acc.flags);
            if (a.accept_prob && acc.prob >= 0.f) a.accept_prob[(size_t)b * a.k + lane] = acc.prob;
            if (lane == 0) a.n_accepted[b] = acc.r;
        }
    }
    if constexpr (!TILES) {
        __shared__ LocateLds loc;
        __shared__ double at_target;
        __shared__ int at_slice;
        if (tid == 0) {
            at_slice = slice;
            at_target = target;
        }
        __syncthreads();
        if (at_slice < 0) return;                          // not the last workgroup, or all done
        const int fb = at_slice * a.geo_s.tps, fe = min(fb + a.geo_s.tps, a.geo_s.ntiles);
        float wtok;
        if (acc.resid) {
            ResidualWeights<DT> wf{prow, qrow, a.geo_s.V, ep, eq};
            locate_in_slice<N, 2>(wf, fb, fe, at_target, loc, &wtok, NoHook(), true, store);
        } else {
            SoftmaxWeights<DT> wf{prow, a.geo_s.V, ep};
            locate_in_slice<N, 2>(wf, fb, fe, at_target, loc, &wtok, NoHook(), true, store);
        }
    }
}

}  // namespace svip
