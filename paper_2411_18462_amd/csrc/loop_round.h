// What a round of the decoding loop does with one sequence before and after its kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/svip.h"
#include "svip_internal.h"

namespace svip {

// A sequence starts another round while it has produced fewer than max_new tokens and the trace
// still holds cap + 1 rows from its position on (Algorithm 1's loop condition, plus the end of
// the synthetic trace).
__device__ __forceinline__ bool finished(int pos, int n0, int cap, int L, int max_new)
{
    return pos - n0 >= max_new || pos + cap + 1 > L;
}

// What the kernels of sequence b's next round read.
__device__ __forceinline__ void begin_sequence(const RoundBuffers &rb, int b, int pos, int cap, int done)
{
    rb.pos[b] = done ? 0 : pos;
    rb.cap[b] = done ? 1 : cap;
    rb.stop[b] = done ? 1 : 0;
    rb.done[b] = done ? 1 : 0;
    rb.draft_len[b] = 0;
}

// The limit of the round behind one that accepted all of its draft, or did not.
__device__ __forceinline__ int next_cap(const LoopArgs &a, int cap, bool all_accepted)
{
    const int c = cap + (all_accepted ? a.inc : -a.dec);
    return c < 1 ? 1 : (c > a.gamma_max ? a.gamma_max : c);
}

// A round's entry in the log.
__device__ __forceinline__ void log_round(const LoopArgs &a, int b, int round, int pos, int cap, int g, int na)
{
    if (!a.round_log) return;
    int *lg = a.round_log + ((size_t)round * a.B + b) * 4;
    lg[0] = pos;
    lg[1] = cap;
    lg[2] = g;
    lg[3] = na;
}

// Bookkeeping of round `round` for sequence b, which accepted `na` of its g drafted tokens and got `next` behind
// them, and the beginning of its next round.  Returns whether the sequence goes on.
__device__ __forceinline__ bool end_sequence(const LoopArgs &a, int b, int round, int g, int na, int next, const int *tokens)
{
    int *st = a.state + (size_t)b * SVIP_LOOP_NSTATE;
    const int pos = st[0], cap = st[1], start = st[7];
    int *o = a.out_tokens + (size_t)b * a.out_stride + st[6];
    for (int j = 0; j < na; ++j) o[j] = tokens[j];
    o[na] = next;
    log_round(a, b, round, pos, cap, g, na);
    const int ncap = next_cap(a, cap, na == g);
    const int npos = pos + na + 1;
    const int done = finished(npos, start, ncap, a.L, a.max_new) ? 1 : 0;
    st[0] = npos;
    st[1] = ncap;
    st[2] = done;
    st[3] += 1;
    st[4] += g;
    st[5] += na;
    st[6] += na + 1;
    begin_sequence(a.rb, b, npos, ncap, done);
    return !done;
}

// Its entry in the log of a round after a sequence's last one.
__device__ __forceinline__ void log_idle(const LoopArgs &a, int b, int round) { log_round(a, b, round, -1, -1, -1, -1); }

// The message (ticket, value) as one word.
__device__ __forceinline__ void post(const Mail &m, int value)
{
    __hip_atomic_store(m.word, ((unsigned long long)m.ticket << 32) | (unsigned)value, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace svip
