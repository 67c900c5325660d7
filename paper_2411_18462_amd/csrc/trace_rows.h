// Which rows of a sequence's trace the decoding loop's kernels read: plain arithmetic on a sequence's state, which a host compiler takes
// as well, so that the bounds can be checked without a GPU.
#pragma once
#ifdef __HIPCC__
#define SVIP_ROW_RULE __host__ __device__ __forceinline__
#else
#define SVIP_ROW_RULE static inline
#endif

namespace svip {

// The row, counted from the sequence's position, that a draft step requests before it has looked at the stop flag.  A sequence that still
// drafts has step_j < cap, and its row is step_j.  One that has stopped keeps its position while the others of its batch go on to later
// steps, and its trace may end with row cap: it requests its last draft row again, which no result depends on.
SVIP_ROW_RULE int step_row(int step_j, int cap)
{
    const int last = cap > 1 ? cap - 1 : 0;
    return step_j < last ? step_j : last;
}

// Draft rows that a launch of the greedy stream reads of a running sequence whose round began at `pos` with limit `cap` and of which
// `drafted` are known (negative: nothing, not even the first target row): up to where all tokens are there, and `ahead` more for the round
// that gets there last; behind that the unfinished draft, as many rows again as are known of it.  No further than the last row that a
// round of the sequence can reach, and target row n behind draft rows 0 .. n - 1 is the last one of the trace at most.  At least 1,
// whatever the call asks for, as drafted < cap: a call may ask for fewer tokens than a sequence has already, which then goes through
// one more round.  max_new and L: of this call; start: where the sequence began.
SVIP_ROW_RULE int stream_rows(int pos, int drafted, int cap, int start, int L, int gamma_max, int max_new, int ahead, int group)
{
    const int known = drafted > 0 ? drafted : 0;                                         // relative to pos, as all below
    const long long all = (long long)start + max_new, end = (long long)L + gamma_max;
    const int goal = (int)(all < end ? all : end) - pos;
    int n = goal + ahead - known;
    if (known >= goal) {
        n = ahead > known ? ahead : known;
        if (n > cap - known) n = cap - known;
    }
    int most = (L - pos < goal + gamma_max ? L - pos : goal + gamma_max) - 1;
    if (most < cap) most = cap;                                                          // the round at hand
    if (n > most - known) n = most - known;
    return n < group ? n : group;
}

}  // namespace svip
