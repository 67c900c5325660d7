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

}  // namespace svip
