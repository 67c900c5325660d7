// Workspace layout and kernel argument blocks shared by the kernels of libsvip.so.
#pragma once
#include "../../include/svip.h"
#include "row_math.h"

namespace svip {

// ---- workspace layout ----------------------------------------------------------------

struct SeqRec {          // what an acceptance test in a launch of its own hands to the residual pass, one per sequence
    double Lp;           // logsumexp(target row r) * log2(e)
    double Lq;           // logsumexp(draft row r) * log2(e) (residual mode only)
    int r;               // target row to sample from (first rejection, or draft_len for a bonus)
    int resid;           // 1: residual of row r, 0: bonus from row r
};

struct Workspace {
    unsigned *flags;     // sticky device-data flags
    unsigned *tickets;   // END of the ticket counters (see ticket()): they grow downwards from here
    SeqRec *rec;         // [B]
    double *mass;        // [B][slices of the residual pass] masses of half tiles, verification only
    void *part;          // slice statistics (LsePart, though sizes count sizeof(Partial) each), keys or records of the call
};

constexpr int MAX_BATCH = 1 << 20;               // sequences per call (grids are one-dimensional)
constexpr size_t HEADER_BYTES = 256;
#ifndef SVIP_TICKET_STRIDE
#define SVIP_TICKET_STRIDE 16
#endif
constexpr int TICKETS_PER_ROW = SVIP_TICKET_STRIDE;   // words between the counters of consecutive rows
__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static size_t ws_rec_bytes(int B) { return align256((size_t)B * sizeof(SeqRec)); }
static size_t ws_mass_bytes(int B, int slices) { return align256((size_t)B * slices * 2 * TILE_MASSES * sizeof(double)); }
static size_t ws_ticket_bytes(int B) { return align256((size_t)B * TICKETS_PER_ROW * sizeof(unsigned)); }

// Layout: flag word | records | slice masses | slice statistics ...            ... ticket counters.
// The counters sit at the END of the workspace (the given size rounded down to 256 bytes) and counter
// t of row b lies TICKETS_PER_ROW * b + t + 1 words below that end, whatever the batch size of the call.  Every call checks
// front + its own counters <= size, so its regions at the front leave the counters of as many rows alone as it has itself, and they
// keep the zeros that svip_workspace_reset wrote and that every kernel restores.  The counters of a larger batch a call may overwrite
// where the workspace holds little more than what that call needs.  With svip_workspace_bytes of the largest batch, draft and
// vocabulary among the calls that share it none does; a draft step uses counters only where the workspace has svip_workspace_bytes
// of its own sizes, and where the others have as much none of them reaches those either.
static Workspace carve(void *ws, size_t bytes, int B, int mass_slices)
{
    char *p = static_cast<char *>(ws);
    Workspace w;
    w.flags = reinterpret_cast<unsigned *>(p);
    w.tickets = reinterpret_cast<unsigned *>(p + (bytes & ~(size_t)255));
    p += HEADER_BYTES;
    w.rec = reinterpret_cast<SeqRec *>(p);
    p += ws_rec_bytes(B);
    w.mass = reinterpret_cast<double *>(p);
    p += ws_mass_bytes(B, mass_slices);
    w.part = p;
    return w;
}
enum { TICKET_RESID = 0, TICKET_DRAFT = 1 };        // (the draft step has two)
static_assert(TICKETS_PER_ROW >= TICKET_DRAFT + 2, "a row's counters lie side by side");
__device__ __forceinline__ unsigned *ticket(unsigned *tickets_end, int b, int t)
{
    return tickets_end - ((size_t)b * TICKETS_PER_ROW + t + 1);
}

// ---- kernel arguments ------------------------------------------------------------------

// A draft record with the mass of each of its chunks: relative to the record's maximum m, S[q] = sum of
// exp2((z - m) c) over chunk q, t = sum over the record of exp2((z - m) c) (z - m) c.  64 bytes, so that a record fills
// its half line alone: at 48, with the lines' halves written by different waves, a step of 64 rows took 0.16 us longer.
struct QuarterRec {
    double S[4];
    double t;
    float m;
    float pad[5];
};
static_assert(sizeof(QuarterRec) == 64, "one store of six lanes, one half line");
// A draft record of one sum.  32 bytes instead of 24: where records of different waves share a sector of a cache line, the
// greedy draft step of 64 rows took 0.17 us longer.  (The slices of the other passes are written by workgroups, further
// apart in time; they stay at 24.)
struct alignas(32) WaveRec : Partial {};
static_assert(sizeof(WaveRec) == 32, "a sector each");

struct DraftArgs {
    const void *logits;
    long long row_stride;   // between the rows of consecutive sequences
    const int *pos;         // optional [B]: sequence b reads trace row pos[b] + step_j of its own trace
    long long pos_stride;   // elements between consecutive trace rows (used with pos)
    const int *cap;         // optional [B], given with pos: per-sequence limit on the draft length (at most k_max)
    int B;
    Geo geo;
    Scale sc;
    float h;
    int step_j, k_max;
    const float *u;
    const unsigned char *stop_in;
    int *token;
    float *entropy;
    float *q_tok;
    double *lse;
    unsigned char *stop;
    int *draft_len;
    long long io_stride;
    void *part;             // [B][ns] records of the row's waves: QuarterRec or WaveRec
    unsigned *tickets;      // k_draft_step: see ticket()
    int common_range;       // 1: the temperature is in the range of wave_tile (draft_kernels.h)
    int rows_by_xcd;        // k_draft_stats: workgroup -> (row, records) mapping, see there
    unsigned div, div_magic;  // its one division, by div: n / div = div == 1 ? n : umulhi(n, div_magic), exact for n * div < 2^32
};

struct VerifyArgs {
    const void *target;
    const void *draft;
    long long seq_t, seq_d, row_stride;
    const int *pos;   // optional [B]: row j of sequence b is trace row pos[b] + j
    const unsigned char *skip;   // optional [B]: sequences to leave alone (no read, no write, no ticket)
    int B, k;
    int kd;        // draft rows per sequence in the statistics pass: k if the draft logsumexps are recomputed, else 0
    int bonus;     // 1: the statistics pass also covers target row draft_len (verification), 0: rows j < draft_len only
    Geo geo;       // slicing of the statistics pass
    int first_half;   // > 0: slices 2 i and 2 i + 1 are the first `first_half` tiles and the rest of the i-th geo.tps tiles
    long long stat_items;   // statistics rows * slices: the work items of the statistics pass
    Geo geo_s;     // slicing of the sampling pass (slices of at most LOCATE_UNROLL tiles when possible)
    Scale sc;
    float m0;      // logits at or below it have sc.c_dn times themselves beyond fp32 (-inf: none has), see accumulate_lse
    const int *tokens;
    const int *draft_len;
    const double *draft_lse;
    const float *u_accept;
    const float *u_resample;
    int *n_accepted;
    int *next_token;
    float *accept_prob;
    Workspace ws;
};

__device__ __forceinline__ int clamp_len(int g, int k) { return g < 0 ? 0 : (g > k ? k : g); }

// Element offset of row j of sequence b (seq_stride between sequences, optional trace position).
template <typename A>
__device__ __forceinline__ long long row_offset(const A &a, long long seq_stride, int b, int j)
{
    return (long long)b * seq_stride + (long long)(j + (a.pos ? a.pos[b] : 0)) * a.row_stride;
}

}  // namespace svip
