// Decoding loop over logit traces (Algorithm 1 and Algorithm 6) with the draft-length rules of
// the paper's baselines (Section 3: Constant, Heuristic), built on the draft and verify calls.
//
// Sampling, per round:
//             drafting       -> the rows of a trace are all there, so one pair of launches covers a group of draft
//                               positions of every sequence (draft_group_call); a sequence's draft ends at the
//                               first position of the group that stops it.  In large batches (see below)
//                               svip_draft_step's kernels run once per position.  Flags are chained on the device.
//             verify         -> svip_verify kernels on trace rows pos[b] .. pos[b] + draft_len[b]
//             k_round_end    -> appends the produced tokens, advances positions, applies the length
//                               rule, updates the counters, counts the sequences still running and sets up the next round
// Greedy:     every sequence goes through its own rounds, on rows that are read once, many per pair of launches
//             (greedy_stream_call); the rounds as above only in large batches.
// k_round_begin sets up what the first launches of a call read.
// The counts reach the host as messages: the counting kernel stores (ticket, count) as one 8-byte word
// into pinned host memory and the host reads that word until the ticket shows.  No copy is enqueued and the
// stream is never synchronised inside the loop; the host launches one round ahead of the count it waits for,
// so the GPU always has the next round queued (a round launched after the last sequence finished finds
// every sequence marked done and changes nothing).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <chrono>

#include "../../include/svip.h"
#include "loop_round.h"
#include "svip_internal.h"

namespace svip {

constexpr int LOOP_WG = 256;

// ---- messages from the device to the host ----------------------------------------------------
//
// A host thread's mailbox: MAIL_SLOTS words of pinned host memory, allocated by the thread's first
// svip_loop_run and kept until the process ends.  A message is (ticket << 32 | value), stored by one
// thread of a kernel with a single system-scope store; tickets count up per host thread and never repeat
// within 2^32 messages, message t uses word t % MAIL_SLOTS, and the loop never has more than
// nine messages outstanding, so a word is not reused before it has been read.
constexpr unsigned MAIL_SLOTS = 64;
struct Mailbox {
    unsigned long long *host, *dev;
    unsigned next;
};
static thread_local Mailbox g_mail = {nullptr, nullptr, 0};

struct Ticket {
    unsigned id;
    unsigned long long *dev;            // what the kernel gets
    const unsigned long long *host;     // what the host reads
};

static bool mailbox_ready()
{
    if (g_mail.host) return true;
    void *h = nullptr, *d = nullptr;
    // coherent (fine-grained) memory: a word stored by a running kernel is seen by the host without waiting for
    // the kernel to end; without the flag the other two would make the allocation non-coherent
    if (hipHostMalloc(&h, MAIL_SLOTS * sizeof(unsigned long long),
                      hipHostMallocCoherent | hipHostMallocPortable | hipHostMallocMapped) != hipSuccess)
        return false;
    memset(h, 0, MAIL_SLOTS * sizeof(unsigned long long));
    if (hipHostGetDevicePointer(&d, h, 0) != hipSuccess) {
        (void)hipHostFree(h);
        return false;
    }
    g_mail.host = static_cast<unsigned long long *>(h);
    g_mail.dev = static_cast<unsigned long long *>(d);
    g_mail.next = 0;
    return true;
}

static Mail mail_of(const Ticket &t) { return Mail{t.dev, t.id}; }

static Ticket new_ticket()
{
    Ticket t;
    t.id = ++g_mail.next;
    if (t.id == 0) t.id = ++g_mail.next;       // 0 is what an unused word holds
    t.dev = g_mail.dev + t.id % MAIL_SLOTS;
    t.host = g_mail.host + t.id % MAIL_SLOTS;
    return t;
}

// Waits until the message of ticket t is there.  The kernel that posts it is already in the stream, so the
// wait ends when the GPU gets there; if nothing shows for a while the stream is asked: one that has drained
// without the message has failed.
static svip_status await(const Ticket &t, int *value, hipStream_t st)
{
    typedef std::chrono::steady_clock clock;
    clock::time_point t0 = clock::now();
    for (unsigned spins = 1;; ++spins) {
        unsigned long long v = __atomic_load_n(t.host, __ATOMIC_ACQUIRE);
        if ((unsigned)(v >> 32) == t.id) {
            *value = (int)(unsigned)v;
            return SVIP_OK;
        }
        if ((spins & 4095u) == 0 && clock::now() - t0 > std::chrono::milliseconds(200)) {
            const hipError_t q = hipStreamQuery(st);
            if (q == hipErrorNotReady) {
                (void)hipGetLastError();        // "not ready" is no error of the loop's: do not leave it behind
                t0 = clock::now();
                continue;
            }
            v = __atomic_load_n(t.host, __ATOMIC_ACQUIRE);
            if (q == hipSuccess && (unsigned)(v >> 32) == t.id) {
                *value = (int)(unsigned)v;
                return SVIP_OK;
            }
            return SVIP_ERR_HIP;
        }
    }
}

static inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- which positions of a draft share a pair of launches ---------------------------------------
//
// A launch's time goes up by about 1 us per 1000 waves (records of one tile, 4 KB each) once it has more than about 1500 of
// them, and a pair of launches that finds nothing to do costs about 4.5 us.
//   Sampling: the first group takes what GROUP_WAVES_FIRST waves cover -- a whole draft of a few sequences, 8 positions of 8
//   sequences of 152K bf16 logits, at least 2 -- and the next one, which most rounds find empty, as much of the rest
//   as the buffer for the records holds.
//   Greedy: each row is read once, so a launch reads as many as it is sure to need, up to STREAM_WAVES_MAX draft records (the target
//   rows come on top): with 16384 / 32768 / 65536 of them 8 sequences of 151936 bf16 logits, 32 tokens in drafts of 1.3, take 138 / 122 /
//   122 us, 64 sequences 445 / 396 / 367.  Where a call may only run a few rounds, and behind the last token, it is STREAM_WAVES
//   records, at least 2 positions, and up to eight times as many for a draft that goes on.
// Beyond GROUP_WAVES_FIRST waves per position (64 sequences of 152K logits are just below) positions go one by one.  The line
// stands behind the largest shape measured, where groups are still the faster form: it is not where the two meet.
// us for 32 tokens per sequence, position by position / in groups (greedy; sampling), drafts of 1.3 | 20 positions (greedy with the
// rows of one round per pair of launches, each round reading its own: 352, 327, 458, 637 | 228, 962, 2525, 3813):
//    1 x 32000 fp32      1255 / 97;  958 / 613   | 2227 / 88;  1087 / 297
//    8 x 151936 bf16     1301 / 122; 1479 / 887  | 2581 / 258; 2834 / 965
//   33 x 128256 bf16     1823 / 210; 1961 / 1409 | 3921 / 440; 3669 / 1636
//   64 x 151936 bf16     2211 / 367; 2570 / 1731 | 5386 / 716; 5276 / 2941
constexpr int GROUP_WAVES_FIRST = 4800, GROUP_WAVES_MAX = 32768, STREAM_WAVES = 2400, STREAM_WAVES_MAX = 65536;

// Positions of the first group (0: positions go one by one) and of later ones; greedy: rows of a small launch and of the largest.
struct GroupPlan {
    int first, next;
};
static GroupPlan plan_groups(int B, int k, int V, int dtype, bool greedy)
{
    GroupPlan p = {0, 0};
    const int waves = group_waves(B, V, dtype);
    if (waves == 0 || waves > GROUP_WAVES_FIRST) return p;
    const int rows = group_waves(1, V, dtype) * ((B + 7) / 8 * 8);        // waves per position with rows kept on XCDs
    const int n = (greedy ? STREAM_WAVES : GROUP_WAVES_FIRST) / waves;
    p.first = n > 2 ? n : 2;
    if (greedy && p.first > 64) p.first = 64;
    if (p.first > k) p.first = k;
    p.next = (greedy ? STREAM_WAVES_MAX : GROUP_WAVES_MAX) / rows;
    const int most = greedy ? STREAM_MAX_GROUP : k;
    if (p.next > most) p.next = most;
    if (p.next < p.first) p.next = p.first;
    return p;
}
// Bytes for the records of the largest group; the loop's workspace has to do for every type, sampling and greedy.  least: what
// groups are taken with at all, the greedy ones only as large as a small launch.
static size_t plan_bytes(int B, int k, int V, bool least)
{
    size_t most = 0;
    for (int dtype = SVIP_F32; dtype <= SVIP_F16; ++dtype)
        for (int greedy = 0; greedy < 2; ++greedy) {
            const GroupPlan p = plan_groups(B, k, V, dtype, greedy);
            const size_t n = p.first ? group_bytes(B, V, dtype, least && greedy ? p.first : p.next, greedy) : 0;
            if (n > most) most = n;
        }
    return most;
}

// What a round taken position by position needs: the least a call may bring.
static size_t serial_buffer_bytes(int B, int k)
{
    const size_t n = (size_t)B, nk = n * (size_t)k;
    return up256(nk * 4) + up256(nk * 8) + 2 * up256(n) + 6 * up256(n * 4) + 256;
}

static size_t round_buffer_bytes(int B, int k, int V, bool least)
{
    const size_t n = (size_t)B, nk = n * (size_t)k;
    return serial_buffer_bytes(B, k) + 2 * up256(n * 4) + up256((nk + n) * 4) + plan_bytes(B, k, V, least);
}

// bytes: of the round's buffers.  Where they do only for the serial loop there are none for groups (group is null); what there is
// beyond the least that groups need makes the greedy ones larger.
static RoundBuffers carve_round(char *p, int B, int k, int V, size_t bytes)
{
    const size_t n = (size_t)B, nk = n * (size_t)k;
    RoundBuffers r;
    r.tokens = reinterpret_cast<int *>(p); p += up256(nk * 4);
    r.lse = reinterpret_cast<double *>(p); p += up256(nk * 8);
    r.stop = reinterpret_cast<unsigned char *>(p); p += up256(n);
    r.done = reinterpret_cast<unsigned char *>(p); p += up256(n);
    r.draft_len = reinterpret_cast<int *>(p); p += up256(n * 4);
    r.n_accepted = reinterpret_cast<int *>(p); p += up256(n * 4);
    r.next_token = reinterpret_cast<int *>(p); p += up256(n * 4);
    r.pos = reinterpret_cast<int *>(p); p += up256(n * 4);
    r.cap = reinterpret_cast<int *>(p); p += up256(n * 4);
    r.counter = reinterpret_cast<int *>(p); p += 256;
    r.drafted = r.round = r.argmax = nullptr;
    r.group = nullptr;
    r.group_bytes = 0;
    const size_t least = round_buffer_bytes(B, k, V, true);
    if (bytes >= least) {
        r.drafted = reinterpret_cast<int *>(p); p += up256(n * 4);
        r.round = reinterpret_cast<int *>(p); p += up256(n * 4);
        r.argmax = reinterpret_cast<int *>(p); p += up256((nk + n) * 4);
        r.group = p;
        r.group_bytes = plan_bytes(B, k, V, true) + (bytes - least);
    }
    return r;
}

__device__ __forceinline__ int block_count(int mine, int *lds)
{
    // one workgroup: sum of `mine` over its threads, valid in thread 0
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_down(mine, o, 64);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = mine;
    __syncthreads();
    int total = 0;
    if (threadIdx.x == 0)
        for (int w = 0; w < LOOP_WG / 64; ++w) total += lds[w];
    return total;
}

// one workgroup
__global__ __launch_bounds__(LOOP_WG) void k_loop_init(int *state, int B, int n0, int gamma0, int L, int max_new,
                                                       int *counter)
{
    __shared__ int lds[LOOP_WG / 64];
    int running = 0;
    for (int b = threadIdx.x; b < B; b += LOOP_WG) {
        int *st = state + (size_t)b * SVIP_LOOP_NSTATE;
        const int done = finished(n0, n0, gamma0, L, max_new) ? 1 : 0;
        st[0] = n0;
        st[1] = gamma0;
        st[2] = done;
        st[3] = st[4] = st[5] = st[6] = 0;
        st[7] = n0;
        running += !done;
    }
    const int total = block_count(running, lds);
    if (threadIdx.x == 0) {
        counter[0] = total;
        counter[1] = 0;
    }
}

// one workgroup: what the kernels of a call's first round read
__global__ __launch_bounds__(LOOP_WG) void k_round_begin(LoopArgs a)
{
    __shared__ int lds[LOOP_WG / 64];
    int running = 0;
    for (int b = threadIdx.x; b < a.B; b += LOOP_WG) {
        const int *st = a.state + (size_t)b * SVIP_LOOP_NSTATE;
        begin_sequence(a.rb, b, st[0], st[1], st[2]);
        if (a.rb.group) {
            a.rb.drafted[b] = -1;
            a.rb.round[b] = a.round;
        }
        running += st[2] ? 0 : 1;
    }
    const int total = block_count(running, lds);
    if (threadIdx.x == 0) {
        a.rb.counter[0] = a.rb.counter[1] = total;
        a.rb.counter[2] = a.round;
    }
}

// one workgroup: number of sequences that are still drafting
__global__ __launch_bounds__(LOOP_WG) void k_count_drafting(const unsigned char *stop, int B, int *counter, Mail mail)
{
    __shared__ int lds[LOOP_WG / 64];
    int n = 0;
    for (int b = threadIdx.x; b < B; b += LOOP_WG) n += stop[b] ? 0 : 1;
    const int total = block_count(n, lds);
    if (threadIdx.x == 0) {
        counter[1] = total;
        post(mail, total);
    }
}

// one workgroup: bookkeeping of the round for every running sequence
__global__ __launch_bounds__(LOOP_WG) void k_round_end(LoopArgs a)
{
    __shared__ int lds[LOOP_WG / 64];
    int running = 0;
    for (int b = threadIdx.x; b < a.B; b += LOOP_WG) {
        const int *tokens = a.rb.tokens + (size_t)b * a.gamma_max;
        if (a.rb.done[b]) log_idle(a, b, a.round);
        else running += end_sequence(a, b, a.round, a.rb.draft_len[b], a.rb.n_accepted[b], a.rb.next_token[b], tokens);
    }
    const int total = block_count(running, lds);
    if (threadIdx.x == 0) {
        a.rb.counter[0] = total;
        post(a.mail, total);
    }
}

static svip_status read_counter(const int *dev, int *host, hipStream_t st)
{
    if (hipMemcpyAsync(host, dev, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess) return SVIP_ERR_HIP;
    return hipStreamSynchronize(st) == hipSuccess ? SVIP_OK : SVIP_ERR_HIP;
}

static LoopArgs loop_args(const svip_loop_config *c, const RoundBuffers &rb, int round)
{
    LoopArgs a;
    a.state = c->state;
    a.B = c->B;
    a.L = c->L;
    a.gamma_max = c->gamma_max;
    a.inc = c->gamma_inc;
    a.dec = c->gamma_dec;
    a.max_new = c->max_new;
    a.round = round;
    a.rb = rb;
    a.out_tokens = c->out_tokens;
    a.out_stride = c->out_stride;
    a.round_log = c->round_log;
    a.mail = Mail{nullptr, 0};
    return a;
}

// The draft call of round `round` for position j (of a group: its first); base: bytes of the kernels' own workspace.
static DraftCall draft_call(const svip_loop_config *c, const RoundBuffers &rb, size_t base, int round, int j)
{
    DraftCall d;
    d.greedy = c->greedy != 0;
    d.logits = c->draft_trace;
    d.dtype = c->dtype;
    d.B = c->B;
    d.V = c->V;
    d.row_stride = c->seq_stride;
    d.pos = rb.pos;
    d.pos_stride = c->row_stride;
    d.cap = rb.cap;
    d.temperature = c->temperature;
    d.h = c->h;
    d.step_j = j;
    d.k_max = c->gamma_max;
    d.u_sample = c->greedy ? nullptr : c->u_sample + (size_t)round * c->B * c->gamma_max + j;
    d.stop_in = rb.stop;
    d.token_out = rb.tokens + j;
    d.entropy_out = nullptr;
    d.q_tok_out = nullptr;
    d.lse_out = rb.lse + j;
    d.stop_out = rb.stop;
    d.draft_len_out = rb.draft_len;
    d.io_stride = c->gamma_max;
    d.workspace = c->workspace;
    d.workspace_bytes = base;
    d.stream = c->hip_stream;
    d.counters = true;
    return d;
}

// The greedy loop: pairs of launches until no sequence is active any more.  Each pair's first kernel reports what the pairs
// before it left, so the next pair is launched while the GPU works on this one.  The first launches are large, until every
// sequence has the rows of max_new tokens; what comes behind them serves rounds that reach further.
static svip_status run_greedy_stream(const svip_loop_config *c, const RoundBuffers &rb, size_t base, const GroupPlan &plan,
                                     int first_round, int max_rounds, int *rounds_run, int *running)
{
    // a round may use no more than its first rows: a call of few rounds reads accordingly
    int most = plan.next;
    if ((long long)plan.first * max_rounds < most) most = plan.first * max_rounds;
    while (most > plan.first && group_bytes(c->B, c->V, c->dtype, most, true) > rb.group_bytes) --most;
    const long long sure = (long long)c->max_new + plan.first;
    const int large = sure < most ? (int)sure : most;
    int small = plan.first;
    hipStream_t st = static_cast<hipStream_t>(c->hip_stream);
    const LoopArgs a = loop_args(c, rb, first_round);
    hipLaunchKernelGGL(k_round_begin, dim3(1), dim3(LOOP_WG), 0, st, a);
    if (hipPeekAtLastError() != hipSuccess) return SVIP_ERR_HIP;
    const DraftCall d = draft_call(c, rb, base, first_round, 0);
    long long covered = 0;
    for (int active = 1; active > 0;) {
        const Ticket t0 = new_ticket(), t1 = new_ticket(), t2 = new_ticket();
        int group = large;
        if (covered >= sure) {
            group = small;
            if (2 * small <= most && 2 * small <= 8 * plan.first) small *= 2;      // (the last launch finds nothing to do)
        }
        covered += group;
        svip_status r = greedy_stream_call(d, c->target_trace, group, plan.first, a, first_round + max_rounds, mail_of(t0), mail_of(t1),
                                           mail_of(t2));
        if (r == SVIP_OK) r = await(t0, &active, st);
        if (r == SVIP_OK) r = await(t1, running, st);
        if (r == SVIP_OK) r = await(t2, rounds_run, st);
        if (r != SVIP_OK) return r;
    }
    *rounds_run -= first_round;
    return hipStreamSynchronize(st) == hipSuccess ? SVIP_OK : SVIP_ERR_HIP;
}

static svip_status check_config(const svip_loop_config *c)
{
    if (!c) return SVIP_ERR_NULL;
    if (!c->target_trace || !c->draft_trace || !c->state || !c->out_tokens) return SVIP_ERR_NULL;
    if (!c->greedy && (!c->u_sample || !c->u_accept || !c->u_resample)) return SVIP_ERR_NULL;
    if (c->B <= 0 || c->V <= 0 || c->gamma_max < 1 || c->gamma_max > SVIP_MAX_K || c->gamma0 < 1 ||
        c->gamma0 > c->gamma_max || c->L < c->gamma_max + 1 || c->n0 < 0 || c->n0 >= c->L || c->max_new < 0 ||
        c->row_stride < c->V || c->seq_stride < (long long)c->L * c->row_stride - (c->row_stride - c->V) ||
        c->out_stride < (long long)c->max_new + c->gamma_max || c->rounds < 1)
        return SVIP_ERR_SHAPE;
    if (c->gamma_inc < 0 || c->gamma_dec < 0 || c->check_every < 0) return SVIP_ERR_PARAM;
    const size_t base = up256(svip_workspace_bytes(c->B, c->gamma_max, c->V));
    if (!c->workspace || (reinterpret_cast<uintptr_t>(c->workspace) & 255u) || base == 0 ||
        c->workspace_bytes < base + serial_buffer_bytes(c->B, c->gamma_max))
        return SVIP_ERR_WORKSPACE;
    return SVIP_OK;
}

}  // namespace svip

using namespace svip;

extern "C" {

size_t svip_loop_workspace_bytes(int B, int gamma_max, int V)
{
    const size_t base = svip_workspace_bytes(B, gamma_max, V);
    if (base == 0) return 0;
    return up256(base) + round_buffer_bytes(B, gamma_max, V, false);
}

svip_status svip_loop_init(const svip_loop_config *c)
{
    const svip_status s = check_config(c);
    if (s != SVIP_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(c->hip_stream);
    const size_t base = up256(svip_workspace_bytes(c->B, c->gamma_max, c->V));
    const RoundBuffers rb = carve_round(static_cast<char *>(c->workspace) + base, c->B, c->gamma_max, c->V,
                                        c->workspace_bytes - base);
    const svip_status r = svip_workspace_reset(c->workspace, base, c->hip_stream);
    if (r != SVIP_OK) return r;
    hipLaunchKernelGGL(k_loop_init, dim3(1), dim3(LOOP_WG), 0, st, c->state, c->B, c->n0, c->gamma0, c->L,
                       c->max_new, rb.counter);
    return hipPeekAtLastError() == hipSuccess ? SVIP_OK : SVIP_ERR_HIP;
}

svip_status svip_loop_run(const svip_loop_config *c, int first_round, int max_rounds, int *rounds_run_host,
                          int *running_host)
{
    const svip_status s = check_config(c);
    if (s != SVIP_OK) return s;
    if (first_round < 0 || max_rounds < 0 || (long long)first_round + max_rounds > c->rounds) return SVIP_ERR_SHAPE;
    hipStream_t st = static_cast<hipStream_t>(c->hip_stream);
    const size_t base = up256(svip_workspace_bytes(c->B, c->gamma_max, c->V));
    const RoundBuffers rb = carve_round(static_cast<char *>(c->workspace) + base, c->B, c->gamma_max, c->V,
                                        c->workspace_bytes - base);
    const int B = c->B, k = c->gamma_max;
    const GroupPlan plan = draft_shape_forced() || !rb.group ? GroupPlan{0, 0} : plan_groups(B, k, c->V, c->dtype, c->greedy != 0);

    int running = 0, done_rounds = 0;
    svip_status r;
    if (c->greedy && plan.first != 0 && max_rounds > 0) {
        if (!mailbox_ready()) return SVIP_ERR_HIP;
        r = run_greedy_stream(c, rb, base, plan, first_round, max_rounds, &done_rounds, &running);
        if (r != SVIP_OK) return r;
        if (rounds_run_host) *rounds_run_host = done_rounds;
        if (running_host) *running_host = running;
        return SVIP_OK;
    }
    r = read_counter(rb.counter, &running, st);
    if (r != SVIP_OK) return r;
    if (running > 0 && max_rounds > 0 && !mailbox_ready()) return SVIP_ERR_HIP;
    // `running` is the count after the last round whose message has been read; `before` is the ticket of the
    // round launched since, whose message has not been read yet.  Round i is launched on the strength of
    // the count after round i - 2; if the count after round i - 1 then turns out to be zero, round i has
    // run (or is being dropped) with every sequence marked done and is not counted.
    Ticket before = {0, nullptr, nullptr};
    bool have_before = false;
    for (int i = 0; i < max_rounds && running > 0; ++i) {
        const int round = first_round + i;
        const Ticket mine = new_ticket();
        LoopArgs a = loop_args(c, rb, round);
        a.mail = mail_of(mine);
        if (i == 0) hipLaunchKernelGGL(k_round_begin, dim3(1), dim3(LOOP_WG), 0, st, a);

        bool idle = false;        // the round before this one finished the last sequence
        int polled = 0;           // draft positions launched when the device was last asked
        for (int j = 0, n = 1; j < k; j += n) {
            // asked before a launch that may find nothing to do, but not where it is the last pair of the round: that costs
            // less than the answer (about 7 us)
            n = plan.first == 0 ? 1 : (j == 0 ? plan.first : (k - j < plan.next ? k - j : plan.next));
            const bool last_pair = plan.first != 0 && j + n == k;
            if (j > 0 && c->check_every > 0 && j / c->check_every > polled / c->check_every && !last_pair) {
                polled = j;
                const Ticket poll = new_ticket();
                hipLaunchKernelGGL(k_count_drafting, dim3(1), dim3(LOOP_WG), 0, st, rb.stop, B, rb.counter, mail_of(poll));
                if (hipPeekAtLastError() != hipSuccess) return SVIP_ERR_HIP;
                int drafting = 0;
                r = await(poll, &drafting, st);
                if (r != SVIP_OK) return r;
                if (have_before) {                // the GPU is inside this round: the one before has posted
                    r = await(before, &running, st);
                    if (r != SVIP_OK) return r;
                    have_before = false;
                    if (running == 0) {
                        idle = true;
                        break;
                    }
                }
                if (drafting == 0) break;
            }
            const DraftCall d = draft_call(c, rb, base, round, j);
            r = plan.first == 0 ? draft_step_call(d) : draft_group_call(d, n, rb.group, rb.group_bytes);
            if (r != SVIP_OK) return r;
        }
        if (idle) break;

        VerifyCall v;
        v.greedy = c->greedy != 0;
        v.target = c->target_trace;
        v.draft = c->draft_trace;
        v.dtype = c->dtype;
        v.B = B;
        v.k_max = k;
        v.V = c->V;
        v.seq_stride_t = c->seq_stride;
        v.seq_stride_d = c->seq_stride;
        v.row_stride = c->row_stride;
        v.pos = rb.pos;
        v.temperature = c->temperature;
        v.draft_tokens = rb.tokens;
        v.draft_len = rb.draft_len;
        v.draft_lse = rb.lse;
        v.u_accept = c->greedy ? nullptr : c->u_accept + (size_t)round * B * k;
        v.u_resample = c->greedy ? nullptr : c->u_resample + (size_t)round * B;
        v.n_accepted_out = rb.n_accepted;
        v.next_token_out = rb.next_token;
        v.accept_prob_out = nullptr;
        v.skip = rb.done;
        v.workspace = c->workspace;
        v.workspace_bytes = base;
        v.stream = c->hip_stream;
        r = verify_call(v);
        if (r != SVIP_OK) return r;

        hipLaunchKernelGGL(k_round_end, dim3(1), dim3(LOOP_WG), 0, st, a);
        if (hipPeekAtLastError() != hipSuccess) return SVIP_ERR_HIP;
        if (have_before) {        // with this round queued behind it, wait for the count of the round before
            r = await(before, &running, st);
            if (r != SVIP_OK) return r;
            have_before = false;
            if (running == 0) break;              // this round was idle
        }
        before = mine;
        have_before = true;
        ++done_rounds;
    }
    if (have_before) {
        r = await(before, &running, st);
        if (r != SVIP_OK) return r;
    }
    if (hipStreamSynchronize(st) != hipSuccess) return SVIP_ERR_HIP;
    if (rounds_run_host) *rounds_run_host = done_rounds;
    if (running_host) *running_host = running;
    return SVIP_OK;
}

}  // extern "C"
