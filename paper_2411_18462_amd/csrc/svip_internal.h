// Calls shared by the sources of libsvip.so: the public entry points of include/svip.h and the
// decoding loop are thin wrappers around these.  Compared with the public signatures they add
// the optional per-sequence trace positions and draft-length limits the loop needs.
#pragma once
#include <stddef.h>

#include "../../include/svip.h"

namespace svip {

struct DraftCall {
    bool greedy;                 // argmax instead of a draw (u_sample unused)
    const void *logits;          // device
    int dtype;
    int B, V;
    long long row_stride;        // elements between the rows (or traces) of consecutive sequences
    const int *pos;              // device [B] or nullptr: sequence b reads trace row pos[b] + step_j
    long long pos_stride;        // elements between consecutive trace rows
    const int *cap;              // device [B] or nullptr, given with pos: per-sequence draft-length limit (<= k_max)
    float temperature, h;
    int step_j, k_max;
    const float *u_sample;
    const unsigned char *stop_in;
    int *token_out;
    float *entropy_out;
    float *q_tok_out;
    double *lse_out;
    unsigned char *stop_out;
    int *draft_len_out;
    long long io_stride;
    void *workspace;
    size_t workspace_bytes;
    void *stream;
    bool counters;               // the workspace has hand-over counters that svip_workspace_reset clears
};

// A message to the host: the word of its mailbox and the ticket that shows it has arrived.
struct Mail {
    unsigned long long *word;
    unsigned ticket;
};

// Buffers of a round of the decoding loop, carved from the loop workspace after the kernels' own.
struct RoundBuffers {
    int *tokens;               // [B, gamma_max]
    double *lse;               // [B, gamma_max]
    unsigned char *stop;       // [B]
    unsigned char *done;       // [B] 1: the sequence has finished, verification skips it
    int *draft_len;            // [B]
    int *n_accepted;           // [B]
    int *next_token;           // [B]
    int *pos;                  // [B] trace position of the round (0 for finished sequences)
    int *cap;                  // [B] length limit of the round
    int *counter;              // [3]: sequences not finished; still drafting (greedy stream: taking part in this call);
                               //      rounds begun before this call + the most that any sequence has ended in it
    int *drafted, *round;      // greedy stream [B]: positions of the round whose draft rows have been read, none of which ends the
                               //      draft, and the target rows up to one behind them (-1: nothing); the sequence's round
    int *argmax;               // greedy stream [B, gamma_max + 1]: argmax of those target rows (the drafted tokens: `tokens`)
    char *group;               // grouped positions: draft records, then (greedy) keys
    size_t group_bytes;
};

struct LoopArgs {
    int *state;                // [B, SVIP_LOOP_NSTATE]
    int B, L, gamma_max, inc, dec, max_new, round;
    RoundBuffers rb;
    int *out_tokens;
    long long out_stride;
    int *round_log;            // [rounds, B, 4] or nullptr
    Mail mail;                 // k_round_end: where the count of running sequences goes
};

struct VerifyCall {
    bool greedy;                 // Algorithms 3 and 5: only the target, tokens and lengths are used
    const void *target, *draft;  // device
    int dtype;
    int B, k_max, V;
    long long seq_stride_t, seq_stride_d, row_stride;
    const int *pos;              // device [B] or nullptr: row j of sequence b is trace row pos[b] + j
    const unsigned char *skip;   // device [B] or nullptr: sequences with skip[b] != 0 are neither read nor written
    float temperature;
    const int *draft_tokens;
    const int *draft_len;
    const double *draft_lse;
    const float *u_accept;
    const float *u_resample;
    int *n_accepted_out;
    int *next_token_out;
    float *accept_prob_out;
    void *workspace;
    size_t workspace_bytes;
    void *stream;
};

svip_status draft_step_call(const DraftCall &c);
// Several positions per pair of launches (loop_kernels.h), for the decoding loop: calls with pos, cap, stop_in and
// draft_len_out; their records go to `buffer` and the call's workspace is only used for its flag word.
// group_waves: waves per position, 0 where rows are too long; group_bytes: the buffer that `group` positions need.
int group_waves(int B, int V, int dtype);
size_t group_bytes(int B, int V, int dtype, int group, bool greedy);
bool draft_shape_forced();           // an experiment's override asks for records of another size
svip_status draft_group_call(const DraftCall &c, int group, void *buffer, size_t bytes);
// Greedy: every active sequence up to `group` rows further, `ahead` where its next round may be its last; step_j is not used.
svip_status greedy_stream_call(const DraftCall &c, const void *target, int group, int ahead, const LoopArgs &l, int last_round,
                               Mail active, Mail running, Mail rounds);
constexpr int STREAM_MAX_GROUP = 128;
svip_status verify_call(const VerifyCall &c);

}  // namespace svip
