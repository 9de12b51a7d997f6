// Internal launch interface between the translation units of libqrnnt.  The
// public entry points validate and then call these; the decoder calls them
// directly.  Nothing here is exported.
#pragma once

#include "qrnnt_common.h"

#define QR_HIDDEN __attribute__((visibility("hidden")))

struct QrStepArgs {
    const v4i *wih, *whh;             // TILED_GATES blobs
    const float *s_wih, *s_whh, *bias;
    const int8_t *x;  int64_t ld_x;   // input codes, row pitch in bytes
    const int32_t *x_row;  int n_x_rows; // optional row index into x (or into gx) per hypothesis; rows available
    const int32_t *gx;  int64_t ld_gx; // precomputed input projection [rows, 4H], tiled-row order (USE_GX only)
    const float *tabf;                 // optional fp32 form of gx with scales, bias and exp2 constants folded in
    const int32_t *parent;  int n_slots;
    const int8_t *h_prev;  int64_t ld_hp;
    const float *c_prev;
    const uint8_t *active;
    int8_t *h_next;  int64_t ld_hn;
    float *c_next;
    int8_t *h_copy;                    // optional second copy of the output codes [N, H]
    int32_t *dbg_accx, *dbg_acch;
    float *dbg_gates;
    int I, H, N, nkc_x, nkc_h;
    int n_out;                         // rows of h_next / c_next (N, or more where a list names them: see QrStepGroup.rows)
    float x_scale, h_scale, h_inv;
};

#define QR_MAX_GROUP 3
struct QrStepGroup {
    QrStepArgs p[QR_MAX_GROUP];
    int n;
    const int32_t *gate;               // optional [device]: the launch does nothing when *gate == 0
    // optional [device] (same N, parent and x_row arrays for all members): the launch advances the hypotheses
    // listed in rows[0 .. *n_rows) and leaves every other row of the outputs untouched.  An entry is
    // (output row n < n_out, parent[n], x_row[n], unused): what the kernel would otherwise fetch through n, so that
    // the list adds no link to its chain of dependent loads.  Entries beyond the end may hold anything.  N is the
    // largest length the list can have; of parent and x_row only whether they are null matters.
    const v4i *rows = nullptr;
    const int32_t *n_rows = nullptr;
    // filled in by the launcher of the tiled kernel: row blocks of all members together, workgroups the device holds at once,
    // and (launches without a list) log2 of how many times narrower than the full column block a workgroup's share is
    int row_blocks = 0, n_resident = 0, width = 0;
    int n_short = 0;                   // (likewise) lists up to this length are contracted with K split over the waves
    int through = 0;                   // (likewise) states are written through the L2
    int col_block0 = 0;                // first column block of this launch (a grid's z extent is limited to 65535)
};

struct QrLinearArgs {
    const v4i *w;  int nkc, rows;
    const float *s_w, *bias;
    float a_scale;
    const int8_t *act;  int K, N;
    int n_out;                         // rows of act and of the outputs (N, or more where a list names them)
    float *y;  int32_t *dbg_acc;
    int log_softmax;
    int8_t *q_out;  float q_inv;  int q_bits;   // optional: codes of y under the next layer's input quantizer, [N, rows]
    int w8;                            // 8-bit weights
};

struct QrLinearGroup {
    QrLinearArgs p[QR_MAX_GROUP];
    int n;
    const int32_t *gate;               // optional [device]: the launch does nothing when *gate == 0
    // optional [device] (same N for all members), as in QrStepGroup: only the activation rows n listed in
    // rows[0 .. *n_rows) (first word of an entry) are computed, every other row of the outputs stays as it is.
    const v4i *rows = nullptr;
    const int32_t *n_rows = nullptr;
};

struct QrJointArgs {
    const float *enc;  int n_enc_rows;
    const int32_t *frame_row;          // per-row encoder row, or null: row = frame_base + n / rows_per_utt
    int frame_base, rows_per_utt;
    const float *pred;
    const v4i *w;  const float *s_w;  const float *b_out;
    float z_scale, z_inv;
    const float *lp_src, *lp_ext;
    float lambda_src, lambda_ext, rho;
    int N, J, V, blank, nkc;
    float *lp_out;  int8_t *dbg_zq;  float *fused;
    int w8;                            // 8-bit output layer: 8-bit weights and an 8-bit quantizer on z
};

// A decoding round (joint.hip): output layers, joint and fusion of every utterance's hypotheses.
struct QrHeadArgs {                    // output layer of one network
    const v4i *w;                      // null: the network is not used
    const float *s_w, *bias;
    const int8_t *act;                 // [pool][K] codes it reads
    int K, nkc, w8, log_softmax;
    float a_scale;
};
struct QrMidArgs {                     // bottleneck in front of a language model's output layer
    const v4i *w;                      // null: none, or its codes lie where the head reads them
    const float *s_w, *bias;
    const int8_t *act;                 // [pool][K] codes it reads
    int K, nkc, rows, w8, q_bits;
    float a_scale, q_inv;
};
struct QrRoundArgs {
    QrHeadArgs head[3];                // prediction network (J rows), source and external LM (V rows)
    QrMidArgs mid[2];                  // of the source and the external LM, where the round takes them in (qr_round_takes)
    const float *enc;  int frame_base; // time-synchronous search: utterance b reads row frame_base + b
    const int32_t *row;                // [N] pool row of every hypothesis
    const v4i *w;  const float *s_w;  const float *b_out;   // the joint's output layer
    float z_scale, z_inv;
    float lambda_src, lambda_ext, rho;
    int J, V, blank, nkc, w8;
    // Several workgroups to an utterance: values on their way between them (joint.hip), n_words (qr_round_words) of value and
    // round number (never 0, no two rounds of a search the same) each, [16][64] to a source; zeroed before the first round.
    unsigned long long *words;
    size_t n_words;
    unsigned round;
    int parts;                         // workgroups that share the joint, and (a round with language models, one without) all of
    int wgs_lm, wgs_last;              // an utterance, 0 where it has one that does it all (qr_plan_round)
    int ticks;                         // how long to wait for the others, in 10 ns
    int n_xcd;                         // XCDs that the workgroups of a launch go to in turn
    int come;                          // diagnostic: how many of an utterance's workgroups there are, the first one included (0: all)
    // (Last: between what every workgroup reads first it cost one utterance 0.6 % of its search.)
    int32_t *late;                     // [B] rounds so far in which a word had not come in time
};
#define QR_ROUND_PARTS 4
#define QR_ALSD_ROWS 2                 // rows of the state pool to a slot of the alignment-length search's beam
QR_HIDDEN size_t qr_round_words(int J, bool use_lm, bool mids, int B, int W);   // of an utterance, 0 where it has one workgroup on any device
QR_HIDDEN void qr_plan_round(QrRoundArgs &a, int B, int W, bool alsd);
QR_HIDDEN bool qr_round_takes(int mid_rows, int n_mids, int B, int W, bool alsd);   // bottlenecks of so many rows

struct QrRouteArgs {
    const float *score_src;                         // [B,W] of the current round
    int B, W, V, R, blank, last_round, node_base;
    const int32_t *node_src, *len_src, *row_src;    // [N] of the current round; row: where the networks' states and outputs are
    float *score_dst;  int32_t *node_dst, *len_dst, *row_dst;   // [N] of the next round
    // Rows of the state pool: utterance b owns rows b*P .. b*P + P-1.  free_rows[b*P + i]: its free ones;
    // n_taken[b]: how many of them this frame's earlier rounds have taken.
    int P;  int32_t *free_rows, *n_taken;
    float *nx_score;  v4i *nx_info;  int32_t *nx_count;   // the frame's candidate list; info = (pool row, trie node, length, -)
    int32_t *node_tok, *node_prev;                  // label trie
    // end of the frame (used when last_round): the W best of the candidate list become the beam in buffer fe_dst_buf
    int fe_dst_buf;
    float *fe_score_all;  int32_t *fe_node_all_w, *fe_len_all_w, *fe_row_all_w;
    // early stop (all optional): the round is dead when *gate == 0; an utterance that picked a label
    // adds 1 to *live_next; workgroup 0 clears *live_clear for a later frame
    const int32_t *gate;  int32_t *live_next, *live_clear;
    // list of the hypotheses that took a label (see QrStepGroup.rows): every utterance appends its own at
    // rows_next[old *n_rows_next ...]; workgroup 0 clears *n_rows_clear for a later frame
    v4i *rows_next;  int32_t *n_rows_next, *n_rows_clear;
    // Which label sequence a row's states belong to (route.h): [B][P] (serial of the sequence one label shorter, -1: none;
    // the label; the sequence's own serial; `now` of the last round that named the row).
    v4i *tags;
    int serial0, now;                               // serials of this round's sequences: from serial0 + 1 on, W at most; the frame
};

// Time-synchronous search that runs ahead (joint.hip): an utterance's state between launches, and what it writes.
struct QrRunArgs {
    int B, W, P, T, max_sym;
    int n_entries;                                  // W * (max_sym + 1)
    int max_rounds;                                 // of a launch
    int every_round;                                // diagnostic: one round to a launch, none of them empty by knowledge
    v4i *prog;                                      // [B]: frame and round that are pending, row to be taken next, candidates so far
    float *score;  int32_t *node, *len, *row;       // [N]: hypotheses of the pending round
    v4i *tags;                                      // [B][P]: see QrRouteArgs.tags
    float *nx_score;  v4i *nx_info;                 // [B][n_entries]: the frame's candidates so far
    int32_t *node_tok, *node_prev;
    float *pred_out, *lm_out;                       // [B * P][J], [B * P][2][64]: outputs of a row of the state pool
    v4i *rows_next;  int32_t *n_rows_next, *n_rows_clear;   // as in QrRouteArgs; cleared for the next launch
    int32_t *n_through;                             // utterances that are through
    unsigned long long *told;                       // host memory, or null: takes ticket << 32 | launch, ~0u when all are through
    unsigned ticket;
};
// What it takes on any device (taken to hold 512 workgroups at most, as for the words; a search of more utterances keeps no
// outputs and has a launch to a round); the workgroups of an utterance on this one, 0: it does not.
inline bool qr_run_takes(int J, bool use_lm, int B, int W)
{
    const int wgs = (J + 63) / 64 + (use_lm ? 1 : 0);
    return W <= 16 && J <= 64 * QR_ROUND_PARTS && (wgs == 1 ? B <= 512 : 6 * (int64_t)B * wgs <= 5 * 512);
}
QR_HIDDEN int qr_plan_run(const QrRoundArgs &a, int B, int W);
// Where a search on stream st can tell the host how far it is (r.told, r.ticket), if there is such a place; 0: not started,
// ~0u: through, else the last launch that has begun (round: from 1 on).
QR_HIDDEN void qr_take_ticket(QrRunArgs &r, hipStream_t st);
inline unsigned qr_how_far(const QrRunArgs &r)
{
    const unsigned long long w = r.told ? __atomic_load_n(r.told, __ATOMIC_RELAXED) : 0ull;
    return (unsigned)(w >> 32) == r.ticket ? (unsigned)w : 0u;
}
QR_HIDDEN void qr_launch_search_run(const QrRoundArgs &a, const QrRunArgs &r, int wgs, hipStream_t st);

// Alignment-length synchronous search: what one iteration needs beyond QrRouteArgs (of which it uses score/node/len/row
// src and dst, the pool rows, the label trie, node_base, gate, live_next and the list of rows).
struct QrAlsdArgs {
    int iter, T, u_max;                              // hypothesis w stands at frame iter - len[w]
    const unsigned long long *hash_src;              // [N] hash of the label sequence (recombination key, with the length)
    unsigned long long *hash_dst;
    float *fin_score;  int32_t *fin_node, *fin_len;  // [B,W] the W best finished hypotheses so far, best first
    // label picks whose sequence a live hypothesis of the beam holds are looked for by hash: to name its row where rows are not
    // looked for by their tags (launch_round), and to be counted where there are stats
    int reuse;
    int32_t *stats;                                  // optional [device] int32[2]: += label picks that kept their slot, += those
};

// One direction of the persistent recurrence (see recurrence.hip).
struct QrRecArgs {
    const v4i *whh;  const float *s_wih, *s_whh, *bias;
    const v4i *wih;                    // used when gx is null: the kernel projects the input itself
    const int8_t *x;  int64_t ld_x;    // input codes [T*B, I], row pitch in bytes
    int I, nkc_x;
    const int32_t *gx;                 // [T*B, 4H] gate-interleaved input projection, or null (qr_rec_projects(I))
    const int8_t *h0;  const float *c0;
    int8_t *h_out;  int64_t ld_out;  int col_off;
    int8_t *h_last;  float *c_last;  float *dbg_c_all;
    char *xbuf;                        // exchange area (qr_rec_xbuf_bytes), zeroed before the launch
    unsigned long long *admit;         // one word per utterance group (qr_rec_admit_bytes), zeroed before the launch
    float *c_buf;                      // [B][H]: cell states of a group whose members are not resident together
    int *err;                          // set to 1 when a bounded wait ran out
    int T, B, H, nkc_h, reverse, spin_limit;
    int admit_ticks;                   // how long a group waits for all of its members, in 10 ns
    int spread, n_come;                // diagnostics: exchange at system scope; only so many members of a group come in time
    float x_scale, h_scale, h_inv;
    int w8;                            // 8-bit layer: 8-bit W_hh blob and an 8-bit hidden-state quantizer
};
struct QrRecGroup {
    QrRecArgs d[2];
    int n;
    int group0 = 0, group_end = 0;     // filled in by the launcher: which groups (direction + n * utterance group) go out
};
QR_HIDDEN bool qr_rec_supported(int H, int B);
QR_HIDDEN bool qr_rec_projects(int I);   // whether the recurrence can take input codes of I columns instead of their projection
QR_HIDDEN size_t qr_rec_xbuf_bytes(int H, int B);
QR_HIDDEN size_t qr_rec_admit_bytes(int B);
QR_HIDDEN bool qr_launch_recurrence(const QrRecGroup &g, hipStream_t st);

QR_HIDDEN void qr_fill_lstm_weights(QrStepArgs &a, const qrnnt_lstm *L);
QR_HIDDEN qrnnt_status qr_check_lstm(const qrnnt_lstm *L);
QR_HIDDEN void qr_launch_lstm_step(const QrStepArgs &a, bool use_gx, hipStream_t st);
QR_HIDDEN void qr_launch_lstm_step_group(const QrStepGroup &g, bool use_gx, hipStream_t st);
QR_HIDDEN void qr_launch_gx_table(const qrnnt_lstm *L, const int32_t *gx, int M, float *tab, hipStream_t st);
QR_HIDDEN void qr_launch_input_projection(const qrnnt_lstm *L, const int8_t *x_codes, int M, int32_t *gx, int32_t *dbg_accx,
                                          hipStream_t st);
QR_HIDDEN void qr_launch_linear_group(const QrLinearGroup &g, hipStream_t st);
QR_HIDDEN void qr_launch_linear(const QrLinearArgs &a, hipStream_t st);
QR_HIDDEN void qr_launch_joint(const QrJointArgs &a, hipStream_t st);
QR_HIDDEN void qr_launch_search_round(const QrRoundArgs &a, const QrRouteArgs &r, hipStream_t st);
QR_HIDDEN void qr_launch_search_round_alsd(const QrRoundArgs &a, const QrRouteArgs &r, const QrAlsdArgs &s, hipStream_t st);
QR_HIDDEN void qr_launch_beam(const float *score, const float *fused, int B, int W, int V, int blank, int force_blank,
                              int32_t *parent_out, int32_t *token_out, float *score_out, hipStream_t st);
