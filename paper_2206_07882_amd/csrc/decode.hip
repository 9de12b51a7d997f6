// The decoding loop, entirely on the device: joint + fusion (Eq. 1), beam
// selection, hypothesis bookkeeping and the advance of the prediction network
// and both language models (Sec. 2).  The paper's simulated system sorts
// hypotheses on an attached CPU and is limited by the link to it (Sec. 4.1);
// here the selection and the bookkeeping are kernels and the host only enqueues,
// as many launches as the longest search can need, and waits for nothing.
#include "kernels.h"
#include "select.h"

namespace {


struct NetBuf {
    int8_t *h[QRNNT_MAX_LAYERS];   // [pool + 1][H]; the last row stays zero: the state before the first symbol
    float *c[QRNNT_MAX_LAYERS];    // [pool + 1][H]
    bool mid_in_round;             // the round contracts the bottleneck itself
    int32_t *gx0;                  // [V][4*H0]: input projection of layer 0 for every token
    float *tab0;                   // the same as fp32 pre-activation contributions (scales, bias folded in)
    int8_t *mid_q;                 // [pool][M]: codes of the bottleneck's output
};

struct Plan {
    int T, B, W, N, R, NB, V, J, max_sym;
    int P;               // rows of the state pool per utterance (route.h): the beam's and those of the labels of a frame / an iteration
    NetBuf net[3];
    float *score;        // [NB][B][W]
    int32_t *node, *len, *row; // [NB][N]
    int32_t *free_rows, *n_taken;                         // [B][P], [B]
    v4i *tags;                                            // [B][P]: see QrRouteArgs.tags
    v4i *prog;  float *pred_out, *lm_out;                 // see QrRunArgs; null where the search does not run ahead
    float *nx_score;  v4i *nx_info;  int32_t *nx_count; // [B][R*W], [B]
    int32_t *node_tok, *node_prev;   // [1 + T*max_sym*N]
    int32_t *live;       // [2][max_sym+2]: utterances that carried a label into round v of the frame (early stop)
    v4i *rows;  int32_t *n_rows;   // [N], [2][max_sym+2]: the hypotheses that carry a label into round v of the frame, and how many
    unsigned long long *words;     // [B][n_words]: see QrRoundArgs.words
    size_t n_words;
    int32_t *late;                 // [B]
    size_t n_clear;                // 32-bit words from `live` on that start at zero: live, n_rows, late, words
    size_t total;
};

struct Carver {
    char *base;  size_t off;
    template <typename Tp> Tp *take(size_t n)
    {
        off = (off + 255) / 256 * 256;
        Tp *p = base ? (Tp *)(base + off) : nullptr;
        off += n * sizeof(Tp);
        return p;
    }
};

const qrnnt_net *net_of(const qrnnt_model *m, int k) { return k == 0 ? &m->pred : (k == 1 ? &m->lm_src : &m->lm_ext); }
bool net_used(const qrnnt_model *m, int k) { return k == 0 || (k == 1 ? m->use_src != 0 : m->use_ext != 0); }

// Network buffers: states and outputs of P rows per utterance, one row of zeros behind them.
void take_nets(const qrnnt_model *m, Plan &p, Carver &cv)
{
    const size_t pool = (size_t)p.B * p.P;
    for (int k = 0; k < 3; ++k) {
        if (!net_used(m, k)) continue;
        const qrnnt_net *net = net_of(m, k);
        for (int l = 0; l < net->n_layers; ++l) {
            p.net[k].h[l] = cv.take<int8_t>((pool + 1) * net->layer[l].hidden_size);
            p.net[k].c[l] = cv.take<float>((pool + 1) * net->layer[l].hidden_size);
        }
        p.net[k].gx0 = cv.take<int32_t>((size_t)m->V * 4 * net->layer[0].hidden_size);
        p.net[k].tab0 = cv.take<float>((size_t)m->V * 4 * net->layer[0].hidden_size);
        p.net[k].mid_q = net->mid.packed ? cv.take<int8_t>(pool * net->mid.rows) : nullptr;
    }
}

// What starts at zero, in one piece: two sets of counters, and the words on their way between an utterance's workgroups.
void take_cleared(const qrnnt_model *m, Plan &p, Carver &cv, size_t n_counters)
{
    bool mids = false;
    for (int k = 1; k < 3; ++k) mids = mids || (net_used(m, k) && net_of(m, k)->mid.packed);
    p.n_words = qr_round_words(p.J, net_used(m, 1) || net_used(m, 2), mids, p.B, p.W);
    p.live = cv.take<int32_t>(n_counters);
    const size_t start = cv.off - n_counters * sizeof(int32_t);
    p.n_rows = cv.take<int32_t>(n_counters);
    p.late = p.n_words ? cv.take<int32_t>(p.B) : nullptr;
    p.words = p.n_words ? cv.take<unsigned long long>(p.B * p.n_words) : nullptr;
    p.n_clear = (cv.off - start) / 4;
}

// Which bottlenecks the rounds take in: those of the language models, if there is none in front of the joint.
void place_mids(const qrnnt_model *m, Plan &p, bool alsd)
{
    int n = 0, rows = 0;
    for (int k = 0; k < 3; ++k) {
        p.net[k].mid_in_round = false;
        if (!net_used(m, k) || net_of(m, k)->mid.packed == nullptr) continue;
        ++n;
        rows = k == 0 || net_of(m, k)->mid.rows > rows ? (k == 0 ? 1 << 30 : net_of(m, k)->mid.rows) : rows;
    }
    if (n == 0 || !qr_round_takes(rows, n, p.B, p.W, alsd)) return;
    for (int k = 1; k < 3; ++k) p.net[k].mid_in_round = net_used(m, k) && net_of(m, k)->mid.packed != nullptr;
}

void make_plan(const qrnnt_model *m, int T, int B, int W, int max_sym, void *ws, Plan &p)
{
    p.T = T; p.B = B; p.W = W; p.N = B * W; p.max_sym = max_sym;
    p.R = max_sym + 1; p.NB = max_sym + 2; p.V = m->V; p.J = m->joint_out.cols;
    p.P = W * (max_sym + 1);
    Carver cv{(char *)ws, 0};
    const size_t N = (size_t)p.N, NB = (size_t)p.NB;
    take_nets(m, p, cv);
    p.score = cv.take<float>(NB * N);
    p.node = cv.take<int32_t>(NB * N);
    p.len = cv.take<int32_t>(NB * N);
    p.row = cv.take<int32_t>(NB * N);
    p.free_rows = cv.take<int32_t>((size_t)B * p.P);
    p.n_taken = cv.take<int32_t>(B);
    p.tags = cv.take<v4i>((size_t)B * p.P);
    p.nx_score = cv.take<float>((size_t)B * p.R * W);
    p.nx_info = cv.take<v4i>((size_t)B * p.R * W);
    p.nx_count = cv.take<int32_t>(B);
    const size_t pool = 1 + (size_t)T * max_sym * N;
    p.node_tok = cv.take<int32_t>(pool);
    p.node_prev = cv.take<int32_t>(pool);
    p.rows = cv.take<v4i>(N);
    const bool use_lm = net_used(m, 1) || net_used(m, 2), runs = qr_run_takes(p.J, use_lm, B, W);
    p.pred_out = runs ? cv.take<float>((size_t)B * p.P * p.J) : nullptr;
    p.lm_out = runs && use_lm ? cv.take<float>((size_t)B * p.P * 128) : nullptr;
    p.prog = runs ? cv.take<v4i>(B) : nullptr;
    take_cleared(m, p, cv, 2 * (size_t)(max_sym + 2));
    p.total = (cv.off + 255) / 256 * 256;
}

__global__ void fill_words_kernel(uint32_t *p, size_t n_words, uint32_t v)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_words) p[i] = v;
}

// Start of an utterance: slot 0 holds the empty sequence with score 0 and advances from the zero state (row B*P) into
// the utterance's first row with the start symbol; the other slots are empty.
__global__ void decode_init_kernel(float *score0, int32_t *node0, int32_t *len0, int32_t *row0, int32_t *free_rows, int32_t *n_taken,
                                   v4i *tags, v4i *prog, int32_t *nx_count, v4i *rows, int32_t *n_rows, int32_t *node_tok, int32_t *node_prev,
                                   int W, int B, int P, int start_symbol)
{
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n == 0) { node_tok[0] = -1; node_prev[0] = 0; *n_rows = B; }
    if (n < B) {
        if (nx_count) nx_count[n] = 0;
        if (n_taken) n_taken[n] = 0;
        if (prog) prog[n] = v4i{0, 0, 1 < P ? 1 : 0, 0};
        rows[n] = v4i{n * P, B * P, start_symbol, 0};
    }
    if (n < B * P) {   // (the last entry of an utterance is never looked at)
        const int i = n % P;
        free_rows[n] = i + 1 < P ? n + 1 : n;
        tags[n] = v4i{-1, -1, 0, i == 0 ? 0 : -1};   // the first row's sequence, the empty one, has serial 0
    }
    if (n >= B * W) return;
    score0[n] = (n % W == 0) ? 0.0f : -INFINITY;
    node0[n] = 0;
    len0[n] = 0;
    row0[n] = (n / W) * P;
}

__global__ void backtrack_kernel(const float *__restrict__ score, const int32_t *__restrict__ node,
                                 const int32_t *__restrict__ len, const int32_t *__restrict__ node_tok,
                                 const int32_t *__restrict__ node_prev, int N, int max_len,
                                 int32_t *__restrict__ tokens_out, int32_t *__restrict__ len_out, float *__restrict__ score_out)
{
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    const float sc = score[n];
    const bool live = sc > -INFINITY;
    const int L = live ? len[n] : 0;
    int32_t *out = tokens_out + (size_t)n * max_len;
    for (int i = (L < max_len ? L : max_len); i < max_len; ++i) out[i] = -1;
    int id = node[n];
    for (int i = L - 1; i >= 0; --i) {
        if (i < max_len) out[i] = node_tok[id];
        id = node_prev[id];
    }
    len_out[n] = live ? L : -1;
    score_out[n] = sc;
}

qrnnt_status check_net(const qrnnt_net *net, int V, int out_rows)
{
    QR_REQUIRE(net->embed_codes != nullptr, QRNNT_ERR_NULL);
    QR_REQUIRE(net->n_layers >= 1 && net->n_layers <= QRNNT_MAX_LAYERS, QRNNT_ERR_RANGE);
    QR_REQUIRE(qr_aligned(net->embed_codes, 16), QRNNT_ERR_ALIGN);
    for (int l = 0; l < net->n_layers; ++l) {
        qrnnt_status s = qr_check_lstm(&net->layer[l]);
        if (s != QRNNT_OK) return s;
        QR_REQUIRE(qr_bits(&net->layer[l].w_hh) == 4, QRNNT_ERR_UNSUPPORTED);   // the step kernels unpack nibbles
        if (l > 0) QR_REQUIRE(net->layer[l].input_size == net->layer[l - 1].hidden_size, QRNNT_ERR_SHAPE);
    }
    qrnnt_status s = qr_check_qmat(&net->out, QRNNT_LAYOUT_TILED);
    if (s != QRNNT_OK) return s;
    if (net->mid.packed) {
        s = qr_check_qmat(&net->mid, QRNNT_LAYOUT_TILED);
        if (s != QRNNT_OK) return s;
        QR_REQUIRE(net->mid.cols == net->layer[net->n_layers - 1].hidden_size, QRNNT_ERR_SHAPE);
        QR_REQUIRE(net->mid.rows % 16 == 0 && net->out.cols == net->mid.rows, QRNNT_ERR_SHAPE);
        QR_REQUIRE(net->mid_scale > 0.0f && net->mid_inv_scale > 0.0f, QRNNT_ERR_RANGE);
    } else {
        QR_REQUIRE(net->out.cols == net->layer[net->n_layers - 1].hidden_size, QRNNT_ERR_SHAPE);
    }
    QR_REQUIRE(net->out.rows == out_rows, QRNNT_ERR_SHAPE);
    QR_REQUIRE(!net->log_softmax || net->out.rows <= 64, QRNNT_ERR_UNSUPPORTED);
    QR_REQUIRE(net->out_a_scale > 0.0f, QRNNT_ERR_RANGE);
    (void)V;
    return QRNNT_OK;
}

qrnnt_status check_model(const qrnnt_model *m)
{
    QR_REQUIRE(m != nullptr, QRNNT_ERR_NULL);
    qrnnt_status s = qr_check_qmat(&m->joint_out, QRNNT_LAYOUT_TILED);
    if (s != QRNNT_OK) return s;
    QR_REQUIRE(m->V > 0 && m->V <= 64 && m->joint_out.rows == m->V, QRNNT_ERR_SHAPE);
    QR_REQUIRE(m->joint_out.cols % 16 == 0, QRNNT_ERR_SHAPE);
    QR_REQUIRE(m->blank >= 0 && m->blank < m->V, QRNNT_ERR_RANGE);
    QR_REQUIRE(m->z_scale > 0.0f && m->z_inv_scale > 0.0f, QRNNT_ERR_RANGE);
    s = check_net(&m->pred, m->V, m->joint_out.cols);
    if (s != QRNNT_OK) return s;
    QR_REQUIRE(!m->pred.log_softmax, QRNNT_ERR_RANGE);
    if (m->use_src) { s = check_net(&m->lm_src, m->V, m->V); if (s != QRNNT_OK) return s; }
    if (m->use_ext) { s = check_net(&m->lm_ext, m->V, m->V); if (s != QRNNT_OK) return s; }
    return QRNNT_OK;
}

// The launches of an advance, the same in every round but for the gate and the count: prepared once a search.
struct Advance {
    QrStepGroup layer[QRNNT_MAX_LAYERS];
    int n_layers;
    QrLinearGroup mids;
};

// The networks advance for the *n_rows hypotheses listed in p.rows, (row written, row read, token) each.  Layer l
// of every network goes out as one grouped launch (the networks are independent).
void prepare_advance(const qrnnt_model *m, const Plan &p, Advance &ad)
{
    const int pool = p.B * p.P;
    const int32_t *const from_list = (const int32_t *)p.rows;   // row and token of an entry take the place of these arrays
    int max_layers = 0;
    for (int k = 0; k < 3; ++k)
        if (net_used(m, k) && net_of(m, k)->n_layers > max_layers) max_layers = net_of(m, k)->n_layers;
    ad.n_layers = max_layers;
    for (int l = 0; l < max_layers; ++l) {
        QrStepGroup &g = ad.layer[l];
        g.n = 0;
        g.rows = p.rows;
        for (int k = 0; k < 3; ++k) {
            if (!net_used(m, k)) continue;
            const qrnnt_net *net = net_of(m, k);
            if (l >= net->n_layers) continue;
            const qrnnt_lstm *L = &net->layer[l];
            const size_t H = (size_t)L->hidden_size;
            QrStepArgs &a = g.p[g.n++];
            a = QrStepArgs{};
            qr_fill_lstm_weights(a, L);
            if (l == 0) {
                // The input of layer 0 is one of V embedding rows, so its integer input
                // projection is a table lookup (exactly the sums the contraction would give).
                a.x = net->embed_codes;  a.ld_x = qr_act_pitch(L->input_size);  a.x_row = from_list;  a.n_x_rows = p.V;
                a.gx = p.net[k].gx0;  a.ld_gx = 4 * (int64_t)H;  a.tabf = p.net[k].tab0;
            } else {
                a.x = p.net[k].h[l - 1];  a.ld_x = L->input_size;
                a.x_row = nullptr;  a.n_x_rows = pool;
            }
            a.parent = from_list;  a.n_slots = pool + 1;
            a.h_prev = a.h_next = p.net[k].h[l];  a.ld_hp = a.ld_hn = (int64_t)H;   // no row is both read and written
            a.c_prev = a.c_next = p.net[k].c[l];
            a.N = p.N;  a.n_out = pool;
        }
    }
    // The output layers belong to the round that reads them (joint.hip); a bottleneck in front of one is a layer of the
    // advance, fused with the quantizer of its output.
    QrLinearGroup &lg = ad.mids;
    lg.n = 0;
    lg.rows = p.rows;
    for (int k = 0; k < 3; ++k) {
        if (!net_used(m, k) || net_of(m, k)->mid.packed == nullptr || p.net[k].mid_in_round) continue;
        const qrnnt_net *net = net_of(m, k);
        QrLinearArgs &la = lg.p[lg.n++];
        la = QrLinearArgs{};
        la.w = (const v4i *)net->mid.packed;
        la.nkc = qr_round_up(net->mid.cols, QRNNT_KCHUNK) / QRNNT_KCHUNK;
        la.rows = net->mid.rows;  la.s_w = net->mid.row_scale;  la.bias = net->mid_bias;  la.a_scale = net->out_a_scale;
        la.act = p.net[k].h[net->n_layers - 1];  la.K = net->mid.cols;  la.N = p.N;  la.n_out = pool;
        la.q_out = p.net[k].mid_q;  la.q_inv = net->mid_inv_scale;  la.q_bits = qr_bits(&net->out);  la.w8 = qr_bits(&net->mid) == 8;
    }
}

void advance_nets(Advance &ad, const int32_t *gate, const int32_t *n_rows, hipStream_t st)
{
    for (int l = 0; l < ad.n_layers; ++l) {
        ad.layer[l].gate = gate;
        ad.layer[l].n_rows = n_rows;
        qr_launch_lstm_step_group(ad.layer[l], l == 0, st);
    }
    ad.mids.gate = gate;
    ad.mids.n_rows = n_rows;
    if (ad.mids.n) qr_launch_linear_group(ad.mids, st);
}

// What a diagnostic call changes (qrnnt_diag_decode_shared).
struct RoundDiag {
    int come = 0, n_xcd = 0;
    int32_t *late_out = nullptr;
};

// What a decoding round reads of the model.
QrRoundArgs round_args(const qrnnt_model *m, const Plan &p, const float *enc_proj, const RoundDiag &diag, bool alsd)
{
    QrRoundArgs ja = {};
    for (int k = 0; k < 3; ++k) {
        if (!net_used(m, k)) continue;
        const qrnnt_net *net = net_of(m, k);
        QrHeadArgs &h = ja.head[k];
        h.w = (const v4i *)net->out.packed;  h.s_w = net->out.row_scale;  h.bias = net->out_bias;
        h.K = net->out.cols;  h.nkc = qr_round_up(net->out.cols, QRNNT_KCHUNK) / QRNNT_KCHUNK;
        h.w8 = qr_bits(&net->out) == 8;  h.log_softmax = net->log_softmax;
        h.act = net->mid.packed ? p.net[k].mid_q : p.net[k].h[net->n_layers - 1];
        h.a_scale = net->mid.packed ? net->mid_scale : net->out_a_scale;
        if (!p.net[k].mid_in_round) continue;
        QrMidArgs &d = ja.mid[k - 1];
        d.w = (const v4i *)net->mid.packed;  d.s_w = net->mid.row_scale;  d.bias = net->mid_bias;
        d.act = p.net[k].h[net->n_layers - 1];  d.K = net->mid.cols;  d.nkc = qr_round_up(net->mid.cols, QRNNT_KCHUNK) / QRNNT_KCHUNK;
        d.rows = net->mid.rows;  d.w8 = qr_bits(&net->mid) == 8;  d.q_bits = qr_bits(&net->out);
        d.a_scale = net->out_a_scale;  d.q_inv = net->mid_inv_scale;
    }
    ja.enc = enc_proj;
    ja.w = (const v4i *)m->joint_out.packed;  ja.s_w = m->joint_out.row_scale;  ja.b_out = m->joint_bias;
    ja.z_scale = m->z_scale;  ja.z_inv = m->z_inv_scale;
    ja.lambda_src = m->lambda_src;  ja.lambda_ext = m->lambda_ext;  ja.rho = m->rho;
    ja.J = p.J;  ja.V = p.V;  ja.blank = m->blank;
    ja.nkc = qr_round_up(p.J, QRNNT_KCHUNK) / QRNNT_KCHUNK;
    ja.w8 = qr_bits(&m->joint_out) == 8;
    ja.words = p.words;  ja.n_words = p.n_words;  ja.late = p.late;
    ja.ticks = diag.come == 1 ? 10 : 1000;   // 10 us; the other workgroups need 3
    ja.come = diag.come;
    qr_plan_round(ja, p.B, p.W, alsd);
    ja.n_xcd = diag.n_xcd ? diag.n_xcd : ja.n_xcd;
    return ja;
}

// The end of a diagnostic call: how many rounds of each utterance had a word come late.
void report_late(const Plan &p, const RoundDiag &diag, hipStream_t st)
{
    if (diag.late_out && p.late) (void)hipMemcpyAsync(diag.late_out, p.late, (size_t)p.B * sizeof(int32_t), hipMemcpyDeviceToDevice, st);
}

// Everything a search starts from: a row of zero states, the first layers' input tables, empty counters and lists
// and the start symbol consumed by the empty sequence of every utterance.
void start_decode(const qrnnt_model *m, const Plan &p, Advance &ad, int32_t *n_taken, int32_t *nx_count, hipStream_t st)
{
    auto fill = [&](void *at, size_t nw) {
        fill_words_kernel<<<(unsigned)((nw + 255) / 256), 256, 0, st>>>((uint32_t *)at, nw, 0u);
    };
    const size_t pool = (size_t)p.B * p.P;
    for (int k = 0; k < 3; ++k) {
        if (!net_used(m, k)) continue;
        const qrnnt_net *net = net_of(m, k);
        for (int l = 0; l < net->n_layers; ++l) {
            const size_t H = (size_t)net->layer[l].hidden_size;
            fill(p.net[k].h[l] + pool * H, H / 4);
            fill(p.net[k].c[l] + pool * H, H);
        }
        qr_launch_input_projection(&net->layer[0], net->embed_codes, p.V, p.net[k].gx0, nullptr, st);
        qr_launch_gx_table(&net->layer[0], p.net[k].gx0, p.V, p.net[k].tab0, st);
    }
    fill(p.live, p.n_clear);
    // the start symbol's list is counted in the first counter, which no round uses
    decode_init_kernel<<<(unsigned)((pool + 255) / 256), 256, 0, st>>>(p.score, p.node, p.len, p.row, p.free_rows, n_taken, p.tags, p.prog, nx_count,
                                                                       p.rows, p.n_rows, p.node_tok, p.node_prev, p.W, p.B, p.P,
                                                                       m->blank);
    prepare_advance(m, p, ad);
    advance_nets(ad, nullptr, p.n_rows, st);
}

}  // namespace

extern "C" size_t qrnnt_decode_workspace(const qrnnt_model *m, int32_t T, int32_t B, int32_t W, int32_t max_sym)
{
    if (check_model(m) != QRNNT_OK || T <= 0 || B <= 0 || W <= 0 || W > 64 || max_sym < 0) return 0;
    Plan p;
    make_plan(m, T, B, W, max_sym, nullptr, p);
    return p.total;
}

extern "C" qrnnt_status qrnnt_decode(const qrnnt_model *m, const float *enc_proj, int32_t T, int32_t B, int32_t W,
                                     int32_t max_sym, int32_t max_len, int32_t *tokens_out, int32_t *len_out,
                                     float *score_out, void *workspace, size_t workspace_bytes, void *stream)
{
    return qrnnt_decode_ex(m, enc_proj, T, B, W, max_sym, max_len, 0u, tokens_out, len_out, score_out, workspace,
                           workspace_bytes, stream);
}

static qrnnt_status time_synchronous(const qrnnt_model *m, const float *enc_proj, int32_t T, int32_t B, int32_t W,
                                     int32_t max_sym, int32_t max_len, uint32_t flags, int32_t *tokens_out,
                                     int32_t *len_out, float *score_out, void *workspace, size_t workspace_bytes,
                                     void *stream, const RoundDiag &diag = {})
{
    qrnnt_status s = check_model(m);
    if (s != QRNNT_OK) return s;
    QR_REQUIRE(enc_proj && tokens_out && len_out && score_out && workspace, QRNNT_ERR_NULL);
    QR_REQUIRE(T > 0 && B > 0 && W > 0 && max_len > 0, QRNNT_ERR_SHAPE);
    QR_REQUIRE(W <= 64, QRNNT_ERR_UNSUPPORTED);
    QR_REQUIRE(max_sym >= 0 && max_sym <= 16, QRNNT_ERR_RANGE);
    QR_REQUIRE((flags & ~(uint32_t)QRNNT_DECODE_EARLY_STOP) == 0u, QRNNT_ERR_RANGE);
    const bool early = (flags & QRNNT_DECODE_EARLY_STOP) != 0u;
    QR_REQUIRE((double)T * (max_sym > 0 ? max_sym : 1) * B * W < 2.0e9, QRNNT_ERR_UNSUPPORTED);
    QR_REQUIRE(qr_aligned(enc_proj, 16) && qr_aligned(workspace, 256), QRNNT_ERR_ALIGN);
    Plan p;
    make_plan(m, T, B, W, max_sym, workspace, p);
    QR_REQUIRE(workspace_bytes >= p.total, QRNNT_ERR_WORKSPACE);
    place_mids(m, p, false);
    hipStream_t st = (hipStream_t)stream;
    const int N = p.N, V = p.V;
    const size_t Ns = (size_t)N;
    const int ZB = p.NB - 1;   // the beam's buffer in every second frame (else 0)

    Advance ad;
    start_decode(m, p, ad, p.n_taken, p.nx_count, st);

    QrRoundArgs ja = round_args(m, p, enc_proj, diag, false);

    // Beams of up to 16 run ahead until the networks have to advance, which is after a frame's last round never the case.
    if (const int wgs = p.prog ? qr_plan_run(ja, B, W) : 0) {
        QrRunArgs r = {};
        r.B = B;  r.W = W;  r.P = p.P;  r.T = T;  r.max_sym = max_sym;  r.n_entries = p.R * W;
        r.every_round = diag.come > 0 && diag.late_out;   // (rounds to be counted)
        r.prog = p.prog;  r.score = p.score;  r.node = p.node;  r.len = p.len;  r.row = p.row;
        r.tags = p.tags;  r.nx_score = p.nx_score;  r.nx_info = p.nx_info;
        r.node_tok = p.node_tok;  r.node_prev = p.node_prev;
        r.pred_out = p.pred_out;  r.lm_out = p.lm_out;  r.rows_next = p.rows;
        // An utterance that does not have to wait makes the others wait for the launch it is in: six rounds of a large batch
        // (64 x 1000 frames, ms: 4 rounds 73.3, 6 69.9, 8 74.3, 12 81.6, 20 98; 13 x 301, wider networks: 26.6, 24.0, 25.0, 26.8,
        // 31.1), more of few utterances (5 at beam 1: 5.3, -, 4.5, 4.7, 4.3, 40 4.2; 1 x 152: 8.9, -, 8.0, 7.3, 7.1, 40 7.1).
        r.max_rounds = 64 / B < 6 ? 6 : (64 / B > 20 ? 20 : 64 / B);
        const int64_t n = r.every_round ? (int64_t)T * p.R : (int64_t)T * max_sym + (T + r.max_rounds - 1) / r.max_rounds + 1;
        r.n_through = p.live;
        // As many launches as the search can need, of which it mostly needs a small part.  The host never waits for the search;
        // where it happens to see that the search is through, it leaves out what it has not enqueued yet.
        qr_take_ticket(r, st);
        for (int64_t i = 0; i < n && qr_how_far(r) != ~0u; ++i) {
            ja.round = 1u + (unsigned)i;
            r.n_rows_next = p.n_rows + 1 + i % 3;   // (the first counter is the start symbol's)
            r.n_rows_clear = p.n_rows + 1 + (i + 1) % 3;
            ja.row = p.row;
            qr_launch_search_run(ja, r, wgs, st);
            if (i + 1 < n) advance_nets(ad, nullptr, r.n_rows_next, st);
        }
        backtrack_kernel<<<(N + 63) / 64, 64, 0, st>>>(p.score, p.node, p.len, p.node_tok, p.node_prev, N, max_len, tokens_out, len_out, score_out);
        report_late(p, diag, st);
        return qr_launch_status();
    }

    int a0 = 0;   // buffer of the beam at the current frame
    for (int t = 0; t < T; ++t) {
        for (int v = 0; v <= max_sym; ++v) {
            const int cur = (v == 0) ? a0 : v;
            const int nxt = v + 1;   // only used when v < max_sym
            ja.frame_base = t * B;
            ja.row = p.row + (size_t)cur * Ns;
            ja.round = 1u + (unsigned)t * p.R + v;
            const int last = (v == max_sym);
            QrRouteArgs ra = {};
            ra.score_src = p.score + (size_t)cur * Ns;
            ra.B = B;  ra.W = W;  ra.V = V;  ra.R = p.R;  ra.blank = m->blank;  ra.last_round = last;
            ra.node_base = 1 + (t * max_sym + v) * N;
            ra.node_src = p.node + (size_t)cur * Ns;  ra.len_src = p.len + (size_t)cur * Ns;
            ra.score_dst = p.score + (size_t)nxt * Ns;  ra.node_dst = p.node + (size_t)nxt * Ns;
            ra.len_dst = p.len + (size_t)nxt * Ns;
            ra.row_src = p.row + (size_t)cur * Ns;  ra.row_dst = p.row + (size_t)nxt * Ns;
            ra.P = p.P;  ra.free_rows = p.free_rows;  ra.n_taken = p.n_taken;
            ra.tags = p.tags;  ra.serial0 = (t * max_sym + v) * W;  ra.now = t;
            ra.nx_score = p.nx_score;  ra.nx_info = p.nx_info;  ra.nx_count = p.nx_count;
            ra.node_tok = p.node_tok;  ra.node_prev = p.node_prev;
            ra.fe_dst_buf = (a0 == 0) ? ZB : 0;
            ra.fe_score_all = p.score;
            ra.fe_node_all_w = p.node;  ra.fe_len_all_w = p.len;  ra.fe_row_all_w = p.row;
            if (early) {   // live[t&1][v] = utterances that carried a label into round v of this frame
                int32_t *lv = p.live + (size_t)(t & 1) * (max_sym + 2), *lo = p.live + (size_t)((t + 1) & 1) * (max_sym + 2);
                ra.gate = v > 0 ? lv + v : nullptr;
                ra.live_next = lv + v + 1;
                ra.live_clear = lo + v + 1;
            }
            // n_rows[t&1][v] = hypotheses that carry a label into round v of this frame, listed in p.rows
            ra.rows_next = p.rows;
            ra.n_rows_next = p.n_rows + (size_t)(t & 1) * (max_sym + 2) + v + 1;
            ra.n_rows_clear = p.n_rows + (size_t)((t + 1) & 1) * (max_sym + 2) + v + 1;
            qr_launch_search_round(ja, ra, st);
            if (!last) advance_nets(ad, early ? ra.live_next : nullptr, ra.n_rows_next, st);
        }
        a0 = (a0 == 0) ? ZB : 0;   // the new beam's buffer
    }
    backtrack_kernel<<<(N + 63) / 64, 64, 0, st>>>(p.score + (size_t)a0 * Ns, p.node + (size_t)a0 * Ns,
                                                   p.len + (size_t)a0 * Ns, p.node_tok, p.node_prev, N, max_len,
                                                   tokens_out, len_out, score_out);
    report_late(p, diag, st);
    return qr_launch_status();
}

extern "C" qrnnt_status qrnnt_decode_ex(const qrnnt_model *m, const float *enc_proj, int32_t T, int32_t B, int32_t W,
                                        int32_t max_sym, int32_t max_len, uint32_t flags, int32_t *tokens_out,
                                        int32_t *len_out, float *score_out, void *workspace, size_t workspace_bytes,
                                        void *stream)
{
    return time_synchronous(m, enc_proj, T, B, W, max_sym, max_len, flags, tokens_out, len_out, score_out, workspace,
                            workspace_bytes, stream);
}

// ---------------------------------------------------------------------------------------------------------
// Alignment-length synchronous search with recombination (Sec. 2: the search the paper decodes with).

namespace {

struct AlsdPlan {
    Plan p;                        // network buffers, beam (2 buffers), label trie, lists
    unsigned long long *hash;      // [2][N]
    float *fin_score;  int32_t *fin_node, *fin_len;   // [N]
    int n_iter;
};

void make_alsd_plan(const qrnnt_model *m, int T, int B, int W, int u_max, void *ws, AlsdPlan &ap)
{
    Plan &p = ap.p;
    p = Plan{};
    p.T = T; p.B = B; p.W = W; p.N = B * W; p.max_sym = 0;
    p.R = 1; p.NB = 2; p.V = m->V; p.J = m->joint_out.cols;
    p.P = QR_ALSD_ROWS * W;   // the beam's rows and those of an iteration's labels
    ap.n_iter = T + u_max;
    Carver cv{(char *)ws, 0};
    const size_t N = (size_t)p.N, NB = 2;
    take_nets(m, p, cv);
    p.score = cv.take<float>(NB * N);
    p.node = cv.take<int32_t>(NB * N);
    p.len = cv.take<int32_t>(NB * N);
    ap.hash = cv.take<unsigned long long>(NB * N);
    p.row = cv.take<int32_t>(NB * N);
    p.free_rows = cv.take<int32_t>((size_t)B * p.P);
    p.tags = cv.take<v4i>((size_t)B * p.P);
    ap.fin_score = cv.take<float>(N);
    ap.fin_node = cv.take<int32_t>(N);
    ap.fin_len = cv.take<int32_t>(N);
    const size_t pool = 1 + (size_t)ap.n_iter * N;
    p.node_tok = cv.take<int32_t>(pool);
    p.node_prev = cv.take<int32_t>(pool);
    p.rows = cv.take<v4i>(N);
    take_cleared(m, p, cv, (size_t)ap.n_iter + 2);
    p.total = (cv.off + 255) / 256 * 256;
}

bool alsd_args_ok(int32_t T, int32_t B, int32_t W, int32_t u_max)
{
    return T > 0 && B > 0 && W > 0 && W <= 64 && u_max >= 0 && (double)(T + (double)u_max) * B * W < 2.0e9;
}

}  // namespace

extern "C" size_t qrnnt_decode_alsd_workspace(const qrnnt_model *m, int32_t T, int32_t B, int32_t W, int32_t u_max)
{
    if (check_model(m) != QRNNT_OK || !alsd_args_ok(T, B, W, u_max)) return 0;
    AlsdPlan ap;
    make_alsd_plan(m, T, B, W, u_max, nullptr, ap);
    return ap.p.total;
}

extern "C" qrnnt_status qrnnt_decode_alsd(const qrnnt_model *m, const float *enc_proj, int32_t T, int32_t B, int32_t W,
                                          int32_t u_max, int32_t max_len, int32_t *tokens_out, int32_t *len_out,
                                          float *score_out, void *workspace, size_t workspace_bytes, void *stream)
{
    return qrnnt_decode_alsd_ex(m, enc_proj, T, B, W, u_max, max_len, 0u, nullptr, tokens_out, len_out, score_out,
                                workspace, workspace_bytes, stream);
}

static qrnnt_status alignment_length_synchronous(const qrnnt_model *m, const float *enc_proj, int32_t T, int32_t B, int32_t W,
                                                 int32_t u_max, int32_t max_len, uint32_t flags, int32_t *stats,
                                                 int32_t *tokens_out, int32_t *len_out, float *score_out, void *workspace,
                                                 size_t workspace_bytes, void *stream, const RoundDiag &diag = {})
{
    qrnnt_status s = check_model(m);
    if (s != QRNNT_OK) return s;
    QR_REQUIRE((flags & ~(uint32_t)QRNNT_ALSD_REUSE) == 0u, QRNNT_ERR_RANGE);
    QR_REQUIRE(qr_aligned(stats, 4), QRNNT_ERR_ALIGN);
    QR_REQUIRE(enc_proj && tokens_out && len_out && score_out && workspace, QRNNT_ERR_NULL);
    QR_REQUIRE(T > 0 && B > 0 && W > 0 && max_len > 0 && u_max >= 0, QRNNT_ERR_SHAPE);
    QR_REQUIRE(W <= 64, QRNNT_ERR_UNSUPPORTED);
    QR_REQUIRE(alsd_args_ok(T, B, W, u_max), QRNNT_ERR_UNSUPPORTED);
    QR_REQUIRE(qr_aligned(enc_proj, 16) && qr_aligned(workspace, 256), QRNNT_ERR_ALIGN);
    AlsdPlan ap;
    make_alsd_plan(m, T, B, W, u_max, workspace, ap);
    const Plan &p = ap.p;
    QR_REQUIRE(workspace_bytes >= p.total, QRNNT_ERR_WORKSPACE);
    place_mids(m, ap.p, true);
    hipStream_t st = (hipStream_t)stream;
    const int N = p.N, V = p.V;
    const size_t Ns = (size_t)N;

    {
        const size_t nw = 2 * Ns * 2;
        fill_words_kernel<<<(unsigned)((nw + 255) / 256), 256, 0, st>>>((uint32_t *)ap.hash, nw, 0u);
        fill_words_kernel<<<(unsigned)((Ns + 255) / 256), 256, 0, st>>>((uint32_t *)ap.fin_score, Ns, 0xFF800000u);   // -inf
        fill_words_kernel<<<(unsigned)((Ns + 255) / 256), 256, 0, st>>>((uint32_t *)ap.fin_node, Ns, 0u);
        fill_words_kernel<<<(unsigned)((Ns + 255) / 256), 256, 0, st>>>((uint32_t *)ap.fin_len, Ns, 0u);
    }
    Advance ad;
    start_decode(m, p, ad, nullptr, nullptr, st);

    QrRoundArgs ja = round_args(m, p, enc_proj, diag, true);

    int cur = 0;
    for (int i = 0; i < ap.n_iter; ++i) {
        const int nxt = cur ^ 1;
        ja.row = p.row + (size_t)cur * Ns;
        ja.round = 1u + (unsigned)i;
        QrRouteArgs ra = {};
        ra.score_src = p.score + (size_t)cur * Ns;
        ra.B = B;  ra.W = W;  ra.V = V;  ra.R = 1;  ra.blank = m->blank;  ra.last_round = 0;
        ra.node_base = 1 + i * N;
        ra.node_src = p.node + (size_t)cur * Ns;  ra.len_src = p.len + (size_t)cur * Ns;
        ra.score_dst = p.score + (size_t)nxt * Ns;  ra.node_dst = p.node + (size_t)nxt * Ns;
        ra.len_dst = p.len + (size_t)nxt * Ns;
        ra.row_src = p.row + (size_t)cur * Ns;  ra.row_dst = p.row + (size_t)nxt * Ns;
        ra.P = p.P;  ra.free_rows = p.free_rows;
        ra.tags = p.tags;  ra.serial0 = i * W;  ra.now = i;
        ra.node_tok = p.node_tok;  ra.node_prev = p.node_prev;
        ra.gate = i > 0 ? p.live + i : nullptr;   // live[i]: utterances with a live hypothesis entering iteration i
        ra.live_next = p.live + i + 1;
        ra.rows_next = p.rows;  ra.n_rows_next = p.n_rows + i + 1;
        QrAlsdArgs sa = {};
        sa.iter = i;  sa.T = T;  sa.u_max = u_max;
        sa.hash_src = ap.hash + (size_t)cur * Ns;  sa.hash_dst = ap.hash + (size_t)nxt * Ns;
        sa.fin_score = ap.fin_score;  sa.fin_node = ap.fin_node;  sa.fin_len = ap.fin_len;
        sa.reuse = (flags & QRNNT_ALSD_REUSE) ? 1 : 0;  sa.stats = stats;
        qr_launch_search_round_alsd(ja, ra, sa, st);
        if (i + 1 < ap.n_iter) advance_nets(ad, ra.live_next, ra.n_rows_next, st);
        cur = nxt;
    }
    backtrack_kernel<<<(N + 63) / 64, 64, 0, st>>>(ap.fin_score, ap.fin_node, ap.fin_len, p.node_tok, p.node_prev, N,
                                                   max_len, tokens_out, len_out, score_out);
    report_late(p, diag, st);
    return qr_launch_status();
}

extern "C" qrnnt_status qrnnt_decode_alsd_ex(const qrnnt_model *m, const float *enc_proj, int32_t T, int32_t B, int32_t W,
                                             int32_t u_max, int32_t max_len, uint32_t flags, int32_t *stats,
                                             int32_t *tokens_out, int32_t *len_out, float *score_out, void *workspace,
                                             size_t workspace_bytes, void *stream)
{
    return alignment_length_synchronous(m, enc_proj, T, B, W, u_max, max_len, flags, stats, tokens_out, len_out, score_out,
                                        workspace, workspace_bytes, stream);
}

static qrnnt_status diag_decode(const qrnnt_model *m, const float *enc_proj, int32_t T, int32_t B, int32_t W, int32_t alsd, int32_t limit,
                                int32_t max_len, int32_t *tokens_out, int32_t *len_out, float *score_out, void *workspace,
                                size_t workspace_bytes, void *stream, const RoundDiag &diag)
{
    return alsd ? alignment_length_synchronous(m, enc_proj, T, B, W, limit, max_len, 0u, nullptr, tokens_out, len_out, score_out,
                                               workspace, workspace_bytes, stream, diag)
                : time_synchronous(m, enc_proj, T, B, W, limit, max_len, 0u, tokens_out, len_out, score_out, workspace,
                                   workspace_bytes, stream, diag);
}

extern "C" qrnnt_status qrnnt_diag_decode(const qrnnt_model *m, const float *enc_proj, int32_t T, int32_t B, int32_t W,
                                          int32_t alsd, int32_t limit, int32_t max_len, int32_t *tokens_out, int32_t *len_out,
                                          float *score_out, void *workspace, size_t workspace_bytes, void *stream)
{
    RoundDiag diag;
    diag.come = 1;
    return diag_decode(m, enc_proj, T, B, W, alsd, limit, max_len, tokens_out, len_out, score_out, workspace, workspace_bytes, stream, diag);
}

extern "C" qrnnt_status qrnnt_diag_decode_shared(const qrnnt_model *m, const float *enc_proj, int32_t T, int32_t B, int32_t W,
                                                 int32_t alsd, int32_t limit, int32_t max_len, int32_t come, int32_t n_xcd,
                                                 int32_t *late_out, int32_t *tokens_out, int32_t *len_out, float *score_out,
                                                 void *workspace, size_t workspace_bytes, void *stream)
{
    QR_REQUIRE(come >= 0 && n_xcd >= 0 && n_xcd <= 32, QRNNT_ERR_RANGE);
    RoundDiag diag;
    diag.come = come;
    diag.n_xcd = n_xcd;
    diag.late_out = late_out;
    return diag_decode(m, enc_proj, T, B, W, alsd, limit, max_len, tokens_out, len_out, score_out, workspace, workspace_bytes, stream, diag);
}
