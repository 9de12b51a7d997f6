// Joint network, log-softmax and density-ratio fusion in one kernel (Sec. 2:
// encoder and prediction outputs are combined multiplicatively, a linear layer
// and a log-softmax follow; Eq. 1 adds the weighted LM log-probabilities).
#include <atomic>
#include <mutex>
#include <type_traits>

#include "head.h"
#include "kernels.h"
#include "round.h"
#include "route.h"
#include "select.h"

namespace {

// The 16 encoder and 16 prediction values of one lane's K block, as loaded.
struct QrJointRaw {
    v4f e[4], p[4];
};

// One block (4 waves) per 16 hypotheses; the J columns are dealt to the waves in
// 64-column blocks.  Lane (col, grp) produces the 16 codes of z that are its own
// MFMA operand for that block, so z never leaves registers; partial sums meet in
// wave 0, which holds all V <= 64 rows of the output layer for the log-softmax.
__global__ __launch_bounds__(256) void joint_fuse_kernel(const QrJointArgs a)
{
    __shared__ v4i lds[4 * 4 * 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, grp = lane >> 4;
    int n = blockIdx.x * 16 + col;
    const bool nv = n < a.N;
    n = nv ? n : a.N - 1;
    int fr = a.frame_row ? a.frame_row[n] : a.frame_base + n / a.rows_per_utt;
    fr = fr < 0 ? 0 : (fr >= a.n_enc_rows ? a.n_enc_rows - 1 : fr);
    const float *e = a.enc + (int64_t)fr * a.J + grp * 16;
    const float *p = a.pred + (int64_t)n * a.J + grp * 16;
    int8_t *zq = a.dbg_zq ? a.dbg_zq + (int64_t)n * a.J + grp * 16 : nullptr;
    const int J = a.J;
    const float z_inv = a.z_inv;
    const int zbits = a.w8 ? 8 : 4;
    auto bload = [&](int kb) -> QrJointRaw {
        QrJointRaw raw = {};
        if (kb * 64 + grp * 16 < J) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                raw.e[d] = *(const v4f *)(e + kb * 64 + 4 * d);
                raw.p[d] = *(const v4f *)(p + kb * 64 + 4 * d);
            }
        }
        return raw;
    };
    auto bmake = [&](const QrJointRaw &raw, int kb) -> v4i {
        v4i b = {0, 0, 0, 0};
        if (kb * 64 + grp * 16 < J) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t word = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float z = qr_tanh(raw.e[d][i] * raw.p[d][i]);
                    word |= (uint32_t)(qr_quant(z, z_inv, zbits) & 0xFF) << (8 * i);
                }
                b[d] = (int)word;
            }
            if (zq && nv) *(v4i *)(zq + kb * 64) = b;
        }
        return b;
    };
    const int n_row_tiles = (a.V + 15) >> 4;
    v4i acc[4];
    qr_head_mma<1>(a.w, a.nkc, n_row_tiles, 0, J, bload, bmake, [] {}, acc, lds, a.w8 != 0);
    if (wave != 0) return;

    float v[4][4];
    float m = -INFINITY;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = mt * 16 + grp * 4 + i;
            if (k < a.V) {
                v[mt][i] = (a.z_scale * a.s_w[k]) * (float)acc[mt][i] + (a.b_out ? a.b_out[k] : 0.0f);
                m = fmaxf(m, v[mt][i]);
            } else {
                v[mt][i] = -INFINITY;
            }
        }
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    float sum = 0.0f;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) sum += (mt * 16 + grp * 4 + i < a.V) ? qr_exp(v[mt][i] - m) : 0.0f;
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    const float lse = m + qr_log(sum);
    if (!nv) return;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = mt * 16 + grp * 4 + i;
            if (k >= a.V) continue;
            const float lp = v[mt][i] - lse;
            float f = lp;
            if (k != a.blank) {
                if (a.lp_src) f -= a.lambda_src * a.lp_src[(int64_t)n * a.V + k];
                if (a.lp_ext) f += a.lambda_ext * a.lp_ext[(int64_t)n * a.V + k];
                f += a.rho;
            }
            if (a.lp_out) a.lp_out[(int64_t)n * a.V + k] = lp;
            a.fused[(int64_t)n * a.V + k] = f;
        }
}

// An utterance's workgroups (512 threads) beside the first: contractions whose results go to it as words.  The first one
// uses the same pieces where they have not come in time.
struct QrShare {
    const QrRoundArgs &a;
    v4i (*sums)[4][64];              // LDS, [8]: partial sums of the waves
    int8_t (*mid_code)[16][272];     // LDS, [2]: codes of the language models' bottlenecks
    float (*jc)[2][64];              // LDS, [3]: row scales and biases of the joint, source LM, external LM
    int *missed;                     // LDS
    int b, V;

    __device__ __forceinline__ int lane() const { return threadIdx.x & 63; }
    __device__ __forceinline__ int wave() const { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
    // this thread's hypothesis and first column of 64, where a workgroup deals 64 rows of 16 hypotheses to its threads
    __device__ __forceinline__ int z_lane() const { return (threadIdx.x >> 1) & 63; }
    __device__ __forceinline__ int z_hyp() const { return z_lane() & 15; }
    __device__ __forceinline__ int z_col() const { return (int)(threadIdx.x >> 7) * 16 + 4 * (z_lane() >> 4) + 2 * (int)(threadIdx.x & 1); }
    __device__ __forceinline__ int row_tiles() const { return (V + 15) >> 4; }

    // Words on their way between the workgroups: source q, hypothesis, token (of a bottleneck: four codes to a word).
    __device__ __forceinline__ unsigned long long *word_at(int q, int hyp, int token) const
    {
        return a.words + b * a.n_words + (q * 16 + hyp) * 64 + token;
    }
    // A wait for words has lasted `limit` (a quarter of the time at first): true if it is enough.
    __device__ __forceinline__ bool enough(unsigned &limit) const
    {
        if (limit == (unsigned)a.ticks || a.late[b] >= 8) return true;   // uniform
        limit = (unsigned)a.ticks;
        return false;
    }
    // row scales and biases of the joint (q = 0) or a language model into LDS, by one wave
    __device__ __forceinline__ void row_constants(int q) const
    {
        const int kk = lane() < V ? lane() : V - 1;
        const float *sw = q == 0 ? a.s_w : a.head[q].s_w, *bs = q == 0 ? a.b_out : a.head[q].bias;
        jc[q][0][lane()] = sw ? (q == 0 ? a.z_scale : a.head[q].a_scale) * sw[kk] : 0.0f;
        jc[q][1][lane()] = bs ? bs[kk] : 0.0f;
    }
    // Contraction of output layer h by this wave: chunks c0, c0 + step, ...; NB of them in flight
    template <int NB>
    __device__ __forceinline__ void head_mma(const QrHeadArgs &h, int row, int c0, int step, v4i (&acc)[4]) const
    {
        constexpr int NB8 = NB > 1 ? NB / 2 : 1;
        unsigned woff[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const int rt = mt < row_tiles() ? mt : row_tiles() - 1;
            woff[mt] = (unsigned)rt * h.nkc * (h.w8 ? 2048 : 1024) + lane() * 16;
        }
        const int grp = lane() >> 4;
        if (h.w8) qr_chunk_mma<true, NB8>(h.w, woff, h.act, row, h.K, h.nkc, c0, step, grp, acc, [] {});
        else qr_chunk_mma<false, NB>(h.w, woff, h.act, row, h.K, h.nkc, c0, step, grp, acc, [] {});
    }
    // where a lane's sums of row tile mt go, and where the thread of the scores with hypothesis hc finds those of its quad
    __device__ __forceinline__ void put_sums(const v4i (&acc)[4]) const
    {
        const int col = lane() & 15, grp = lane() >> 4;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) sums[wave()][mt][grp * 16 + (col ^ (4 * mt + grp))] = acc[mt];
    }
    // 64 rows (block `part`) of output layer or bottleneck h (K dealt to the eight waves), added up: this thread's two sums.
    // meanwhile(): loads that arrive while the sums meet
    template <int NB, class Args, class Meanwhile>
    __device__ __forceinline__ void block_sums(const Args &h, int n_tiles, int part, int row, int &s0, int &s1, Meanwhile &&meanwhile) const
    {
        unsigned woff[4];   // (a matrix of 2 GiB would have to have 4 million rows)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const int rt = 4 * part + mt < n_tiles ? 4 * part + mt : n_tiles - 1;
            woff[mt] = (unsigned)rt * h.nkc * (h.w8 ? 2048 : 1024) + lane() * 16;
        }
        const v4i zero = {0, 0, 0, 0};
        const int grp = lane() >> 4;
        v4i acc[4] = {zero, zero, zero, zero};
        if (h.w8) qr_chunk_mma<true, 1>(h.w, woff, h.act, row, h.K, h.nkc, wave(), 8, grp, acc, [] {});
        else qr_chunk_mma<false, NB>(h.w, woff, h.act, row, h.K, h.nkc, wave(), 8, grp, acc, [] {});
        meanwhile();
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) sums[wave()][mt][lane()] = acc[mt];
        __syncthreads();
        s0 = s1 = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const int *const q = (const int *)&sums[w][threadIdx.x >> 7][z_lane()] + 2 * (threadIdx.x & 1);
            s0 += q[0];
            s1 += q[1];
        }
        s0 = h.w8 ? s0 : (s0 >> 4);   // 4-bit operands carry a factor 16
        s1 = h.w8 ? s1 : (s1 >> 4);
    }
    // 64 rows of the bottleneck of language model 1 + net: this thread's two codes.
    __device__ __forceinline__ unsigned mid_part(int net, int part, int row) const
    {
        const QrMidArgs &h = a.mid[net];
        const int j = part * 64 + z_col() < h.rows ? part * 64 + z_col() : 0;
        float sw0, sw1, bs0, bs1;
        int s0, s1;
        block_sums<2>(h, h.rows >> 4, part, row, s0, s1, [&]() {
            sw0 = h.a_scale * h.s_w[j];
            sw1 = h.a_scale * h.s_w[j + 1];
            bs0 = h.bias ? h.bias[j] : 0.0f;
            bs1 = h.bias ? h.bias[j + 1] : 0.0f;
        });
        const int c0 = qr_quant(sw0 * (float)s0 + bs0, h.q_inv, h.q_bits), c1 = qr_quant(sw1 * (float)s1 + bs1, h.q_inv, h.q_bits);
        return (unsigned)(c0 & 0xFF) | (unsigned)(c1 & 0xFF) << 8;
    }
    // Output layer of language model 1 + net by this wave, chunks c0, c0 + step, ...; its operand may lie in mid_code.
    __device__ __forceinline__ void lm_mma(int net, int row, int c0, int step, v4i (&acc)[4]) const
    {
        const QrHeadArgs &h = a.head[1 + net];
        if (!h.w) return;   // uniform
        if (!a.mid[net].w) {
            head_mma<2>(h, row, c0, step, acc);
            return;
        }
        const int m = (int)0xF0F0F0F0u, col = lane() & 15, grp = lane() >> 4;
        for (int kc = c0; kc < h.nkc; kc += step) {   // (at most two chunks; columns beyond K meet zero weights)
            const int k = kc * QRNNT_KCHUNK + grp * 16;
            const v4i x0 = *(const v4i *)&mid_code[net][col][k], x1 = *(const v4i *)&mid_code[net][col][k + 64];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const int rt = mt < row_tiles() ? mt : row_tiles() - 1;
                const v4i *const w = h.w + ((size_t)rt * h.nkc + kc) * (h.w8 ? 128 : 64) + lane();
                const v4i f = w[0];
                acc[mt] = qr_mfma(h.w8 ? f : ((f << 4) & m), x0, acc[mt]);
                acc[mt] = qr_mfma(h.w8 ? w[64] : (f & m), x1, acc[mt]);
            }
        }
    }
    // The work of a workgroup for the language models: p = 0, their values (waves 0-3 source, 4-7 external, K split in four);
    // p > 0, 64 rows of a bottleneck.
    __device__ __forceinline__ void send_lm(int p, int row) const
    {
        const int tid = threadIdx.x;
        if (p > 0) {
            --p;
            const int n0 = a.mid[0].w ? (a.mid[0].rows + 63) >> 6 : 0, net = p < n0 ? 0 : 1;
            p -= net ? n0 : 0;
            const unsigned code = mid_part(net, p, row);
            const unsigned next = (unsigned)__builtin_amdgcn_update_dpp(0, (int)code, 0xB1 /* the neighbour's */, 0xf, 0xf, true);
            if ((tid & 1) == 0 && p * 64 + z_col() < a.mid[net].rows)
                qr_send(word_at(QR_ROUND_PARTS + 1 + net, z_hyp(), (p * 64 + z_col()) >> 2), code | next << 16, a.round);
            return;
        }
        const int net = wave() >> 2;
        const QrHeadArgs &h = a.head[1 + net];
        const v4i zero = {0, 0, 0, 0};
        v4i acc[4] = {zero, zero, zero, zero};
        if ((wave() & 3) == 3) row_constants(1 + net);
        if (a.mid[0].w || a.mid[1].w) {                // uniform: the bottlenecks' codes, 16 of a hypothesis to a thread
            if (tid == 0) *missed = 0;
            __syncthreads();
            if (a.mid[net].w) {                        // uniform
                const int hyp = (tid & 255) >> 4, c0 = (tid & 15) * 16;
                const __amdgpu_buffer_rsrc_t area = __builtin_amdgcn_make_buffer_rsrc((void *)word_at(QR_ROUND_PARTS + 1 + net, 0, 0), 0,
                                                                                      16 * 64 * 8, 0x00020000 /* raw bytes */);
                const bool mine = c0 < a.mid[net].rows;
                unsigned limit = (unsigned)a.ticks / 4;
                for (const unsigned long long t0 = wall_clock64();;) {
                    const unsigned off = (unsigned)(hyp * 64 + (tid & 15) * 4) * 8;
                    const v4i u = (v4i)__builtin_amdgcn_raw_buffer_load_b128(area, off, 0, 16 /* sc1 */);
                    const v4i v = (v4i)__builtin_amdgcn_raw_buffer_load_b128(area, off + 16, 0, 16);
                    asm volatile("" ::: "memory");     // every poll loads anew
                    const bool ok = !mine || ((unsigned)u[1] == a.round && (unsigned)u[3] == a.round && (unsigned)v[1] == a.round &&
                                              (unsigned)v[3] == a.round);
                    if (__all(ok)) {
                        *(v4i *)&mid_code[net][hyp][c0] = v4i{u[0], u[2], v[0], v[2]};
                        break;
                    }
                    if (wall_clock64() - t0 > limit && enough(limit)) {
                        if (lane() == 0) *missed = 1;
                        break;
                    }
                }
            }
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(*missed)) return;   // uniform: the first workgroup does it all then
        }
        lm_mma(net, row, wave() & 3, 4, acc);
        put_sums(acc);
        __syncthreads();
        const int hc = (tid & 255) >> 4, quad = lane() & 15, mt = quad >> 2, at = (quad & 3) * 16 + (hc ^ quad);
        v4i t = zero;
#pragma unroll
        for (int k = 0; k < 4; ++k) t += sums[4 * net + k][mt][at];
        const v4f v = qr_token_values(t, h.w8 != 0, jc[1 + net][0], jc[1 + net][1], 4 * quad, V, h.log_softmax != 0);
        qr_send(word_at(net == 0 ? 0 : QR_ROUND_PARTS, hc, 4 * quad),
                v4i{__float_as_int(v[0]), __float_as_int(v[1]), __float_as_int(v[2]), __float_as_int(v[3])}, a.round);
    }
};

// One decoding round of an utterance in one workgroup (or several: see CL): output layers of the three networks, joint,
// log-softmax and fusion for its W hypotheses (NTW column tiles of 16), selection of the W best (parent, token) extensions, routing
// (route.h), and after the last round of a frame the new beam.  In one workgroup nothing touches memory between the networks'
// top hidden codes and the picks.
//   contraction, waves 0-3: the prediction network's output layer and the joint.  A wave owns 64-column blocks of the
//     joint: it contracts the 64 rows of the output layer that produce them, 16 to an MFMA, dealt so that a lane ends
//     up with the 16 consecutive columns that are its operand of the joint's contraction (row r of tile mt is row
//     16*(r/4) + 4*mt + r%4 of the block).
//   contraction, waves 4-5, 6-7: output layer of the source and of the external LM, K split in two.
//   scores, waves 0-3: the partial sums meet in LDS (16-byte pieces swizzled by token quartet); 16 lanes share a
//     hypothesis, four tokens each, and form the three log-softmaxes and the fused score together.
//   selection, waves 0-3: the W-th best of the best ones of 64 groups of candidates or more bounds the W-th best
//     candidate from below; what passes the bound is gathered in LDS and ranked by counting.
// One workgroup (beams of more than 16, more than about 100 utterances) is bound by its chain of dependent steps, and the
// chain by one compute unit's path to L2 (145 KB of weights and 80 KB of codes: 44 KB of them, the prediction network's
// fetched by four waves; 36 bytes a cycle measured) and by single waves running straight-line code, hence the split of every
// step over four waves.  Measured in this form, one utterance at beam 16: 10.1 us, where a launch for the output layers and
// one for joint, selection and routing in single waves took 7.0 + 10.9 us.
// ALSD: the same inside the alignment-length synchronous search (route.h, qr_alsd_route): every hypothesis reads its
// own encoder frame (iteration - labels so far), a blank at the last frame finishes a hypothesis instead of being a
// candidate, labels beyond the cap are no candidates.
// CL (up to 16 hypotheses, and five sixths of the device hold all workgroups; nearer to its limit one workgroup each is the
// faster form, 100 utterances at beam 1 30.7 us a round against 32.1): an utterance has up to QR_ROUND_PARTS workgroups that
// share the joint, 64 columns at a time (its output layer's sums add up), and one that contracts the language models' output
// layers and forms their log-probabilities; the first one collects and goes on alone.  One compute unit's path to L2 no
// longer bounds the round: 36 KB to a share of the joint and 80 KB to the language models (base networks) instead of 225.
// What they send goes through the L2 of the XCD they run on (ids congruent modulo the number of XCDs; nothing but the time
// depends on that), value and round number in one 8-byte word, so that every word says by itself whether it is there: no
// flag, no order of stores.  The others wait for nobody (the one with the language models for bottlenecks only), and nobody
// waits for long: what has not come after `ticks` the first one does itself, and counts the round; where this keeps happening
// (words that stay in another XCD's L2, say) a quarter of the time has to do from then on.  A bottleneck in front of a
// language model's output layer is contracted in the round too, 64 rows to a workgroup (qr_round_takes).  The last round of a
// frame has blanks to offer only, and no use for the language models.  Stamps of the first workgroup (one utterance at beam
// 16, ns after its start, one workgroup -> several): sums of the output layers 5000 -> 2100, scores begin 6100 -> 3600, end
// 9900 -> 7500; a round of three launches 23.3 -> 20.5 us, of 64 utterances (batch of 1000 frames, all rounds) 37.3 -> 36.5.
// (Two workgroups, the second with the language models: the first one's share still took 4.2 us, no gain.)
// TAGS: label picks look for rows that hold their states (route.h); see launch_round.
template <int NTW, bool ALSD, bool CL, bool TAGS = true>
__global__ __launch_bounds__(512, CL ? 4 : 2) void search_round_kernel(const QrRoundArgs a, const QrRouteArgs r, const QrAlsdArgs s)
{
    constexpr int MAX_LIST = ALSD ? 1 : 16 * NTW * 17;   // a frame's candidates: W blanks in each of at most 17 rounds
    __shared__ v4i sums[8][4][64];          // [wave][row tile][lane, swizzled] partial sums; then the gathered candidates
    __shared__ unsigned group_best[NTW * 256];
    __shared__ QrCand list[MAX_LIST], best[64], best_fe[64];
    __shared__ int list_row[MAX_LIST], list_node[MAX_LIST], list_len[MAX_LIST];
    __shared__ float fin_new[64];           // ALSD: value of hypothesis w finishing now
    __shared__ __attribute__((aligned(16))) float jc[3][2][64];   // row scales and biases: joint, source LM, external LM
    __shared__ __attribute__((aligned(16))) float pc[4][2][64];   // [wave] those of the prediction network's 64 rows at hand
    __shared__ __attribute__((aligned(16))) int8_t z_code[CL ? 16 : 1][80];   // a block's codes (the pitch spreads the rows over the banks)
    __shared__ __attribute__((aligned(16))) int8_t mid_code[CL ? 2 : 1][CL ? 16 : 1][272];   // codes of the language models' bottlenecks
    __shared__ v4f lm_val[CL ? 2 : 1][CL ? 256 : 1];   // the language models' values for each thread of the scores
    __shared__ unsigned mask[64];
    constexpr int LOG_SLOTS = !TAGS ? 1 : (NTW == 1 ? 9 : 11);
    __shared__ v4i tag_lds[TAGS ? (16 * NTW * (ALSD ? QR_ALSD_ROWS : 17) + 63) / 64 * 64 : 1];   // (a row of the pool for every candidate of a frame)
    __shared__ unsigned short tag_slot[1 << LOG_SLOTS];
    __shared__ unsigned char tag_twin[1 << LOG_SLOTS];
    const QrTags tags = {tag_lds, tag_slot, tag_twin};
    __shared__ int n_cand, n_list, missed;
    QrCand *const gathered = (QrCand *)&sums[0][0][0];
    static_assert(sizeof(sums) >= 16 * 4 * 64 * sizeof(QrCand), "all candidates of 64 hypotheses x 64 tokens");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    // Grid: x = utterance; CL with several workgroups: x = XCD (workgroups go out with x fastest, each to the next XCD), y =
    // workgroup of the utterance, the first one last (the ones that are waited for go out first), z = XCD's next utterance
    const int b = CL ? (int)(blockIdx.z * gridDim.x + blockIdx.x) : (int)blockIdx.x;
    if (CL && b >= r.B) return;   // uniform
    const int W = r.W, V = a.V, J = a.J;
    const bool frame_end = !ALSD && r.last_round;
    const bool use_lm = !frame_end && (a.head[1].w || a.head[2].w);   // (the last round's candidates are blanks)
    const int n_entries = r.R * W;
    const size_t nx = (size_t)b * n_entries;
    const v4i zero = {0, 0, 0, 0};
    const int m = (int)0xF0F0F0F0u;

    // The new beam of the frame: the W best of the candidate list in LDS (n_list of them) by (score descending,
    // insertion order), each with its trie node, length and pool row; the rows it does not name are free again.
    int first_free = 0;
    // where the next frame's list of free rows begins: behind the row that this one's took last
    auto load_first_free = [&](int taken) {
        const int f = r.free_rows[(size_t)b * r.P + (taken > 0 ? taken - 1 : 0)] - b * r.P + (taken > 0 ? 1 : 0);
        first_free = f < r.P ? f : 0;
    };
    auto finish_frame = [&]() {
        __syncthreads();
        if (wave < 4) qr_rank(list, n_list, W, tid, best_fe);
        __syncthreads();
        if (wave != 0) return;
        const QrCand p = best_fe[lane];
        const bool found = lane < W && p != 0;
        const int c = found ? qr_cand_index(p) : 0;
        int row = b * r.P;
        if (lane < W) {
            const size_t o = (size_t)r.fe_dst_buf * r.B * W + b * W + lane;
            row = found ? list_row[c] : row;
            r.fe_score_all[o] = found ? qr_cand_value(p) : -INFINITY;
            r.fe_node_all_w[o] = found ? list_node[c] : 0;
            r.fe_len_all_w[o] = found ? list_len[c] : 0;
            r.fe_row_all_w[o] = row;
        }
        if (lane == 0) {
            r.nx_count[b] = 0;
            r.n_taken[b] = 0;
        }
        qr_list_free_rows(r, b, lane, found, row, mask, first_free);
    };
    auto list_entry = [&](int e, float v, const v4i &info) {
        list[e] = qr_cand(qr_float_key(v + 0.0f), e);   // + 0: one key per value
        list_row[e] = info[0];
        list_node[e] = info[1];
        list_len[e] = info[2];
    };

    const int n_row_tiles = (V + 15) >> 4;
    const int my_n = b * W + (col < W ? col : W - 1);   // this lane's column of the (first) tile
    QrShare share = {a, sums, (int8_t(*)[16][272])mid_code, jc, &missed, b, V};   // what the workgroups of an utterance do for one another
    auto word_at = [&](int q, int hyp, int token) { return share.word_at(q, hyp, token); };
    auto enough = [&](unsigned &limit) { return share.enough(limit); };

    // CL: this workgroup's share of the joint: blocks of 64 columns first, first + a.parts, ...  A block: the 64 rows of the
    // prediction network's output layer, K dealt to the eight waves; a thread adds up two columns of a hypothesis and forms
    // their codes; waves 0-3 contract the codes with a row tile each of the joint's output layer and return its sums.
    const int z_lane = (tid >> 1) & 63, z_hyp = z_lane & 15, z_col = (tid >> 7) * 16 + 4 * (z_lane >> 4) + 2 * (tid & 1);
    auto joint_part = [&](int first, int row, int len) -> v4i {
        const QrHeadArgs &h = a.head[0];
        const int n_tiles = J >> 4, zbits = a.w8 ? 8 : 4;
        int64_t fr = a.frame_base + b;
        if (ALSD) {   // this hypothesis' own frame
            int t_w = s.iter - len;
            t_w = t_w < 0 ? 0 : (t_w > s.T - 1 ? s.T - 1 : t_w);
            fr = (int64_t)t_w * r.B + b;
        }
        v4i sum = zero;
        for (int jb = first; jb * 64 < J; jb += a.parts) {   // uniform
            const bool jv = jb * 64 + z_col < J;
            const int j = jv ? jb * 64 + z_col : 0;
            unsigned woff[4];   // (a matrix of 2 GiB would have to have 4 million rows)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const int rt = 4 * jb + mt < n_tiles ? 4 * jb + mt : n_tiles - 1;
                woff[mt] = (unsigned)rt * h.nkc * (h.w8 ? 2048 : 1024) + lane * 16;
            }
            v4i acc[4] = {zero, zero, zero, zero};
            if (h.w8) qr_chunk_mma<true, 1>(h.w, woff, h.act, row, h.K, h.nkc, wave, 8, grp, acc, [] {});
            else qr_chunk_mma<false, 1>(h.w, woff, h.act, row, h.K, h.nkc, wave, 8, grp, acc, [] {});
            // what the codes need arrives while the sums meet
            const float *const e = a.enc + fr * J + j;
            const float e0 = e[0], e1 = e[1], sw0 = h.s_w[j], sw1 = h.s_w[j + 1];
            const float bs0 = h.bias ? h.bias[j] : 0.0f, bs1 = h.bias ? h.bias[j + 1] : 0.0f;
            v4i wj = zero;
            if (wave < 4) {
                const int rt = wave < n_row_tiles ? wave : n_row_tiles - 1;
                wj = a.w8 ? a.w[((size_t)rt * a.nkc * 2 + jb) * 64 + lane] : a.w[((size_t)rt * a.nkc + (jb >> 1)) * 64 + lane];
            }
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) sums[wave][mt][lane] = acc[mt];
            __syncthreads();
            int s0 = 0, s1 = 0;
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                const int *const q = (const int *)&sums[w][tid >> 7][z_lane] + 2 * (tid & 1);
                s0 += q[0];
                s1 += q[1];
            }
            s0 = h.w8 ? s0 : (s0 >> 4);   // 4-bit operands carry a factor 16
            s1 = h.w8 ? s1 : (s1 >> 4);
            const float p0 = (h.a_scale * sw0) * (float)s0 + bs0, p1 = (h.a_scale * sw1) * (float)s1 + bs1;
            const int c0 = qr_quant(qr_tanh(e0 * p0), a.z_inv, zbits), c1 = qr_quant(qr_tanh(e1 * p1), a.z_inv, zbits);
            *(unsigned short *)&z_code[z_hyp][z_col] = (unsigned short)(jv ? (c0 & 0xFF) | (c1 & 0xFF) << 8 : 0);
            __syncthreads();
            if (wave < 4) {   // uniform
                const v4i z = *(const v4i *)&z_code[col][grp * 16];
                sum = qr_mfma(a.w8 ? wj : ((jb & 1) ? (wj & m) : ((wj << 4) & m)), z, sum);
            }
        }
        return sum;
    };
    if (CL && blockIdx.y + 1 < gridDim.y) {   // uniform: not the first workgroup
        if (!ALSD && r.gate && *r.gate == 0) return;   // uniform
        const int row = a.row[my_n];
        const int part = (int)(gridDim.y - 1 - blockIdx.y);   // first workgroup 0, shares of the joint, language models, bottlenecks
        if (part >= a.parts) {
            share.send_lm(part - a.parts, row);
            return;
        }
        const v4i sum = joint_part(part, row, ALSD ? r.len_src[b * W + (z_hyp < W ? z_hyp : W - 1)] : 0);   // a share of the joint
        if (wave < 4) qr_send(word_at(part, col, wave * 16 + 4 * grp), sum, a.round);
        return;
    }

    if (!ALSD && r.gate && *r.gate == 0) {   // uniform: no utterance carried a label into this round, nothing can be picked
        if (tid == 0 && b == 0 && r.live_clear) *r.live_clear = 0;
        if (tid == 0 && b == 0 && r.n_rows_clear) *r.n_rows_clear = 0;
        if (!frame_end) return;
        const int n0 = r.nx_count[b];
        for (int e = tid; e < n0; e += 512) list_entry(e, r.nx_score[nx + e], r.nx_info[nx + e]);
        if (tid == 0) n_list = n0;
        if (tid < 64) best_fe[tid] = 0;
        if (wave == 0) load_first_free(r.n_taken[b]);
        finish_frame();
        return;
    }

    if (wave >= 4) {   // (the waves with less to do)
        const int k = (wave - 4) * 64 + lane;
        if (k < 64) best[k] = 0;
        else if (k < 128) best_fe[k - 64] = 0;
        else if (k < 192) fin_new[k - 128] = -INFINITY;
        else if (k == 192) n_cand = missed = 0;
        if (wave < 7) share.row_constants(wave - 4);   // joint, source LM, external LM
    }
    // What the routing wave and the scoring threads will need: requested first, used last.
    QrOwn own = {};
    QrAlsdOwn alsd_own = {};
    QrAlsdFinished finished = {};
    int nx0 = 0;                // length of the utterance's candidate list before this round
    float sc[NTW];              // the thread's hypotheses in the scores (16 * nt + tid / 16): running score, length
    int len_t[NTW];
    if (wave == 0) {
        own = qr_load_own(r, b, lane);
        if (ALSD) alsd_own = qr_alsd_load_own(r, s, b, lane);
        else nx0 = r.nx_count[b];
    }
    if (TAGS && !frame_end && wave == 6) qr_request_tags(r.tags + (size_t)b * r.P, r.P, lane, tags);
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
        const int w = nt * 16 + ((tid >> 4) & 15);
        const int n = b * W + (w < W ? w : W - 1);
        sc[nt] = wave < 4 ? r.score_src[n] : 0.0f;
        len_t[nt] = (ALSD && wave < 4) ? r.len_src[n] : 0;
    }
    unsigned key[4 * NTW];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
        const int w = nt * 16 + col;
        const int n = b * W + (w < W ? w : W - 1);
        const int row = a.row[n];
        if (nt > 0) __syncthreads();   // what the previous tile left in LDS has been read
        v4i acc[4] = {zero, zero, zero, zero};
        // waves 4-7, besides: the frame's candidates so far (the last round's list), the list of finished hypotheses
        float e_score = 0.0f;
        v4i e_info = zero;
        const int e0 = tid - 256;
        auto load_rest = [&]() {
            if (frame_end && nt == 0 && e0 >= 0 && e0 < n_entries) {
                e_score = r.nx_score[nx + e0];
                e_info = r.nx_info[nx + e0];
            }
            if (ALSD && nt == 0 && wave == 5) finished = qr_alsd_load_finished(r, s, b, lane);
        };
        auto enter_rest = [&]() {
            if (frame_end && nt == 0 && e0 >= 0) {
                if (e0 < n_entries) list_entry(e0, e_score, e_info);   // (entries behind the end of the list are overwritten or not counted)
                for (int e = e0 + 256; e < n_entries; e += 256) list_entry(e, r.nx_score[nx + e], r.nx_info[nx + e]);
            }
        };
        if (CL) load_rest();
        // CL: the words of the other workgroups that this thread of the scores (waves 0-3: shares of the joint; waves 4-7, for
        // the same thread of waves 0-3: language models) waits for, past this CU's cache
        v4i word[2 * (CL ? QR_ROUND_PARTS - 1 : 1)];
        const int n_src = wave < 4 ? a.parts - 1 : (use_lm ? 2 : 0);   // uniform
        auto source = [&](int i) { return wave < 4 ? 1 + i : (i == 0 ? 0 : QR_ROUND_PARTS); };
        auto request = [&]() {
            const __amdgpu_buffer_rsrc_t area = __builtin_amdgcn_make_buffer_rsrc(
                (void *)word_at(0, 0, 0), 0, (QR_ROUND_PARTS + 1) * 16 * 64 * 8, 0x00020000 /* raw bytes */);
#pragma unroll
            for (int i = 0; i < QR_ROUND_PARTS - 1; ++i)
                if (i < n_src) {
                    const unsigned off = (unsigned)((source(i) * 16 + ((tid >> 4) & 15)) * 64 + 4 * (lane & 15)) * 8;
                    word[2 * i] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(area, off, 0, 16 /* sc1 */);
                    word[2 * i + 1] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(area, off + 16, 0, 16);
                }
            asm volatile("" ::: "memory");   // every poll loads anew
        };
        v4i t = zero;   // CL: sums of the other shares
        if (CL) {
            const v4i sum = joint_part(0, row, ALSD ? r.len_src[b * W + (z_hyp < W ? z_hyp : W - 1)] : 0);
            request();
            if (wave < 4) sums[0][wave][grp * 16 + (col ^ (4 * wave + grp))] = sum;
            unsigned limit = (unsigned)a.ticks / 4;
            for (const unsigned long long t0 = wall_clock64();; request()) {
                bool ok = true;
#pragma unroll
                for (int i = 0; i < 2 * (QR_ROUND_PARTS - 1); ++i)
                    if (i < 2 * n_src) ok = ok && (unsigned)word[i][1] == a.round && (unsigned)word[i][3] == a.round;
                if (__all(ok)) break;
                if (wall_clock64() - t0 > limit && enough(limit)) {
                    if (lane == 0) missed = 1;
                    break;
                }
            }
#pragma unroll
            for (int i = 0; i < QR_ROUND_PARTS - 1; ++i) {
                const v4i v = i < n_src ? v4i{word[2 * i][0], word[2 * i][2], word[2 * i + 1][0], word[2 * i + 1][2]} : zero;
                if (wave < 4) t += v;
                else if (i < 2) lm_val[i][e0] = v4f{__int_as_float(v[0]), __int_as_float(v[1]), __int_as_float(v[2]), __int_as_float(v[3])};
            }
        } else if (wave < 4) {
            const QrHeadArgs &h = a.head[0];
            const int n_pred_tiles = J >> 4;
            const int zbits = a.w8 ? 8 : 4;
            const int len = ALSD ? r.len_src[n] : 0;
            for (int jb = wave; jb * 64 < J; jb += 4) {
                const bool jv = jb * 64 + grp * 16 < J;
                const int j0 = jv ? jb * 64 + grp * 16 : 0;   // this lane's 16 columns
                // row constants of the block
                const int j = jb * 64 + lane < J ? jb * 64 + lane : J - 1;
                const float sw = h.s_w[j], bs = h.bias ? h.bias[j] : 0.0f;   // of row `lane` of the block
                int rt = 4 * jb + (col >> 2);
                rt = rt < n_pred_tiles ? rt : n_pred_tiles - 1;
                unsigned woff[4];   // (a matrix of 2 GiB would have to have 4 million rows)
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) woff[mt] = (unsigned)rt * h.nkc * (h.w8 ? 2048 : 1024) + (grp * 16 + 4 * mt + (col & 3)) * 16;
                v4f e[4];
                auto load_frame = [&]() {
                    int64_t fr = a.frame_base + b;
                    if (ALSD) {   // this hypothesis' own frame
                        int t_w = s.iter - len;
                        t_w = t_w < 0 ? 0 : (t_w > s.T - 1 ? s.T - 1 : t_w);
                        fr = (int64_t)t_w * r.B + b;
                    }
#pragma unroll
                    for (int d = 0; d < 4; ++d) e[d] = *(const v4f *)(a.enc + fr * J + j0 + 4 * d);
                };
                v4i accp[4] = {zero, zero, zero, zero};
                if (h.w8) qr_chunk_mma<true, NTW == 1 ? 3 : 1>(h.w, woff, h.act, row, h.K, h.nkc, 0, 1, grp, accp, load_frame);
                else qr_chunk_mma<false, NTW == 1 ? 6 : 2>(h.w, woff, h.act, row, h.K, h.nkc, 0, 1, grp, accp, load_frame);
                // the block's weights of the joint arrive while its codes are formed
                v4i wj[4];
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const int rt = mt < n_row_tiles ? mt : n_row_tiles - 1;
                    wj[mt] = a.w8 ? a.w[((size_t)rt * a.nkc * 2 + jb) * 64 + lane] : a.w[((size_t)rt * a.nkc + (jb >> 1)) * 64 + lane];
                }
                // the wave's own 64 constants change places: a lane takes those of its 16 columns
                pc[wave][0][lane] = h.a_scale * sw;
                pc[wave][1][lane] = bs;
                __builtin_amdgcn_wave_barrier();
                v4i z = zero;
                if (jv)
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const v4f swd = *(const v4f *)&pc[wave][0][grp * 16 + 4 * d], bsd = *(const v4f *)&pc[wave][1][grp * 16 + 4 * d];
                        uint32_t word = 0;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int sum = h.w8 ? accp[d][i] : (accp[d][i] >> 4);   // 4-bit operands carry a factor 16
                            const float p = swd[i] * (float)sum + bsd[i];
                            word |= (uint32_t)(qr_quant(qr_tanh(e[d][i] * p), a.z_inv, zbits) & 0xFF) << (8 * i);
                        }
                        z[d] = (int)word;
                    }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
                    acc[mt] = qr_mfma(a.w8 ? wj[mt] : ((jb & 1) ? (wj[mt] & m) : ((wj[mt] << 4) & m)), z, acc[mt]);
            }
        } else {
            const QrHeadArgs &h = a.head[wave >= 6 ? 2 : 1];
            load_rest();
            if (h.w && !frame_end) share.head_mma<NTW == 1 ? 4 : 2>(h, row, wave & 1, 2, acc);   // uniform
            enter_rest();
        }
        if (CL) enter_rest();
        if (!CL) share.put_sums(acc);
        if (ALSD && nt == 0 && r.gate && *r.gate == 0) return;   // uniform: no live hypothesis anywhere, the finals stay as they are
        __syncthreads();

        // ---- scores: hypothesis 16 * nt + hc, tokens 4 * quad .. 4 * quad + 3
        const int hc = (tid >> 4) & 15, quad = lane & 15, mt = quad >> 2;
        const int at = (quad & 3) * 16 + (hc ^ quad), k0 = 4 * quad;
        v4f v[3];   // joint, source LM, external LM
        bool own_lm = !CL;   // the language models' sums lie in LDS
        if (!CL && wave >= 4) continue;
        if (!CL) t = (sums[0][mt][at] + sums[1][mt][at]) + (sums[2][mt][at] + sums[3][mt][at]);
        if (CL && wave < 4) t += sums[0][mt][at];
        if (CL && __builtin_amdgcn_readfirstlane(missed)) {   // uniform: everything that should have come
            if (tid == 0) a.late[b] += 1;
            if (wave < 4) t = sums[0][mt][at];
            own_lm = use_lm;
            __syncthreads();
            for (int part = 1; part < a.parts; ++part) {
                const v4i sum = joint_part(part, row, ALSD ? r.len_src[b * W + (z_hyp < W ? z_hyp : W - 1)] : 0);
                if (wave < 4) sums[0][wave][grp * 16 + (col ^ (4 * wave + grp))] = sum;
                __syncthreads();
                if (wave < 4) t += sums[0][mt][at];
                __syncthreads();
            }
            for (int net = 0; net < 2; ++net)
                for (int p = 0; use_lm && a.mid[net].w && p * 64 < a.mid[net].rows; ++p) {
                    const unsigned code = share.mid_part(net, p, row);
                    *(unsigned short *)&mid_code[net][z_hyp][p * 64 + z_col] = (unsigned short)code;
                    __syncthreads();
                }
            if (wave >= 4 && use_lm) {
                share.lm_mma(wave >= 6 ? 1 : 0, row, wave & 1, 2, acc);
                share.put_sums(acc);
            }
            __syncthreads();
        }
        if (CL && wave >= 4) continue;
        v[0] = qr_token_values(t, a.w8 != 0, jc[0][0], jc[0][1], k0, V, true);
#pragma unroll
        for (int q = 1; q < 3; ++q) {
            if (!own_lm)   // uniform
                v[q] = lm_val[q - 1][tid];
            else
                v[q] = qr_token_values(sums[2 + 2 * q][mt][at] + sums[3 + 2 * q][mt][at], a.head[q].w8 != 0, jc[q][0], jc[q][1], k0, V,
                                       a.head[q].log_softmax != 0);
        }
        const int ws_ = nt * 16 + hc;
        int t_w = s.iter - len_t[nt];
        t_w = t_w < 0 ? 0 : (t_w > s.T - 1 ? s.T - 1 : t_w);
        unsigned top = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = k0 + i;
            float f = v[0][i];
            if (k != a.blank) {
                if (a.head[1].w) f -= a.lambda_src * v[1][i];
                if (a.head[2].w) f += a.lambda_ext * v[2][i];
                f += a.rho;
            }
            // an empty slot (score -inf) offers nothing, whatever its row of the networks' states holds
            bool ok = ws_ < W && k < V && sc[nt] > -INFINITY && (ALSD || !r.last_round || k == a.blank);
            if (ALSD) {
                if (k != a.blank && len_t[nt] >= s.u_max) ok = false;      // label cap
                if (k == a.blank && t_w == s.T - 1) {                      // a blank at the last frame finishes the hypothesis
                    if (ok) fin_new[ws_] = sc[nt] + f;
                    ok = false;
                }
            }
            const float val = (sc[nt] + f) + 0.0f;   // + 0: one key per value
            key[nt * 4 + i] = (ok && val > -INFINITY) ? qr_float_key(val) : 0u;
            top = key[nt * 4 + i] > top ? key[nt * 4 + i] : top;
        }
        group_best[nt * 256 + tid] = top;
    }
    if (wave == 0) {
        if (frame_end) load_first_free(own.taken);
        else own.free_row = qr_free_row(r, b, lane, own.taken);
    }
    if (TAGS && !frame_end && wave == 6) qr_enter_tags<LOG_SLOTS>(r.P, lane, tags);
    __syncthreads();
    if (TAGS && !frame_end && wave == 0) own.serial = tag_lds[own.row - b * r.P][2];

    // ---- the W best under (value descending, flat index ascending)
    if (wave < 4) {
        // Up to 16 hypotheses: 64 groups, lane l looks at quartet l % 16 of hypotheses l / 16 + 4, 8, ...  More: every
        // quartet of every hypothesis is a group (with 64 groups 64 picks would bound nothing: 1.6 ms a frame at W = 64).
        constexpr int NG = NTW == 1 ? 1 : 4 * NTW;   // groups per lane
        unsigned g[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) g[i] = 0u;
#pragma unroll
        for (int i = 0; i < 4 * NTW; ++i) {
            const unsigned o = group_best[i * 64 + lane];
            g[i % NG] = o > g[i % NG] ? o : g[i % NG];
        }
        const QrBound bound(g, W);
        qr_gather<4 * NTW>(key, bound, [&](int i) { return ((i >> 2) * 16 + (tid >> 4)) * V + 4 * (lane & 15) + (i & 3); }, lane, &n_cand,
                           gathered);
    }
    __syncthreads();
    if (wave < 4) qr_rank(gathered, n_cand, W, tid, best);
    __syncthreads();
    if (wave == 0) {
        const QrCand p = best[lane];
        const bool found = lane < W && p != 0;
        const int my_c = found ? qr_cand_index(p) : -1;
        const float my_v = found ? qr_cand_value(p) : -INFINITY;
        if (ALSD) {
            alsd_own.h = own;
            qr_alsd_route<LOG_SLOTS, TAGS>(r, s, b, lane, my_c, my_v, alsd_own, tags, mask);
        } else {
            const int cnt = qr_route_picks<LOG_SLOTS, TAGS>(r, b, lane, my_c, my_v, own, nx0, tags, mask, [&](int e, float v, const v4i &info) {
                if (frame_end) {
                    list_entry(e, v, info);
                } else {
                    r.nx_score[nx + e] = v;
                    r.nx_info[nx + e] = info;
                }
            });
            if (lane == 0) {
                if (frame_end) n_list = cnt;
                else r.nx_count[b] = cnt;
            }
        }
    }
    if (ALSD && wave == 5) qr_alsd_finish(s, b, W, lane, fin_new[lane], finished);
    if (frame_end) finish_frame();
}

}  // namespace

namespace {

// Workgroups of search_round_kernel<1, ALSD, true> that the device holds at once; taken to be no more than two to each of 256
// compute units (registers), so that the size of a search's workspace does not hang on the device.
constexpr int MOST_RESIDENT = 512;
struct RoundRoom {
    int n_xcd, wgs;
};
template <bool ALSD>
RoundRoom resident()
{
    static std::atomic<int> known[QR_MAX_DEVICES];   // 0: not asked yet, -1: none, else wgs * 64 + n_xcd
    const int dev = qr_current_device();
    int n = known[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        int n_cu = 0, per_cu = 0, n_xcd = 0;
        if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipDeviceGetAttribute(&n_xcd, hipDeviceAttributeNumberOfXccs, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, search_round_kernel<1, ALSD, true>, 512, 0) != hipSuccess)
            return {1, 0};
        n_xcd = n_xcd < 1 || n_xcd > 32 ? 8 : n_xcd;
        n = n_cu * per_cu < MOST_RESIDENT ? n_cu * per_cu : MOST_RESIDENT;
        n = n > 0 ? n * 64 + n_xcd : -1;
        known[dev].store(n, std::memory_order_relaxed);
    }
    return n > 0 ? RoundRoom{n & 63, n >> 6} : RoundRoom{1, 0};
}

bool fit_together(int B, int W, int wgs, int room) { return W <= 16 && 6 * (int64_t)B * wgs <= 5 * (int64_t)room; }

int joint_parts(int J) { return (J + 63) / 64 < QR_ROUND_PARTS ? (J + 63) / 64 : QR_ROUND_PARTS; }

template <bool ALSD>
void launch_round(const QrRoundArgs &a, const QrRouteArgs &r, const QrAlsdArgs &s, hipStream_t st)
{
    int wgs = ALSD || !r.last_round ? a.wgs_lm : a.wgs_last;
    if (a.come > 0 && a.come < wgs) wgs = a.come;
    // No label pick looks for its states at beam 1, where every one stays and no sequence comes back (looking and not looking, ms:
    // time-synchronous, 60 frames, 100 utterances 6.38 and 6.27, 300 9.00 and 8.83; alignment-length search, 180 iterations, 32
    // utterances 4.07 and 4.01, 100 4.76 and 4.72; at beam 2 looking takes 64 utterances of 150 frames from 5.85 to 5.10), and none in
    // an alignment-length search of up to 16 hypotheses, whose step kernels take as long for one as for all of them and whose
    // list is hardly ever empty (228 iterations at beam 4 2 %, 60 us).
    const bool tags = r.W > 1 && !(ALSD && r.B * r.W <= 16);
    // (one workgroup to an utterance: any number of utterances, and a grid's z extent ends at 65535)
    const dim3 grid = wgs == 1 ? dim3(r.B) : dim3(a.n_xcd, wgs, (r.B + a.n_xcd - 1) / a.n_xcd);
    if (wgs && tags) search_round_kernel<1, ALSD, true><<<grid, 512, 0, st>>>(a, r, s);
    else if (wgs) search_round_kernel<1, ALSD, true, false><<<grid, 512, 0, st>>>(a, r, s);
    else if (r.W <= 16 && tags) search_round_kernel<1, ALSD, false><<<r.B, 512, 0, st>>>(a, r, s);
    else if (r.W <= 16) search_round_kernel<1, ALSD, false, false><<<r.B, 512, 0, st>>>(a, r, s);
    else if (r.W <= 32) search_round_kernel<2, ALSD, false><<<r.B, 512, 0, st>>>(a, r, s);
    else search_round_kernel<4, ALSD, false><<<r.B, 512, 0, st>>>(a, r, s);
}

}  // namespace

// Sources of words: shares of the joint (of the first one: the source LM), external LM, bottlenecks.
size_t qr_round_words(int J, bool use_lm, bool mids, int B, int W)
{
    const int parts = joint_parts(J);
    if (!(parts > 1 && fit_together(B, W, parts, MOST_RESIDENT)) && !(use_lm && fit_together(B, W, parts + 1, MOST_RESIDENT))) return 0;
    return (size_t)(mids ? QR_ROUND_PARTS + 3 : (use_lm ? QR_ROUND_PARTS + 1 : parts)) * 16 * 64;
}

void qr_plan_round(QrRoundArgs &a, int B, int W, bool alsd)
{
    const RoundRoom on = alsd ? resident<true>() : resident<false>();
    const int room = on.wgs;
    a.n_xcd = on.n_xcd;
    a.parts = joint_parts(a.J);
    a.wgs_lm = a.wgs_last = 0;
    // One workgroup to an utterance (a joint of up to 64 columns and no language model) is the faster form at any number of
    // them, K over eight waves and half the registers: 40 frames, ms, 64 utterances at beam 16 3.46 -> 3.39, 420 5.65 -> 3.79,
    // 4000 33.8 -> 19.3.
    auto fits = [&](int wgs) { return wgs == 1 ? W <= 16 : fit_together(B, W, wgs, room); };
    const bool use_lm = a.head[1].w || a.head[2].w;
    if (fits(a.parts)) a.wgs_last = a.parts;
    if (fits(a.parts + (use_lm ? 1 : 0))) {
        a.wgs_lm = a.parts + (use_lm ? 1 : 0);
        for (int net = 0; net < 2; ++net) a.wgs_lm += a.mid[net].w ? (a.mid[net].rows + 63) / 64 : 0;
    }
}

// A bottleneck in the round saves its own launch (6 us) and delays the language models by 2 us, as long as two thirds of the
// workgroups are resident at once.  External language model of 2 x 2048 cells, bottleneck of 256, beam 16, us a round of
// joint, steps and (before) bottleneck: 1 utterance 25.0 -> 22.4, 48 57.3 -> 54.8, 64 65.4 -> 62.6, 85 77.5 -> 74.9.
bool qr_round_takes(int mid_rows, int n_mids, int B, int W, bool alsd)
{
    const int room = (alsd ? resident<true>() : resident<false>()).wgs;
    return mid_rows <= 256 && fit_together(B, W, QR_ROUND_PARTS + 1, room) &&
           2 * B * (QR_ROUND_PARTS + 1 + n_mids * ((mid_rows + 63) / 64)) <= 3 * room;
}

void qr_launch_search_round(const QrRoundArgs &a, const QrRouteArgs &r, hipStream_t st) { launch_round<false>(a, r, QrAlsdArgs{}, st); }

void qr_launch_search_round_alsd(const QrRoundArgs &a, const QrRouteArgs &r, const QrAlsdArgs &s, hipStream_t st)
{
    launch_round<true>(a, r, s, st);
}

namespace {

// Time-synchronous search, beams of up to 16 hypotheses: an utterance runs ahead, round after round and frame after frame,
// until a label pick leads to a sequence whose states no row of the pool holds (route.h).  Only then does it need the networks;
// it leaves what is pending in memory and goes on in the next launch, behind the step kernels.  The utterances of a batch
// are in different frames.  (64 x 1000 frames at beam 16, with a launch to a round 104.5 ms, now 70; 13 x 301, wider
// networks and 8-bit layers 33.9 / 24.0; 1 x 152 11.1 / 7.1; 5 x 237 at beam 1, early stop 12.1 / 4.3.)
//
// The outputs of a row (prediction network's output layer, language models' log-probabilities) depend on the row alone, as its
// states do: they are formed in the round after the networks have advanced into it and kept beside it.  So only the first
// round of a launch contracts output layers (by the workgroups of the utterance: shares of the prediction network's rows, the
// language models, bottlenecks, as in search_round_kernel, whose words and waits these are); the others read 24 KB and are
// bound by their chain of dependent steps: outputs and codes, the joint, scores, selection, routing.  Whatever passes
// from round to round lies in LDS.
// Nobody but the first workgroup writes outputs, and it reads them in rounds behind its own stores only.
// A round whose hypotheses can offer blanks only (the last one of a frame) has nothing to select: they join the frame's
// candidates in slot order, which is the order of ties.  Without a label pick the frame's remaining rounds are empty.
// Rows: those that nothing names in this frame (the beam's, and the rows of the frame's picks) are free, and taken in turn.
__global__ __launch_bounds__(512, 4) void search_run_kernel(const QrRoundArgs a, const QrRunArgs r)
{
    constexpr int MAX_LIST = 16 * 17, LOG_SLOTS = 9;
    __shared__ v4i sums[8][4][64];          // partial sums; the words of the language models; gathered candidates
    __shared__ v4f p_lds[16][65];           // outputs of the prediction network: [hypothesis][column]
    __shared__ __attribute__((aligned(16))) int8_t mid_code[2][16][272];   // codes of the bottlenecks; the joint's codes
    __shared__ unsigned group_best[256];
    __shared__ QrCand list[MAX_LIST], best[64], best_fe[64];
    __shared__ int list_row[MAX_LIST], list_node[MAX_LIST], list_len[MAX_LIST];
    __shared__ __attribute__((aligned(16))) float jc[3][2][64];            // row scales and biases: joint, source LM, external LM
    __shared__ v4i tag_lds[(MAX_LIST + 63) / 64 * 64];
    __shared__ unsigned short tag_slot[1 << LOG_SLOTS];
    __shared__ unsigned char tag_twin[1 << LOG_SLOTS];
    __shared__ unsigned mask[64];
    __shared__ float own_score[16], blank_value[16];   // hypotheses of the round
    __shared__ int own_node[16], own_len[16], own_row[16];
    __shared__ int n_cand, n_list, n_lab, n_new, cursor, missed;
    QrCand *const gathered = (QrCand *)&sums[2][0][0];
    v4f *const lm_words = (v4f *)&sums[6][0][0];       // [2][256]
    static_assert(2 * sizeof(sums[0]) >= 16 * 64 * sizeof(QrCand) && 2 * sizeof(sums[0]) >= 2 * 256 * sizeof(v4f), "parts of the sums");
    int8_t (*const z_code)[272] = mid_code[0];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int b = (int)(blockIdx.z * gridDim.x + blockIdx.x);   // (grid as search_round_kernel's)
    if (b >= r.B) return;   // uniform
    const int part = (int)(gridDim.y - 1 - blockIdx.y);
    const int W = r.W, V = a.V, J = a.J, P = r.P;
    auto tell = [&](unsigned what) {
        if (r.told) __hip_atomic_store(r.told, (unsigned long long)r.ticket << 32 | what, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };
    if (b == 0 && part == 0 && tid == 0) {
        *r.n_rows_clear = 0;
        tell(*r.n_through >= r.B ? ~0u : a.round);
    }
    const v4i prog = r.prog[b];
    const int row = r.row[b * W + (col < W ? col : W - 1)];
    int t = __builtin_amdgcn_readfirstlane(prog[0]), v = __builtin_amdgcn_readfirstlane(prog[1]);
    if (t >= r.T) return;   // uniform: the utterance is through
    QrShare share = {a, sums, mid_code, jc, &missed, b, V};
    auto word_at = [&](int q, int hyp, int token) { return share.word_at(q, hyp, token); };
    const int z_hyp = share.z_hyp(), z_col = share.z_col();
    const v4i zero = {0, 0, 0, 0};

    // 64 columns (block `part`) of the prediction network's outputs: this thread's two
    auto pred_part = [&](int part, float &p0, float &p1) {
        const QrHeadArgs &h = a.head[0];
        const int j = part * 64 + z_col < J ? part * 64 + z_col : 0;
        float sw0, sw1, bs0, bs1;
        int s0, s1;
        share.block_sums<1>(h, J >> 4, part, row, s0, s1, [&]() {
            sw0 = h.s_w[j];
            sw1 = h.s_w[j + 1];
            bs0 = h.bias ? h.bias[j] : 0.0f;
            bs1 = h.bias ? h.bias[j + 1] : 0.0f;
        });
        p0 = (h.a_scale * sw0) * (float)s0 + bs0;
        p1 = (h.a_scale * sw1) * (float)s1 + bs1;
    };
    auto put_pred = [&](int part, float p0, float p1) {
        float *const to = (float *)&p_lds[z_hyp][0] + part * 64 + z_col;
        to[0] = p0;
        to[1] = p1;
    };
    if (part > 0) {   // uniform: not the first workgroup
        if (part >= a.parts) {
            share.send_lm(part - a.parts, row);
            return;
        }
        float p0, p1;
        pred_part(part, p0, p1);
        qr_send(word_at(part, z_hyp, z_col), p0, p1, a.round);
        return;
    }

    const bool use_lm = a.head[1].w || a.head[2].w;
    const int row0 = b * P;
    const QrTags tags = {tag_lds, tag_slot, tag_twin};
    auto list_entry = [&](int e, float value, int row, int node, int len) {
        list[e] = qr_cand(qr_float_key(value + 0.0f), e);   // + 0: one key per value
        list_row[e] = row;
        list_node[e] = node;
        list_len[e] = len;
    };

    // ---- what the first round needs beside the outputs
    if (wave == 6) qr_request_tags(r.tags + (size_t)row0, P, lane, tags);
    if (wave >= 4) {
        if (wave < 7) {
            share.row_constants(wave - 4);
        } else if (lane < 16) {
            const int o = b * W + (lane < W ? lane : W - 1);
            own_score[lane] = lane < W ? r.score[o] : -INFINITY;
            own_node[lane] = r.node[o];
            own_len[lane] = r.len[o];
            own_row[lane] = r.row[o];
        } else if (lane == 16) {
            missed = 0;
            n_list = prog[3];
            cursor = prog[2];
        }
        for (int e = tid - 256; e < prog[3]; e += 256) {
            const v4i info = r.nx_info[(size_t)b * r.n_entries + e];
            list_entry(e, r.nx_score[(size_t)b * r.n_entries + e], info[0], info[1], info[2]);
        }
    }
    // the joint: wave w has row tile w % 4 and 128 columns of K
    v4i wj[2] = {zero, zero};
    {
        const int rt = (wave & 3) < share.row_tiles() ? (wave & 3) : share.row_tiles() - 1, kc = wave >> 2, m = (int)0xF0F0F0F0u;
        if (kc < a.nkc) {   // uniform
            if (a.w8) {
                wj[0] = a.w[((size_t)rt * a.nkc + kc) * 128 + lane];
                wj[1] = a.w[((size_t)rt * a.nkc + kc) * 128 + 64 + lane];
            } else {
                const v4i f = a.w[((size_t)rt * a.nkc + kc) * 64 + lane];
                wj[0] = (f << 4) & m;
                wj[1] = f & m;
            }
        }
    }
    // this thread's eight columns of a hypothesis' codes, and of the encoder's frames t and t + 1
    const int h8 = tid >> 5, c8 = (tid & 31) * 8;
    const bool c_ok = c8 < J;
    v4f e[2], e_next[2];
    auto load_frame = [&](int t, v4f (&to)[2]) {
        const float *const f = a.enc + ((int64_t)(t < r.T ? t : r.T - 1) * r.B + b) * J + (c_ok ? c8 : 0);
        to[0] = *(const v4f *)f;
        to[1] = *(const v4f *)(f + 4);
    };
    // scores: hypothesis hc, tokens 4 * quad .. (waves 0-3)
    const int hc = (tid >> 4) & 15, quad = lane & 15, mt = quad >> 2, at = (quad & 3) * 16 + (hc ^ quad), k0 = 4 * quad;
    v4f p8[2], lm[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};

    // ---- the first round's outputs
    {
        float p0, p1;
        pred_part(0, p0, p1);
        load_frame(t, e);
        load_frame(t + 1, e_next);
        __syncthreads();   // (the sums have been read: words may take their place)
        put_pred(0, p0, p1);
        // words that this thread waits for, past this CU's cache: waves 0-3 the other shares', waves 4-7 the language models'
        v4i word[2 * (QR_ROUND_PARTS - 1)];
        const int n_src = wave < 4 ? a.parts - 1 : (use_lm ? 2 : 0);   // uniform
        auto request = [&]() {
            const __amdgpu_buffer_rsrc_t area = __builtin_amdgcn_make_buffer_rsrc((void *)word_at(0, 0, 0), 0,
                                                                                  (QR_ROUND_PARTS + 1) * 16 * 64 * 8, 0x00020000 /* raw bytes */);
#pragma unroll
            for (int i = 0; i < QR_ROUND_PARTS - 1; ++i)
                if (i < n_src) {
                    const int q = wave < 4 ? 1 + i : (i == 0 ? 0 : QR_ROUND_PARTS);
                    const unsigned off = (unsigned)((q * 16 + hc) * 64 + k0) * 8;
                    word[2 * i] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(area, off, 0, 16 /* sc1 */);
                    word[2 * i + 1] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(area, off + 16, 0, 16);
                }
            asm volatile("" ::: "memory");   // every poll loads anew
        };
        request();
        unsigned limit = (unsigned)a.ticks / 4;
        for (const unsigned long long t0 = wall_clock64();; request()) {
            bool ok = true;
#pragma unroll
            for (int i = 0; i < 2 * (QR_ROUND_PARTS - 1); ++i)
                if (i < 2 * n_src) ok = ok && (unsigned)word[i][1] == a.round && (unsigned)word[i][3] == a.round;
            if (__all(ok)) break;
            if (wall_clock64() - t0 > limit && share.enough(limit)) {
                if (lane == 0) missed = 1;
                break;
            }
        }
#pragma unroll
        for (int i = 0; i < QR_ROUND_PARTS - 1; ++i)
            if (i < n_src) {
                const v4f w = {__int_as_float(word[2 * i][0]), __int_as_float(word[2 * i][2]), __int_as_float(word[2 * i + 1][0]),
                               __int_as_float(word[2 * i + 1][2])};
                if (wave < 4) p_lds[hc][(1 + i) * 16 + quad] = w;
                else if (i < 2) lm_words[i * 256 + tid - 256] = w;
            }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(missed)) {   // uniform: everything that should have come
            if (tid == 0) a.late[b] += 1;
            for (int k = 1; k < a.parts; ++k) {
                pred_part(k, p0, p1);
                put_pred(k, p0, p1);
                __syncthreads();
            }
            for (int net = 0; net < 2; ++net)
                for (int k = 0; a.mid[net].w && k * 64 < a.mid[net].rows; ++k) {
                    const unsigned code = share.mid_part(net, k, row);
                    *(unsigned short *)&mid_code[net][z_hyp][k * 64 + z_col] = (unsigned short)code;
                    __syncthreads();
                }
            if (wave >= 4 && use_lm) {
                v4i acc[4] = {zero, zero, zero, zero};
                share.lm_mma(wave >= 6 ? 1 : 0, row, wave & 1, 2, acc);
                share.put_sums(acc);
            }
            __syncthreads();
            if (wave < 4 && use_lm)
#pragma unroll
                for (int q = 1; q < 3; ++q)
                    lm[q - 1] = qr_token_values(sums[2 + 2 * q][mt][at] + sums[3 + 2 * q][mt][at], a.head[q].w8 != 0, jc[q][0], jc[q][1], k0, V,
                                                a.head[q].log_softmax != 0);
            __syncthreads();
        } else if (wave < 4 && use_lm) {
            lm[0] = lm_words[tid];
            lm[1] = lm_words[256 + tid];
        }
        p8[0] = p_lds[h8][c8 >> 2];
        p8[1] = p_lds[h8][(c8 >> 2) + 1];
        if (h8 < W && c_ok) {
            float *const to = r.pred_out + (int64_t)own_row[h8] * J + c8;
            *(v4f *)to = p8[0];
            *(v4f *)(to + 4) = p8[1];
        }
        if (wave < 4 && use_lm && hc < W) {
            float *const to = r.lm_out + (int64_t)own_row[hc] * 128 + k0;
            *(v4f *)to = lm[0];
            *(v4f *)(to + 64) = lm[1];
        }
    }

    int n_rounds = 0;
    for (bool first = true;; first = false) {
        const bool last = v == r.max_sym;   // uniform
        if (!first) {
            const float *const p = r.pred_out + (int64_t)own_row[h8] * J + (c_ok ? c8 : 0);
            p8[0] = *(const v4f *)p;
            p8[1] = *(const v4f *)(p + 4);
            if (wave < 4 && use_lm && !last) {
                const float *const l = r.lm_out + (int64_t)own_row[hc] * 128 + k0;
                lm[0] = *(const v4f *)l;
                lm[1] = *(const v4f *)(l + 64);
            }
        }
        if (wave == 5) best[lane] = 0;
        if (wave == 7) best_fe[lane] = 0;
        // ---- codes
        {
            const int zbits = a.w8 ? 8 : 4;
            uint2 z = {0, 0};
            if (c_ok) {
                unsigned w[2] = {0, 0};
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[d] |= (unsigned)(qr_quant(qr_tanh(e[d][i] * p8[d][i]), a.z_inv, zbits) & 0xFF) << (8 * i);
                z = {w[0], w[1]};
            }
            *(uint2 *)&z_code[h8][c8] = z;
        }
        __syncthreads();
        // ---- joint
        if (tid == 256) n_cand = n_new = n_lab = 0;   // (behind the barrier: the round before has read them)
        {
            const int kc = wave >> 2, rt = wave & 3;
            const v4i z0 = *(const v4i *)&z_code[col][kc * 128 + grp * 16], z1 = *(const v4i *)&z_code[col][kc * 128 + 64 + grp * 16];
            v4i acc = qr_mfma(wj[0], z0, zero);
            acc = qr_mfma(wj[1], z1, acc);
            sums[kc][rt][grp * 16 + (col ^ (4 * rt + grp))] = acc;
        }
        __syncthreads();
        // ---- scores
        unsigned key[4];
        if (wave < 4) {
            const v4f joint = qr_token_values(sums[0][mt][at] + sums[1][mt][at], a.w8 != 0, jc[0][0], jc[0][1], k0, V, true);
            const float sc = own_score[hc];
            unsigned top = 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = k0 + i;
                float f = joint[i];
                if (k != a.blank) {
                    if (a.head[1].w) f -= a.lambda_src * lm[0][i];
                    if (a.head[2].w) f += a.lambda_ext * lm[1][i];
                    f += a.rho;
                }
                // an empty slot (score -inf) offers nothing, whatever its row of the networks' states holds
                const bool ok = hc < W && k < V && sc > -INFINITY;
                const float val = (sc + f) + 0.0f;   // + 0: one key per value
                key[i] = (ok && val > -INFINITY) ? qr_float_key(val) : 0u;
                top = key[i] > top ? key[i] : top;
                if (k == a.blank) blank_value[hc] = key[i] ? val : -INFINITY;
            }
            group_best[tid] = top;
        } else if (first && wave == 6) {
            qr_enter_tags<LOG_SLOTS>(P, lane, tags);
        }
        __syncthreads();
        if (last) {
            if (wave == 0) {
                const float val = lane < W ? blank_value[lane] : -INFINITY;
                const bool ok = val > -INFINITY;
                const unsigned long long om = __ballot(ok);
                const int n = n_list;
                if (ok) list_entry(n + (int)__popcll(om & ((1ull << lane) - 1ull)), val, own_row[lane], own_node[lane], own_len[lane]);
                if (lane == 0) n_list = n + (int)__popcll(om);
            }
        } else {
            // ---- the W best under (value descending, flat index ascending), as in search_round_kernel
            if (wave < 4) {
                unsigned g[1] = {0u};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const unsigned o = group_best[i * 64 + lane];
                    g[0] = o > g[0] ? o : g[0];
                }
                const QrBound bound(g, W);
                qr_gather<4>(key, bound, [&](int i) { return hc * V + k0 + i; }, lane, &n_cand, gathered);
            }
            __syncthreads();
            if (wave < 4) qr_rank(gathered, n_cand, W, tid, best);
            __syncthreads();
            if (wave == 0) {
                // ---- routing (see qr_route_picks): blanks join the frame's candidates, labels are the next round's slots
                const QrCand pick = best[lane];
                const bool found = lane < W && pick != 0;
                const int c = found ? qr_cand_index(pick) : 0, par = c / V, tok = c - par * V;
                const float val = found ? qr_cand_value(pick) : -INFINITY;
                const bool is_blank = found && tok == a.blank, is_lab = found && tok != a.blank;
                const unsigned long long lt = (1ull << lane) - 1ull, bm = __ballot(is_blank), lm_ = __ballot(is_lab);
                const int par_node = own_node[par], par_len = own_len[par], par_row = own_row[par];
                const int par_serial = tag_lds[par_row - row0][2];
                const int n = n_list, labels = (int)__popcll(lm_), k_lab = (int)__popcll(lm_ & lt);
                if (is_blank) list_entry(n + (int)__popcll(bm & lt), val, par_row, par_node, par_len);
                bool steps = false;
                int new_row = row0, n_steps = 0, k_step = 0, base = 0;
                if (labels > 0) {   // uniform
                    int from = cursor;
                    new_row = qr_find_rows_in_turn<LOG_SLOTS>(P, row0, lane, is_lab, par_serial, tok, t, (t * r.max_sym + v) * W, from, tags, mask, steps);
                    const unsigned long long sm = __ballot(steps);
                    n_steps = (int)__popcll(sm);
                    k_step = (int)__popcll(sm & lt);
                    if (lane == 0) {
                        cursor = from;
                        if (n_steps > 0) {
                            if (r.B == 1) *r.n_rows_next = n_steps;
                            else base = atomicAdd(r.n_rows_next, n_steps);
                        }
                    }
                }
                __builtin_amdgcn_wave_barrier();
                if (is_lab) {
                    const int id = 1 + (t * r.max_sym + v) * (r.B * W) + b * W + k_lab;
                    r.node_tok[id] = tok;
                    r.node_prev[id] = par_node;
                    own_score[k_lab] = val;
                    own_node[k_lab] = id;
                    own_len[k_lab] = par_len + 1;
                    own_row[k_lab] = new_row;
                }
                if (lane < 16 && lane >= labels) {
                    own_score[lane] = -INFINITY;
                    own_node[lane] = 0;
                    own_len[lane] = 0;
                    own_row[lane] = row0;   // any row of the utterance
                }
                if (lane == 0) {
                    n_list = n + (int)__popcll(bm);
                    n_lab = labels;
                    n_new = n_steps;
                }
                if (n_steps > 0) {   // uniform
                    base = __builtin_amdgcn_readfirstlane(base);
                    if (steps) r.rows_next[base + k_step] = v4i{new_row, par_row, tok, 0};
                }
            }
        }
        __syncthreads();
        const bool wants = __builtin_amdgcn_readfirstlane(n_new) > 0;   // the networks, before anything else
        if (last || (__builtin_amdgcn_readfirstlane(n_lab) == 0 && !r.every_round)) {
            // ---- the new beam: the W best of the frame's candidates by (score descending, insertion order)
            const int n = __builtin_amdgcn_readfirstlane(n_list);
            if (wave < 4) qr_rank(list, n, W, tid, best_fe);
            __syncthreads();
            if (wave == 0 && lane < 16) {
                const QrCand pick = best_fe[lane];
                const bool found = lane < W && pick != 0;
                const int c = found ? qr_cand_index(pick) : 0;
                const int beam_row = found ? list_row[c] : row0;
                own_score[lane] = found ? qr_cand_value(pick) : -INFINITY;
                own_node[lane] = found ? list_node[c] : 0;
                own_len[lane] = found ? list_len[c] : 0;
                own_row[lane] = beam_row;
                if (found) tag_lds[beam_row - row0][3] = t + 1;   // no row of the beam is taken in the next frame
            } else if (wave == 0 && lane == 16) {
                n_list = 0;
            }
            ++t;
            v = 0;
            e[0] = e_next[0];
            e[1] = e_next[1];
            load_frame(t + 1, e_next);
            __syncthreads();
        } else {
            ++v;
        }
        if (wants || t >= r.T || ++n_rounds >= r.max_rounds || r.every_round) break;   // uniform
    }

    // ---- what is pending
    if (wave == 0) {
        if (lane < W) {
            const int o = b * W + lane;
            r.score[o] = own_score[lane];
            r.node[o] = own_node[lane];
            r.len[o] = own_len[lane];
            r.row[o] = own_row[lane];
        }
        if (lane == 0) {
            r.prog[b] = v4i{t, v, cursor, n_list};
            if (t >= r.T && atomicAdd(r.n_through, 1) == r.B - 1) tell(~0u);
        }
    } else if (wave == 1) {
        for (int i = lane; i < P; i += 64) r.tags[(size_t)row0 + i] = tag_lds[i];
    } else {
        for (int i = tid - 128; i < n_list; i += 384) {
            r.nx_score[(size_t)b * r.n_entries + i] = qr_cand_value(list[i]);
            r.nx_info[(size_t)b * r.n_entries + i] = v4i{list_row[i], list_node[i], list_len[i], 0};
        }
    }
}

}  // namespace

int qr_plan_run(const QrRoundArgs &a, int B, int W)
{
    static std::atomic<int> room_of[QR_MAX_DEVICES];   // workgroups that the device holds at once; 0: not asked yet, -1: none
    const int dev = qr_current_device();
    int room = room_of[dev].load(std::memory_order_relaxed);
    if (room == 0) {
        int n_cu = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, search_run_kernel, 512, 0) != hipSuccess)
            return 0;
        room = n_cu * per_cu > 0 ? n_cu * per_cu : -1;
        room_of[dev].store(room, std::memory_order_relaxed);
    }
    const int wgs = a.parts + (a.head[1].w || a.head[2].w ? 1 : 0);   // (those of bottlenecks: qr_round_takes)
    return wgs == 1 || 6 * (int64_t)B * wgs <= 5 * (int64_t)room ? a.wgs_lm : 0;
}

// One page of pinned host memory for all searches of the process, kept to its end.  Taken under the relaxed capture mode, so that
// another thread's capture does not mind; a failure is not kept, the next search tries again.
static std::atomic<unsigned long long *> ticket_words{nullptr};
constexpr int TICKET_WORDS = 64, TICKET_APART = 8;   // a cache line each

static unsigned long long *take_ticket_words()
{
    static std::mutex one;
    std::unique_lock<std::mutex> lock(one, std::try_to_lock);
    if (!lock) return nullptr;   // another thread is at it; this search does without
    if (unsigned long long *const w = ticket_words.load(std::memory_order_acquire)) return w;
    constexpr size_t n = (size_t)TICKET_WORDS * TICKET_APART;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return nullptr;
    void *at = nullptr;
    const hipError_t e = hipHostMalloc(&at, n * sizeof(unsigned long long), hipHostMallocPortable | hipHostMallocMapped);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess) return nullptr;
    unsigned long long *const w = (unsigned long long *)at;
    for (size_t i = 0; i < n; ++i) w[i] = 0;
    ticket_words.store(w, std::memory_order_release);
    return w;
}

// A word of that page for a call, by turns: a search that ends late may write into the word of another one, which then enqueues
// more launches than it needs.  None while a graph is captured (a graph's launches are all of them anyway).
void qr_take_ticket(QrRunArgs &r, hipStream_t st)
{
    static std::atomic<unsigned> next{1};
    const bool clean = hipPeekAtLastError() == hipSuccess;   // (what the call's launches left is reported at its end)
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    r.told = nullptr;
    if (hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone) {
        unsigned long long *w = ticket_words.load(std::memory_order_acquire);
        if (!w) w = take_ticket_words();
        r.ticket = next.fetch_add(1, std::memory_order_relaxed);
        r.told = w ? w + r.ticket % TICKET_WORDS * TICKET_APART : nullptr;
    }
    if (clean) (void)hipGetLastError();
}

void qr_launch_search_run(const QrRoundArgs &a, const QrRunArgs &r, int wgs, hipStream_t st)
{
    if (a.come > 0 && a.come < wgs) wgs = a.come;
    const dim3 grid = wgs == 1 ? dim3(r.B) : dim3(a.n_xcd, wgs, (r.B + a.n_xcd - 1) / a.n_xcd);
    search_run_kernel<<<grid, 512, 0, st>>>(a, r);
}

void qr_launch_joint(const QrJointArgs &a, hipStream_t st)
{
    joint_fuse_kernel<<<(a.N + 15) / 16, 256, 0, st>>>(a);
}

extern "C" qrnnt_status qrnnt_joint_fuse(const float *enc_proj, int32_t n_enc_rows, const int32_t *frame_row,
                                         const float *pred_proj, const qrnnt_qmat *w_out, const float *b_out,
                                         float z_scale, float z_inv_scale, const float *lp_src, const float *lp_ext,
                                         float lambda_src, float lambda_ext, float rho, int32_t N, int32_t blank,
                                         float *lp_rnnt_out, int8_t *dbg_zq, float *fused_out, void *stream)
{
    qrnnt_status s = qr_check_qmat(w_out, QRNNT_LAYOUT_TILED);
    if (s != QRNNT_OK) return s;
    QR_REQUIRE(enc_proj && frame_row && pred_proj && fused_out, QRNNT_ERR_NULL);
    QR_REQUIRE(N > 0 && n_enc_rows > 0, QRNNT_ERR_SHAPE);
    QR_REQUIRE(w_out->cols % 16 == 0, QRNNT_ERR_SHAPE);
    QR_REQUIRE(w_out->rows <= 64, QRNNT_ERR_UNSUPPORTED);
    QR_REQUIRE(blank >= 0 && blank < w_out->rows, QRNNT_ERR_RANGE);
    QR_REQUIRE(z_scale > 0.0f && z_inv_scale > 0.0f, QRNNT_ERR_RANGE);
    QR_REQUIRE(qr_aligned(enc_proj, 16) && qr_aligned(pred_proj, 16), QRNNT_ERR_ALIGN);
    QR_REQUIRE(dbg_zq == nullptr || qr_aligned(dbg_zq, 16), QRNNT_ERR_ALIGN);
    QrJointArgs a = {};
    a.enc = enc_proj;  a.n_enc_rows = n_enc_rows;  a.frame_row = frame_row;  a.pred = pred_proj;
    a.w = (const v4i *)w_out->packed;  a.s_w = w_out->row_scale;  a.b_out = b_out;
    a.z_scale = z_scale;  a.z_inv = z_inv_scale;
    a.lp_src = lp_src;  a.lp_ext = lp_ext;
    a.lambda_src = lambda_src;  a.lambda_ext = lambda_ext;  a.rho = rho;
    a.N = N;  a.J = w_out->cols;  a.V = w_out->rows;  a.blank = blank;
    a.nkc = qr_round_up(w_out->cols, QRNNT_KCHUNK) / QRNNT_KCHUNK;
    a.w8 = qr_bits(w_out) == 8;
    a.lp_out = lp_rnnt_out;  a.dbg_zq = dbg_zq;  a.fused = fused_out;
    a.rows_per_utt = 1;
    qr_launch_joint(a, (hipStream_t)stream);
    return qr_launch_status();
}
