// Time-synchronous search, beams of up to 16 hypotheses: an utterance runs ahead, round after round and frame after frame,
// until a label pick leads to a sequence whose states no row of the pool holds (route.h).  Only then does it need the networks;
// it leaves what is pending in memory and goes on in the next launch, behind the step kernels.  The utterances of a batch
// are in different frames.  (64 x 1000 frames at beam 16, with a launch to a round 104.5 ms, now 66 to 71; 13 x 301, wider
// networks and 8-bit layers 33.9 / 23; 1 x 152 11.1 / 5.8 to 7.3; 5 x 237 at beam 1, early stop 12.1 / 2.8.)
#include <atomic>

#include "round.h"
#include "route.h"
#include "select.h"

namespace {

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
        qr_send(share.word_at(part, z_hyp, z_col), p0, p1, a.round);
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
            const __amdgpu_buffer_rsrc_t area = __builtin_amdgcn_make_buffer_rsrc((void *)share.word_at(0, 0, 0), 0,
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

// A word of host memory for a call, by turns: a search that ends late may write into the word of another one, which then
// enqueues more launches than it needs.  One allocation in a process, of one page, kept to its end; none while a graph is
// captured (a graph's launches are all of them anyway).
void qr_take_ticket(QrRunArgs &r, hipStream_t st)
{
    constexpr int WORDS = 64, APART = 8;   // a cache line each
    static std::atomic<unsigned> next{1};
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    r.told = nullptr;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return;
    static unsigned long long *const words = [] {
        void *at = nullptr;
        if (hipHostMalloc(&at, WORDS * APART * sizeof(unsigned long long), hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
            (void)hipGetLastError();
            return (unsigned long long *)nullptr;
        }
        for (int i = 0; i < WORDS * APART; ++i) ((unsigned long long *)at)[i] = 0;
        return (unsigned long long *)at;
    }();
    r.ticket = next.fetch_add(1, std::memory_order_relaxed);
    r.told = words ? words + r.ticket % WORDS * APART : nullptr;
}

void qr_launch_search_run(const QrRoundArgs &a, const QrRunArgs &r, int wgs, hipStream_t st)
{
    if (a.come > 0 && a.come < wgs) wgs = a.come;
    const dim3 grid = wgs == 1 ? dim3(r.B) : dim3(a.n_xcd, wgs, (r.B + a.n_xcd - 1) / a.n_xcd);
    search_run_kernel<<<grid, 512, 0, st>>>(a, r);
}
