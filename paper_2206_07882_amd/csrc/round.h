// What the kernels of a decoding round share: log-probabilities of an utterance's hypotheses, sixteen lanes to each, and, where
// an utterance has several workgroups, what those do for the first one.
#pragma once

#include <type_traits>

#include "head.h"
#include "kernels.h"

// Maximum over the 16 lanes of a row, in each of them.
__device__ __forceinline__ float qr_row_max(float x)
{
#define QR_ROW_STEP(ctrl) x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, true)));
    QR_ROW_STEP(0xB1)    // quad_perm [1,0,3,2]
    QR_ROW_STEP(0x4E)    // quad_perm [2,3,0,1]
    QR_ROW_STEP(0x141)   // row_half_mirror
    QR_ROW_STEP(0x140)   // row_mirror
#undef QR_ROW_STEP
    return x;
}

// Sum over the 16 x 4 values of a row, in each of its lanes, in the order of the kernels that hold a hypothesis' tokens
// in four lanes (linear.hip): lane 4*mt + g has tokens 16*mt + 4*g + i; for each g one chain over mt and i, then
// (g0 + g1) + (g2 + g3).  The same bits as there matter: equal hypotheses tie, and a tie decides a beam.
__device__ __forceinline__ float qr_row_sum(const v4f &e)
{
    float sum = 0.0f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {   // after t passes the lanes of mt < t hold their chain's value (row_shr:4 brings 0 to mt = 0)
        const float from = t == 0 ? 0.0f : __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(sum), 0x114, 0xf, 0xf, true));
        sum = (((from + e[0]) + e[1]) + e[2]) + e[3];
    }
    int x = __float_as_int(sum);   // of interest: lanes 12..15 of the row
#define QR_ROW_ADD(ctrl) x = __float_as_int(__int_as_float(x) + __int_as_float(__builtin_amdgcn_update_dpp(0, x, ctrl, 0xf, 0xf, true)));
    QR_ROW_ADD(0xB1)
    QR_ROW_ADD(0x4E)
#undef QR_ROW_ADD
    x = __builtin_amdgcn_update_dpp(x, x, 0x128 /* row_ror:8 */, 0xf, 0x2, false);   // lanes 4..7
    x = __builtin_amdgcn_update_dpp(x, x, 0x124 /* row_ror:4 */, 0xf, 0x5, false);   // lanes 0..3 and 8..11
    return __int_as_float(x);
}

// Four tokens (k0 ..) of an output layer from the sums of their rows, as log-probabilities if it ends in a log-softmax; the
// 16 lanes of a row hold all tokens of a hypothesis.
__device__ __forceinline__ v4f qr_token_values(v4i t, bool w8, const float *scale, const float *bias, int k0, int V, bool log_softmax)
{
    t = w8 ? t : (t >> 4);   // 4-bit operands carry a factor 16
    const v4f ws = *(const v4f *)(scale + k0), wb = *(const v4f *)(bias + k0);
    float mx = -INFINITY;
    v4f v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = k0 + i < V ? ws[i] * (float)t[i] + wb[i] : -INFINITY;
        mx = fmaxf(mx, v[i]);
    }
    mx = qr_row_max(mx);
    v4f e;
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = qr_exp(v[i] - mx);   // (0 behind the last token)
    float lse = mx + qr_log(qr_row_sum(e));
    if (!log_softmax) lse = 0.0f;
    return v - lse;
}

// Words of value and round number for another workgroup, one, two or four next to each other.  What a reader finds is a whole word
// or none of it: the store is one instruction, here and not by the compiler's leave, and its 8-byte words are aligned.  It
// reaches the XCD's L2; at the scope of the device, as 8-byte atomics or as these with sc1, the same stores cost 3 to 11 % of a
// search (64 x 300 frames, alignment-length search, ms: 16.65, sc1 17.19, atomics 18.42).
__device__ __forceinline__ void qr_send(unsigned long long *to, unsigned v, unsigned round)
{
    asm volatile("global_store_dwordx2 %0, %1, off" ::"v"(to), "v"((unsigned long long)round << 32 | v) : "memory");
}
__device__ __forceinline__ void qr_send(unsigned long long *to, v4i v, unsigned round)
{
    const v4i lo = {v[0], (int)round, v[1], (int)round}, hi = {v[2], (int)round, v[3], (int)round};
    asm volatile("global_store_dwordx4 %0, %1, off\n\tglobal_store_dwordx4 %0, %2, off offset:16\n\ts_nop 1" ::"v"(to), "v"(lo), "v"(hi)
                 : "memory");   // (s_nop: see qr_store_through)
}
__device__ __forceinline__ void qr_send(unsigned long long *to, float v0, float v1, unsigned round)
{
    const v4i w = {__float_as_int(v0), (int)round, __float_as_int(v1), (int)round};
    asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 1" ::"v"(to), "v"(w) : "memory");
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
