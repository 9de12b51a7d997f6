// "W best of C candidates" under the total order (value descending, index ascending), shared by the decoding round's
// selection, the end of a frame and the beam selection.  -inf and NaN candidates are never picked.
// Up to some thousand candidates in the registers of 256 threads: a bound from below for the W-th best (QrBound), what
// passes it gathered in LDS (qr_gather), and the rank of each by counting (qr_rank), every step over four waves.
// Any number: W rounds of arg-best over memory by one wave (qr_select_from_mem).
#pragma once

#include "qrnnt_common.h"

__device__ __forceinline__ bool qr_better(float v, int c, float bv, int bc) { return v > bv || (v == bv && c < bc); }

__device__ __forceinline__ bool qr_select_round(float bv, int bc, int r, int lane, float &last_v, int &last_c, int &my_c,
                                                float &my_v)
{
    const unsigned key = bc != 0x7fffffff ? qr_float_key(bv) : 0u;
    const unsigned gmax = qr_wave_reduce_u32<true>(key);
    if (gmax == 0u) return false;   // uniform: nothing left
    const unsigned gidx = qr_wave_reduce_u32<false>(key == gmax ? (unsigned)bc : 0xFFFFFFFFu);
    last_v = qr_key_float(gmax);
    last_c = (int)gidx;
    if (lane == r) { my_c = last_c; my_v = last_v; }
    return true;
}

// Any size: value(c) re-forms candidate c in every round.
template <class Value>
__device__ __forceinline__ void qr_select_from_mem(Value &&value, int C, int W, int lane, int &my_c, float &my_v)
{
    float last_v = INFINITY;
    int last_c = -1;
    my_c = -1;
    my_v = -INFINITY;
    for (int r = 0; r < W; ++r) {
        float bv = -INFINITY;
        int bc = 0x7fffffff;
        for (int c = lane; c < C; c += 64) {
            const float v = value(c);
            const bool ok = v > -INFINITY && (v < last_v || (v == last_v && c > last_c));
            if (ok && qr_better(v, c, bv, bc)) { bv = v; bc = c; }
        }
        if (!qr_select_round(bv, bc, r, lane, last_v, last_c, my_c, my_v)) break;
    }
}

// A candidate of a selection in one word: larger is better under (value descending, index ascending); 0: none.
typedef unsigned long long QrCand;
__device__ __forceinline__ QrCand qr_cand(unsigned key, int idx) { return ((QrCand)key << 32) | (unsigned)~idx; }
__device__ __forceinline__ int qr_cand_index(QrCand c) { return (int)~(unsigned)c; }
__device__ __forceinline__ float qr_cand_value(QrCand c) { return qr_key_float((unsigned)(c >> 32)); }

// Lower bound of the W-th best candidate, from keys (qr_float_key, 0: none) of groups of candidates: the best of each
// group, NG groups per lane of a wave.  The W-th best of the groups' best ones has W candidates that are no worse.
// Distances from the best of all make the bits that tell candidates apart come early, and 16 of them will do.
struct QrBound {
    unsigned top;        // key of the best of all
    float v_max;
    unsigned T;

    template <int NG>
    __device__ __forceinline__ QrBound(const unsigned (&g)[NG], int W)
    {
        top = 0u;
#pragma unroll
        for (int i = 0; i < NG; ++i) top = g[i] > top ? g[i] : top;
        top = qr_wave_reduce_u32<true>(top);
        v_max = qr_key_float(top);
        unsigned near[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) near[i] = nearness(g[i]);
        T = 0u;
        for (int bit = 30; bit >= 15; --bit) {
            const unsigned trial = T | (1u << bit);
            int cnt = 0;
#pragma unroll
            for (int i = 0; i < NG; ++i) cnt += (int)__popcll(__ballot(near[i] >= trial));
            if (cnt >= W) T = trial;   // uniform
            if (cnt == W) break;
        }
        T = T ? T : 1u;   // fewer than W groups hold a candidate: every candidate passes
    }
    // Larger is nearer to the best; 0: no candidate.  (The best may be +inf: no difference is formed for its equals.)
    __device__ __forceinline__ unsigned nearness(unsigned k) const
    {
        return k == 0u ? 0u : (k == top ? 0x7FFFFFFFu : 0x7FFFFFFFu - __float_as_uint(v_max - qr_key_float(k)));
    }
    __device__ __forceinline__ bool passes(unsigned k) const { return nearness(k) >= T; }
};

// This wave's candidates that pass go to list[old *n ...], in any order (n and list in LDS).
template <int PER, class IndexOf>
__device__ __forceinline__ void qr_gather(const unsigned (&key)[PER], const QrBound &bound, IndexOf &&index_of, int lane, int *n, QrCand *list)
{
    unsigned long long pass[PER];
    bool in[PER];
    int n_pass = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        in[i] = bound.passes(key[i]);
        pass[i] = __ballot(in[i]);
        n_pass += (int)__popcll(pass[i]);
    }
    int base = 0;
    if (lane == 0 && n_pass) base = atomicAdd(n, n_pass);
    base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int pos = base + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(pass[i] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)pass[i], 0u));
        if (in[i]) list[pos] = qr_cand(key[i], index_of(i));
        base += (int)__popcll(pass[i]);
    }
}

// Rank of every one of the M candidates in list[] (no two equal): the best W go to best[rank].  256 threads: four count
// for one candidate, 64 candidates at a time.
__device__ __forceinline__ void qr_rank(const QrCand *list, int M, int W, int tid, QrCand *best)
{
    for (int i0 = 0; i0 < M; i0 += 64) {   // uniform
        const int i = i0 + (tid >> 2);
        const QrCand mine = list[i < M ? i : 0];
        int rank = 0;
#pragma unroll 4
        for (int j = tid & 3; j < M; j += 4) rank += list[j] > mine ? 1 : 0;
        rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xf, 0xf, true);
        rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xf, 0xf, true);
        if ((tid & 3) == 0 && i < M && rank < W) best[rank] = mine;
    }
}

