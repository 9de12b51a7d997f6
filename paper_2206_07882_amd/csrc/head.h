// Split-K contraction for "head" layers: few weight rows (a block owns 64 of them),
// 16 activation rows per block, the 64-column K blocks dealt round-robin to the 4
// waves, partial sums reduced through LDS into wave 0.  All loads of a wave are
// issued before its first MFMA, so a block exposes one memory latency.
#pragma once

#include "qrnnt_common.h"

// bload(kb) issues the loads of this lane's 16 activation values of K block kb and returns them raw;
// bmake(raw, kb) turns them into the 16 codes (zero beyond K).  after_issue() runs once, after the first
// batch of loads has been issued and before anything waits for it: the place for loads that only the
// caller's epilogue needs (issued earlier they would sit in front of the operands in the in-order
// memory counter and the contraction would wait for them too).
// w8 (uniform): the weights are 8-bit (two blocks per chunk, operands as stored).
template <int BATCH, class BLoad, class BMake, class AfterIssue>
__device__ __forceinline__ void qr_head_mma(const v4i *__restrict__ w, int nkc, int n_row_tiles, int rt0, int K,
                                            BLoad &&bload, BMake &&bmake, AfterIssue &&after_issue, v4i (&acc)[4],
                                            v4i *lds /* [4][4][64] */, bool w8 = false)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: MFMAs below sit under wave-uniform branches
    const int nkb = (K + 63) >> 6;
    const v4i zero = {0, 0, 0, 0};
    const int m = (int)0xF0F0F0F0u;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) acc[mt] = zero;
    for (int kb0 = wave; kb0 == wave || kb0 < nkb; kb0 += 4 * BATCH) {   // at least once: after_issue must run
        v4i pa[BATCH][4], pb[BATCH];
        decltype(bload(0)) raw[BATCH];
#pragma unroll
        for (int it = 0; it < BATCH; ++it) {
            const int kb = kb0 + 4 * it;
            const bool ok = kb < nkb;
            const int kc = ok ? (kb >> 1) : 0;
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                int rt = rt0 + mt;
                rt = rt < n_row_tiles ? rt : n_row_tiles - 1;
                pa[it][mt] = w8 ? w[(((size_t)rt * nkc + kc) * 2 + (kb & 1)) * 64 + lane] : w[((size_t)rt * nkc + kc) * 64 + lane];
            }
            raw[it] = bload(ok ? kb : 0);
        }
        if (kb0 == wave) after_issue();
#pragma unroll
        for (int it = 0; it < BATCH; ++it) {
            const int kb = kb0 + 4 * it;
            pb[it] = kb < nkb ? bmake(raw[it], kb) : zero;
        }
#pragma unroll
        for (int it = 0; it < BATCH; ++it) {
            const int kb = kb0 + 4 * it;
            if (kb < nkb) {
                const bool hi = kb & 1;
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const v4i a = w8 ? pa[it][mt] : (hi ? (pa[it][mt] & m) : ((pa[it][mt] << 4) & m));
                    acc[mt] = qr_mfma(a, pb[it], acc[mt]);
                }
            }
        }
    }
    // reduce the four partial sums into wave 0
    if (wave != 0) {
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) lds[(wave * 4 + mt) * 64 + lane] = acc[mt];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int wv = 1; wv < 4; ++wv)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) acc[mt] += lds[(wv * 4 + mt) * 64 + lane];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[mt] = w8 ? acc[mt] : (acc[mt] >> 4);   // 4-bit operands carry a factor 16
    }
}

// Contraction of up to 4 row tiles with 16 activation rows by one wave: NB chunks of 128 columns per batch, all loads of a
// batch before its first MFMA.  w + woff[mt]: this lane's 16 bytes of chunk 0 of row tile mt; act: this
// lane's 16 columns of chunk 0 of its hypothesis' codes (K columns in all).  Chunks c0, c0 + step, ...
// Memory answers in order: the caller requests the row number behind `row` before this asks for the weights, so that
// the codes follow the weights without a second round trip.  then(): more loads to go with the first batch's codes.
template <bool W8, int NB, class Then>
__device__ __forceinline__ void qr_chunk_mma(const v4i *w, const unsigned (&woff)[4], const int8_t *acts, int row, int K, int nkc,
                                             int c0, int step, int grp, v4i (&acc)[4], Then &&then)
{
    const int m = (int)0xF0F0F0F0u;
    for (int kc0 = c0; kc0 < nkc; kc0 += NB * step) {
        v4i p[NB][4][W8 ? 2 : 1], x0[NB], x1[NB];
#pragma unroll
        for (int it = 0; it < NB; ++it) {
            int kc = kc0 + it * step;
            kc = kc < nkc ? kc : nkc - 1;   // uniform; what lies beyond the end is not contracted
            const char *base = (const char *)w + (size_t)kc * (W8 ? 2048 : 1024);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                p[it][mt][0] = *(const v4i *)(base + woff[mt]);
                if (W8) p[it][mt][W8 ? 1 : 0] = *(const v4i *)(base + 1024 + woff[mt]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (kc0 == c0) then();
        const int8_t *act = acts + (int64_t)row * K + grp * 16;
#pragma unroll
        for (int it = 0; it < NB; ++it) {
            int kc = kc0 + it * step;
            kc = kc < nkc ? kc : nkc - 1;
            // (columns beyond K meet zero weights: any valid bytes do)
            const int k = kc * QRNNT_KCHUNK;
            x0[it] = *(const v4i *)(act + (k + grp * 16 < K ? k : -grp * 16));
            x1[it] = *(const v4i *)(act + (k + 64 + grp * 16 < K ? k + 64 : -grp * 16));
        }
#pragma unroll
        for (int it = 0; it < NB; ++it)
            if (kc0 + it * step < nkc)   // uniform
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const v4i f = p[it][mt][0];
                    acc[mt] = qr_mfma(W8 ? f : ((f << 4) & m), x0[it], acc[mt]);
                    acc[mt] = qr_mfma(W8 ? p[it][mt][W8 ? 1 : 0] : (f & m), x1[it], acc[mt]);
                }
    }
}
