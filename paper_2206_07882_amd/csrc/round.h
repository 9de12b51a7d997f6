// What the kernels of a decoding round share: log-probabilities of an utterance's hypotheses, sixteen lanes to each, and words
// on their way between an utterance's workgroups.
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
