// The time loop of an LSTM layer as one persistent kernel (Sec. 3.4: the hidden
// state is quantized once at the cell output and that code feeds the next step).
//
// The recurrence is a chain of T dependent steps, each far too small to fill the
// GPU, so its cost is the latency of one step: exchange of the new hidden codes,
// contraction, cell.  Design:
//   - a group is one direction of 16 utterances; groups never exchange anything.  A
//     workgroup owns 32 cells (128 gate rows) of one group for all T steps;
//   - the members of a group sit on one XCD, so the codes travel through that XCD's L2
//     (stores reach it, loads marked sc1 go past the CU's own cache to it) and not through
//     the memory side of the device.  Workgroup ids are dealt to the XCDs in turn, so the
//     launch lays group g's members out at ids congruent to g mod 8; nothing relies on it:
//     at the start every workgroup counts itself in for the XCD it runs on, and a group that
//     finds itself spread over several exchanges at system scope instead (same words, sc0 sc1);
//   - the code of a cell travels in one byte of a 4-bit layer: code in the high nibble, step
//     number mod 16 in the low one (8-bit layer: two bytes).  Every byte says by itself
//     whether it is current, so data and flag arrive in the same store whatever its width,
//     without fence, atomic or grid barrier, and the bytes are the MFMA operand as they are:
//     code and weight both sit in the high nibble (sums come out x 256), and what the step
//     number adds is known beforehand (number x sum of the row's weights), so the accumulators
//     start at minus that;
//   - four waves carry the recurrence.  They split K in two and the rows in two: a wave holds
//     4 row tiles x half of K of W_hh in registers, hands two row tiles' partial sums to its K
//     partner through LDS (one barrier per step, double-buffered) and finishes the cells of the
//     other two: two adjacent cells x one utterance per lane, cell state in registers;
//   - four more waves, one beside each of them on its SIMD, bring the input part of the next
//     step: they hold W_ih the same way and contract the next frame's codes while the others
//     wait for the exchange (the matrix unit is idle most of a step), so a layer needs no
//     projection pass and no array of sums.  Layers with more input columns than the registers
//     hold get the sums from memory (qrnnt_input_projection), fetched by the same waves one step
//     ahead.  Either way the recurrence waves load nothing but the exchanged codes: a wave's
//     memory counter is in order, and a load from HBM in front of a poll holds the poll up;
//   - both directions of a bidirectional layer run in the same launch.
// A workgroup spins on its group's members, so these have to be resident together.  A launch
// asks for no more than an idle device holds (more utterances go in several launches), but
// recurrences of several streams, graphs or processes can each get part of an XCD and then
// wait for each other.  So a group first counts its members in; when they have not all come
// after about the time the layer takes, those that have come divide the group's cells among
// them and whoever comes later leaves at once (shared_steps: slower, the same results).
// Behind that every wait is for a resident workgroup; it is bounded by spin_limit polls all
// the same, after which the error flag is set and the workgroup leaves, so the grid drains.
#include <hip/hip_runtime.h>

#include <atomic>
#include <type_traits>

#include "kernels.h"
#include "mma_pipe.h"

namespace {

// A group's admission word: how many of its members have come, 6 bits for each XCD they run on (the ninth field: any
// other), whether it went ahead without the rest, and with how many.
typedef unsigned long long u64;
constexpr u64 ADMIT_SHORT = 1ull << 63;
constexpr int ADMIT_FIELDS = 9, ADMIT_N_SHIFT = 54;
static_assert(6 * ADMIT_FIELDS <= ADMIT_N_SHIFT && ADMIT_N_SHIFT + 6 <= 63, "fields do not overlap");
__device__ __forceinline__ int admit_count(u64 w)
{
    int n = 0;
#pragma unroll
    for (int i = 0; i < ADMIT_FIELDS; ++i) n += (int)((w >> (6 * i)) & 63);
    return n;
}
__device__ __forceinline__ bool admit_one_xcd(u64 w, int members)
{
    bool one = false;
#pragma unroll
    for (int i = 0; i < ADMIT_FIELDS - 1; ++i) one = one || (int)((w >> (6 * i)) & 63) == members;
    return one;
}

// What a workgroup does: all members have come, on one XCD or not; or it is one of the first `n` and takes the cells
// (32 at a time) number rank, rank + n, ...; or it is not needed.
enum { REC_LOCAL, REC_SPREAD, REC_SHARED, REC_LEAVE };
struct RecAdmission {
    int mode, rank, n;
};
// What a workgroup adds to the word to count itself in.
__device__ __forceinline__ u64 admit_field()
{
    int xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(xcc));
    return 1ull << (6 * (xcc < ADMIT_FIELDS - 1 ? xcc : ADMIT_FIELDS - 1));
}
// One wave, w: what counting itself in returned to lane 0.  All that happens to the word are atomics, and both ends (all
// have come; ADMIT_SHORT) are final.
__device__ __forceinline__ RecAdmission admit(u64 *word, u64 w, int members, int max_ticks, int lane)
{
    const u64 t0 = wall_clock64();   // 100 MHz
    auto uniform = [](u64 v) {
        return ((u64)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | (unsigned)__builtin_amdgcn_readfirstlane((int)v);
    };
    w = uniform(w);
    RecAdmission r = {REC_LEAVE, admit_count(w), 0};
    if (w & ADMIT_SHORT) return r;
    w += admit_field();
    while (true) {
        const int n = admit_count(w);
        if (w & ADMIT_SHORT) {
            r.mode = REC_SHARED;
            r.n = (int)((w >> ADMIT_N_SHIFT) & 63);
            return r;
        }
        if (n == members) {
            r.mode = admit_one_xcd(w, members) ? REC_LOCAL : REC_SPREAD;
            return r;
        }
        if (wall_clock64() - t0 > (u64)max_ticks) {
            u64 seen = w;
            if (lane == 0)
                __hip_atomic_compare_exchange_strong(word, &seen, w | ADMIT_SHORT | ((u64)n << ADMIT_N_SHIFT), __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            seen = uniform(seen);
            w = seen == w ? (w | ADMIT_SHORT | ((u64)n << ADMIT_N_SHIFT)) : seen;
        } else {
            __builtin_amdgcn_s_sleep(1);
            w = uniform(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
    }
}

// PER 128-bit loads from `bytes` bytes at base at each off[k].  LOCAL: past the CU's cache to the XCD's L2; otherwise past every
// cache that is not coherent.  What a lane finds says by itself whether it is current, so the time between the loads and
// the first use of v[] can be used; the compiler places the wait, in front of whatever touches v[] first, a spill included.
template <int KH, int PER, bool LOCAL>
__device__ __forceinline__ void load_words(const char *base, unsigned bytes, const unsigned (&off)[KH], v4i (&v)[KH * PER])
{
    constexpr int SC0 = 1, SC1 = 16;
    const __amdgpu_buffer_rsrc_t area = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00020000 /* raw bytes */);
#pragma unroll
    for (int i = 0; i < KH * PER; ++i)
        v[i] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(area, off[i / PER] + 16 * (i % PER), 0, LOCAL ? SC1 : SC0 | SC1);
    asm volatile("" ::: "memory");   // every poll loads anew
    __builtin_amdgcn_sched_barrier(0);
}

// Stores with the lanes outside `mask` left out, in one block instead of under a branch: the instructions around it stay
// one stretch for the scheduler.
#define QR_MASKED_ST(op, addr, F, ...)                                                                                   \
    asm volatile("s_mov_b64 %[keep], exec\n\ts_mov_b64 exec, %[mask]\n\tglobal_store_" op " %[o], %[v], " addr " " F    \
                 "\n\ts_mov_b64 exec, %[keep]" : [keep] "=&s"(keep) : [v] "v"(v), [mask] "s"(mask), __VA_ARGS__ : "memory")

// A lane's new codes for its group's members: NB bytes at base + off.
template <int NB>
__device__ __forceinline__ void store_codes(char *base, unsigned off, unsigned v, unsigned long long mask, bool local)
{
    unsigned long long keep;
#define QR_ST(op)                                                              \
    if (local) QR_MASKED_ST(op, "%[b]", "", [o] "v"(off), [b] "s"(base));      \
    else QR_MASKED_ST(op, "%[b]", "sc0 sc1", [o] "v"(off), [b] "s"(base));
    if constexpr (NB == 1) { QR_ST("byte") }
    if constexpr (NB == 2) { QR_ST("short") }
    if constexpr (NB == 4) { QR_ST("dword") }
#undef QR_ST
}

// A lane's codes to the layer's output.
template <int NB>
__device__ __forceinline__ void store_out(int8_t *p, unsigned v, unsigned long long mask)
{
    unsigned long long keep;
    if constexpr (NB == 1) QR_MASKED_ST("byte", "off", "", [o] "v"(p));
    else QR_MASKED_ST("short", "off", "", [o] "v"(p));
}

// a | (b ^ c)
__device__ __forceinline__ unsigned or_xor(unsigned a, unsigned b, unsigned c)
{
    unsigned r;
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0xf6" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}

// A pointer that is the same in all lanes, in scalar registers.
__device__ __forceinline__ char *scalar(char *p)
{
    const u64 v = (u64)(size_t)p;
    return (char *)(size_t)(((u64)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | (unsigned)__builtin_amdgcn_readfirstlane((int)v));
}

// Workgroup barrier that orders LDS accesses only: no wait for the memory operations in flight.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Lanes of the upper utterance half take b from the lane 8 columns below, the others keep a.
__device__ __forceinline__ v4i upper_from(v4i a, v4i b)
{
    v4i r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_update_dpp(a[i], b[i], 0x128 /* row_ror:8 */, 0xf, 0xc, false);
    return r;
}

// The cell of Sec. 3.4 from the sums of its gates; returns the code of its output.
template <bool W8, bool C_FIRST>
__device__ __forceinline__ int rec_cell(const v4f &sx, const v4f &sh, const v4f &bb, const float (&gx)[4], const v4i &ah, float h_inv, float &c)
{
    float p[4];
#pragma unroll
    for (int gt = 0; gt < 4; ++gt) p[gt] = __builtin_fmaf(sx[gt], gx[gt], __builtin_fmaf(sh[gt], (float)ah[gt], bb[gt]));
    const float gi = qr_sigmoid(p[0]), gf = qr_sigmoid(p[1]), gg = qr_tanh(p[2]), go = qr_sigmoid(p[3]);
    c = C_FIRST ? __builtin_fmaf(gi, gg, gf * c) : __builtin_fmaf(gf, c, gi * gg);
    return qr_quant(go * qr_tanh(c), h_inv, W8 ? 8 : 4);
}

// K step ks of row tile rt as an MFMA operand.
template <bool W8>
__device__ __forceinline__ v4i rec_weight(const v4i *w, int nkc, int rt, int ks, int lane)
{
    if (W8) return w[(((size_t)rt * nkc + (ks >> 1)) * 2 + (ks & 1)) * 64 + lane];   // as stored, two blocks per 128-column chunk
    const int m = (int)0xF0F0F0F0u;
    const v4i p = w[((size_t)rt * nkc + (ks >> 1)) * 64 + lane];
    return (ks & 1) ? (p & m) : ((p << 4) & m);
}

// All T steps of a group by n of its workgroups (this one is number rank), each taking 32 cells at a time: the way out
// when the group's members are not resident together.  Weights come from L2 in every step (all of a tile's before the
// first is used), the cell states stay in memory, the codes go through the exchange area at device scope, 16 columns to
// a 16-cell group.  hl, xl: LDS for the operands of a step, 64 * 2 * KH and 64 * 2 * KX pieces.
// Bound by the weight stream of the workgroup with the most cells, 2 us for 32 cells: 640 cells, 1280 inputs, one utterance
// take 38 us a step with one workgroup, 10.3 with 4, 5.4 with 10; 0.96 with all 20.
template <int KH, int KX, bool W8, bool C_FIRST>
__device__ __forceinline__ void shared_steps(const QrRecArgs &a, int ug, int members, int rank, int n, char *xb0, char *xb1, v4i *hl,
                                             v4i *xl, int *s_fail)
{
    constexpr int PER = W8 ? 2 : 1, KXA = KX > 0 ? KX : 1;
    constexpr float X_UNIT = (W8 || KX == 0) ? 1.0f : 0.0625f, H_UNIT = W8 ? 1.0f : 0.00390625f;
    const int H = a.H, B = a.B, T = a.T;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int n_groups = H >> 4, x_pieces = KX > 0 ? (int)(a.ld_x >> 4) : 0;
    const int u = ug * 16 + col, uu = u < B ? u : B - 1;
    const v4i zero = {0, 0, 0, 0};
    const int m = (int)0xF0F0F0F0u;
    for (int e = tid; e < KH * 128; e += 512) hl[e] = zero;    // what lies behind the layer's last group and
    for (int e = tid; e < KX * 128; e += 512) xl[e] = zero;    // column stays zero
    __syncthreads();
    for (int s = 0; s < T; ++s) {
        const int t = a.reverse ? T - 1 - s : s;
        // ---- the frame and the codes of the step before, as MFMA operands: piece 16 * group + utterance
        for (int e = tid; e < x_pieces * 16; e += 512) {
            const int n0 = ug * 16 + (e & 15) < B ? ug * 16 + (e & 15) : B - 1;
            xl[e] = *(const v4i *)(a.x + ((int64_t)t * B + n0) * a.ld_x + (e >> 4) * 16);
        }
        for (int e = tid; e < n_groups * 16; e += 512) {
            v4i v = zero;
            if (s == 0) {
                const int n0 = ug * 16 + (e & 15) < B ? ug * 16 + (e & 15) : B - 1;
                if (a.h0) v = *(const v4i *)(a.h0 + (int64_t)n0 * H + (e >> 4) * 16);
                hl[e] = W8 ? v : ((v << 4) & m);
                continue;
            }
            const u64 *src = (const u64 *)(((s - 1) & 1 ? xb1 : xb0) + (size_t)e * 16 * PER);
            const u64 want = W8 ? 0x0100010001000100ull * (u64)(s & 0xFF) : 0x0101010101010101ull * (u64)(s & 15);
            const u64 tags = W8 ? 0xFF00FF00FF00FF00ull : 0x0F0F0F0F0F0F0F0Full;
            u64 q[2 * PER];
            for (int spins = 0;; ++spins) {
                u64 bad = 0;
#pragma unroll
                for (int i = 0; i < 2 * PER; ++i) {
                    q[i] = __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    bad |= (q[i] ^ want) & tags;
                }
                if (bad == 0) break;
                if (spins >= a.spin_limit) {
                    atomicExch(a.err, 1);
                    *s_fail = 1;
                    break;
                }
            }
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                if (W8) v[d] = (int)__builtin_amdgcn_perm((unsigned)(q[d * PER / 2] >> 32), (unsigned)q[d * PER / 2], 0x06040200u);
                else v[d] = (int)(unsigned)(q[d / 2] >> (32 * (d & 1))) & m;
            }
            hl[e] = v;
        }
        __syncthreads();
        if (*s_fail) break;   // uniform
        for (int sl = rank; sl < members; sl += n) {
            const int cg = 2 * sl + (wave >> 2), rt = cg * 4 + (wave & 3);
            if (cg >= n_groups) continue;   // uniform
            const int j = qr_gates_cell(rt, grp);
            v4i wh[KH][PER], wx[KXA][PER];
            auto fetch = [&](const v4i *w, int nkc, int k, v4i (&f)[PER]) {   // (a chunk that the layer does not have meets zeros)
                const v4i *p = w + ((size_t)rt * nkc + (k < nkc ? k : nkc - 1)) * (64 * PER);
#pragma unroll
                for (int i = 0; i < PER; ++i) f[i] = p[64 * i + lane];
            };
#pragma unroll
            for (int k = 0; k < KH; ++k) fetch(a.whh, a.nkc_h, k, wh[k]);
#pragma unroll
            for (int k = 0; k < KX; ++k) fetch(a.wih, a.nkc_x, k, wx[k]);
            v4i ah = zero, ax = zero;
            if (KX == 0) ax = *(const v4i *)(a.gx + ((int64_t)t * B + uu) * 4 * H + rt * 16 + 4 * grp);
            v4f sx, sh, bb;
#pragma unroll
            for (int gt = 0; gt < 4; ++gt) {
                sx[gt] = a.x_scale * a.s_wih[gt * H + j] * X_UNIT;
                sh[gt] = a.h_scale * a.s_whh[gt * H + j] * H_UNIT;
                bb[gt] = a.bias[gt * H + j];
            }
            float *c_at = a.c_buf + (int64_t)uu * H + j;
            float c = s > 0 ? *c_at : (a.c0 ? a.c0[(int64_t)uu * H + j] : 0.0f);
            __builtin_amdgcn_sched_barrier(0);
            auto tile = [&](const v4i (&f)[PER], const v4i *op, int k, v4i &acc) {   // 128 columns
                const v4i *o = op + (8 * k + grp) * 16 + col;
                acc = qr_mfma(W8 ? f[0] : ((f[0] << 4) & m), o[0], acc);
                acc = qr_mfma(W8 ? f[PER - 1] : (f[0] & m), o[64], acc);
            };
#pragma unroll
            for (int k = 0; k < KH; ++k) tile(wh[k], hl, k, ah);
#pragma unroll
            for (int k = 0; k < KX; ++k) tile(wx[k], xl, k, ax);
            float gx[4];
#pragma unroll
            for (int gt = 0; gt < 4; ++gt) gx[gt] = (float)ax[gt];
            const unsigned code = (unsigned)rec_cell<W8, C_FIRST>(sx, sh, bb, gx, ah, a.h_inv, c);
            char *dst = (s & 1 ? xb1 : xb0) + (size_t)((cg * 16 + col) * 16 + (j & 15)) * PER;
            const unsigned tag = (unsigned)(s + 1);
            if (W8) __hip_atomic_store((unsigned short *)dst, (unsigned short)((code & 0xFFu) | tag << 8), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else __hip_atomic_store((unsigned char *)dst, (unsigned char)(code << 4 | (tag & 15u)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (u < B) {
                *c_at = c;
                a.h_out[((int64_t)t * B + u) * a.ld_out + a.col_off + j] = (int8_t)code;
                if (a.dbg_c_all) a.dbg_c_all[((int64_t)t * B + u) * H + j] = c;
                if (s == T - 1 && a.h_last) a.h_last[(int64_t)u * H + j] = (int8_t)code;
                if (s == T - 1 && a.c_last) a.c_last[(int64_t)u * H + j] = c;
            }
        }
        __syncthreads();   // the operands have been read
    }
}

// Exchange area of a direction: [parity][utterance group][16-cell group][utterance][16 cells], one byte per cell (two
// in an 8-bit layer): a lane's MFMA operand for a K step (16 cells of one utterance) is contiguous.  A layer of B < 16
// utterances keeps its columns closer together (the next power of two): lanes of absent utterances read what a present
// one reads, and a poll touches that many fewer cache lines.
// KH: K steps (64 cells) of h per wave, H <= 128 * KH.  KX: K steps of the input per wave, I <= 128 * KX; 0: sums from memory.
// CELLS: cells per lane in the cell update: 2, or 1 if there are at most 8 utterances: the lanes of the absent upper
// eight then take the second cell of the lower eight.
// C_FIRST: which product of c' = f*c + i*g is rounded before the sum (see launch_rec_w).
// NG: groups of 16 utterances that a workgroup has under way, 1, or 2 in turn (the second one need not exist): while the codes
// of one are on their way the other one's step is done, with the same weights in registers.
// Returns without a step done when the group's members have not all come (adm.mode).
template <int KH, int KX, bool W8, int CELLS, bool C_FIRST, int NG>
__device__ __forceinline__ void member_steps(const QrRecArgs &a, int ug, int mem, int members, char *xb0, char *xb1, size_t ug_bytes,
                                             v4i (&px)[2][2][2][4][64], v4i (&xs)[KX > 0 ? 3 * 2 * KX : 1][64], int (&s_fail)[2],
                                             RecAdmission &adm)
{
    constexpr int PER = W8 ? 2 : 1;    // bytes per exchanged cell
    constexpr int NL = KH * PER;       // 128-bit loads per wave and poll
    __shared__ v4i part[2][4][CELLS][64];   // [parity][wave][row tile][lane] partial sums on their way to the K partner
    // Where the weights leave no registers for them (up to 57 spilled), what a lane needs once a step lies in LDS: row
    // scales and biases of its cells, row sums of its wave's weights.  50 steps of 2 x 768 cells at 320 inputs and 32
    // utterances: 4-bit 88 -> 76 us, 8-bit 158 -> 119 us.
    constexpr bool PARK = KH >= 8 && (W8 || CELLS == 2);
    __shared__ v4f pk[PARK ? CELLS : 1][3][PARK ? 256 : 1];
    __shared__ v4i pk_rsum[PARK && !W8 ? 4 : 1][PARK && !W8 ? 256 : 1];
    static_assert(NG == 1 || (KX > 0 && CELLS == 2 && !PARK), "the forms that two groups in turn are made for");
    const int H = a.H, B = a.B, T = a.T;
    const int ng = NG == 1 || (ug + 1) * 16 >= B ? 1 : 2;   // groups there are: turn q is step q / ng of group q % ng
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave8 & 3;                 // 0..3 of either kind
    const int col = lane & 15, grp = lane >> 4;
    const int kh = wave & 1, rh = wave >> 1;
    const int n_groups = H >> 4;                // 16-cell groups of the layer
    const int cg = 2 * mem + rh;                // this wave's
    const bool have = cg < n_groups;            // (an odd number of groups leaves half of the last workgroup without cells)
    const int cgc = have ? cg : 0;
    const int64_t dir = a.reverse ? -1 : 1, t0 = a.reverse ? T - 1 : 0;
    const v4i zero = {0, 0, 0, 0};
    const int m = (int)0xF0F0F0F0u;
    auto weight = [&](const v4i *w, int nkc, int rt, int ks) -> v4i { return rec_weight<W8>(w, nkc, rt, ks, lane); };

    if (tid == 0) s_fail[0] = s_fail[1] = 0;
    __syncthreads();

    if (wave8 >= 4) {
        // ================= input part: K half kh of cell group rh, one step ahead of the recurrence
        const int n = ug * 16 + col, nn = n < B ? n : B - 1;
        if constexpr (KX > 0) {
            // A frame's codes go global -> LDS directly, 8 utterances x 128 columns to an instruction: whole cache lines
            // (as MFMA operands straight from memory they would be 16 half lines to an instruction, and the other waves'
            // polls would queue behind them), 16-byte pieces swizzled by row.  Three frames are on their way or in use.
            constexpr int CH = KX;                       // 128-column chunks
            constexpr int LOADS = (2 * CH + 3) / 4;      // per wave and frame
            v4i Ax[4][KX > 0 ? KX : 1];
#pragma unroll
            for (int k = 0; k < KX; ++k) {
                const int ks = kh + 2 * k;
#pragma unroll
                for (int i = 0; i < 4; ++i) Ax[i][k] = (have && ks < 2 * a.nkc_x) ? weight(a.wih, a.nkc_x, cg * 4 + i, ks) : zero;
            }
            const unsigned lds0 = (unsigned)(size_t)&xs[0][0];
            const int8_t *src[LOADS], *src2[NG > 1 ? LOADS : 1];   // of the group whose frame is fetched next, of the other one
#pragma unroll
            for (int q = 0; q < LOADS; ++q) {
                int blk = wave + 4 * q;                  // (chunk, utterance half); the last few repeat the last block
                blk = blk < 2 * CH ? blk : 2 * CH - 1;
                int nr = ug * 16 + (blk & 1) * 8 + (lane >> 3);
                const int o = (blk >> 1) * 128 + ((lane & 7) ^ (lane >> 3)) * 16;
                const int8_t *const x = a.x + t0 * B * a.ld_x + (o < a.ld_x ? o : 0);   // beyond the row: any valid bytes, they meet zero weights
                src[q] = x + (int64_t)(nr < B ? nr : B - 1) * a.ld_x;
                nr += 16;
                if (NG > 1) src2[NG > 1 ? q : 0] = x + (int64_t)(nr < B ? nr : B - 1) * a.ld_x;
            }
            const int64_t x_step = dir * B * a.ld_x;
            auto fetch = [&](int buf, bool advance) {
#pragma unroll
                for (int q = 0; q < LOADS; ++q) {
                    int blk = wave + 4 * q;
                    blk = blk < 2 * CH ? blk : 2 * CH - 1;
                    qr_load_lds16(src[q], lds0 + (unsigned)(buf * 2 * CH + blk) * 1024);
                    src[q] += advance ? x_step : 0;
                    if (NG > 1 && ng > 1) {   // uniform
                        const int8_t *const other = src2[NG > 1 ? q : 0];
                        src2[NG > 1 ? q : 0] = src[q];
                        src[q] = other;
                    }
                }
            };
            const int at = (col >> 3) * 64 + (col & 7) * 8;   // this lane's row within a chunk's two blocks, in 16-byte pieces
            auto produce = [&](int buf, int par) {
                v4i acc[4] = {zero, zero, zero, zero}, b[KX > 0 ? KX : 1];
#pragma unroll
                for (int k = 0; k < KX; ++k) b[k] = xs[buf * 2 * CH + 2 * k][at + ((4 * kh + grp) ^ (col & 7))];
                __builtin_amdgcn_sched_barrier(0);   // all of them first: two at a time a turn of two groups waited for LDS five times
#pragma unroll
                for (int k = 0; k < KX; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[i] = qr_mfma(Ax[i][k], b[k], acc[i]);
#pragma unroll
                for (int i = 0; i < 4; ++i) px[par][kh][rh][i][lane] = acc[i];
            };
            const int turns = T * ng, left = turns - ng;   // (a frame behind a group's last one: the last one again)
            fetch(0, 0 < left);
            fetch(1, 1 < left);
            fetch(2, 2 < left);
            qr_wait_vmcnt<0>();
            lds_barrier();
            produce(0, 0);
            lds_barrier();
            if (adm.mode >= REC_SHARED) return;          // uniform
            int b1 = 1, b3 = 0;                          // buffers of frames s + 1 and s + 3
            for (int s = 0; s < turns; ++s) {
                fetch(b3, s + 3 < left);
                if (s + 1 < turns) produce(b1, (s + 1) & 1);
                qr_wait_vmcnt<LOADS>();                  // all but the newest fetch: frame s + 2 is there
                lds_barrier();
                if (__builtin_amdgcn_readfirstlane(s_fail[s & 1])) break;
                b1 = b1 == 2 ? 0 : b1 + 1;
                b3 = b3 == 2 ? 0 : b3 + 1;
            }
            qr_wait_vmcnt<0>();
        } else {
            // two of the group's four row tiles; the other K half's slot stays zero
            const int32_t *gq = a.gx + (t0 * B + nn) * 4 * H + (cgc * 4 + 2 * kh) * 16 + 4 * grp;
            const int64_t gx_step = dir * B * 4 * H;
#pragma unroll
            for (int i = 0; i < 2; ++i) px[0][1][rh][2 * kh + i][lane] = px[1][1][rh][2 * kh + i][lane] = zero;
            v4i v0 = *(const v4i *)gq, v1 = *(const v4i *)(gq + 16);
            auto produce = [&](int par, bool more) {
                px[par][0][rh][2 * kh][lane] = v0;
                px[par][0][rh][2 * kh + 1][lane] = v1;
                gq += more ? gx_step : 0;
                v0 = *(const v4i *)gq;
                v1 = *(const v4i *)(gq + 16);
            };
            lds_barrier();
            produce(0, T > 1);
            lds_barrier();
            if (adm.mode >= REC_SHARED) return;          // uniform
            for (int s = 0; s < T; ++s) {
                if (s + 1 < T) produce((s + 1) & 1, s + 2 < T);
                lds_barrier();
                if (__builtin_amdgcn_readfirstlane(s_fail[s & 1])) break;
            }
        }
        return;
    }

    // ================= recurrence
    u64 *const admit_word = a.admit + ug;
    u64 found = 0;
    if (wave == 0 && members > 1) {
        if (a.n_come > 0 && mem >= a.n_come)    // diagnostic: this one comes when the others have gone ahead (or after 0.1 s)
            for (const u64 t0 = wall_clock64(); wall_clock64() - t0 < 10000000ull;)
                if (__hip_atomic_load(admit_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ADMIT_SHORT) break;
        if (lane == 0) found = __hip_atomic_fetch_add(admit_word, admit_field(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // ---- stationary operands: this wave's K steps (kh, kh + 2, ...) of its four row tiles; tiles 0 and 1 are the ones
    // whose cells it finishes (row tiles 2*kh, 2*kh + 1 of the cell group), tiles 2 and 3 its K partner's
    const int nks = (H + 63) >> 6;              // K steps in total (the blob pads to whole steps)
    v4i A[4][KH];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            const int ks = kh + 2 * k, rt = cg * 4 + (i < 2 ? 2 * kh + i : 2 * (1 - kh) + i - 2);
            A[i][k] = (have && ks < nks) ? weight(a.whh, a.nkc_h, rt, ks) : zero;   // absent: contributes nothing, whatever it reads
        }
    // 4-bit: minus the row sums of the weights (x 16), which a step number in the low nibbles multiplies
    v4i nrsum[4];
    const int pt = wave * 64 + lane;            // this lane's place in what is parked
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        nrsum[i] = zero;
        const v4i minus_ones = {-1, -1, -1, -1};
        if (!W8)
#pragma unroll
            for (int k = 0; k < KH; ++k) nrsum[i] = qr_mfma(A[i][k], minus_ones, nrsum[i]);
        if constexpr (PARK && !W8) pk_rsum[i][pt] = nrsum[i];
    }
    // ---- the cells this lane finishes: j0 .. j0 + CELLS - 1 of utterance n
    const int my_col = CELLS == 1 ? col & 7 : col;
    int n[NG], nn[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        n[g] = (ug + g) * 16 + my_col;
        nn[g] = n[g] < B ? n[g] : B - 1;
    }
    const int sub = CELLS == 1 ? col >> 3 : 0;
    const int j0 = 16 * cgc + 4 * grp + 2 * kh + sub;
    // exact powers of two undo what the 4-bit operands carry: 16 (x as it is) and 256
    constexpr float X_UNIT = (W8 || KX == 0) ? 1.0f : 0.0625f, H_UNIT = W8 ? 1.0f : 0.00390625f;
    v4f sx[CELLS], sh[CELLS], bb[CELLS];
    float c[NG][CELLS];
#pragma unroll
    for (int ct = 0; ct < CELLS; ++ct) {
#pragma unroll
        for (int gt = 0; gt < 4; ++gt) {
            sx[ct][gt] = a.x_scale * a.s_wih[gt * H + j0 + ct] * X_UNIT;
            sh[ct][gt] = a.h_scale * a.s_whh[gt * H + j0 + ct] * H_UNIT;
            bb[ct][gt] = a.bias[gt * H + j0 + ct];
        }
        if constexpr (PARK) {
            pk[ct][0][pt] = sx[ct];
            pk[ct][1][pt] = sh[ct];
            pk[ct][2][pt] = bb[ct];
        }
#pragma unroll
        for (int g = 0; g < NG; ++g) c[g][ct] = a.c0 ? a.c0[(int64_t)nn[g] * H + j0 + ct] : 0.0f;
    }
    // ---- exchange addresses
    int ncol = 16;                              // columns kept per 16-cell group
    if (CELLS == 1)
        for (ncol = 8; ncol >= 2 * B; ncol >>= 1) {}
    unsigned off[KH];
#pragma unroll
    for (int k = 0; k < KH; ++k) {
        int q = 4 * (kh + 2 * k) + grp;         // 16-cell group of this lane's operand; beyond the layer: any valid one (it meets zero weights)
        q = q < n_groups ? q : 0;
        off[k] = (unsigned)((q * ncol + (col & (ncol - 1))) * 16 * PER);
    }
    const unsigned st_off = (unsigned)(((cgc * ncol + (my_col & (ncol - 1))) * 16 + 4 * grp + 2 * kh + sub) * PER);
    const unsigned long long pub_mask = __ballot(have && my_col < ncol);
    bool store_ok[NG];
    unsigned long long out_mask[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        store_ok[g] = have && n[g] < B;
        out_mask[g] = __ballot(store_ok[g]);
    }
    // where this lane's sums of the input part lie in px[parity][K half]
    const int px_at = (rh * 4 + 2 * kh + sub) * 64 + grp * 16 + my_col;

    // ---- running pointers: output row of the step before, debug output
    const int64_t h_step = dir * B * a.ld_out;
    const bool dbg = a.dbg_c_all != nullptr;
    int8_t *hq[NG];
    float *dq[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        hq[g] = a.h_out + (t0 * B + nn[g]) * a.ld_out + a.col_off + j0;
        dq[g] = dbg ? a.dbg_c_all + (t0 * B + nn[g]) * H + j0 : nullptr;
    }

    if (wave == 0) {                            // (the weights were on their way meanwhile)
        RecAdmission r = {REC_LOCAL, 0, 0};
        if (members > 1) r = admit(admit_word, found, members, a.admit_ticks, lane);
        if (lane == 0) adm = r;
    }
    lds_barrier();
    lds_barrier();
    if (adm.mode >= REC_SHARED) return;         // uniform
    __builtin_amdgcn_s_setprio(3);              // these waves are the chain, the input waves fill its gaps
    const bool local = adm.mode == REC_LOCAL && !a.spread;   // uniform over the group
    unsigned codes[NG] = {};                    // the codes of the step before, one per byte
    v4i acc[4];
    float gx[CELLS][4];                         // this step's sums of the input part
    // What a step can do while its operands are on their way: its sums of the input part, and the start of its
    // accumulators, minus what the step number in the operands adds.  (The empty blocks keep the compiler from moving
    // this in front of the loads or behind the wait for them.)  Where registers are short the sums wait for the end of
    // the contraction.
    constexpr bool LATE_X = PARK && W8;
    auto load_x = [&](int turn, v4i (&x0)[CELLS], v4i (&x1)[CELLS]) {
        const v4i *p0 = &px[__builtin_amdgcn_readfirstlane(turn & 1)][0][0][0][0] + px_at, *p1 = p0 + 2 * 4 * 64;
#pragma unroll
        for (int ct = 0; ct < CELLS; ++ct) {
            x0[ct] = p0[64 * ct];
            x1[ct] = p1[64 * ct];
        }
    };
    auto add_x = [&](const v4i (&x0)[CELLS], const v4i (&x1)[CELLS]) {
#pragma unroll
        for (int ct = 0; ct < CELLS; ++ct) {
#pragma unroll
            for (int gt = 0; gt < 4; ++gt) gx[ct][gt] = (float)(x0[ct][gt] + x1[ct][gt]);
            asm volatile("" : "+v"(gx[ct][0]), "+v"(gx[ct][1]), "+v"(gx[ct][2]), "+v"(gx[ct][3]));
        }
    };
    auto prepare = [&](int s, int turn) {
        int tag = s & 15;
        if (!W8) asm volatile("" : "+s"(tag));
        v4i x0[CELLS], x1[CELLS];
        if (!LATE_X) load_x(turn, x0, x1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (PARK && !W8) nrsum[i] = pk_rsum[i][pt];
#pragma unroll
            for (int gt = 0; gt < 4; ++gt) acc[i][gt] = W8 ? 0 : __mul24(nrsum[i][gt], tag);
        }
        if (!LATE_X) add_x(x0, x1);
        if (!W8) asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]));
    };
    // The K partner's tiles of a step, from its operands; their way through LDS then runs under the own tiles' contraction.
    auto partner_tiles = [&](const v4i (&bf)[KH]) {
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            acc[2] = qr_mfma(A[2][k], bf[k], acc[2]);
            acc[3] = qr_mfma(A[3][k], bf[k], acc[3]);
        }
    };
    // The rest of the step; true: a wait ran out somewhere in the workgroup, leave.
    // ask(): more loads, once the sums have changed hands.
    auto step = [&](auto g_tag, const v4i (&bf)[KH], int s, int turn, auto &&ask) __attribute__((always_inline)) -> bool {
        constexpr int G = decltype(g_tag)::value;
        const int par = __builtin_amdgcn_readfirstlane(turn & 1);
        constexpr int K0 = KH < 2 ? KH : 2;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < K0; ++k) {
            acc[0] = qr_mfma(A[0][k], bf[k], acc[0]);
            acc[1] = qr_mfma(A[1][k], bf[k], acc[1]);
        }
        if (CELLS == 1) {
            part[par][wave][0][lane] = upper_from(acc[2], acc[3]);
        } else {
            part[par][wave][0][lane] = acc[2];
            part[par][wave][CELLS - 1][lane] = acc[3];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = K0; k < KH; ++k) {
            acc[0] = qr_mfma(A[0][k], bf[k], acc[0]);
            acc[1] = qr_mfma(A[1][k], bf[k], acc[1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (LATE_X) {                               // (in front of the barrier behind which they are overwritten)
            v4i x0[CELLS], x1[CELLS];
            load_x(turn, x0, x1);
            add_x(x0, x1);
        }
        store_out<CELLS>(hq[G], codes[G], s > 0 ? out_mask[G] : 0ull);   // the codes of the step before: here they hold nothing up
        hq[G] += s > 0 ? h_step : 0;
        lds_barrier();
        int fail_now = s_fail[par];   // a slot is written before its step's barrier only, and again two steps later: uniform
        v4i asum[CELLS];
#pragma unroll
        for (int ct = 0; ct < CELLS; ++ct)
            asum[ct] = (CELLS == 1 ? upper_from(acc[0], acc[1]) : acc[ct]) + part[par][wave ^ 1][ct][lane];
        asm volatile("" : "+v"(fail_now), "+v"(asum[0]));       // (both reads now, not one of them in front of the next poll)
        ask();
        codes[G] = 0u;
        unsigned word = W8 ? (unsigned)((s + 1) & 0xFF) * 0x01000100u : (unsigned)((s + 1) & 15) * 0x0101u;
#pragma unroll
        for (int ct = 0; ct < CELLS; ++ct) {
            if constexpr (PARK) {
                sx[ct] = pk[ct][0][pt];
                sh[ct] = pk[ct][1][pt];
                bb[ct] = pk[ct][2][pt];
            }
            const unsigned code = (unsigned)rec_cell<W8, C_FIRST>(sx[ct], sh[ct], bb[ct], gx[ct], asum[ct], a.h_inv, c[G][ct]);
            codes[G] |= (code & 0xFFu) << (8 * ct);
            word |= W8 ? (code & 0xFFu) << (16 * ct) : ((code & 15u) << 4) << (8 * ct);
        }
        if constexpr (NG == 1) store_codes<CELLS * PER>(par ? xb1 : xb0, st_off, word, pub_mask, local);
        else store_codes<CELLS * PER>(scalar((s & 1 ? xb1 : xb0) + G * ug_bytes), st_off, word, pub_mask, local);
        if (dbg) {
            if (store_ok[G])
#pragma unroll
                for (int ct = 0; ct < CELLS; ++ct) dq[G][ct] = c[G][ct];
            dq[G] += dir * B * H;
        }
        return __builtin_amdgcn_readfirstlane(fail_now) != 0;
    };
    // All steps but the first: the operands come from the exchange area.
    auto later_steps = [&](auto local_tag) __attribute__((always_inline)) {
        constexpr bool LOCAL = decltype(local_tag)::value;
        // Group G's words for step s.  Two groups in turn: they are requested in the turn before, late enough for them to be there.
        v4i v[NL];
        auto request = [&](auto g_tag, int s) __attribute__((always_inline)) {
            load_words<KH, PER, LOCAL>((__builtin_amdgcn_readfirstlane(s & 1) ? xb0 : xb1) + decltype(g_tag)::value * ug_bytes, (unsigned)ug_bytes, off, v);
        };
        const bool early = NG > 1 && ng > 1;   // uniform
        auto turn_of = [&](auto g_tag, int s, int turn) __attribute__((always_inline)) -> bool {
            constexpr int G = decltype(g_tag)::value;
            // words written at step s-1 carry tag s
            const int par = __builtin_amdgcn_readfirstlane(s & 1);
            const unsigned want = W8 ? (unsigned)(s & 0xFF) * 0x01000100u : (unsigned)(s & 15) * 0x01010101u;
            v4i bf[KH];
            asm volatile(".p2align 6");   // the poll on a cache line of its own: where it lay otherwise cost up to 3 % of a step
            for (int spins = 0;; ++spins) {
                if (!early || spins > 0) request(g_tag, s);
                prepare(s, turn);
                __builtin_amdgcn_sched_barrier(0);
                unsigned bad0 = 0u, bad1 = 0u;
#pragma unroll
                for (int i = 0; i < NL; ++i)
#pragma unroll
                    for (int d = 0; d < 4; d += 2) {
                        bad0 = or_xor(bad0, (unsigned)v[i][d], want);
                        bad1 = or_xor(bad1, (unsigned)v[i][d + 1], want);
                    }
                const unsigned bad = (bad0 | bad1) & (W8 ? 0xFF00FF00u : 0x0F0F0F0Fu);
#pragma unroll
                for (int k = 0; k < KH; ++k) {
                    if (W8) {
#pragma unroll
                        for (int d = 0; d < 4; ++d)   // the code bytes of two words
                            bf[k][d] = (int)__builtin_amdgcn_perm((unsigned)v[PER * k + (d >> 1) * (PER - 1)][(2 * (d & 1) + 1) & 3],
                                                                  (unsigned)v[PER * k + (d >> 1) * (PER - 1)][2 * (d & 1)], 0x06040200u);
                    } else {
                        bf[k] = v[k];
                    }
                }
                partner_tiles(bf);   // whether the words were current or not: the check runs under these
                if (__all(bad == 0u)) break;
                if (spins >= a.spin_limit) {
                    if (lane == 0) {
                        atomicExch(a.err, 1);
                        s_fail[NG == 1 ? par : turn & 1] = 1;
                    }
                    break;
                }
            }
            return step(g_tag, bf, s, turn, [&]() __attribute__((always_inline)) {
                if (NG > 1 && early) request(std::integral_constant<int, 1 - G>{}, s + G);   // uniform
            });
        };
        if (early) request(std::integral_constant<int, 0>{}, 1);
        for (int s = 1; s < T; ++s) {
            if (turn_of(std::integral_constant<int, 0>{}, s, s * ng)) break;
            if constexpr (NG > 1)
                if (ng > 1 && turn_of(std::integral_constant<int, 1>{}, s, s * ng + 1)) break;   // uniform
        }
    };
    // first step: the caller's initial state
    auto first = [&](auto g_tag) __attribute__((always_inline)) -> bool {
        v4i bf[KH];
        const int nc = (ug + decltype(g_tag)::value) * 16 + col, n0 = nc < B ? nc : B - 1;
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            const int k0 = (kh + 2 * k) * 64 + grp * 16;
            bf[k] = (a.h0 && k0 < H) ? *(const v4i *)(a.h0 + (int64_t)n0 * H + k0) : zero;
            if (!W8) bf[k] = (bf[k] << 4) & m;
        }
        prepare(0, decltype(g_tag)::value);
        partner_tiles(bf);
        return step(g_tag, bf, 0, decltype(g_tag)::value, [] {});
    };
    bool failed = first(std::integral_constant<int, 0>{});
    if constexpr (NG > 1)
        if (!failed && ng > 1) failed = first(std::integral_constant<int, 1>{});   // uniform
    if (!failed) {
        if (local) later_steps(std::true_type{}); else later_steps(std::false_type{});
    }
#pragma unroll
    for (int g = 0; g < NG; ++g)
        if (store_ok[g])
#pragma unroll
            for (int ct = 0; ct < CELLS; ++ct) {
                const int8_t code = (int8_t)(codes[g] >> (8 * ct));
                hq[g][ct] = code;
                if (a.h_last) a.h_last[(int64_t)n[g] * H + j0 + ct] = code;
                if (a.c_last) a.c_last[(int64_t)n[g] * H + j0 + ct] = c[g][ct];
            }
}

template <int KH, int KX, bool W8, int CELLS, bool C_FIRST, int NG>
__global__ __launch_bounds__(512, 2) void lstm_rec_kernel(const QrRecGroup g)
{
    __shared__ v4i px[2][2][2][4][64];      // [parity][K half][cell group][row tile][lane] sums of the input part
    __shared__ __attribute__((aligned(1024))) v4i xs[KX > 0 ? 3 * 2 * KX : 1][64];   // three frames of input codes, blocks of 8 utterances x 128 columns
    __shared__ int s_fail[2];
    __shared__ RecAdmission adm;
    // Grid: x = XCD (workgroups go out with x fastest, each to the next XCD), y = member, z = XCD's next group
    const int gi = g.group0 + (int)(blockIdx.z * gridDim.x + blockIdx.x), mem = (int)blockIdx.y, members = (int)gridDim.y;
    if (gi >= g.group_end) return;   // uniform
    const int ug = (gi >> (g.n - 1)) * NG;  // one or two directions
    const size_t ug_bytes = (size_t)(g.d[0].H >> 4) * 256 * (W8 ? 2 : 1);
    {
        const QrRecArgs a = g.d[gi & (g.n - 1)];   // a copy: a few wide scalar loads
        char *const xb = a.xbuf + (size_t)ug * ug_bytes;   // this group's exchange area, even steps
        member_steps<KH, KX, W8, CELLS, C_FIRST, NG>(a, ug, mem, members, xb, xb + (size_t)((a.B + 15) >> 4) * ug_bytes, ug_bytes, px, xs,
                                                 s_fail, adm);
    }
    if (adm.mode == REC_SHARED) {   // uniform
        int d = gi & (g.n - 1);
        asm volatile("" : "+s"(d));   // a copy of its own: the one above need not outlive the loop
        const QrRecArgs a = g.d[d];
        for (int i = 0; i < NG && (ug + i) * 16 < a.B; ++i) {   // uniform
            char *const xb = a.xbuf + (size_t)(ug + i) * ug_bytes;
            shared_steps<KH, KX, W8, C_FIRST>(a, ug + i, members, adm.rank, adm.n, xb, xb + (size_t)((a.B + 15) >> 4) * ug_bytes,
                                              &px[0][0][0][0][0], &xs[0][0], s_fail);
        }
    }
}

// XCDs of the current device and workgroups of this kernel that each holds at once; 0: none (or the device does not answer).
struct RecRoom {
    int n_xcd, per_xcd;
};
template <int KH, int KX, bool W8, int CELLS, bool C_FIRST, int NG>
RecRoom room()
{
    static std::atomic<int> known[QR_MAX_DEVICES];   // 0: not asked yet, -1: none, else per_xcd * 64 + n_xcd
    const int dev = qr_current_device();
    int v = known[dev].load(std::memory_order_relaxed);
    if (v == 0) {
        int n_cu = 0, n_xcd = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipDeviceGetAttribute(&n_xcd, hipDeviceAttributeNumberOfXccs, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, lstm_rec_kernel<KH, KX, W8, CELLS, C_FIRST, NG>, 512, 0) != hipSuccess)
            return {0, 0};
        n_xcd = n_xcd < 1 || n_xcd > 32 ? 8 : n_xcd;
        v = n_cu / n_xcd * per_cu * 64 + n_xcd;
        v = v >= 64 ? v : -1;
        known[dev].store(v, std::memory_order_relaxed);
    }
    return v > 0 ? RecRoom{v & 63, v >> 6} : RecRoom{0, 0};
}

template <int KH, int KX, bool W8, int CELLS, bool C_FIRST, int NG>
bool launch_rec_n(const QrRecGroup &g, hipStream_t st)
{
    QrRecGroup gg = g;
    const int members = (g.d[0].H + 31) / 32;
    const RecRoom r = room<KH, KX, W8, CELLS, C_FIRST, NG>();
    const int q = r.per_xcd / members;   // groups that an XCD holds together; beyond H = 512 it is one
    if (q < 1) return false;
    const int n_groups = g.n * (((g.d[0].B + 15) / 16 + NG - 1) / NG), most = q * r.n_xcd;
    // Two groups in turn take 1.6 to 1.75 times as long as one (2 x 640 cells, us a step, 64 -> 77 utterances: 320 inputs 0.95 ->
    // 1.49, 1280 inputs 0.99 -> 1.72, two launches 1.90 and 1.99), so they pay where they save more than three launches of seven:
    // 2 -> 1 and 4 -> 2, but not 3 -> 2 or 5 -> 3.  Narrower layers, 100 steps of two directions at 320 inputs, us: 272 cells and 300
    // utterances 227 -> 180, 400 and 130 224 -> 176, 512 and 130 229 -> 180, 576 and 80 228 -> 176.  (More than 640 cells leave no
    // registers for a second state.  Up to 256, where an XCD holds four groups or more, a second launch begins at 257
    // utterances and more, and 100 steps of 300 take 190 us against 99 of 130: not built.)
    if constexpr (NG == 1 && KH == 5 && KX > 0 && CELLS == 2) {
        const int n_pairs = g.n * (((g.d[0].B + 15) / 16 + 1) / 2);
        if (4 * ((n_groups + most - 1) / most) > 7 * ((n_pairs + most - 1) / most) && launch_rec_n<KH, KX, W8, CELLS, C_FIRST, 2>(g, st))
            return true;
    }
    if (NG > 1)
        for (int d = 0; d < g.n; ++d) gg.d[d].admit_ticks = gg.d[d].admit_ticks < (1 << 29) ? 2 * gg.d[d].admit_ticks : 1 << 30;
    for (int g0 = 0; g0 < n_groups; g0 += most) {
        gg.group0 = g0;
        gg.group_end = n_groups - g0 < most ? n_groups : g0 + most;
        const int turns = (gg.group_end - g0 + r.n_xcd - 1) / r.n_xcd;
        lstm_rec_kernel<KH, KX, W8, CELLS, C_FIRST, NG><<<dim3(r.n_xcd, members, turns), 512, 0, st>>>(gg);
    }
    return true;
}

template <int KH, int KX, bool W8, int CELLS, bool C_FIRST>
bool launch_rec_t(const QrRecGroup &g, hipStream_t st)
{
    return launch_rec_n<KH, KX, W8, CELLS, C_FIRST, 1>(g, st);
}

template <int KH, int KX>
bool launch_rec_w(const QrRecGroup &g, hipStream_t st)
{
    const int H = g.d[0].H, B = g.d[0].B;
    const bool few = B <= 8, w8 = g.d[0].w8 != 0;
    // One of the two products of c' = f*c + i*g is rounded before the fused multiply-add.  Which one follows an earlier
    // kernel, where the compiler had picked f*c in the form with two cells per lane and i*g in the other (up to 512 cells in
    // both).  The former ran where 16-cell x 16-utterance tiles outnumbered 256 compute units, beyond 768 cells only as
    // long as half of them did not.  So the last bit of a cell, and a code that sits on a rounding tie, can depend on the
    // batch that an utterance is in; but a tie is carried on through all later steps and layers, and one order for all
    // sizes would change what layers return.
    const int tiles = (H / 16) * ((B + 15) / 16) * g.n;
    if constexpr (KH >= 5)
        if (H > 512 && H % 32 == 0 && tiles > 256 && (H <= 768 || tiles <= 512))
            return w8 ? launch_rec_t<KH, KX, true, 2, true>(g, st) : launch_rec_t<KH, KX, false, 2, true>(g, st);
    if (w8) return few ? launch_rec_t<KH, KX, true, 1, false>(g, st) : launch_rec_t<KH, KX, true, 2, false>(g, st);
    return few ? launch_rec_t<KH, KX, false, 1, false>(g, st) : launch_rec_t<KH, KX, false, 2, false>(g, st);
}

template <int KH>
bool launch_rec_x(const QrRecGroup &g, hipStream_t st)
{
    if (g.d[0].gx) return launch_rec_w<KH, 0>(g, st);
    return g.d[0].I <= 384 ? launch_rec_w<KH, 3>(g, st) : launch_rec_w<KH, 10>(g, st);
}

}  // namespace

bool qr_rec_supported(int H, int B) { return H % 16 == 0 && H <= 1024 && B >= 1; }

size_t qr_rec_xbuf_bytes(int H, int B)
{
    return (size_t)2 * ((B + 15) / 16) * ((H + 63) / 64) * 64 * 4 * 8;
}

bool qr_rec_projects(int I) { return I <= 1280; }

size_t qr_rec_admit_bytes(int B) { return (size_t)((B + 15) / 16) * sizeof(u64); }

// Launches the recurrence of 1 or 2 directions (same H, B, T, width).  Returns false if it
// cannot run (size or residency): the caller then takes the step-by-step path.
bool qr_launch_recurrence(const QrRecGroup &g, hipStream_t st)
{
    const int kh = ((g.d[0].H + 63) / 64 + 1) / 2;
    if (kh <= 2) return launch_rec_x<2>(g, st);
    if (kh <= 5) return launch_rec_x<5>(g, st);
    if (kh <= 8) return launch_rec_x<8>(g, st);
    return false;
}
