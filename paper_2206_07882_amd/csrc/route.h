// Routing of one utterance's W picks inside the decoding loop (Sec. 2: every
// decoding iteration keeps the W best extensions).  Blank picks join the frame's
// candidate list, label picks become the slots of the next round in selection
// order (prefix counts by ballot), the remaining slots die.  Runs in one wave:
// lane r < W holds pick r as (flat candidate index c = parent*V + token, or -1; score v).
//
// The networks' states and outputs after a label sequence are written once, into a row of a pool, and never move: a
// hypothesis names its row.  A label pick takes a free row of its utterance, a blank pick goes on with its parent's,
// and what no hypothesis of the new beam names is free again.  Only label picks cost an advance of the networks.
// (64 x 16 hypotheses: copying a new beam's rows was 25 MB read and written per frame, 4.5 us of the frame's 224 us;
// the alignment-length search passed every row through the networks, 63 us an iteration against 50.)
#pragma once

#include "kernels.h"
#include "mma_pipe.h"
#include "select.h"

// What lane w < W of the routing wave knows about hypothesis w of the current round: fetched at the start of the
// kernel, so that nothing in the routing waits for memory.
struct QrOwn {
    int node, len, row;
    int taken;                         // entries of the list of free rows that earlier rounds of the frame have passed (uniform)
    int free_row;                      // the w-th entry after those (qr_free_row)
    int serial;                        // of its sequence (QrTags)
};

__device__ __forceinline__ int qr_free_row(const QrRouteArgs &a, int b, int lane, int taken);

// States that are already there.  What the networks hold after a label sequence depends on the sequence alone, and a row
// keeps it until another sequence takes the row: a free one still has it.  So every row carries a tag (QrRouteArgs.tags) that
// says which sequence it stands for, and a label pick whose parent's row and label lead to a tag of the utterance names that
// row, be it in use or free, instead of taking one and advancing the networks; of several picks with the same sequence in one
// round one advances.  Sequences are compared exactly: by the label and the serial of the sequence before it, which a row
// gets together with its states and never shares with an earlier owner.  The same proposals come back from frame to frame,
// as most of them fall out of the beam again: of 64 utterances at beam 16 and 4 labels a frame (base networks) 29 of 32 label
// picks a frame find their states, and the launches of an advance are those of a list a tenth as long.  Finding a row takes
// three dependent LDS reads.  Whole calls, ms: 64 x 1000 frames 168.0 -> 104.5, 13 x 301 (2 x 2048 LM) 51.8 -> 33.9, 1 x 152
// 13.28 -> 11.1 (its rounds without a row to advance cost two launches that return); which searches look: launch_round (joint.hip).  Alignment-length search
// (its pool of two rows to a slot of the beam; three, four and six find no more), 64 x 300 16.65 -> 14.56, 1 x 152 at beam 4 level.
struct QrTags {
    v4i *tag;                          // LDS, [P rounded up to 64]: the utterance's
    unsigned short *slot;              // LDS, [1 << LOG]: hash table, row (relative) or anything at all
    unsigned char *twin;               // LDS, [1 << LOG]: the lane of a pick without a row
};

template <int LOG>
__device__ __forceinline__ unsigned qr_tag_hash(int serial, int tok)
{
    return ((unsigned)serial * 64u + (unsigned)tok) * 0x9E3779B1u >> (32 - LOG);
}

// The tags of utterance b go to LDS, by one wave: requested at the kernel's start, straight into LDS (wanted much later, and
// registers are short), and entered in the table when they are there.  (Of rows that share a place in the table one is found.)
__device__ __forceinline__ void qr_request_tags(const v4i *tags, int P, int lane, const QrTags &t)
{
    for (int i0 = 0; i0 < P; i0 += 64) {
        const int i = i0 + lane < P ? i0 + lane : P - 1;
        qr_load_lds16(tags + i, (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)(t.tag + i0));
    }
}

template <int LOG>
__device__ __forceinline__ void qr_enter_tags(int P, int lane, const QrTags &t)
{
    qr_wait_vmcnt<0>();
    for (int i = lane; i < P; i += 64) {
        const v4i g = t.tag[i];
        if (g[0] >= 0) t.slot[qr_tag_hash<LOG>(g[0], g[1])] = (unsigned short)i;
    }
}

// The row (relative) that holds the sequence of this lane's label pick, P: none.  steps: none, and the networks have to advance;
// first: the lane of the pick that does so for this one's sequence.
template <int LOG, bool TWINS>
__device__ __forceinline__ int qr_held_row(int P, int lane, bool is_lab, int serial, int tok, int now, const QrTags &t, bool &steps, int &first)
{
    const unsigned at = qr_tag_hash<LOG>(serial, tok);
    int held = is_lab ? t.slot[at] : P;      // (an entry that nobody has written may be any number)
    if (held < P) {
        const v4i g = t.tag[held];
        held = g[0] == serial && g[1] == tok ? held : P;
    } else {
        held = P;
    }
    const bool hit = held < P;
    if (hit) t.tag[held][3] = now;
    first = lane;
    if (TWINS) {
        if (is_lab && !hit) t.twin[at] = (unsigned char)lane;
        __builtin_amdgcn_wave_barrier();
        first = is_lab && !hit ? t.twin[at] : lane;
        const int first_serial = __shfl(serial, first), first_tok = __shfl(tok, first);
        first = first_serial == serial && first_tok == tok ? first : lane;
    }
    steps = is_lab && !hit && first == lane;
    return held;
}

// Rows for this round's label picks (lanes with is_lab: parent's row, label): a row that holds the sequence, or the next
// free one that no pick of this frame names.  Returns the row; steps: the networks have to advance into it.  n_passed: how
// much of the list of free rows lies behind the round.  There is always enough of it: a frame's picks name or take
// W * max_sym rows at most (an iteration's of the alignment-length search W), the list is that long.  last: the row
// (relative) that was taken last, if any.  mask: 64 words of LDS, private to the wave.
// TWINS: two hypotheses may have one sequence, so that two picks want one new row.
template <int LOG, bool TWINS>
__device__ __forceinline__ int qr_find_rows(const QrRouteArgs &a, int b, int lane, bool is_lab, int par_serial, int tok, const QrOwn &own,
                                            const QrTags &t, unsigned *mask, bool &steps, int &n_passed, int &last)
{
    const int row0 = b * a.P;
    const int serial = is_lab ? par_serial : -1;
    int first;
    const int held = qr_held_row<LOG, TWINS>(a.P, lane, is_lab, serial, tok, a.now, t, steps, first);
    const bool hit = held < a.P;
    if (hit) a.tags[(size_t)row0 + held][3] = a.now;
    const unsigned long long sm = __ballot(steps);
    const int n_new = (int)__popcll(sm);
    int row = row0 + held;
    n_passed = own.taken;
    if (n_new > 0) {   // uniform
        const int k_new = (int)__popcll(sm & ((1ull << lane) - 1ull));
        int got = 0, entry = own.free_row, new_row;
        bool ok = t.tag[entry - row0][3] != a.now;
        unsigned long long om = __ballot(ok);
        if ((~om & ((2ull << (n_new - 1)) - 1ull)) == 0ull) {   // uniform: the next ones are all there to take
            new_row = __shfl(entry, k_new < n_new ? k_new : 0);
            last = __builtin_amdgcn_readlane(entry, n_new - 1) - row0;
            n_passed += n_new;
        } else {
            for (;;) {     // (once, unless most of the next 64 free rows are named already)
                const int k = got + (int)__popcll(om & ((1ull << lane) - 1ull));
                if (ok && k < n_new) mask[k] = (unsigned)(entry - row0) | (unsigned)lane << 16;
                got += (int)__popcll(om);
                if (got >= n_new) break;
                n_passed += 64;
                entry = qr_free_row(a, b, lane, n_passed);
                ok = t.tag[entry - row0][3] != a.now;
                om = __ballot(ok);
            }
            __builtin_amdgcn_wave_barrier();
            const unsigned mine = mask[k_new < n_new ? k_new : 0], end = mask[n_new - 1];
            n_passed += (int)(end >> 16) + 1;
            last = (int)(end & 0xFFFFu);
            new_row = row0 + (int)(mine & 0xFFFFu);
        }
        if (steps) a.tags[new_row] = v4i{serial, tok, a.serial0 + 1 + k_new, a.now};
        const int first_row = TWINS ? __shfl(new_row, first) : new_row;
        row = hit ? row : first_row;
    }
    return row;
}

__device__ __forceinline__ QrOwn qr_load_own(const QrRouteArgs &a, int b, int lane)
{
    const int o = b * a.W + (lane < a.W ? lane : 0);
    QrOwn own;
    own.node = a.node_src[o];
    own.len = a.len_src[o];
    own.row = a.row_src[o];
    own.taken = a.n_taken ? a.n_taken[b] : 0;
    own.free_row = 0;
    return own;
}

__device__ __forceinline__ int qr_free_row(const QrRouteArgs &a, int b, int lane, int taken)
{
    int f = taken + lane;              // (a pick never needs more than there are, see the pool's size in decode.hip)
    f = f < a.P ? f : a.P - 1;
    return a.free_rows[(size_t)b * a.P + f];
}

// The same where the tags stay in LDS and no list is kept: a row is free if it has not been named in frame `now` (those of the
// beam are marked when the frame begins), and the free ones are taken in turn from row `cursor` (relative) on.  There is always
// one: a frame names W * (max_sym + 1) = P rows at most.  Serials serial0 + 1 ... go to the new sequences.
template <int LOG>
__device__ __forceinline__ int qr_find_rows_in_turn(int P, int row0, int lane, bool is_lab, int par_serial, int tok, int now, int serial0,
                                                    int &cursor, const QrTags &t, unsigned *mask, bool &steps)
{
    const int serial = is_lab ? par_serial : -1;
    int first;
    const int held = qr_held_row<LOG, true>(P, lane, is_lab, serial, tok, now, t, steps, first);
    const unsigned long long sm = __ballot(steps), lt = (1ull << lane) - 1ull;
    const int n_new = (int)__popcll(sm);
    int row = held;
    if (n_new > 0) {   // uniform
        const int k_new = (int)__popcll(sm & lt);
        int got = 0;
        for (int i0 = 0; i0 < P; i0 += 64) {
            int i = cursor + i0 + lane;
            i = i < P ? i : i - P;
            i = i0 + lane < P ? i : 0;
            const bool ok = i0 + lane < P && t.tag[i][3] != now;
            const unsigned long long om = __ballot(ok);
            const int k = got + (int)__popcll(om & lt);
            if (ok && k < n_new) mask[k] = (unsigned)i;
            got += (int)__popcll(om);
            if (got >= n_new) break;   // uniform
        }
        __builtin_amdgcn_wave_barrier();
        const int new_row = (int)mask[k_new < n_new ? k_new : 0], last = (int)mask[n_new - 1];
        cursor = last + 1 < P ? last + 1 : 0;
        if (steps) t.tag[new_row] = v4i{serial, tok, serial0 + 1 + k_new, now};
        const int first_row = __shfl(new_row, first);
        row = held < P ? held : first_row;
    }
    return row0 + row;
}

// The utterance's free rows for what follows: all of its P rows except the ones that lanes with `held` name, from row
// `first` (relative) on, so that what was taken last is taken again last.
// mask: 64 words of LDS, private to the calling wave (P <= 64 * 17 bits).
__device__ __forceinline__ void qr_list_free_rows(const QrRouteArgs &a, int b, int lane, bool held, int row, unsigned *mask, int first = 0)
{
    __builtin_amdgcn_wave_barrier();
    mask[lane] = 0u;
    __builtin_amdgcn_wave_barrier();
    const int rel = row - b * a.P;
    if (held && rel >= 0 && rel < a.P) atomicOr(mask + (rel >> 5), 1u << (rel & 31));
    __builtin_amdgcn_wave_barrier();
    int n = 0;
    for (int i0 = 0; i0 < a.P; i0 += 64) {
        const bool in = i0 + lane < a.P;
        int i = i0 + lane + first;
        i = i < a.P ? i : i - a.P;
        i = in ? i : 0;
        const bool is_free = in && ((mask[i >> 5] >> (i & 31)) & 1u) == 0u;
        const unsigned long long fm = __ballot(is_free);
        const int pos = n + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(fm >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)fm, 0u));
        if (is_free) a.free_rows[(size_t)b * a.P + pos] = b * a.P + i;
        n += (int)__popcll(fm);
    }
    __builtin_amdgcn_wave_barrier();
}

// Returns the length of the utterance's candidate list after this round (uniform).
// own: hypothesis `lane` of the current round; a pick reads its parent's from that lane.
// nx0: the length of the utterance's candidate list before this round (a.nx_count[b], fetched early as well);
// add(e, score, info) puts a candidate at its end.
template <int LOG, bool TAGS, class Add>
__device__ __forceinline__ int qr_route_picks(const QrRouteArgs &a, int b, int lane, int c, float v, const QrOwn &own, int nx0,
                                              const QrTags &tags, unsigned *mask, Add &&add)
{
    if (lane == 0 && b == 0 && a.live_clear) *a.live_clear = 0;
    if (lane == 0 && b == 0 && a.n_rows_clear) *a.n_rows_clear = 0;
    const int W = a.W, V = a.V;
    const bool in = lane < W;
    const bool found = in && c >= 0;
    const int par = found ? c / V : 0, tok = found ? c - (c / V) * V : 0;
    const bool is_blank = found && tok == a.blank;
    const bool is_lab = found && tok != a.blank && !a.last_round;
    const unsigned long long bm = __ballot(is_blank), lm = __ballot(is_lab);
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int par_node = __shfl(own.node, par), par_len = __shfl(own.len, par), par_row = __shfl(own.row, par);
    const int par_serial = __shfl(own.serial, par);
    const int k_lab = (int)__popcll(lm & lt);            // this pick's number among the label picks
    if (is_blank) {
        add(nx0 + (int)__popcll(bm & lt), v, v4i{par_row, par_node, par_len, 0});
    }
    const int cnt = nx0 + (int)__popcll(bm);
    if (a.last_round) return cnt;
    const int n_lab = __popcll(lm);
    if (lane == 0 && n_lab > 0 && a.live_next) atomicAdd(a.live_next, 1);
    // Rows for the labels, and the place of those that advance in the list (the order of the utterances in it does not
    // matter): asked for now, used last.  A single utterance has the list to itself.
    int base = 0, row = 0, n_new = 0, k_new = 0;
    bool steps = false;
    if (n_lab > 0) {   // uniform
        int n_passed = own.taken + n_lab, last;
        if (TAGS) {
            row = qr_find_rows<LOG, true>(a, b, lane, is_lab, par_serial, tok, own, tags, mask, steps, n_passed, last);
        } else {
            row = __shfl(own.free_row, k_lab);
            steps = is_lab;
        }
        const unsigned long long sm = __ballot(steps);
        n_new = (int)__popcll(sm);
        k_new = (int)__popcll(sm & lt);
        if (lane == 0 && n_new > 0) {
            if (a.B == 1) *a.n_rows_next = n_new;
            else base = atomicAdd(a.n_rows_next, n_new);
            a.n_taken[b] = n_passed;
        }
    }
    if (is_lab) {
        const int dst = b * W + k_lab;
        const int id = a.node_base + dst;
        a.node_tok[id] = tok;
        a.node_prev[id] = par_node;
        a.score_dst[dst] = v;
        a.node_dst[dst] = id;
        a.len_dst[dst] = par_len + 1;
        a.row_dst[dst] = row;
    }
    if (in && lane >= n_lab) {
        const int dst = b * W + lane;
        a.score_dst[dst] = -INFINITY;
        a.node_dst[dst] = 0;
        a.len_dst[dst] = 0;
        a.row_dst[dst] = b * a.P;   // any row of the utterance
    }
    if (n_new > 0) {   // uniform
        base = __builtin_amdgcn_readfirstlane(base);
        if (steps) a.rows_next[base + k_new] = v4i{row, par_row, tok, 0};
    }
    return cnt;
}

// One iteration of the alignment-length synchronous search for utterance b (one wave; Sec. 2 names the search,
// the algorithm is the published one).  Lane r < W holds pick r (flat candidate index c = parent*V + token or -1,
// score v).
//   - pick r becomes slot r of the next beam: a blank keeps the parent's sequence and state, a label extends it;
//   - recombination: picks that stand for the same label sequence (same length and same 64-bit sequence hash)
//     are one hypothesis; the best-ranked keeps its slot with log(sum exp(scores)), the others die;
//   - a label that stays takes a free row of the state pool and joins the list of those the networks advance for, or
//     (reuse) names the row of a live hypothesis that holds its sequence; a blank goes on with its parent's row;
//   - the rows that no slot of the next beam names are free again.
// Hypotheses that finish (a blank at the last frame) are no candidates: qr_alsd_finish takes them.

// What lane w < W of the routing wave knows, beyond QrOwn, about hypothesis w of the current beam.
struct QrAlsdOwn {
    QrOwn h;
    unsigned long long hash;
    float score;
};

__device__ __forceinline__ QrAlsdOwn qr_alsd_load_own(const QrRouteArgs &a, const QrAlsdArgs &s, int b, int lane)
{
    const int own = b * a.W + (lane < a.W ? lane : 0);
    QrAlsdOwn o;
    o.hash = s.hash_src[own];  o.score = a.score_src[own];
    return o;
}

template <int LOG, bool TAGS>
__device__ __forceinline__ void qr_alsd_route(const QrRouteArgs &a, const QrAlsdArgs &s, int b, int lane, int c, float v,
                                              const QrAlsdOwn &o, const QrTags &tags, unsigned *mask)
{
    const int W = a.W, V = a.V;
    const bool in = lane < W;
    const bool found = in && c >= 0;
    const int par = found ? c / V : 0, tok = found ? c - (c / V) * V : a.blank;
    const bool is_lab = found && tok != a.blank;
    // the parent's sequence, taken from the lane that holds it
    const int len_p = __shfl(o.h.len, par);
    const int node_p = __shfl(o.h.node, par);
    const int row_p = __shfl(o.h.row, par);
    const int serial_p = __shfl(o.h.serial, par);
    const unsigned long long hash_p = ((unsigned long long)(unsigned)__shfl((int)(unsigned)(o.hash >> 32), par) << 32) |
                                      (unsigned long long)(unsigned)__shfl((int)(unsigned)o.hash, par);
    const int new_len = len_p + (is_lab ? 1 : 0);
    const unsigned long long new_hash = is_lab ? hash_p * 0x9E3779B97F4A7C15ull + (unsigned long long)(tok + 1) : hash_p;
    const int h_lo = (int)(unsigned)new_hash, h_hi = (int)(unsigned)(new_hash >> 32);
    // length and "is a pick" in one word: a lane without a pick gets a value no other lane has
    const int lw = found ? new_len : -1 - lane;
    // Picks that may share a sequence with another one, by one word of theirs (nearly always just those that do); only
    // these are compared in full and merged, one after the other.  (Comparing and merging all W with all W took 4 us of
    // an iteration's 42 at 64 x 16 hypotheses.)
    const int word = h_lo ^ (h_hi * (int)0x9E3779B1u) ^ (lw * (int)0x85EBCA6Bu);
    int alike = 0;
    for (int j = 0; j < W; ++j) alike += __builtin_amdgcn_readlane(word, j) == word ? 1 : 0;
    const unsigned long long twins = __ballot(found && alike > 1);
    int leader = lane;
    float m = v, sum = 1.0f;        // alone: log(exp(v - v)) = 0
    if (twins != 0ull) {            // uniform
        unsigned long long eq = 0ull;   // the picks that stand for this lane's label sequence
        for (unsigned long long t = twins; t != 0ull; t &= t - 1ull) {
            const int j = __ffsll((long long)t) - 1;
            const bool same = __builtin_amdgcn_readlane(lw, j) == lw && __builtin_amdgcn_readlane(h_lo, j) == h_lo &&
                              __builtin_amdgcn_readlane(h_hi, j) == h_hi;
            const float vj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
            if (same) {
                eq |= 1ull << j;
                leader = j < leader ? j : leader;
                m = fmaxf(m, vj);
            }
        }
        float s2 = 0.0f;
        for (unsigned long long t = twins; t != 0ull; t &= t - 1ull) {
            const int j = __ffsll((long long)t) - 1;
            const float vj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
            if ((eq >> j) & 1ull) s2 += qr_exp(vj - m);
        }
        sum = eq != 0ull ? s2 : sum;
    }
    const bool keep = found && leader == lane;
    const unsigned long long km = __ballot(keep);
    if (lane == 0 && km != 0ull && a.live_next) atomicAdd(a.live_next, 1);
    // Reuse of cached hypotheses (Sec. 4.1): when a live hypothesis of the current beam already holds the sequence this label
    // pick produces (y + k is in the beam and y proposes k again one frame later), the new slot names that hypothesis' row.
    // Looked for in this way, by the sequences' hashes, only where the caller counts them or rows are not looked for by their
    // tags, which find nearly all of these and others.
    int reuse_slot = -1;
    if (s.reuse && (s.stats || !TAGS)) {   // uniform
        const int o_hlo = (int)(unsigned)o.hash, o_hhi = (int)(unsigned)(o.hash >> 32);
        for (int j = 0; j < W; ++j) {
            const bool live_j = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(o.score), j)) > -INFINITY;
            const bool same = live_j && __builtin_amdgcn_readlane(o.h.len, j) == new_len &&
                              __builtin_amdgcn_readlane(o_hlo, j) == h_lo && __builtin_amdgcn_readlane(o_hhi, j) == h_hi;
            if (same && keep && is_lab && reuse_slot < 0) reuse_slot = j;
        }
    }
    if (s.stats) {   // uniform
        const int n_req = (int)__popcll(__ballot(keep && is_lab)), n_hit = (int)__popcll(__ballot(reuse_slot >= 0));
        if (lane == 0 && n_req) atomicAdd(s.stats, n_req);
        if (lane == 0 && n_hit) atomicAdd(s.stats + 1, n_hit);
    }
    const bool wants = keep && is_lab && reuse_slot < 0;   // a row that holds the sequence, or one that the networks advance into
    bool steps = false;
    int first = TAGS ? __shfl(o.h.free_row, 0) - b * a.P : 0;   // where the next list of free rows begins
    const int reuse_row = __shfl(o.h.row, reuse_slot >= 0 ? reuse_slot : 0);
    int row = reuse_slot >= 0 ? reuse_row : row_p;
    if (!TAGS) {
        const unsigned long long wm = __ballot(wants);
        const int new_row = __shfl(o.h.free_row, (int)__popcll(wm & ((1ull << lane) - 1ull)));
        row = wants ? new_row : row;
        steps = wants;
    } else if (__ballot(wants) != 0ull) {   // uniform
        int n_passed, last = -1;
        const int found_row = qr_find_rows<LOG, false>(a, b, lane, wants, serial_p, tok, o.h, tags, mask, steps, n_passed, last);
        row = wants ? found_row : row;
        if (last >= 0) first = last + 1 < a.P ? last + 1 : 0;   // uniform
    }
    const unsigned long long sm = __ballot(steps);
    const int k_step = (int)__popcll(sm & ((1ull << lane) - 1ull));
    int base = 0;   // the place of the utterance's labels in the list: asked for now, used last (see qr_route_picks)
    if (sm != 0ull && lane == 0) {
        if (a.B == 1) *a.n_rows_next = (int)__popcll(sm);
        else base = atomicAdd(a.n_rows_next, (int)__popcll(sm));
    }
    if (in) {
        const int dst = b * W + lane;
        if (keep) {
            int node = node_p;
            if (is_lab) {
                node = a.node_base + dst;
                a.node_tok[node] = tok;
                a.node_prev[node] = node_p;
            }
            a.score_dst[dst] = m + qr_log(sum);
            a.node_dst[dst] = node;
            a.len_dst[dst] = new_len;
            s.hash_dst[dst] = new_hash;
            a.row_dst[dst] = row;
        } else {
            a.score_dst[dst] = -INFINITY;
            a.node_dst[dst] = 0;
            a.len_dst[dst] = 0;
            s.hash_dst[dst] = 0ull;
            a.row_dst[dst] = b * a.P;   // any row of the utterance
        }
    }
    qr_list_free_rows(a, b, lane, keep, row, mask, first);
    if (sm != 0ull) {   // uniform
        base = __builtin_amdgcn_readfirstlane(base);
        if (steps) a.rows_next[base + k_step] = v4i{row, row_p, tok, 0};
    }
}

// The running list of the W best finished hypotheses of utterance b (one wave) takes the new ones in, ordered by (score
// descending, insertion order), new ones in slot order.  Lane w < W holds rank w of the list and, as fin_new, the score
// with which hypothesis w of the current beam finishes now (-inf: it does not); node, len: that hypothesis'.
struct QrAlsdFinished {
    float score;  int node, len;       // rank w of the list
    int new_node, new_len;             // hypothesis w
};

__device__ __forceinline__ QrAlsdFinished qr_alsd_load_finished(const QrRouteArgs &a, const QrAlsdArgs &s, int b, int lane)
{
    const int own = b * a.W + (lane < a.W ? lane : 0);
    return QrAlsdFinished{s.fin_score[own], s.fin_node[own], s.fin_len[own], a.node_src[own], a.len_src[own]};
}

__device__ __forceinline__ void qr_alsd_finish(const QrAlsdArgs &s, int b, int W, int lane, float fin_new, const QrAlsdFinished &f)
{
    const bool in = lane < W;
    const float fn = in ? fin_new : -INFINITY;
    if (__ballot(fn > -INFINITY) == 0ull) return;   // uniform
    const float fo = in ? f.score : -INFINITY;
    int rank_o = 0, rank_n = 0;
    for (int j = 0; j < W; ++j) {
        const float oj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(fo), j));
        const float nj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(fn), j));
        rank_o += ((oj > fo) || (oj == fo && j < lane)) ? 1 : 0;
        rank_o += (nj > fo) ? 1 : 0;
        rank_n += (oj >= fn) ? 1 : 0;
        rank_n += ((nj > fn) || (nj == fn && j < lane)) ? 1 : 0;
    }
    if (in && rank_o < W) {
        const int o = b * W + rank_o;
        s.fin_score[o] = fo;  s.fin_node[o] = f.node;  s.fin_len[o] = f.len;
    }
    if (in && rank_n < W) {
        const int o = b * W + rank_n;
        s.fin_score[o] = fn;  s.fin_node[o] = fn > -INFINITY ? f.new_node : 0;  s.fin_len[o] = fn > -INFINITY ? f.new_len : 0;
    }
}
