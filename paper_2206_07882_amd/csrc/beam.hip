// Beam selection: per utterance the W best (parent, token) extensions (Sec. 2:
// the beam width is the number of hypotheses kept per decoding iteration).
// Selection runs on the GPU so that the decoding loop never returns to the host.
#include "kernels.h"
#include "select.h"

namespace {

// One workgroup (4 waves) per utterance; thread t forms the candidates t, t + 256, ... (fp32 add) and keeps their keys in
// registers: 256 groups for the bound, at most PER candidates each, so that rarely more than W * PER pass it.
// Bound by the chain of its steps; in one wave, which this was, 64 x 16 x 46 candidates took 17.4 us; a decoding
// round driven by the caller went from 87 to 76 us.
template <int PER>
__global__ __launch_bounds__(256) void beam_step_kernel(const float *__restrict__ score, const float *__restrict__ fused,
                                                         int W, int V, int blank, int force_blank,
                                                         int32_t *__restrict__ parent_out, int32_t *__restrict__ token_out,
                                                         float *__restrict__ score_out)
{
    __shared__ QrCand list[256 * PER], best[64];
    __shared__ unsigned group_best[256];
    __shared__ int n_list;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int C = W * V;
    const float *sc = score + (int64_t)b * W, *fu = fused + (int64_t)b * C;
    const int dw = 256 / V, dk = 256 - dw * V;   // uniform: from one candidate of a thread to its next
    int w = tid / V, k = tid - w * V;
    float f[PER], s[PER];
    bool ok[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int c = tid + 256 * i;
        ok[i] = c < C && (!force_blank || k == blank);
        f[i] = fu[c < C ? c : C - 1];
        s[i] = sc[w < W ? w : W - 1];
        w += dw;
        k += dk;
        if (k >= V) { k -= V; ++w; }
    }
    unsigned key[PER], top = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const float v = (s[i] + f[i]) + 0.0f;   // + 0: -0 becomes +0, one key per value
        key[i] = (ok[i] && v > -INFINITY) ? qr_float_key(v) : 0u;
        top = key[i] > top ? key[i] : top;
    }
    group_best[tid] = top;
    if (tid < 64) best[tid] = 0;
    if (tid == 0) n_list = 0;
    __syncthreads();
    unsigned g[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = group_best[i * 64 + lane];
    const QrBound bound(g, W);
    qr_gather<PER>(key, bound, [&](int i) { return tid + 256 * i; }, lane, &n_list, list);
    __syncthreads();
    qr_rank(list, n_list, W, tid, best);
    __syncthreads();
    if (tid < W) {
        const QrCand p = best[tid];
        const int c = p != 0 ? qr_cand_index(p) : 0;
        parent_out[(int64_t)b * W + tid] = p != 0 ? c / V : -1;
        token_out[(int64_t)b * W + tid] = p != 0 ? c % V : -1;
        score_out[(int64_t)b * W + tid] = p != 0 ? qr_cand_value(p) : -INFINITY;
    }
}

// Any number of candidates: one wave re-forms them from memory in every round.
__global__ __launch_bounds__(64) void beam_step_any_kernel(const float *__restrict__ score, const float *__restrict__ fused,
                                                            int W, int V, int blank, int force_blank,
                                                            int32_t *__restrict__ parent_out, int32_t *__restrict__ token_out,
                                                            float *__restrict__ score_out)
{
    const int b = blockIdx.x, lane = threadIdx.x;
    const float *sc = score + (int64_t)b * W, *fu = fused + (int64_t)b * W * V;
    auto value = [&](int c) -> float {
        const int w = c / V, k = c - w * V;
        return (force_blank && k != blank) ? -INFINITY : (sc[w] + fu[c]) + 0.0f;
    };
    int c;
    float v;
    qr_select_from_mem(value, W * V, W, lane, c, v);
    if (lane < W) {
        parent_out[(int64_t)b * W + lane] = c >= 0 ? c / V : -1;
        token_out[(int64_t)b * W + lane] = c >= 0 ? c % V : -1;
        score_out[(int64_t)b * W + lane] = v;
    }
}

}  // namespace

void qr_launch_beam(const float *score, const float *fused, int B, int W, int V, int blank, int force_blank,
                    int32_t *parent_out, int32_t *token_out, float *score_out, hipStream_t st)
{
    const int64_t C = (int64_t)W * V;
    // (16 candidates a thread are what LDS holds should all of them pass)
#define QR_BEAM(kernel, threads) kernel<<<B, threads, 0, st>>>(score, fused, W, V, blank, force_blank, parent_out, token_out, score_out)
    if (C <= 256) QR_BEAM(beam_step_kernel<1>, 256);
    else if (C <= 256 * 3) QR_BEAM(beam_step_kernel<3>, 256);
    else if (C <= 256 * 6) QR_BEAM(beam_step_kernel<6>, 256);
    else if (C <= 256 * 16) QR_BEAM(beam_step_kernel<16>, 256);
    else QR_BEAM(beam_step_any_kernel, 64);
#undef QR_BEAM
}

extern "C" qrnnt_status qrnnt_beam_step(const float *score, const float *fused, int32_t B, int32_t W, int32_t V,
                                        int32_t blank, int32_t force_blank, int32_t *parent_out, int32_t *token_out,
                                        float *score_out, void *stream)
{
    QR_REQUIRE(score && fused && parent_out && token_out && score_out, QRNNT_ERR_NULL);
    QR_REQUIRE(B > 0 && W > 0 && V > 0, QRNNT_ERR_SHAPE);
    QR_REQUIRE(W <= 64, QRNNT_ERR_UNSUPPORTED);
    QR_REQUIRE(blank >= 0 && blank < V, QRNNT_ERR_RANGE);
    qr_launch_beam(score, fused, B, W, V, blank, force_blank, parent_out, token_out, score_out, (hipStream_t)stream);
    return qr_launch_status();
}
