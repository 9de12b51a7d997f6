"""End-to-end parity: encoder stack and the on-device beam search against the
oracle, free-running (no teacher forcing).  The sizes are small enough that a
rounding tie of a hidden code is improbable; the seeds are fixed, so the outcome
is deterministic."""
import os

import numpy as np
import pytest
import torch

import oracle
from oracle import models as omodels
from paper_2206_07882_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    return t.detach().cpu().numpy()


def _compare_beams(got, ref, atol=2e-3):
    tok_g, len_g, sc_g = (host(x) for x in got)
    tok_r, len_r, sc_r = ref
    assert np.array_equal(len_g, len_r)
    L = min(tok_g.shape[2], tok_r.shape[2])
    assert np.array_equal(tok_g[:, :, :L], tok_r[:, :, :L])
    fin = np.isfinite(sc_r)
    assert np.array_equal(np.isfinite(sc_g), fin)
    assert np.abs(sc_g[fin] - sc_r[fin]).max() < atol


@pytest.mark.parametrize("std", [0.1, 0.6])
def test_config0_end_to_end_beams_identical(gpu_lib, std):
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(0, weight_std=std)
    T, B = 20, 2
    feats = synth.features(0, T, B, m.feat_dim)
    # oracle
    layers, proj = omodels.encoder_from_float(m)
    x_r, e_r = omodels.encoder_forward(layers, proj, feats, m.alpha_x)
    ref = oracle.decode(omodels.model_from_float(m), e_r, m.beam, m.max_sym)
    # GPU
    enc = gmodel.Encoder(m, DEV)
    x_g, e_g = enc.forward(dev(feats))
    assert np.array_equal(host(x_g), x_r)
    assert np.abs(host(e_g) - e_r).max() < 1e-5
    G = gmodel.model_from_float(m, DEV)
    got = gpu_lib.decode(G, e_g, m.beam, m.max_sym)
    _compare_beams(got, ref)
    # the stored golden beams say the same
    path = os.path.join(os.path.dirname(__file__), "golden", "cfg0_decode.txt")
    lines = [l for l in open(path).read().splitlines() if l.startswith(f"{std} ")]
    tok_g, len_g, _ = (host(x) for x in got)
    for l in lines:
        head, labs = l.split("|")
        _, b, w, _ = head.split()
        want = [int(t) for t in labs.split()]
        assert tok_g[int(b), int(w), :len_g[int(b), int(w)]].tolist() == want


@pytest.mark.parametrize("T,B", [(12, 3), (9, 1)])
def test_encoder_stack_full_widths_layer_by_layer(gpu_lib, T, B):
    """The encoder of configuration 1 (6 bidirectional layers of 640 cells over 240 features, then the
    projection to the joint) on a short batch: every layer is compared with the oracle's layer run on the
    GPU's own output of the layer below, so that a rounding tie in one layer cannot travel upwards; the
    projection is compared on the GPU's final codes; the whole stack is also compared free-running."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    m = synth.make_model(1)
    feats = synth.features(1, T, B, m.feat_dim)
    layers, proj = omodels.encoder_from_float(m)
    enc = gmodel.Encoder(m, DEV)
    x_free, e_free = omodels.encoder_forward(layers, proj, feats, m.alpha_x)
    x_g, e_g = enc.forward(dev(feats))
    assert (host(x_g) == x_free).mean() >= 0.995
    # layer by layer on the GPU's own inputs
    ws = enc.workspace(T, B, DEV)
    x = q.quantize_act(dev(feats), enc.inv_s_x)
    assert np.array_equal(host(x), oracle.quant_sym(feats, enc.inv_s_x, 4))
    for li, (dirs_g, dirs_o) in enumerate(zip(enc.layers, layers)):
        H = dirs_g[0].H
        out = torch.empty((T, B, 2 * H), dtype=torch.int8, device=DEV)
        q.bilstm_layer(dirs_g[0], dirs_g[1], x, h_out=out, workspace=ws)
        ref = np.zeros((T, B, 2 * H), np.int8)
        for d, L in enumerate(dirs_o):
            oracle.lstm_layer(L, host(x), reverse=(d == 1), h_out=ref, col_off=d * H)
        og = host(out)
        assert np.abs(og.astype(np.int32) - ref).max() <= 1, f"layer {li}"
        assert (og == ref).mean() >= 0.999, f"layer {li}: {(og == ref).mean()}"
        x = out
    assert np.array_equal(host(x), host(x_g))
    e_ref = oracle.linear(proj, host(x).reshape(T * B, -1)).reshape(T, B, -1)
    assert np.abs(host(e_g) - e_ref).max() <= 1e-5 * np.abs(e_ref).max() + 1e-6


@pytest.mark.parametrize("B,W,max_sym,T,lms,std", [(3, 4, 2, 12, True, 0.6), (2, 1, 3, 10, True, 0.6),
                                                   (4, 16, 4, 6, True, 0.5), (2, 3, 0, 8, False, 0.6),
                                                   (5, 8, 1, 9, False, 0.4), (5, 16, 2, 6, True, 0.5),
                                                   (3, 33, 2, 5, True, 0.5), (2, 64, 1, 4, True, 0.5),
                                                   (1, 16, 4, 1, True, 0.6), (16, 64, 2, 4, True, 0.5)])
def test_decode_variants_match_oracle(gpu_lib, B, W, max_sym, T, lms, std):
    """Beam widths on both sides of the 16-column tile and up to the maximum of 64, a single frame, no LMs, no
    labels (max_sym 0), and 16 x 64 = 1024 hypotheses of the tiny networks: the tiled step kernel with partial
    K chunks running over the device-built list of advancing hypotheses."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(0, weight_std=std)
    if not lms:
        m.lm_src = m.lm_ext = None
    m.rho = 0.1
    e = synth.normal(100 + B + W, (T, B, m.J), 1.0)
    ref = oracle.decode(omodels.model_from_float(m), e, W, max_sym, max_len=max(1, T * max(max_sym, 1)))
    G = gmodel.model_from_float(m, DEV)
    got = gpu_lib.decode(G, dev(e), W, max_sym, max_len=max(1, T * max(max_sym, 1)))
    _compare_beams(got, ref)


def test_decode_full_width_networks_small_batch(gpu_lib):
    """The measured layer widths (pred 768, LMs 2 x 1024, joint 256, V 46) on a
    short, narrow problem the oracle finishes in seconds."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(4, enc_layers=1)
    T, B, W, max_sym = 6, 2, 4, 2
    e = synth.normal(200, (T, B, m.J), 1.0)
    ref = oracle.decode(omodels.model_from_float(m), e, W, max_sym)
    got = gpu_lib.decode(gmodel.model_from_float(m, DEV), dev(e), W, max_sym)
    _compare_beams(got, ref)


def test_decode_full_width_networks_128_hypotheses(gpu_lib):
    """Same widths at 8 utterances x beam 16 = 128 hypotheses: the compute-bound step
    kernel with full tiles and the per-token table of layer-0 input projections."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(4, enc_layers=1)
    T, B, W, max_sym = 2, 8, 16, 2
    e = synth.normal(201, (T, B, m.J), 1.0)
    ref = oracle.decode(omodels.model_from_float(m), e, W, max_sym)
    got = gpu_lib.decode(gmodel.model_from_float(m, DEV), dev(e), W, max_sym)
    _compare_beams(got, ref)


@pytest.mark.parametrize("B,W,max_sym,T", [(3, 4, 2, 8), (5, 16, 3, 5)])
def test_decode_with_bottleneck_and_unequal_depths(gpu_lib, B, W, max_sym, T):
    """Networks of unequal depth and an external LM with a bottleneck layer (Sec. 2) on the tiny
    configuration: source LM 1 layer, external LM 2 layers + bottleneck 16."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(0, weight_std=0.5)
    rng = np.random.default_rng(77)
    m.lm_ext = synth._net(rng, m.V, 64, 64, 2, m.V, 0.5, mid=16)
    m.lm_ext.alpha_mid = 2.0
    m.rho = 0.2
    e = synth.normal(300 + B, (T, B, m.J), 1.0)
    ref = oracle.decode(omodels.model_from_float(m), e, W, max_sym)
    got = gpu_lib.decode(gmodel.model_from_float(m, DEV), dev(e), W, max_sym)
    _compare_beams(got, ref)
    assert (ref[1] > 0).any()


def test_decode_paper_shapes_small_batch(gpu_lib):
    """The layer shapes of Sec. 2 (prediction network and source LM 1 x 768 over a padded 10-dimensional
    embedding, external LM 2 x 2048 + bottleneck 256, fusion weights 0.7 / 0.5 / 0.2) on a short, narrow
    problem the oracle finishes in seconds; once at 8 hypotheses (weight-streaming step kernel) and once
    at 128 (tiled step kernel)."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(5, enc_layers=1)
    M = omodels.model_from_float(m)
    G = gmodel.model_from_float(m, DEV)
    for (T, B, W, max_sym) in ((4, 2, 4, 2), (2, 8, 16, 1)):
        e = synth.normal(310 + B, (T, B, m.J), 1.0)
        ref = oracle.decode(M, e, W, max_sym)
        got = gpu_lib.decode(G, dev(e), W, max_sym)
        _compare_beams(got, ref)


@pytest.mark.parametrize("blank_bias", [0.0, 1.5])
def test_decode_benchmark_shape_sampled_utterances(gpu_lib, blank_bias):
    """The decoder in the launch configuration the benchmark times (64 utterances x beam 16 = 1024
    hypotheses, at most 4 labels per frame, full layer widths), on a few frames.  Utterances do not
    interact, so the oracle decodes two sampled ones alone and must find the GPU's beams for them.
    The networks advance only for the hypotheses that took a label (a list built on the device): with
    the plain model nearly all of them do in some rounds and one per utterance in others, with the
    blank's joint bias raised the lists are short and of uneven length."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(4, enc_layers=1)
    m.joint_out.bias = m.joint_out.bias.copy()
    m.joint_out.bias[0] += np.float32(blank_bias)   # blank is token 0
    T, B, W, max_sym = 3, 64, 16, 4
    e = synth.normal(202, (T, B, m.J), 1.0)
    got = gpu_lib.decode(gmodel.model_from_float(m, DEV), dev(e), W, max_sym)
    tok_g, len_g, sc_g = (host(x) for x in got)
    M = omodels.model_from_float(m)
    for b in (5, 41):
        ref = oracle.decode(M, np.ascontiguousarray(e[:, b:b + 1]), W, max_sym)
        _compare_beams((torch.from_numpy(tok_g[b:b + 1]), torch.from_numpy(len_g[b:b + 1]), torch.from_numpy(sc_g[b:b + 1])), ref)


@pytest.mark.parametrize("B,W,max_sym,blank_bias", [(70, 17, 3, 0.0), (64, 16, 4, 2.0), (64, 64, 2, 1.0), (24, 7, 4, 4.0),
                                                    (8, 33, 1, 0.0)])
def test_decode_utterance_alone_equals_batched(gpu_lib, B, W, max_sym, blank_bias):
    """Utterances do not interact (Sec. 2: the search is per utterance), so an utterance decoded alone must give,
    bit for bit, the rows it gives inside a batch.  The two runs go through different kernels (few hypotheses: the
    weight-streaming step kernel or narrow instances of the tiled one; many: full-width tiles, longer lists), so
    this holds only if all of those compute the same step; and one of the sampled utterances is checked against
    the oracle, so that "the same" is also "right"."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(0, weight_std=0.5)
    m.joint_out.bias = m.joint_out.bias.copy()
    m.joint_out.bias[0] += np.float32(blank_bias)   # blank is token 0
    T = 6
    e = synth.normal(230 + B + W, (T, B, m.J), 1.0)
    G = gmodel.model_from_float(m, DEV)
    for flags in (0, gpu_lib.DECODE_EARLY_STOP):
        batched = [host(x) for x in gpu_lib.decode(G, dev(e), W, max_sym, flags=flags)]
        for b in sorted({0, B // 3, B - 1}):
            alone = [host(x) for x in gpu_lib.decode(G, dev(e[:, b:b + 1]), W, max_sym, flags=flags)]
            for x, y in zip(alone, batched):
                assert np.array_equal(x[0], y[b]), (b, flags)
    ref = oracle.decode(omodels.model_from_float(m), np.ascontiguousarray(e[:, :1]), W, max_sym)
    _compare_beams(tuple(torch.from_numpy(x[:1]) for x in batched), ref)


@pytest.mark.parametrize("blank_bias", [0.0, 6.0])
def test_decode_early_stop_gives_the_same_beams(gpu_lib, blank_bias):
    """With the early-stop flag the kernels of a round return at once when no utterance carried a label
    into it (not of a search that runs ahead, as this one does: those that do not are in
    test_gpu_search_round.py).  Same beams as the fixed-round search and as the oracle; the blank-heavy variant (joint bias
    of blank raised) makes most rounds after the first die, the plain one keeps them all alive."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(0, weight_std=0.6)
    m.joint_out.bias = m.joint_out.bias.copy()
    m.joint_out.bias[0] += np.float32(blank_bias)   # blank is token 0
    T, B, W, max_sym = 14, 5, 4, 3
    e = synth.normal(210, (T, B, m.J), 1.0)
    ref = oracle.decode(omodels.model_from_float(m), e, W, max_sym)
    G = gmodel.model_from_float(m, DEV)
    fixed = gpu_lib.decode(G, dev(e), W, max_sym)
    early = gpu_lib.decode(G, dev(e), W, max_sym, flags=gpu_lib.DECODE_EARLY_STOP)
    _compare_beams(fixed, ref)
    for a, b in zip(fixed, early):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,W,u_max,T,lms,std", [(3, 4, 6, 8, True, 0.5), (2, 1, 5, 10, True, 0.6), (4, 16, 8, 6, True, 0.5),
                                                 (2, 3, 0, 8, False, 0.6), (5, 8, 3, 9, False, 0.4), (3, 33, 4, 4, True, 0.5),
                                                 (2, 64, 3, 3, True, 0.5), (16, 64, 3, 4, True, 0.5), (5, 8, 6, 7, True, 0.6)])
def test_alsd_matches_oracle(gpu_lib, B, W, u_max, T, lms, std):
    """Alignment-length synchronous search with recombination (Sec. 2) on the tiny configuration: the finished
    lists (label sequences, lengths, merged scores) must be the oracle's; beams 1 to 64, up to 1024 slots."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(0, weight_std=std)
    if not lms:
        m.lm_src = m.lm_ext = None
    m.rho = 0.1
    e = synth.normal(400 + B + W, (T, B, m.J), 1.0)
    ref = oracle.decode_alsd(omodels.model_from_float(m), e, W, u_max)
    got = gpu_lib.decode_alsd(gmodel.model_from_float(m, DEV), dev(e), W, u_max)
    _compare_beams(got, ref)
    if u_max > 0 and W > 1:
        assert (ref[1] > 0).any()


def test_alsd_recombination_is_exercised_and_matters(gpu_lib):
    """With a small vocabulary the picks of an iteration hold many duplicates of one label sequence: the merged
    scores differ from the scores of the search without merging, and the GPU has the merged ones."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(0, weight_std=0.5)
    T, B, W, u_max = 6, 2, 16, 4
    e = synth.normal(420, (T, B, m.J), 1.0)
    M = omodels.model_from_float(m)
    ref = oracle.decode_alsd(M, e, W, u_max)
    got = gpu_lib.decode_alsd(gmodel.model_from_float(m, DEV), dev(e), W, u_max)
    _compare_beams(got, ref)
    # the best finished hypothesis carries more probability mass than any single alignment of it can
    for b in range(B):
        L = int(ref[1][b, 0])
        y = ref[0][b, 0, :L].tolist()
        # the single best alignment found by the time-synchronous search without merging
        ts = oracle.decode(M, np.ascontiguousarray(e[:, b:b + 1]), W, u_max)
        same = [r for r in range(W) if ts[1][0, r] == L and ts[0][0, r, :L].tolist() == y]
        if same:
            assert ref[2][b, 0] > ts[2][0, same[0]] + 1e-3


def test_alsd_full_width_networks(gpu_lib):
    """The measured layer widths (and the Sec. 2 shapes with the mixed-precision map) under the alignment-length
    synchronous search: 8 hypotheses (weight-streaming step kernel) and 128 (tiled step kernel)."""
    from paper_2206_07882_amd import model as gmodel
    for m in (synth.make_model(4, enc_layers=1), synth.make_model(5, enc_layers=1, mixed=True)):
        M = omodels.model_from_float(m)
        G = gmodel.model_from_float(m, DEV)
        for (T, B, W, u_max) in ((4, 2, 4, 3), (2, 8, 16, 2)):
            e = synth.normal(430 + B, (T, B, m.J), 1.0)
            ref = oracle.decode_alsd(M, e, W, u_max)
            got = gpu_lib.decode_alsd(G, dev(e), W, u_max)
            _compare_beams(got, ref)


@pytest.mark.parametrize("B,W,u_max", [(64, 16, 6), (70, 17, 4), (8, 33, 5)])
def test_alsd_utterance_alone_equals_batched(gpu_lib, B, W, u_max):
    """The same independence for the alignment-length synchronous search: alone (few hypotheses, other kernels)
    and inside a batch an utterance must give the same bits."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(0, weight_std=0.5)
    T = 5
    e = synth.normal(260 + B + W, (T, B, m.J), 1.0)
    G = gmodel.model_from_float(m, DEV)
    batched = [host(x) for x in gpu_lib.decode_alsd(G, dev(e), W, u_max)]
    for b in sorted({0, B // 3, B - 1}):
        alone = [host(x) for x in gpu_lib.decode_alsd(G, dev(e[:, b:b + 1]), W, u_max)]
        for x, y in zip(alone, batched):
            assert np.array_equal(x[0], y[b]), b


@pytest.mark.parametrize("std", [0.1, 0.6])
def test_alsd_config0_end_to_end_matches_golden(gpu_lib, std):
    """Encoder + alignment-length synchronous search on the tiny configuration against the oracle and against the
    stored finished lists (tests/golden/cfg0_alsd.txt, written by the oracle alone)."""
    from paper_2206_07882_amd import model as gmodel
    from tests.golden import make_golden as mg
    m = synth.make_model(0, weight_std=std)
    feats = synth.features(0, mg.T, mg.B, m.feat_dim)
    layers, proj = omodels.encoder_from_float(m)
    _, e_r = omodels.encoder_forward(layers, proj, feats, m.alpha_x)
    ref = oracle.decode_alsd(omodels.model_from_float(m), e_r, mg.ALSD_W, mg.ALSD_UMAX)
    _, e_g = gmodel.Encoder(m, DEV).forward(dev(feats))
    got = gpu_lib.decode_alsd(gmodel.model_from_float(m, DEV), e_g, mg.ALSD_W, mg.ALSD_UMAX)
    _compare_beams(got, ref)
    tok_g, len_g, _ = (host(x) for x in got)
    path = os.path.join(os.path.dirname(__file__), "golden", "cfg0_alsd.txt")
    n = 0
    for l in open(path).read().splitlines():
        if not l.startswith(f"{std} "):
            continue
        head, labs = l.split("|")
        _, b, w, _ = head.split()
        assert tok_g[int(b), int(w), :len_g[int(b), int(w)]].tolist() == [int(t) for t in labs.split()]
        n += 1
    assert n >= 6


def test_config4_slice_encoder_through_decoder_at_full_widths(gpu_lib):
    """The end-to-end configuration at its own parity size: 2 utterances x 50 frames through the whole network at
    full depth and width (240 features -> 6 bidirectional layers of 640 cells -> projection -> time-synchronous
    search at beam 16 with at most 4 labels per frame over the prediction network 768 and both LMs 2 x 1024),
    free-running on both sides.  What may differ, and when, is decided by the oracle's margins and by nothing
    chosen here.  Encoder: ~4 * 10^5 hidden-state decisions per utterance; an utterance none of whose decisions
    lies within the bound of a rounding tie must come out with exactly the oracle's codes; one that has such a
    decision may lose it either way, and a flipped code then travels through the layers above, so for it the
    free-running codes say nothing, and every layer is checked step by step on the GPU's own inputs instead (for
    every utterance).  The decoder then runs on the GPU's own encoder output on both sides, and every utterance
    whose decode margins are clear of the bounds must give the oracle's beams."""
    from paper_2206_07882_amd import model as gmodel
    from tests.test_gpu_sweep import Q_BOUND, S_STEP, _utterance_equal
    from tests.test_gpu_parity import assert_codes_close
    q = gpu_lib
    m = synth.make_model(4)
    T, B, W, max_sym = 50, 2, 16, 4
    feats = synth.features(4, T, B, m.feat_dim)
    layers, proj = omodels.encoder_from_float(m)
    enc_margin = np.full(B, np.inf)
    x_r, e_r = omodels.encoder_forward(layers, proj, feats, m.alpha_x, utt_margin=enc_margin)
    enc = gmodel.Encoder(m, DEV)
    x_g, e_g = enc.forward(dev(feats))
    enc.check()
    xg = host(x_g)
    agree = (xg == x_r).mean(axis=(0, 2))
    for b in range(B):
        if enc_margin[b] >= Q_BOUND:          # no decision of this utterance near a tie: the codes are the oracle's
            assert np.array_equal(xg[:, b], x_r[:, b]), (b, enc_margin[b], agree[b])
    # layer by layer, step by step, on the GPU's own inputs and previous codes
    ws = enc.workspace(T, B, DEV)
    x = q.quantize_act_rows(dev(feats), enc.inv_s_x)
    assert np.array_equal(host(x)[:, :, :m.feat_dim], oracle.quant_sym(feats, enc.inv_s_x, 4))
    for li, (dirs_g, dirs_o) in enumerate(zip(enc.layers, layers)):
        H = dirs_g[0].H
        out = torch.empty((T, B, 2 * H), dtype=torch.int8, device=DEV)
        q.bilstm_layer(dirs_g[0], dirs_g[1], x, h_out=out, workspace=ws)
        og, xin = host(out), host(x)[:, :, :dirs_o[0].I]
        for d, (L, order) in enumerate(((dirs_o[0], range(T)), (dirs_o[1], range(T - 1, -1, -1)))):
            hg = og[:, :, d * H:(d + 1) * H]
            hp = np.zeros((B, H), np.int8); cp = np.zeros((B, H), np.float32)
            for t in order:
                hr, cr, dbg = oracle.lstm_step(L, xin[t], hp, cp, debug=True)
                assert_codes_close(hg[t], hr, dbg["h_real"] * 7.0, f"layer {li} dir {d} t={t}", min_agree=0.999)
                hp, cp = hg[t], cr            # GPU codes forward; cell state from the oracle's step on those codes
        x = out
    assert np.array_equal(host(x), xg)
    # the projection of the GPU's own codes
    e_own = oracle.linear(proj, xg.reshape(T * B, -1)).reshape(T, B, -1)
    assert np.abs(host(e_g) - e_own).max() <= 1e-5 * np.abs(e_own).max() + 1e-6
    # decoder, free-running from the GPU's encoder output on both sides
    eg = host(e_g)
    ref = oracle.decode(omodels.model_from_float(m), eg, W, max_sym, margins=True)
    got = tuple(host(t) for t in gpu_lib.decode(gmodel.model_from_float(m, DEV), e_g, W, max_sym))
    qm, sm = ref[3], ref[4]
    s_bound = S_STEP * T * (max_sym + 1)
    n_equal = 0
    for b in range(B):
        equal = _utterance_equal(got, ref[:3], b, s_bound + 1e-5)
        n_equal += int(equal)
        clear = qm[b] >= Q_BOUND and sm[b] >= s_bound
        assert equal or not clear, (b, qm[b], sm[b])
    print("config-4 slice: free-running encoder agreement", agree, "encoder margins", enc_margin, "decode margins", qm, sm,
          "utterances with the oracle's beams:", n_equal, "of", B)
    # whatever the margins say, a flipped code moves scores by fractions of a unit: the best hypothesis' score
    # must be close for every utterance
    assert np.all(np.abs(got[2][:, 0] - ref[2][:, 0]) < 0.5)


@pytest.mark.parametrize("B,W,u_max,T,std", [(5, 16, 6, 10, 0.5), (3, 4, 8, 12, 0.6), (16, 64, 3, 4, 0.5), (4, 8, 5, 9, 0.4)])
def test_alsd_reuse_of_cached_hypotheses(gpu_lib, B, W, u_max, T, std):
    """Sec. 4.1's reuse of cached hypotheses in the alignment-length synchronous search: a label pick whose sequence
    a live hypothesis of the beam already holds takes over its network states.  Same finished lists as without the
    flag and as the oracle; the counters (label picks that kept their slot, reuses) are the oracle's own for the
    same rule (its cache mode 1)."""
    from paper_2206_07882_amd import model as gmodel
    m = synth.make_model(0, weight_std=std)
    m.rho = 0.1
    e = synth.normal(460 + B + W, (T, B, m.J), 1.0)
    from tests.test_gpu_sweep import Q_BOUND, S_STEP, _utterance_equal
    M = omodels.model_from_float(m)
    ref = oracle.decode_alsd_cached(M, e, W, u_max, 1)
    marg = oracle.decode_alsd(M, e, W, u_max, margins=True)
    G = gmodel.model_from_float(m, DEV)
    plain = gpu_lib.decode_alsd(G, dev(e), W, u_max)
    stats = torch.zeros(2, dtype=torch.int32, device=DEV)
    got = gpu_lib.decode_alsd(G, dev(e), W, u_max, flags=gpu_lib.ALSD_REUSE, stats=stats)
    for a, b in zip(plain, got):
        assert torch.equal(a, b)              # the flag changes the work, not one bit of the result
    # against the oracle under the rule of the free-running sweep: an utterance whose margins are clear must agree
    got_h = tuple(host(x) for x in got)
    s_bound = S_STEP * (T + u_max)
    all_equal = True
    for b in range(B):
        equal = _utterance_equal(got_h, ref[:3], b, s_bound + 1e-5)
        all_equal = all_equal and equal
        assert equal or not (marg[3][b] >= Q_BOUND and marg[4][b] >= s_bound), (b, marg[3][b], marg[4][b])
    n_req, n_hit = (int(v) for v in stats.cpu())
    assert n_hit > 0 and abs(n_req - int(ref[3].sum())) <= 0.05 * n_req
    if all_equal:     # same search, same rule: the same counts
        assert n_req == int(ref[3].sum()) and n_hit == int((ref[3] - ref[4]).sum()), (n_req, n_hit, ref[3].sum(), ref[4].sum())
    # without the flag the counters still count the picks, and no reuse
    stats.zero_()
    gpu_lib.decode_alsd(G, dev(e), W, u_max, stats=stats)
    assert stats.cpu().tolist() == [n_req, 0]
