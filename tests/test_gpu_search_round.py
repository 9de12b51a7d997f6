"""The decoding round's kernel at the edges of what it splits: joint widths that end inside a wave's 64 columns or need
several blocks per wave, output layers that end inside a 128-column chunk, vocabularies at the edges of the 16-row tiles,
beams on both sides of a column tile, and mixed widths."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from oracle import models as omodels
from paper_2206_07882_amd import synth

from .test_gpu_decode import _compare_beams, dev

pytestmark = pytest.mark.gpu


def _linear(seed, rows, cols):
    return synth.LinearF(synth.normal(seed, (rows, cols), 0.6), synth.normal(seed + 1, (rows,), 0.3))


@pytest.mark.parametrize("J,V,B,W,mixed", [(16, 2, 2, 1, False), (48, 16, 2, 4, False), (80, 17, 3, 15, False), (272, 48, 2, 16, True),
                                           (320, 49, 2, 17, False), (528, 64, 1, 16, False), (64, 33, 2, 33, True)])
def test_round_at_the_edges_of_its_tiles(gpu_lib, J, V, B, W, mixed):
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    m = _model(J, V, mixed)
    T = 5
    e = synth.normal(930 + J, (T, B, J), 1.0)
    G, M = gmodel.model_from_float(m, "cuda:0"), omodels.model_from_float(m)
    _compare_beams(q.decode(G, dev(e), W, 2, max_len=2 * T), oracle.decode(M, e, W, 2, max_len=2 * T))
    _compare_beams(q.decode_alsd(G, dev(e), W, 4), oracle.decode_alsd(M, e, W, 4))


def _model(J, V, mixed, mids=()):
    """mids: (network, rows of its bottleneck)."""
    m = synth.make_model(0, weight_std=0.5)
    if mixed:
        m.mixed_precision = True
    m.J, m.V, m.rho = J, V, 0.1
    h = m.pred.layers[-1].w_hh.shape[1]
    m.pred.out = _linear(900, J, h)
    m.joint_out = _linear(902, V, J)
    for i, net in enumerate((m.pred, m.lm_src, m.lm_ext)):
        net.embed = synth.normal(910 + i, (V, net.embed.shape[1]), 0.5)
        if net is not m.pred:
            net.out = _linear(920 + 2 * i, V, net.layers[-1].w_hh.shape[1])
    for i, rows in mids:
        net = (m.pred, m.lm_src, m.lm_ext)[i]
        net.mid, net.alpha_mid = _linear(940 + i, rows, net.layers[-1].w_hh.shape[1]), 4.0
        net.out = _linear(950 + i, J if i == 0 else V, rows)
    return m


@pytest.mark.parametrize("J,V,B,W,mixed,mids", [(256, 46, 1, 16, False, ()), (80, 17, 9, 5, False, ()), (272, 48, 2, 16, True, ()),
                                                (64, 33, 3, 1, False, ()), (256, 46, 1, 16, False, ((2, 256),)),
                                                (80, 17, 3, 7, True, ((1, 80), (2, 144))), (64, 46, 2, 16, False, ((1, 16),)),
                                                (64, 46, 2, 4, False, ((0, 48), (2, 64))), (64, 20, 2, 8, False, ((2, 272),))])
def test_a_workgroup_left_alone_returns_the_same_beams(gpu_lib, J, V, B, W, mixed, mids):
    """The workgroups of a beam exchange whole numbers and the very values one of them would form: the bits are the same
    whether the others come or not.  A launch of more than about 100 utterances has one workgroup for each: the same beams
    (other step kernels run there, so the scores may differ in the last bits)."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    m = _model(J, V, mixed, mids)
    G, M = gmodel.model_from_float(m, "cuda:0"), omodels.model_from_float(m)
    T, many = 6, 264 // B * B
    e = dev(synth.normal(930 + J, (T, B, J), 1.0))
    for alsd, limit, fn, size in ((0, 2, q.decode, q.decode_workspace), (1, 4, q.decode_alsd, q.decode_alsd_workspace)):
        want = fn(G, e, W, limit, max_len=2 * T)
        ws = torch.empty(size(G, T, B, W, limit), dtype=torch.uint8, device="cuda:0")
        got = tuple(torch.empty_like(t) for t in want)
        q._check(q.load().qrnnt_diag_decode(C.byref(G.c()), C.c_void_p(e.data_ptr()), T, B, W, alsd, limit, 2 * T,
                                            *(C.c_void_p(t.data_ptr()) for t in got), C.c_void_p(ws.data_ptr()),
                                            C.c_size_t(ws.numel()), q._stream()), "qrnnt_diag_decode")
        batch = fn(G, e.repeat(1, many // B, 1).contiguous(), W, limit, max_len=2 * T)
        for w, g in zip(want, got):
            assert torch.equal(w, g)
        if mids:   # in the round, or (272 rows, or one in front of the joint) in a launch of their own
            ref = (oracle.decode_alsd if alsd else oracle.decode)(M, e.cpu().numpy(), W, limit, max_len=2 * T)
            _compare_beams(want, ref)
        _compare_beams(batch, [np.tile(w.cpu().numpy(), (many // B,) + (1,) * (w.dim() - 1)) for w in want])


def test_a_search_over_more_utterances_than_a_grid_has_layers(gpu_lib):
    """A joint of 64 columns and no language model: one workgroup to an utterance.  A grid's z extent ends at 65535, and
    8 x 65535 utterances are not the most that a search takes."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    m = _model(64, 17, False)
    G, M = gmodel.model_from_float(m, "cuda:0", use_src=False, use_ext=False), omodels.model_from_float(m, use_src=False, use_ext=False)
    T, few, many = 2, 8, 8 * 65535 + 16
    e = synth.normal(960, (T, few, 64), 1.0)
    E = dev(e).repeat(1, many // few, 1).contiguous()
    for got, ref in ((q.decode(G, E, 1, 1, max_len=T), oracle.decode(M, e, 1, 1, max_len=T)),
                     (q.decode_alsd(G, E, 1, 1), oracle.decode_alsd(M, e, 1, 1))):
        _compare_beams([t[:few] for t in got], ref)
        for t in got:
            assert torch.equal(t.view(many // few, few, *t.shape[1:]), t[:few].expand(many // few, *t[:few].shape))


def _diag_shared(q, G, e, W, alsd, limit, max_len, come, n_xcd=0):
    T, B, _ = e.shape
    size = q.decode_alsd_workspace if alsd else q.decode_workspace
    ws = torch.empty(size(G, T, B, W, limit), dtype=torch.uint8, device="cuda:0")
    late = torch.full((B,), -1, dtype=torch.int32, device="cuda:0")
    out = [torch.empty(s, dtype=d, device="cuda:0") for s, d in (((B, W, max_len), torch.int32), ((B, W), torch.int32), ((B, W), torch.float32))]
    q._check(q.load().qrnnt_diag_decode_shared(C.byref(G.c()), C.c_void_p(e.data_ptr()), T, B, W, alsd, limit, max_len, come, n_xcd,
                                               C.c_void_p(late.data_ptr()), *(C.c_void_p(t.data_ptr()) for t in out),
                                               C.c_void_p(ws.data_ptr()), C.c_size_t(ws.numel()), q._stream()), "qrnnt_diag_decode_shared")
    return out, late.cpu().numpy()


@pytest.mark.parametrize("J,V,B,W,mixed,mids", [(256, 46, 1, 16, False, ()), (272, 48, 2, 16, True, ()), (64, 33, 3, 1, False, ()),
                                                (256, 46, 9, 16, False, ((2, 256),)), (80, 17, 3, 7, True, ((1, 80), (2, 144)))])
@pytest.mark.parametrize("alsd", [0, 1])
def test_some_of_a_beams_workgroups_come(gpu_lib, J, V, B, W, mixed, mids, alsd):
    """Whichever of them stay away (shares of the joint, the language models', the bottlenecks' that those wait for), or do
    their work on other XCDs: the same bits, and the first one has to step in.  When all come it hardly ever has to."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    G = gmodel.model_from_float(_model(J, V, mixed, mids), "cuda:0")
    T, limit = 24, 6 if alsd else 2
    e = dev(synth.normal(970 + J, (T, B, J), 1.0))
    parts = min((J + 63) // 64, 4)
    total = parts + 1 + sum((rows + 63) // 64 for _, rows in mids)
    want = (q.decode_alsd if alsd else q.decode)(G, e, W, limit, max_len=2 * T)
    for come in range(1, total + 1):
        got, late = _diag_shared(q, G, e, W, alsd, limit, 2 * T, come)
        for w, g in zip(want, got):
            assert torch.equal(w, g), come
        if come == total:
            assert late.max() <= T // 4, late
        else:   # every round that has a use for them: all but a frame's last one, and that too for the joint
            assert late.min() >= (T - 1 if alsd else T * (limit + (come < parts))), (come, late)
    got, _ = _diag_shared(q, G, e, W, alsd, limit, 2 * T, 0, n_xcd=7)
    for w, g in zip(want, got):
        assert torch.equal(w, g)


def test_searches_on_several_streams(gpu_lib):
    """Three searches of 48 utterances, each alone worth more than half of the device, and an encoder layer beside them: a
    beam's workgroups come late or one by one, and the results are those of a search on its own."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    T, B, W = 20, 48, 16
    m = _model(256, 46, False, ((2, 256),))
    G = gmodel.model_from_float(m, "cuda:0")
    L = gmodel.lstm_from_float(synth.make_model(4, enc_layers=1).enc_layers[0][0], gmodel.S_H, "cuda:0")
    x = dev(synth.codes(981, (200, 32, L.I)))
    es = [dev(synth.normal(982 + i, (T, B, 256), 1.0)) for i in range(3)]
    want = [fn(G, e, W, 4, max_len=2 * T) for e in es for fn in (q.decode, q.decode_alsd)]
    want_h = q.lstm_layer(L, x)["h_out"]
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()
    got = []
    for e, s in zip(es, streams):
        with torch.cuda.stream(s):
            got += [fn(G, e, W, 4, max_len=2 * T) for fn in (q.decode, q.decode_alsd)]
    with torch.cuda.stream(streams[3]):
        hs = [q.lstm_layer(L, x)["h_out"] for _ in range(4)]
    torch.cuda.synchronize()
    for a, b in zip(want, got):
        for w, g in zip(a, b):
            assert torch.equal(w, g)
    assert all(torch.equal(h, want_h) for h in hs)


@pytest.mark.parametrize("J,B,W", [(272, 2, 16), (272, 3, 1), (32, 5, 20), (32, 2, 40), (256, 105, 2), (256, 110, 2), (256, 110, 1)])
@pytest.mark.parametrize("blank_bias", [0.0, 6.0])
def test_early_stop_where_a_round_is_a_launch(gpu_lib, J, B, W, blank_bias):
    """Searches that do not run ahead (a wide joint, a wide beam, many utterances: one workgroup each, in 105 but for a frame's
    last round): kernels that return because no utterance carried a label into their round leave the same beams.  With the blank
    made likely most rounds after a frame's first are such."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    T, max_sym, few = 6, 3, 5
    m = _model(J, 20, False)
    m.joint_out.bias = m.joint_out.bias.copy()
    m.joint_out.bias[0] += np.float32(blank_bias)   # blank is token 0
    e = synth.normal(990 + J, (T, few, J), 1.0)
    G, M = gmodel.model_from_float(m, "cuda:0"), omodels.model_from_float(m)
    E = dev(e)[:, torch.arange(B, device="cuda:0") % few].contiguous()
    n = min(B, few)
    plain = q.decode(G, E, W, max_sym, max_len=T * max_sym)
    early = q.decode(G, E, W, max_sym, max_len=T * max_sym, flags=q.DECODE_EARLY_STOP)
    _compare_beams([t[:n] for t in early], [r[:n] for r in oracle.decode(M, e, W, max_sym, max_len=T * max_sym)])
    for a, b in zip(plain, early):
        assert torch.equal(a, b)
