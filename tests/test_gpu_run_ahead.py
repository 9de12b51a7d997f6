"""Beams of up to 16 and joints of up to 256 columns: an utterance runs ahead inside a launch.  The edges: one round to a frame,
no label at all, every frame the same, joints that end inside a 64-column share, bottlenecks, beams, joints and numbers of
utterances on both sides of the limits, workgroups that stay away; and the launches of a graph, which are all that can be needed."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from oracle import models as omodels
from paper_2206_07882_amd import synth

from .test_gpu_decode import _compare_beams, dev
from .test_gpu_search_round import _model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J,V,B,W,max_sym,T,rho,mids", [(256, 46, 1, 16, 4, 30, 0.1, ()), (80, 17, 3, 5, 1, 40, 0.4, ()),
                                                        (16, 2, 2, 1, 4, 30, 0.4, ()), (240, 64, 2, 16, 0, 12, 0.1, ()),
                                                        (256, 33, 9, 3, 2, 20, 8.0, ()), (64, 20, 2, 8, 3, 20, 0.4, ((2, 80),)),
                                                        (256, 46, 2, 17, 2, 10, 0.4, ()), (272, 46, 2, 16, 2, 10, 0.4, ()),
                                                        (128, 46, 130, 2, 2, 6, 0.4, ())])
def test_running_ahead(gpu_lib, J, V, B, W, max_sym, T, rho, mids):
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    m = _model(J, V, False, mids)
    m.rho = rho
    e = (synth.normal(1000 + J, (1, B, J), 1.0) + 0.1 * synth.normal(1001 + J, (T, B, J), 1.0)).astype(np.float32)
    G, M = gmodel.model_from_float(m, "cuda:0"), omodels.model_from_float(m)
    max_len = max(1, T * max_sym)
    got = q.decode(G, dev(e), W, max_sym, max_len=max_len)
    _compare_beams(got, oracle.decode(M, e, W, max_sym, max_len=max_len))
    early = q.decode(G, dev(e), W, max_sym, max_len=max_len, flags=q.DECODE_EARLY_STOP)   # (of no effect where it runs ahead)
    for a, b in zip(got, early):
        assert torch.equal(a, b)


# 6 * utterances * workgroups <= 5 * 512 (three workgroups: two shares of the joint, language models); one workgroup: 512 utterances
@pytest.mark.parametrize("J,B,W,lms", [(128, 142, 3, True), (128, 143, 3, True), (64, 1, 16, False), (64, 512, 2, False), (64, 513, 2, False),
                                       (16, 1, 5, False), (16, 512, 1, False), (16, 513, 1, False)])
def test_as_many_utterances_as_run_ahead(gpu_lib, J, B, W, lms):
    """Five utterances, again and again: each is the oracle's, and the same wherever it stands."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    T, max_sym, few = 8, 2, 5
    m = _model(J, 17, False)
    m.rho = 0.4
    e = (synth.normal(1030 + J, (1, few, J), 1.0) + 0.1 * synth.normal(1031 + J, (T, few, J), 1.0)).astype(np.float32)
    use = dict(use_src=lms, use_ext=lms)
    G, M = gmodel.model_from_float(m, "cuda:0", **use), omodels.model_from_float(m, **use)
    at = torch.arange(B, device="cuda:0") % few
    got = q.decode(G, dev(e)[:, at].contiguous(), W, max_sym, max_len=T * max_sym)
    n = min(B, few)
    _compare_beams([t[:n] for t in got], [r[:n] for r in oracle.decode(M, e, W, max_sym, max_len=T * max_sym)])
    for t in got:
        assert torch.equal(t, t[:n][at])


@pytest.mark.parametrize("W", [1, 2, 3, 4, 8, 16])
def test_equal_candidates(gpu_lib, W):
    """Pairs of tokens with the same row of the joint's output layer and no language model: their candidates are equal, and the
    last place of the beam goes to the first of a pair."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    m = _model(80, 17, False)
    for a in (m.joint_out.w, m.joint_out.bias):
        a[2::2] = a[1::2]
    T, max_sym = 10, 3
    e = synth.normal(1200, (T, 3, 80), 1.0)
    G, M = gmodel.model_from_float(m, "cuda:0", use_src=False, use_ext=False), omodels.model_from_float(m, use_src=False, use_ext=False)
    _compare_beams(q.decode(G, dev(e), W, max_sym), oracle.decode(M, e, W, max_sym))


@pytest.mark.parametrize("B,W", [(1, 16), (7, 4)])
def test_a_graph_of_a_search(gpu_lib, B, W):
    """A graph holds the launches of the longest search, and its replays read what is in the inputs then."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    T, max_sym = 12, 3
    G = gmodel.model_from_float(_model(80, 17, False), "cuda:0")
    es = [dev(synth.normal(1100 + i, (T, B, 80), 1.0)) for i in range(3)]
    want = [q.decode(G, e, W, max_sym) for e in es]
    e = es[0].clone()
    ws = torch.empty(q.decode_workspace(G, T, B, W, max_sym), dtype=torch.uint8, device="cuda:0")
    q.decode(G, e, W, max_sym, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = q.decode(G, e, W, max_sym, workspace=ws)
    for i in (1, 0, 2, 1):
        e.copy_(es[i])
        graph.replay()
        torch.cuda.synchronize()
        for w, g in zip(want[i], out):
            assert torch.equal(w, g)
        assert all(torch.equal(a, b) for a, b in zip(q.decode(G, es[i], W, max_sym), want[i]))


@pytest.mark.parametrize("J,V,B,W,mids", [(256, 46, 1, 16, ()), (80, 17, 9, 5, ()), (64, 33, 3, 1, ()), (256, 46, 5, 16, ((2, 256),)),
                                          (80, 17, 3, 7, ((1, 80), (2, 144)))])
def test_running_ahead_alone(gpu_lib, J, V, B, W, mids):
    """Whichever of an utterance's workgroups stay away: the first one does their work and runs ahead with its own results.  The same
    bits as when all come, over frames that change slowly, so that a launch has several rounds and frames."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    T, max_sym = 30, 3
    m = _model(J, V, False, mids)
    m.rho = 0.4
    G = gmodel.model_from_float(m, "cuda:0")
    e = dev((synth.normal(1060 + J, (1, B, J), 1.0) + 0.1 * synth.normal(1061 + J, (T, B, J), 1.0)).astype(np.float32))
    max_len = T * max_sym
    want = q.decode(G, e, W, max_sym, max_len=max_len)
    assert int(want[1].max()) > 2   # there were labels
    ws = torch.empty(q.decode_workspace(G, T, B, W, max_sym), dtype=torch.uint8, device="cuda:0")
    total = min((J + 63) // 64, 4) + 1 + sum((rows + 63) // 64 for _, rows in mids)
    for come in range(1, total + 1):
        got = [torch.empty_like(t) for t in want]
        q._check(q.load().qrnnt_diag_decode_shared(C.byref(G.c()), C.c_void_p(e.data_ptr()), T, B, W, 0, max_sym, max_len, come, 0, None,
                                                   *(C.c_void_p(t.data_ptr()) for t in got), C.c_void_p(ws.data_ptr()),
                                                   C.c_size_t(ws.numel()), q._stream()), "qrnnt_diag_decode_shared")
        for w, g in zip(want, got):
            assert torch.equal(w, g), come
