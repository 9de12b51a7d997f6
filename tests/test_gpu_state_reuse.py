"""Label picks that lead to a sequence whose states a row of the pool still holds name that row.  Frames that change slowly
bring the same proposals back: most picks find their states, in rows of the beam, in free ones, and in a row that another
pick of the same round is about to fill.  The widest beams look for free rows beyond the first 64 of their list."""
import numpy as np
import pytest

import oracle
from oracle import models as omodels
from paper_2206_07882_amd import synth

from .test_gpu_decode import _compare_beams, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,W,max_sym,T", [(1, 16, 4, 40), (3, 16, 4, 24), (2, 5, 1, 60), (2, 1, 4, 60), (2, 20, 4, 20),
                                           (1, 16, 16, 8), (2, 40, 4, 12), (1, 64, 16, 4), (33, 4, 2, 20)])
def test_slow_frames(gpu_lib, B, W, max_sym, T):
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    m = synth.make_model(0, weight_std=0.5)
    m.rho = 0.4
    e = (synth.normal(500 + W, (1, B, m.J), 1.0) + 0.1 * synth.normal(600 + W, (T, B, m.J), 1.0)).astype(np.float32)
    G, M = gmodel.model_from_float(m, "cuda:0"), omodels.model_from_float(m)
    ref = oracle.decode(M, e, W, max_sym, max_len=T * max_sym)
    got = q.decode(G, dev(e), W, max_sym, max_len=T * max_sym)
    _compare_beams(got, ref)
    assert ref[1].max() > 2   # there were labels
    early = q.decode(G, dev(e), W, max_sym, max_len=T * max_sym, flags=q.DECODE_EARLY_STOP)   # (another route at beams of more than 16)
    for a, b in zip(got, early):
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())


@pytest.mark.parametrize("B,W,u_max,T", [(1, 16, 30, 40), (3, 16, 20, 24), (2, 5, 30, 60), (2, 1, 30, 60), (2, 20, 20, 20), (1, 64, 10, 12), (17, 1, 12, 20)])
def test_slow_frames_alignment_length(gpu_lib, B, W, u_max, T):
    import torch
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    m = synth.make_model(0, weight_std=0.5)
    m.rho = 0.4
    e = (synth.normal(700 + W, (1, B, m.J), 1.0) + 0.1 * synth.normal(800 + W, (T, B, m.J), 1.0)).astype(np.float32)
    G, M = gmodel.model_from_float(m, "cuda:0"), omodels.model_from_float(m)
    ref = oracle.decode_alsd(M, e, W, u_max)
    got = q.decode_alsd(G, dev(e), W, u_max)
    _compare_beams(got, ref)
    assert ref[1].max() > 2   # there were labels
    stats = torch.zeros(2, dtype=torch.int32, device="cuda:0")
    for more in (dict(flags=q.ALSD_REUSE), dict(flags=q.ALSD_REUSE, stats=stats)):   # (counting looks for them in another way)
        again = q.decode_alsd(G, dev(e), W, u_max, **more)
        for a, b in zip(got, again):
            assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())


@pytest.mark.parametrize("B", [20, 220])
def test_beams_of_one(gpu_lib, B):
    """Nothing is looked for at beam 1 where a round is a launch: one workgroup to an utterance (220) and several (20; the
    time-synchronous search with a joint that does not run ahead).  The utterances are four, again and again, and short: a value
    whose fp32 error of about 1e-6 of a step takes it over a rounding tie becomes another code than the oracle's and moves the
    scores by 0.1 (ten utterances of 16 frames, 4 rounds and 500 codes: 0.3 such values expected, and one seen; here 0.05)."""
    import torch
    from paper_2206_07882_amd import model as gmodel
    from .test_gpu_search_round import _model
    q = gpu_lib
    T, max_sym, u_max = 6, 3, 6
    m = _model(272 if B == 20 else 256, 46, False)
    m.rho = 0.4
    e = (synth.normal(710, (1, 4, m.J), 1.0) + 0.1 * synth.normal(711, (T, 4, m.J), 1.0)).astype(np.float32)
    G, M = gmodel.model_from_float(m, "cuda:0"), omodels.model_from_float(m)
    E = dev(e).repeat(1, B // 4, 1).contiguous()
    for got, ref in ((q.decode(G, E, 1, max_sym, max_len=T * max_sym), oracle.decode(M, e, 1, max_sym, max_len=T * max_sym)),
                     (q.decode(G, E, 1, max_sym, max_len=T * max_sym, flags=q.DECODE_EARLY_STOP), oracle.decode(M, e, 1, max_sym, max_len=T * max_sym)),
                     (q.decode_alsd(G, E, 1, u_max), oracle.decode_alsd(M, e, 1, u_max)),
                     (q.decode_alsd(G, E, 1, u_max, flags=q.ALSD_REUSE), oracle.decode_alsd(M, e, 1, u_max))):
        _compare_beams([t[:4] for t in got], ref)
        assert ref[1].max() > 2   # there were labels
        for t in got:
            assert torch.equal(t.view(B // 4, 4, *t.shape[1:]), t[:4].expand(B // 4, *t[:4].shape))
