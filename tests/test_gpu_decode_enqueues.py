"""A search is enqueued and its call returns: the host waits for nothing that the device does."""
import time

import pytest
import torch

from paper_2206_07882_amd import synth

from .test_gpu_decode import dev
from .test_gpu_search_round import _model

pytestmark = pytest.mark.gpu


def test_a_search_on_a_busy_stream_is_enqueued_at_once(gpu_lib):
    """A search that runs ahead (joint of 256 columns) has T * (max_sym + 1/20) + 1 iterations to enqueue, one with a launch to a
    round (272 columns) T * (max_sym + 1), of as many launches each: behind work that keeps the stream busy the first one must
    not take longer to enqueue (a fifth is for noise; best of five).  Both return while the stream is busy."""
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    T, W, max_sym = 40, 16, 4   # (the runtime itself holds a call back at about a thousand launches ahead)
    a = torch.zeros((8192, 8192), dtype=torch.bfloat16, device="cuda:0")
    b = torch.empty_like(a)
    calls = []
    for J in (256, 272):
        G = gmodel.model_from_float(_model(J, 46, False), "cuda:0")
        e = dev(synth.normal(1300, (T, 1, J), 1.0))
        ws = torch.empty(q.decode_workspace(G, T, 1, W, max_sym), dtype=torch.uint8, device="cuda:0")
        calls.append((lambda G=G, e=e, ws=ws: q.decode(G, e, W, max_sym, workspace=ws)))
    want = [c() for c in calls]
    torch.cuda.synchronize()
    best, busy, done = [1e9, 1e9], [False, False], torch.cuda.Event()
    for _ in range(5):
        for i, call in enumerate(calls):
            for _ in range(60):   # some 40 ms
                torch.mm(a, a, out=b)
            done.record()
            t0 = time.perf_counter()
            got = call()
            best[i] = min(best[i], time.perf_counter() - t0)
            busy[i] = busy[i] or not done.query()
            torch.cuda.synchronize()
            assert all(torch.equal(g, w) for g, w in zip(got, want[i]))
    assert all(busy)   # (the calls came back in front of what is ahead of them)
    assert best[0] < 1.2 * best[1], best
