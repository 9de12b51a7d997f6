"""The step kernel that splits K over a workgroup's waves, at the edges of its tiles: hypothesis counts around its column
blocks and the counts that choose it, cell counts around its row groups, inputs that end inside a chunk or leave waves
without one, gathered and inactive hypotheses, lists, and a looked-up input part with and without its fp32 table; short
lists in the tiled kernel's launch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2206_07882_amd import synth
from tests.test_gpu_parity import _lstm_pair, assert_codes_close, assert_rel, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,I,H,looked_up,listed", [(33, 16, 16, False, None), (64, 48, 80, False, None), (65, 272, 48, False, None),
                                                    (128, 1040, 144, False, None), (96, 2080, 32, False, None),
                                                    (33, 32, 1040, "sums", None), (64, 64, 272, "table", None),
                                                    (256, 64, 80, False, 1), (200, 144, 64, False, 32), (129, 64, 64, False, 129),
                                                    (128, 64, 96, "table", 77), (100, 64, 1040, "sums", 33), (70, 32, 48, "table", 0),
                                                    (129, 64, 64, "table", 100), (208, 80, 1024, "table", 150),
                                                    (300, 144, 80, False, 192), (300, 144, 80, False, 193), (600, 64, 48, False, 128),
                                                    (600, 64, 48, False, 129), (257, 1040, 16, False, 1), (250, 3200, 32, False, 222),
                                                    (257, 3200, 32, False, 33), (200, 64, 80, "table", 64), (130, 64, 1040, "sums", 65),
                                                    (1030, 80, 272, "table", 63), (300, 64, 1376, False, 160), (300, 64, 1376, False, 161),
                                                    (144, 64, 1376, False, 144), (17, 48, 80, False, None), (20, 272, 48, "sums", None),
                                                    (31, 32, 1040, "table", None), (32, 2080, 32, False, None), (32, 144, 272, False, 17),
                                                    (32, 64, 80, "table", 31), (20, 80, 1040, "sums", 16)])
def test_split_step(gpu_lib, N, I, H, looked_up, listed):
    q = gpu_lib
    s_x = float(np.float32(4) / np.float32(7))
    L, G = _lstm_pair(q, 2300 + N + I + H, I, H, s_x)
    rows = 50
    xt = synth.codes(2301, (rows, I), -8, 7)
    x_row = (np.arange(N, dtype=np.int32) * 7) % rows
    parent = ((np.arange(N, dtype=np.int64) * 5 + 3) % N).astype(np.int32)
    hp, cp = synth.codes(2302, (N, H), -7, 7), synth.normal(2303, (N, H), 0.6)
    active = None if listed is not None else (np.arange(N) % 5 != 1).astype(np.uint8)
    hr, cr, dbg = oracle.lstm_step(L, xt[x_row], hp, cp, parent=parent, active=active, debug=True)
    d = dict(L=G, N=N, x_codes=dev(xt), x_row=dev(x_row), parent=dev(parent), h_prev=dev(hp), c_prev=dev(cp),
             h_next=torch.full((N, H), 99, dtype=torch.int8, device="cuda:0"),
             c_next=torch.full((N, H), 99.0, device="cuda:0"),
             dbg_acch=torch.zeros((N, 4 * H), dtype=torch.int32, device="cuda:0"))
    if active is not None:
        d["active"] = dev(active)
    if looked_up:
        d["gx"] = q.input_projection(G, d["x_codes"])[0]
        if looked_up == "table":
            d["gx_table"] = q.input_table(G, d["gx"])
    else:
        d["dbg_accx"] = torch.zeros((N, 4 * H), dtype=torch.int32, device="cuda:0")
    group = q.StepGroup([d])
    who = np.arange(N)
    if listed is None:
        group.launch()
    else:
        who = np.random.default_rng(N).permutation(N)[:listed]
        entries = np.full((N, 4), 1 << 30, np.int32)   # behind the end: anything
        entries[:listed] = np.stack([who, parent[who], x_row[who], 0 * who], 1)
        group.launch(dev(entries), dev(np.array([listed], np.int32)))
    h, c = host(d["h_next"]), host(d["c_next"])
    others = np.setdiff1d(np.arange(N), who)
    assert (h[others] == 99).all() and (c[others] == 99.0).all()
    if len(who) == 0:
        return
    on = who if active is None else who[active[who] != 0]   # (the oracle forms no sums for the others)
    assert np.array_equal(host(d["dbg_acch"])[on], dbg["acch"][on])
    if not looked_up:
        assert np.array_equal(host(d["dbg_accx"])[on], dbg["accx"][on])
    assert_rel(c[who], cr[who], "c")
    assert_codes_close(h[on], hr[on], dbg["h_real"][on] * 7.0, "h")
    off = np.setdiff1d(who, on)
    assert np.array_equal(h[off], hp[parent[off]])


@pytest.mark.parametrize("I,H", [(48, 80), (1040, 272), (64, 1040)])
@pytest.mark.parametrize("looked_up", [False, "sums", "table"])
def test_up_to_32_hypotheses_one_arithmetic(gpu_lib, I, H, looked_up):
    """Up to 16 hypotheses the weights are streamed, with 17 to 32 K is split: a hypothesis gets the same bits either way."""
    q = gpu_lib
    s_x = float(np.float32(4) / np.float32(7))
    _, G = _lstm_pair(q, 2400 + I + H, I, H, s_x)
    x, hp, cp = dev(synth.codes(2401, (32, I), -8, 7)), dev(synth.codes(2402, (32, H), -7, 7)), dev(synth.normal(2403, (32, H), 0.6))
    active = dev((np.arange(32) % 5 != 1).astype(np.uint8))
    rows = dev(np.arange(32, dtype=np.int32)[::-1].copy())
    first = {}
    for N in (16, 17, 20, 31, 32):
        d = dict(L=G, N=N, x_codes=x, x_row=rows[:N].contiguous(), parent=(rows[:N] % N).contiguous(),
                 h_prev=hp[:N].contiguous(), c_prev=cp[:N].contiguous(), active=active[:N].contiguous(),
                 h_next=torch.empty((N, H), dtype=torch.int8, device="cuda:0"), c_next=torch.empty((N, H), device="cuda:0"))
        d["parent"][:16] = torch.arange(16, dtype=torch.int32, device="cuda:0").flip(0)   # (the first 16 are the same hypotheses in all)
        if looked_up:
            d["gx"] = q.input_projection(G, x)[0]
            if looked_up == "table":
                d["gx_table"] = q.input_table(G, d["gx"])
        q.StepGroup([d]).launch()
        got = d["h_next"][:16], d["c_next"][:16]
        first = first or dict(zip("hc", got))
        for k, v in zip("hc", got):
            assert torch.equal(v, first[k]), (N, k)
