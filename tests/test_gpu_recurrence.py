"""The persistent recurrence at the edges of its dispatch: layers narrower than a workgroup's 32 cells and with an odd
number of 16-cell groups, 1..8 utterances (one cell per lane, columns packed to a power of two) against 9 and more,
input widths on either side of what the kernel projects by itself (384 | 385, 1280 | 1281), sequences longer than the
step number that travels with a code (mod 16, at 8 bits mod 256), more utterances than one launch holds, and two
directions of different width; 641 cells and more (constants in LDS) at both widths, 97 utterances (f*c rounded first).
Every step against one oracle step from the GPU's own previous state.  Then the routes that an idle device does not take:
a refused launch, a group spread over XCDs, a group short of members, several streams at once."""
import numpy as np
import pytest
import torch

import oracle
from paper_2206_07882_amd import synth
from tests.test_gpu_parity import _lstm_pair, assert_codes_close, assert_rel, dev, host, DEV
from tests.test_gpu_int8 import _lstm8_pair

pytestmark = pytest.mark.gpu


def _check(L, x, hg, cg, reverse, h0, c0, unit, what):
    T, B = x.shape[:2]
    hp = np.zeros((B, L.H), np.int8) if h0 is None else h0
    cp = np.zeros((B, L.H), np.float32) if c0 is None else c0
    # A code may differ (by one) only where the quantizer's input lies within 1e-4 of a rounding tie: 2e-4 of all codes.
    # That is the bar for the sequence; one step of a narrow layer has too few codes for a bar of its own.
    same = 0
    for t in (range(T - 1, -1, -1) if reverse else range(T)):
        hr, cr, dbg = oracle.lstm_step(L, x[t], hp, cp, debug=True)
        if cg is not None:
            assert_rel(cg[t], cr, f"{what} c t={t}")
        assert_codes_close(hg[t], hr, dbg["h_real"] * unit, f"{what} h t={t}", 0.9)
        same += int((hg[t] == hr).sum())
        hp, cp = hg[t], (cr if cg is None else cg[t])
    assert same >= 0.999 * T * B * L.H, what
    return hp, cp


@pytest.mark.parametrize("T,B,I,H,bits,reverse,state", [
    (40, 1, 64, 16, 4, False, False), (35, 2, 1280, 48, 4, True, True), (20, 8, 385, 272, 4, False, True),
    (20, 9, 384, 256, 4, True, False), (9, 17, 1281, 640, 4, False, True), (5, 33, 48, 656, 4, True, False),
    (270, 3, 40, 32, 8, False, True), (6, 20, 1300, 48, 8, True, True), (1, 5, 64, 64, 4, False, True),
    (2, 4, 320, 640, 8, False, False), (4, 530, 32, 1024, 4, False, True), (6, 13, 340, 1024, 8, True, True),
    (5, 7, 385, 704, 8, False, True), (4, 97, 64, 704, 8, True, False), (4, 97, 1300, 768, 4, False, True)])
def test_recurrence_edges(gpu_lib, T, B, I, H, bits, reverse, state):
    q = gpu_lib
    q_max = 127 if bits == 8 else 7
    s_x = float(np.float32(4) / np.float32(q_max))
    L, G = (_lstm8_pair if bits == 8 else _lstm_pair)(q, 5171 + I + H, I, H, s_x)
    P = q.act_pitch(I)
    x = synth.codes(5172 + T, (T, B, I), -q_max - 1, q_max)
    xp = np.full((T, B, P), 3, np.int8)   # padding bytes must not matter
    xp[..., :I] = x
    h0 = synth.codes(5173, (B, H), -q_max, q_max) if state else None
    c0 = synth.normal(5174, (B, H), 0.6) if state else None
    kw = dict(reverse=reverse, h0=None if h0 is None else dev(h0), c0=None if c0 is None else dev(c0), want_last=True)
    need = q.lstm_layer_workspace(G, T, B)
    ws = torch.full((need,), 0x55, dtype=torch.uint8, device=DEV)   # whatever an earlier call left there
    out = q.lstm_layer(G, dev(xp), debug=True, workspace=ws, **kw)
    assert q.layer_error_flag(ws, need) == 0
    hg, cg = host(out["h_out"]), host(out["c_all"])
    hl, cl = _check(L, x, hg, cg, reverse, h0, c0, float(q_max), f"I={I} H={H} B={B}")
    assert np.array_equal(host(out["h_last"]), hl) and np.array_equal(host(out["c_last"]), cl)
    again = q.lstm_layer(G, dev(xp), workspace=ws, **kw)   # without debug outputs, on the used workspace
    assert torch.equal(again["h_out"], out["h_out"]) and torch.equal(again["c_last"], out["c_last"])


@pytest.mark.parametrize("T,B,bits", [(18, 130, (4, 4)), (6, 3, (8, 4)), (5, 60, (8, 8)), (17, 65, (4, 4)), (1, 77, (4, 4)),
                                      (6, 100, (8, 8)), (3, 200, (4, 4))])
def test_two_directions(gpu_lib, T, B, bits):
    """130 utterances: 18 groups of 16 utterances and direction, more than one launch's worth; a backward direction of
    another width than the forward one; 60 x 640 cells x 2 directions: the size class whose cell rounds f*c first.  65 to
    200 utterances: workgroups with two groups in turn, the last of them with one."""
    q = gpu_lib
    I, H = 340, 640
    s_x = 0.03
    pairs = [(_lstm8_pair if b == 8 else _lstm_pair)(q, 5271 + d, I, H, s_x) for d, b in enumerate(bits)]
    x = synth.codes(5272 + T, (T, B, I), -7, 7)
    xp = np.zeros((T, B, q.act_pitch(I)), np.int8)
    xp[..., :I] = x
    ws = torch.full((q.bilstm_layer_workspace(pairs[0][1], pairs[1][1], T, B),), 0x33, dtype=torch.uint8, device=DEV)
    out = host(q.bilstm_layer(pairs[0][1], pairs[1][1], dev(xp), workspace=ws))
    assert q.layer_error_flag(ws, q.lstm_layer_workspace(pairs[0][1], T, B)) == 0 and q.layer_error_flag(ws, ws.numel()) == 0
    for d in range(2):
        _check(pairs[d][0], x, out[:, :, d * H:(d + 1) * H], None, d == 1, None, None, 127.0 if bits[d] == 8 else 7.0, f"dir {d}")


@pytest.mark.parametrize("T,B,I,H,reverse,state", [(7, 3, 340, 640, False, True), (5, 20, 1280, 48, True, False),
                                                   (6, 40, 64, 768, False, True)])
def test_refused_recurrence_runs_step_by_step(gpu_lib, T, B, I, H, reverse, state):
    """A device that cannot hold the persistent kernel: the layer goes step by step, with sums of the input part that the
    persistent kernel would have formed by itself (the workspace holds whatever an earlier call left there)."""
    q = gpu_lib
    s_x = float(np.float32(4) / np.float32(7))
    L, G = _lstm_pair(q, 5371 + I + H, I, H, s_x)
    x = synth.codes(5372 + T, (T, B, I), -8, 7)
    xp = np.zeros((T, B, q.act_pitch(I)), np.int8)
    xp[..., :I] = x
    h0 = synth.codes(5373, (B, H), -7, 7) if state else None
    c0 = synth.normal(5374, (B, H), 0.6) if state else None
    need = q.lstm_layer_workspace(G, T, B)
    ws = torch.full((need,), 0x55, dtype=torch.uint8, device=DEV)
    out = q.lstm_layer(G, dev(xp), reverse=reverse, h0=None if h0 is None else dev(h0), c0=None if c0 is None else dev(c0),
                       want_last=True, workspace=ws, route=q.DIAG_STEPWISE)
    assert q.layer_error_flag(ws, need) == 0
    hl, _ = _check(L, x, host(out["h_out"]), None, reverse, h0, c0, 7.0, f"step by step H={H}")
    assert np.array_equal(host(out["h_last"]), hl)


@pytest.mark.parametrize("H,B,bits,f_first", [(640, 96, 4, False), (640, 97, 4, True), (640, 97, 8, True), (640, 8, 8, False),
                                              (704, 80, 4, False), (704, 96, 4, True), (768, 90, 8, True), (784, 96, 4, False),
                                              (512, 140, 4, False), (832, 100, 8, True), (1024, 64, 4, False),
                                              (1024, 65, 4, True), (1024, 128, 4, True), (1024, 129, 4, False)])
def test_which_product_of_the_cell_is_rounded_first(gpu_lib, H, B, bits, f_first):
    """c' = f*c + i*g has one product rounded before the sum, f*c in some size classes and i*g in the others.  With g = 1
    the gates can be read off exactly (c = 0 gives i, c = 2^60 gives f) and the two orders told apart bit for bit."""
    q = gpu_lib
    I = 64
    G = (_lstm8_pair if bits == 8 else _lstm_pair)(q, 5671 + H, I, H, 0.1)[1]
    bias = G.bias.clone()
    bias[2 * H:3 * H] = 60.0
    G = q.Lstm(G.w_ih, G.w_hh, bias, G.x_scale, G.h_scale, G.h_inv_scale)
    x = dev(synth.codes(5672 + B, (1, B, I), -7, 7))

    def cell(c0):
        return host(q.lstm_layer(G, x, c0=dev(c0), want_last=True)["c_last"])

    full = lambda v: np.full((B, H), v, np.float32)
    i, f = cell(full(0.0)), np.ldexp(cell(full(2.0 ** 60)), -60)
    c0 = synth.normal(5673 + B, (B, H), 0.8)
    got = cell(c0)
    exact = np.longdouble(f) * np.longdouble(c0)   # 48 bits of 64
    first = np.float32(np.longdouble(exact.astype(np.float32)) + np.longdouble(i))
    last = (exact + np.longdouble(i)).astype(np.float32)
    assert (first != last).mean() > 0.01
    assert np.array_equal(got, first if f_first else last)


@pytest.mark.parametrize("T,B,I,H,bits,state", [(20, 1, 64, 64, 4, True), (40, 3, 1280, 640, 4, False), (9, 17, 1300, 640, 4, True),
                                                (6, 120, 340, 640, 4, True), (5, 8, 385, 656, 4, False), (280, 5, 40, 80, 8, True), (19, 150, 1280, 640, 4, True),
                                                (3, 400, 384, 272, 8, False), (6, 20, 1281, 48, 8, False), (7, 13, 340, 1024, 8, True), (4, 100, 64, 704, 8, False)])
def test_routes_of_the_recurrence_agree(gpu_lib, T, B, I, H, bits, state):
    """A group whose workgroups run on several XCDs, and one whose workgroups are not resident together (whoever has come
    shares the work), return the very bits of the usual route; 120 and 100 utterances: layers that round f*c first; 150 and
    400: two groups to a workgroup."""
    q = gpu_lib
    q_max = 127 if bits == 8 else 7
    L, G = (_lstm8_pair if bits == 8 else _lstm_pair)(q, 5471 + I + H, I, H, 0.5 / q_max)
    xp = np.full((T, B, q.act_pitch(I)), 3, np.int8)
    xp[..., :I] = synth.codes(5472 + T, (T, B, I), -q_max - 1, q_max)
    h0 = dev(synth.codes(5473, (B, H), -q_max, q_max)) if state else None
    c0 = dev(synth.normal(5474, (B, H), 0.6)) if state else None
    need = q.lstm_layer_workspace(G, T, B)
    x, want = dev(xp), None
    members = (H + 31) // 32
    for route in [0, q.DIAG_SPREAD] + [n << 8 for n in sorted({1, 2, 3, members // 2, members - 1}) if 0 < n < members]:
        ws = torch.full((need,), 0x55, dtype=torch.uint8, device=DEV)
        out = q.lstm_layer(G, x, reverse=state, h0=h0, c0=c0, want_last=True, debug=True, workspace=ws, route=route)
        assert q.layer_error_flag(ws, need) == 0
        del out["accx"]
        want = want or out
        for k, v in out.items():
            assert torch.equal(v, want[k]), f"route {route:#x}: {k}"


@pytest.mark.parametrize("B,I,H,two", [(128, 340, 640, False), (129, 340, 640, True), (150, 1280, 640, True), (256, 340, 640, True),
                                       (257, 340, 640, False), (400, 384, 272, True), (384, 384, 272, False), (150, 340, 656, False),
                                       (300, 64, 256, False), (150, 1296, 640, False)])
def test_when_a_workgroup_has_two_groups_in_turn(gpu_lib, B, I, H, two):
    """Where that saves more than three launches of seven (2 -> 1, not 3 -> 2): the members of a pair count themselves in with
    the first group's admission word only.  (The words lie in front of the exchange area, which the error flag follows.)"""
    q = gpu_lib
    _, G = _lstm_pair(q, 6100 + I + H, I, H, 0.03)
    T, groups, members = 3, (B + 15) // 16, (H + 31) // 32
    need = q.lstm_layer_workspace(G, T, B)
    ws = torch.full((need,), 0x55, dtype=torch.uint8, device=DEV)
    q.lstm_layer(G, dev(synth.codes(6101, (T, B, q.act_pitch(I)), -8, 7)), workspace=ws)
    assert q.layer_error_flag(ws, need) == 0
    exchange = (2 * groups * ((H + 63) // 64) * 64 * 4 * 8 + 255) // 256 * 256
    at = need - 256 - exchange - (8 * groups + 15) // 16 * 16
    words = ws[at:at + 8 * groups].cpu().numpy().view(np.uint64)
    counts = [sum((int(w) >> (6 * i)) & 63 for i in range(9)) for w in words]
    assert counts == [members if not two or g % 2 == 0 else 0 for g in range(groups)]


@pytest.mark.parametrize("B,n_streams,layers", [(1, 4, 6), (40, 3, 4), (77, 3, 2)])
def test_recurrences_on_several_streams(gpu_lib, B, n_streams, layers):
    """Encoders on streams of their own, with workspaces of their own: each launch wants more than half of an XCD, so
    their workgroups meet on the same compute units and groups are cut short of members."""
    q = gpu_lib
    T, I, H = 100, 1280, 640
    L = [_lstm_pair(q, 5571 + d, I, H, 0.1)[1] for d in range(2)]
    xs = [dev(synth.codes(5573 + i, (T, B, I), -7, 7)) for i in range(n_streams)]
    need = q.bilstm_layer_workspace(L[0], L[1], T, B)
    wss = [torch.empty((layers, need), dtype=torch.uint8, device=DEV) for _ in range(n_streams)]

    def run(i):
        x = xs[i]
        for k in range(layers):
            x = q.bilstm_layer(L[0], L[1], x, workspace=wss[i][k])
        return x

    want = []
    for i in range(n_streams):
        want.append(run(i).clone())
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(n_streams)]
    for _ in range(3):
        got = []
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                got.append(run(i))
        torch.cuda.synchronize()
        for i in range(n_streams):
            for k in range(layers):
                assert q.layer_error_flag(wss[i][k], need) == 0
                assert q.layer_error_flag(wss[i][k], q.lstm_layer_workspace(L[0], T, B)) == 0
            assert torch.equal(got[i], want[i])
