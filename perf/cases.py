"""Workloads of the INT4 RNN-T library for timing: what its users have it do, through the Python layer's entry points.

``listed()`` names the representative ones, ``draw(rng)`` gives one more of the same ranges, ``prepare(case, seed)``
makes what a program holds before the call (inputs, packed weights, workspaces), ``run(state)`` is one pass,
``work(case)`` what a pass cannot do without, ``tolerance(case)`` how far two correct builds may be apart.

Kinds of work
  transcribe  features -> encoder -> time-synchronous search (one call of the product)
  alsd        encoder output -> alignment-length synchronous search with recombination
  encode      features -> encoder stack + projection to the joint
  chunk       one unidirectional layer over a chunk of frames with carried state, in the library's own workspace
  step        one round of a caller-driven search: grouped LSTM steps, output layers, joint + fusion, beam selection

Nets: "base" (240 features, prediction network 768, two language models 2 x 1024, all 4-bit), "paper" (the layer
shapes of the paper's Sec. 2 at 4 bits: 340 features, external language model 2 x 2048 with a bottleneck) and "mixed"
(those shapes with the first encoder layer and the RNN-T's linear layers at 8 bits).
"""
from __future__ import annotations

import functools

import torch

from paper_2206_07882_amd import model as gmodel
from paper_2206_07882_amd import qrnnt as q
from paper_2206_07882_amd import synth

DEV = "cuda:0"
V, J, H_ENC = 46, 256, 640
FEAT = {"base": 240, "paper": 340, "mixed": 340}
# (hidden, layers, bottleneck) of the prediction network, the source and the external language model
NETS = {"base": ((768, 1, 0), (1024, 2, 0), (1024, 2, 0)), "paper": ((768, 1, 0), (768, 1, 0), (2048, 2, 256))}
NETS["mixed"] = NETS["paper"]


def listed():
    return [
        # one 152-frame utterance as it arrives at a recogniser: the latency a single speaker sees, beam 16
        dict(name="transcribe_utterance", kind="transcribe", net="base", B=1, T=152, W=16, max_sym=4, early=False),
        # the benchmark's batch: 64 utterances of 40 s, beam 16, at most 4 labels a frame
        dict(name="transcribe_batch", kind="transcribe", net="base", B=64, T=1000, W=16, max_sym=4, early=False),
        # the paper's layer shapes and precision map, a ragged batch as a server collects it
        dict(name="transcribe_mixed_ragged", kind="transcribe", net="mixed", B=13, T=301, W=16, max_sym=4, early=False),
        # greedy decoding of a few utterances, rounds without a label skipped
        dict(name="transcribe_greedy", kind="transcribe", net="base", B=5, T=237, W=1, max_sym=4, early=True),
        # the paper's own search over a full batch
        dict(name="alsd_batch", kind="alsd", net="base", B=64, T=300, W=16, u_max=150, reuse=False),
        # the same for one utterance at a narrow beam, reusing the states of hypotheses already held
        dict(name="alsd_utterance", kind="alsd", net="base", B=1, T=152, W=4, u_max=76, reuse=True),
        # the encoder stack alone: the batch and the single utterance of the encoder configuration, and an odd batch
        # at mixed precision
        dict(name="encode_batch", kind="encode", net="base", B=32, T=500),
        dict(name="encode_utterance", kind="encode", net="base", B=1, T=500),
        dict(name="encode_mixed_ragged", kind="encode", net="mixed", B=77, T=129),
        # a serving loop that feeds a unidirectional layer one second of frames at a time
        dict(name="chunk_4x25", kind="chunk", net="base", B=4, T=25),
        # one decoding round driven by the caller: a single beam of 16, and 64 beams of 16
        dict(name="step_1x16", kind="step", net="base", B=1, W=16),
        dict(name="step_64x16", kind="step", net="base", B=64, W=16),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["transcribe", "transcribe", "alsd", "encode", "encode", "chunk", "step"])
    net = rng.choice(["base", "base", "paper", "mixed"])
    if kind == "transcribe":
        return dict(kind=kind, net=net, B=_log(rng, 1, 64), T=_log(rng, 20, 500), W=rng.choice([1, 2, 4, 5, 8, 10, 16, 16]),
                    max_sym=rng.choice([1, 2, 3, 4, 4]), early=rng.random() < 0.25)
    if kind == "alsd":
        T = _log(rng, 20, 400)
        return dict(kind=kind, net=net, B=_log(rng, 1, 64), T=T, W=rng.choice([1, 2, 4, 5, 8, 10, 16, 16]),
                    u_max=max(1, int(T * rng.uniform(0.2, 1.0))), reuse=rng.random() < 0.25)
    if kind == "encode":
        return dict(kind=kind, net=net, B=_log(rng, 1, 128), T=_log(rng, 20, 700))
    if kind == "chunk":
        T = _log(rng, 4, 200)
        return dict(kind=kind, net="base", B=_log(rng, 1, min(64, 3000 // T)), T=T)
    return dict(kind=kind, net="base" if net == "base" else "paper", B=_log(rng, 1, 128), W=rng.choice([1, 2, 4, 5, 8, 10, 16, 16]))


@functools.lru_cache(maxsize=4)
def _float_model(net, enc_layers):
    """Float weights on the host: the same for every seed, as a trained model's would be."""
    return synth.make_model(4 if net == "base" else 5, enc_layers=enc_layers, mixed=(net == "mixed"))


def _features(case, seed):
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    return torch.randn((case["T"], case["B"], FEAT[case["net"]]), generator=g, device=DEV, dtype=torch.float32)


def _codes(g, shape):
    return torch.randint(-7, 8, shape, generator=g, device=DEV, dtype=torch.int8)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=dict(case))
    if kind in ("transcribe", "alsd", "encode"):
        m = _float_model(case["net"], None)
        enc = gmodel.Encoder(m, DEV)
        feats = _features(case, seed)
        enc.workspace(case["T"], case["B"], DEV)
        if kind != "encode":
            G = s["G"] = gmodel.model_from_float(m, DEV)
        if kind == "transcribe":
            need = q.decode_workspace(G, case["T"], case["B"], case["W"], case["max_sym"])
            s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        if kind == "alsd":
            need = q.decode_alsd_workspace(G, case["T"], case["B"], case["W"], case["u_max"])
            s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
            s["e"] = enc.forward(feats)[1]
        else:
            s["enc"], s["feats"] = enc, feats
        return s
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    if kind == "chunk":
        f = _float_model("base", None).enc_layers[1][0]
        s["L"] = gmodel.lstm_from_float(f, gmodel.S_H, DEV)
        T, B = case["T"], case["B"]
        s["x"] = _codes(g, (T, B, 2 * H_ENC))
        s["h0"] = _codes(g, (B, H_ENC))
        s["c0"] = 0.5 * torch.randn((B, H_ENC), generator=g, device=DEV)
        s["h_out"] = torch.empty((T, B, H_ENC), dtype=torch.int8, device=DEV)
        s["h_last"] = torch.empty((B, H_ENC), dtype=torch.int8, device=DEV)
        s["c_last"] = torch.empty((B, H_ENC), dtype=torch.float32, device=DEV)
        return s
    # one round of a caller-driven search
    m = _float_model(case["net"], 1)
    G = s["G"] = gmodel.model_from_float(m, DEV)
    B, W = case["B"], case["W"]
    N = B * W
    tok = torch.randint(1, V, (N,), generator=g, device=DEV, dtype=torch.int32)
    parent = (torch.randint(0, W, (B, W), generator=g, device=DEV, dtype=torch.int32)
              + torch.arange(B, device=DEV, dtype=torch.int32)[:, None] * W).reshape(-1).contiguous()
    nets = s["nets"] = [G.pred, G.lm_src, G.lm_ext]
    s["h"], s["c"], s["groups"] = [[] for _ in nets], [[] for _ in nets], []
    for layer in range(max(len(n.layers) for n in nets)):
        steps = []
        for i, net in enumerate(nets):
            if layer >= len(net.layers):
                continue
            L = net.layers[layer]
            d = dict(L=L, N=N, parent=parent, h_prev=_codes(g, (N, L.H)),
                     c_prev=0.5 * torch.randn((N, L.H), generator=g, device=DEV),
                     h_next=torch.empty((N, L.H), dtype=torch.int8, device=DEV),
                     c_next=torch.empty((N, L.H), dtype=torch.float32, device=DEV))
            if layer == 0:   # the input part of an embedding-fed layer comes from its per-token table
                d["x_codes"], d["x_row"] = net.embed_codes, tok
                d["gx"] = q.input_projection(L, net.embed_codes)[0]
                d["gx_table"] = q.input_table(L, d["gx"])
            else:
                d["x_codes"] = s["h"][i][layer - 1]
            s["h"][i].append(d["h_next"])
            s["c"][i].append(d["c_next"])
            steps.append(d)
        s["groups"].append(q.StepGroup(steps))
    s["enc"] = torch.randn((B, J), generator=g, device=DEV)
    s["frame"] = torch.arange(B, device=DEV, dtype=torch.int32).repeat_interleave(W).contiguous()
    s["score"] = torch.sort(-3.0 * torch.rand((B, W), generator=g, device=DEV), dim=1, descending=True).values.contiguous()
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "transcribe":
        _, e = s["enc"].forward(s["feats"])
        return q.decode(s["G"], e, case["W"], case["max_sym"], workspace=s["ws"], flags=q.DECODE_EARLY_STOP if case["early"] else 0)
    if kind == "alsd":
        return q.decode_alsd(s["G"], s["e"], case["W"], case["u_max"], workspace=s["ws"], flags=q.ALSD_REUSE if case["reuse"] else 0)
    if kind == "encode":
        return s["enc"].forward(s["feats"])
    if kind == "chunk":
        q.lstm_layer_static(s["L"], s["x"], s["h_out"], h0=s["h0"], c0=s["c0"], h_last=s["h_last"], c_last=s["c_last"])
        return s["h_out"], s["h_last"], s["c_last"]
    G = s["G"]
    for group in s["groups"]:
        group.launch()
    out = []
    for i, net in enumerate(s["nets"]):
        a, a_scale = s["h"][i][-1], net.out_a_scale
        if net.mid is not None:
            a, a_scale = q.linear_quant(net.mid, net.mid_bias, a_scale, a, net.mid_inv_scale), net.mid_scale
        out.append(q.linear(net.out, net.out_bias, a_scale, a, log_softmax=net.log_softmax))
    fused, _, _ = q.joint_fuse(s["enc"], s["frame"], out[0], G.joint_out, G.joint_bias, out[1], out[2], G.lambda_src, G.lambda_ext,
                               G.rho, G.blank, G.z_scale, G.z_inv_scale)
    parent, token, score = q.beam_step(s["score"], fused, blank=G.blank)
    return dict(h=s["h"], c=s["c"], fused=fused, parent=parent, token=token, score=score)


def _net_work(net, N, table):
    """(operations, weight bytes, state bytes) of one advance of all networks of `net` for N hypotheses."""
    ops = wts = st = 0.0
    for (h, layers, mid), rows in zip(NETS[net], (J, V, V)):
        for l in range(layers):
            k = h if (l == 0 and table) else 2 * h
            ops += 2.0 * N * 4 * h * k
            wts += 4 * h * k / 2 + 4 * h * 12
            st += N * h * 10.0
        if mid:
            ops += 2.0 * N * h * mid
            wts += h * mid / 2
        ops += 2.0 * N * (mid or h) * rows
        wts += (mid or h) * rows / 2
    return ops, wts, st


def _enc_work(case):
    T, B = case["T"], case["B"]
    ops = wts = 0.0
    for l in range(6):
        I = FEAT[case["net"]] if l == 0 else 2 * H_ENC
        width = 1.0 if (l == 0 and case["net"] == "mixed") else 0.5
        ops += 2 * 2.0 * T * B * 4 * H_ENC * (I + H_ENC)
        wts += 2 * (4 * H_ENC * (I + H_ENC) * width + 4 * H_ENC * 12)
    ops += 2.0 * T * B * 2 * H_ENC * J
    wts += 2 * H_ENC * J * (1.0 if case["net"] == "mixed" else 0.5)
    return ops, wts + T * B * 4.0 * FEAT[case["net"]]


def work(case):
    """Inputs and weights read once, outputs written once; operations count a multiply-accumulate as two.  A search is
    counted with every slot of its beam alive in every round (joint for all slots, network advance for all slots)."""
    kind = case["kind"]
    if kind == "encode":
        ops, byt = _enc_work(case)
        return dict(flops=ops, bytes=byt + case["T"] * case["B"] * (2.0 * H_ENC + 4 * J))
    if kind == "chunk":
        T, B, h = case["T"], case["B"], H_ENC
        return dict(flops=2.0 * T * B * 4 * h * 3 * h, bytes=4 * h * 3 * h / 2 + 4 * h * 12 + T * B * 3.0 * h + B * h * 10.0)
    N = case["B"] * case["W"]
    ops, wts, st = _net_work(case["net"], N, True)
    joint = 2.0 * N * J * V
    if kind == "step":
        return dict(flops=ops + joint, bytes=wts + st + J * V / 2 + case["B"] * J * 4 + N * V * 4.0)
    if kind == "alsd":
        it = case["T"] + case["u_max"]
        return dict(flops=it * (ops + joint), bytes=wts + 4.0 * case["T"] * case["B"] * J + 4.0 * N * case["u_max"])
    eo, eb = _enc_work(case)
    T, S = case["T"], case["max_sym"]
    return dict(flops=eo + T * (S * ops + (S + 1) * joint), bytes=eb + wts + 4.0 * N * T * S)


def tolerance(case):
    """Measured with every row scale and bias of the cells moved by one unit in the last place, which stands for another
    order of the fp32 sums.  A sum that lies on a rounding tie of the 4-bit quantizer of h then takes the other code, and
    a recurrence carries that on: the differences are few but not small.  One step (nothing carried on): rel 1.2e-7,
    max 1.1e-6, no code differs.  A chunk of one layer: rel 2.7e-3, max 0.056, 5e-4 of the codes.  The search: rel
    4.5e-4, max 2e-3, 3e-4 of the tokens; with recombination 1.3e-2 of them (an equal pair of hypotheses changes places).
    The six-layer encoder: from nothing at all to rel 0.26 and 5e-2 of the codes, so there the bounds are the tightest
    that still leave room for a few flipped codes."""
    kind = case["kind"]
    if kind == "step":
        return {"rel": 5e-7, "max": 5e-6, "differ": 1e-3}
    if kind == "chunk":
        return {"rel": 1e-2, "max": 0.2, "differ": 2e-3}
    if kind == "encode":
        return {"rel": 0.03, "max": 1.0 - 1e-9, "differ": 0.01}
    return {"rel": 2e-3, "max": 1e-2, "differ": 0.01 if kind == "alsd" else 1.5e-3}
