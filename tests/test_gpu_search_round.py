"""The decoding round's kernel at the edges of what it splits: joint widths that end inside a wave's 64 columns or need
several blocks per wave, output layers that end inside a 128-column chunk, vocabularies at the edges of the 16-row tiles,
beams on both sides of a column tile, and mixed widths."""
import numpy as np
import pytest

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
    T = 5
    e = synth.normal(930 + J, (T, B, J), 1.0)
    G, M = gmodel.model_from_float(m, "cuda:0"), omodels.model_from_float(m)
    _compare_beams(q.decode(G, dev(e), W, 2, max_len=2 * T), oracle.decode(M, e, W, 2, max_len=2 * T))
    _compare_beams(q.decode_alsd(G, dev(e), W, 4), oracle.decode_alsd(M, e, W, 4))
