"""Rows of the decoder's state pool: taken by label picks, freed at the end of a frame (or iteration), named by several
rounds in between.  Many frames make every row change hands often; W = 64 with 16 labels a frame is the largest pool
(1088 rows an utterance, the limit of the free-row mask) and W = 1 the smallest."""
import numpy as np
import pytest
import torch

import oracle
from oracle import models as omodels
from paper_2206_07882_amd import synth

from .test_gpu_decode import _compare_beams, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("search,B,W,limit,T", [("frames", 2, 64, 16, 3), ("frames", 3, 1, 16, 30), ("frames", 2, 2, 1, 40),
                                                ("frames", 2, 5, 3, 25), ("alsd", 2, 64, 5, 6), ("alsd", 3, 1, 20, 20),
                                                ("alsd", 2, 5, 12, 30), ("alsd_reuse", 2, 5, 12, 30)])
def test_pool_rows_change_hands(gpu_lib, search, B, W, limit, T):
    from paper_2206_07882_amd import model as gmodel
    q = gpu_lib
    m = synth.make_model(0, weight_std=0.5)
    m.rho = 0.1
    e = synth.normal(300 + B + W, (T, B, m.J), 1.0)
    G, M = gmodel.model_from_float(m, "cuda:0"), omodels.model_from_float(m)
    if search == "frames":
        ref = oracle.decode(M, e, W, limit, max_len=T * limit)
        got = q.decode(G, dev(e), W, limit, max_len=T * limit)
    else:
        ref = oracle.decode_alsd(M, e, W, limit)
        got = q.decode_alsd(G, dev(e), W, limit, flags=q.ALSD_REUSE if search == "alsd_reuse" else 0)
    _compare_beams(got, ref)
