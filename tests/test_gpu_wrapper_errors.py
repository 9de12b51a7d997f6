"""Values of a wrong type at the Python entry points whose argument types are declared to ctypes: a TypeError, as the other
entry points raise, and numpy or torch scalars go in like plain numbers."""
import numpy as np
import pytest
import torch

from paper_2206_07882_amd import synth

from .test_gpu_parity import DEV, dev

pytestmark = pytest.mark.gpu


def test_wrong_types_are_type_errors_and_scalars_are_numbers(gpu_lib):
    q = gpu_lib
    m = q.pack_int4(dev(synth.normal(1, (32, 64), 0.3)), q.LAYOUT_TILED)
    a = dev(synth.codes(2, (5, 64), -7, 7))
    want = q.linear(m, None, 0.25, a)
    assert torch.equal(q.linear(m, None, np.float32(0.25), a), want)
    assert torch.equal(q.linear(m, None, torch.tensor(0.25), a), want)
    score, fused = torch.zeros((1, 2), device=DEV), torch.zeros((2, 8), device=DEV)
    assert torch.equal(q.beam_step(score, fused, blank=np.int64(3), force_blank=True)[1], torch.full((1, 2), 3, dtype=torch.int32, device=DEV))
    e, p, fr = torch.zeros((2, 32), device=DEV), torch.zeros((2, 32), device=DEV), torch.zeros(2, dtype=torch.int32, device=DEV)
    w = q.pack_int4(dev(synth.normal(3, (8, 32), 0.3)), q.LAYOUT_TILED)
    for call in (lambda: q.linear(m, None, "0.25", a), lambda: q.linear(m, None, None, a),
                 lambda: q.linear_quant(m, None, 0.25, a, "7"), lambda: q.linear_quant(m, None, 0.25, a, 7.0, bits=4.0),
                 lambda: q.beam_step(score, fused, blank=1.5), lambda: q.joint_fuse(e, fr, p, w, None, None, None, "0", 0.0)):
        with pytest.raises(TypeError):
            call()
