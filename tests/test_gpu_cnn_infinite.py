"""Activations that have become infinite (a training run that diverges): the
training forward gives what the nine taps give, infinity times a positive
weight staying infinite in every layer, also where a matrix instruction's
spare tap has a weight of zero."""
import numpy as np
import pytest

from oracle import cnn

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402


@pytest.mark.parametrize("size", [(97, 61), (640, 480)])
def test_infinite_activations_stay_infinite(size):
    convs = [(np.full((9, cnn.C, cnn.C), 0.01), np.zeros(cnn.C)) for _ in range(cnn.NL)]
    convs[0] = (np.full((9, cnn.C, cnn.C), 0.01), np.full(cnn.C, 3.4e38))   # above the largest bf16
    P = cnn.pack(convs, np.full((cnn.C, cnn.NH), 0.5), np.zeros(cnn.NH)).astype(np.float32)
    pipe = cd.Pipeline([size])
    pipe.cnn_forward(torch.from_numpy(P).cuda(), tau=0.3)
    torch.cuda.synchronize()
    acts = pipe.d_acts.cpu().numpy().view(np.uint16).reshape(cnn.NL, pipe.ncells, cnn.C)
    for l in range(cnn.NL):
        assert np.all(acts[l] == 0x7F80), l
    assert np.all(np.isposinf(pipe.d_logits.cpu().numpy()))
