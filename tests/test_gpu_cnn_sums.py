"""The sums behind a training step's gradients, and what a step leaves behind.

Gradients of many cells cancel, so the workgroups' rows of sums are added in
64 bits.  Here two images' contributions cancel exactly and a third's, 2e5
times smaller, is what is left: the gradients have to be those of the third
image alone.  Each row is the same in both calls, so the only differences are
the 64-bit additions' (at most 64 of them, 2^-53 of the largest row each) and
one rounding to fp32 each: |a - b| <= 2^-23 |b| + 2^-47 |large|.

A step that starts from the same state gives the same bits, and the forward
pass after an update is the oracle's with the updated parameters, to the bars
of test_gpu_cnn.py (bf16 activations, 1e-2)."""
import numpy as np
import pytest

import synth
from oracle import cnn

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

W4, H4 = 160, 120


def _params(seed):
    convs, Wh, _ = cnn.unpack(cnn.init_params(seed).astype(np.float64))
    rng = np.random.default_rng(seed)
    convs = [(W, rng.uniform(-0.05, 0.1, size=cnn.C)) for W, _ in convs]
    return cnn.pack(convs, Wh, rng.normal(-1, 0.5, size=cnn.NH)).astype(np.float32)


def test_rows_that_cancel():
    pipe = cd.Pipeline([(640, 480)] * 5)
    pipe.cnn_buffers()
    pipe.d_images.fill_(128)
    acts = torch.ones(4 * pipe.ncells * cnn.C, dtype=torch.bfloat16, device="cuda").view(torch.int16)
    P = torch.from_numpy(_params(5)).cuda()
    pw = torch.ones(cnn.NH, device="cuda")
    work = torch.empty(2 * pipe.ncells * cnn.C, dtype=torch.int16, device="cuda")

    def grads(*parts):
        # a logit of -110 gives a gradient of exactly zero, 0 one of +-0.5
        z = torch.full((5, H4, W4, cnn.NH), -110.0, device="cuda")
        y = torch.zeros((5, H4, W4), dtype=torch.int32, device="cuda")
        for img, y0, x0, logit, label in parts:   # blocks of 32 x 16 cells
            z[img, y0:y0 + 16, x0:x0 + 32] = logit
            y[img, y0:y0 + 16, x0:x0 + 32] = label
        grad = torch.empty(cnn.N_PARAMS, device="cuda")
        loss = torch.empty(1, device="cuda")
        cd.cdvs_cnn_backward(pipe.ctx, pipe.d_images, P, acts, z, y, pw, work, grad, loss)
        torch.cuda.synchronize()
        return grad.cpu().numpy().astype(np.float64)

    plus, minus, small = (0, 16, 32, 0.0, 0), (4, 16, 32, 0.0, 63), (2, 64, 64, -12.0, 0)
    large, want, got = grads(plus), grads(small), grads(plus, small, minus)
    assert np.count_nonzero(want) > 0.9 * cnn.N_PARAMS
    assert np.all(np.abs(got - want) <= 2.0 ** -23 * np.abs(want) + 2.0 ** -47 * np.abs(large).max())


def test_steps_from_one_state():
    sizes = [(640, 480), (97, 61), (500, 641)]
    imgs = [synth.image(synth.SEED_TRAIN, i, w, h, nblobs=max(4, w * h // 1500)) for i, (w, h) in enumerate(sizes)]
    pipe = cd.Pipeline(sizes)
    pipe.upload(imgs)
    pipe.cnn_buffers()
    rng = np.random.default_rng(21)
    labels = torch.from_numpy((rng.random((pipe.ncells, 6)) < 0.1).dot(1 << np.arange(6)).astype(np.int32)).cuda()
    pw = torch.full((cnn.NH,), 5.0, device="cuda")
    work = torch.empty(2 * pipe.ncells * cnn.C, dtype=torch.int16, device="cuda")
    grad, loss = torch.empty(cnn.N_PARAMS, device="cuda"), torch.empty(1, device="cuda")
    runs = []
    for _ in range(2):
        p0 = _params(3)
        p, m, v = (torch.from_numpy(a).cuda() for a in (p0, np.zeros_like(p0), np.zeros_like(p0)))
        ref, rm, rv = p0.astype(np.float64), np.zeros(cnn.N_PARAMS), np.zeros(cnn.N_PARAMS)
        for step in (1, 2, 3):
            pipe.cnn_forward(p, tau=None, logits=True)
            cd.cdvs_cnn_backward(pipe.ctx, pipe.d_images, p, pipe.d_acts, pipe.d_logits, labels, pw, work, grad, loss)
            cd.cdvs_cnn_adam(pipe.ctx, p, grad, m, v, step, lr=1e-3)
            torch.cuda.synchronize()
            ref, rm, rv = cnn.adam(ref, grad.cpu().numpy().astype(np.float64), rm, rv, step, lr=1e-3)
            np.testing.assert_allclose(p.cpu().numpy(), ref, atol=1e-6)
        pipe.cnn_forward(p, tau=None, logits=True)
        torch.cuda.synchronize()
        runs.append([t.cpu().numpy().copy() for t in (grad, p, m, v, loss, pipe.d_logits)])
    for a, b in zip(*runs):
        np.testing.assert_array_equal(a, b)
    final, logits = runs[1][1], runs[1][5]
    for i, im in enumerate(imgs):
        c0, w4, h4 = pipe.cell_layout(i)
        Z, _ = cnn.forward(final, im, bf16_mode=True)
        got = logits[c0:c0 + w4 * h4].reshape(h4, w4, cnn.NH)
        assert np.linalg.norm(got - Z) <= 1e-2 * np.linalg.norm(Z), i
