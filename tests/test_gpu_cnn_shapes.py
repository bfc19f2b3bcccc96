"""The mask network's kernels on the batch shapes where their work split
changes: the smallest image, partial tiles and ranges, workgroups that span
several images, and more cells than one pass of the grid covers.

Bars as in test_gpu_cnn.py, which follow from the kernels' bf16 operands
(rounding 2^-9 per operand): gradients cosine >= 0.999 and relative L2
<= 2e-2 of the oracle run with the same roundings, loss within 1e-3."""
import numpy as np
import pytest

import synth
from oracle import cnn

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402


def _params(seed):
    convs, Wh, _ = cnn.unpack(cnn.init_params(seed).astype(np.float64))
    rng = np.random.default_rng(seed)
    convs = [(W, rng.uniform(-0.05, 0.1, size=cnn.C)) for W, _ in convs]
    return cnn.pack(convs, Wh, rng.normal(-1, 0.5, size=cnn.NH)).astype(np.float32)


def _rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


# (16, 16): 16 cells; (97, 61): 25 x 16 cells, partial tiles; 40 images of
# 20 cells in one 256-cell range; 134,400 cells, more than the grid's
# 512 x 256; 548 tiles, more than its 512
SHAPES = {"smallest": [(16, 16)], "partial": [(97, 61), (130, 66), (129, 65)], "many_small": [(20, 16)] * 40,
          "beyond_grid": [(640, 480)] * 7, "beyond_tiles": [(130, 66)] * 9 + [(16, 16)] * 512}


@pytest.mark.parametrize("shape", list(SHAPES))
def test_backward_shapes(shape):
    sizes = SHAPES[shape]
    imgs = [synth.image(synth.SEED_TRAIN, i, w, h, nblobs=max(4, w * h // 1500)) for i, (w, h) in enumerate(sizes)]
    pipe = cd.Pipeline(sizes)
    pipe.upload(imgs)
    P = _params(2)
    dP = torch.from_numpy(P).cuda()
    pipe.cnn_forward(dP)
    rng = np.random.default_rng(9)
    labels = rng.integers(0, 64, size=pipe.ncells).astype(np.uint32)
    pw = rng.uniform(1, 8, size=cnn.NH).astype(np.float32)
    work = torch.empty(2 * pipe.ncells * cnn.C, dtype=torch.int16, device="cuda")
    grad = torch.full((cnn.N_PARAMS,), float("nan"), device="cuda")
    loss = torch.full((1,), float("nan"), device="cuda")
    for _ in range(2):   # overwritten, not added to
        cd.cdvs_cnn_backward(pipe.ctx, pipe.d_images, dP, pipe.d_acts, pipe.d_logits,
                             torch.from_numpy(labels.view(np.int32)).cuda(), torch.from_numpy(pw).cuda(), work, grad, loss)
    torch.cuda.synchronize()
    g_ref, l_ref = np.zeros(cnn.N_PARAMS), 0.0
    for i, im in enumerate(imgs):
        c0, w4, h4 = pipe.cell_layout(i)
        lab = labels[c0:c0 + w4 * h4].reshape(h4, w4).astype(np.uint8)
        l, g = cnn.loss_and_grad(P, im, lab, pw, min(pipe.num_octaves(i), cnn.NH), bf16_mode=True)
        l_ref += l / len(imgs)
        g_ref += g / len(imgs)
    g = grad.cpu().numpy().astype(np.float64)
    assert abs(loss.item() - l_ref) <= 1e-3 * abs(l_ref)
    assert g @ g_ref / np.linalg.norm(g) / np.linalg.norm(g_ref) >= 0.999 and _rel(g, g_ref) <= 2e-2
    off = 0
    for l in range(cnn.NL):
        assert _rel(g[off:off + cnn.CONV_W], g_ref[off:off + cnn.CONV_W]) <= 3e-2, l
        assert _rel(g[off + cnn.CONV_W:off + cnn.CONV_W + cnn.C], g_ref[off + cnn.CONV_W:off + cnn.CONV_W + cnn.C]) <= 3e-2, l
        off += cnn.CONV_W + cnn.C
    assert _rel(g[off:], g_ref[off:]) <= 2e-2
