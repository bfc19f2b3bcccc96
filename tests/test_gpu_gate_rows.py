"""Gated detection's reading of the cell mask: strips that begin within a cell
row, in the octaves where a cell covers four, two, one and half a row.  Bits of
one octave at a time, so that no keypoint is dropped as another octave's
duplicate: a mask's and its complement's keypoints are then the full mask's,
each centre in its own."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

SIZES = [(333, 251), (640, 403), (131, 640)]


def _records(pipe, mask):
    pipe.d_mask.copy_(torch.from_numpy(mask))
    pipe.detect(mask=pipe.d_mask)
    torch.cuda.synchronize()
    assert pipe.sync_status() == cd.CDVS_OK
    return pipe.keypoints()


@pytest.mark.parametrize("copies", [1, 40])
@pytest.mark.parametrize("border", [1, 2, 3, 4, 7])
def test_mask_and_complement_split_the_keypoints(border, copies):
    # (40 copies: taller strips)
    p = cd.default_params()
    p.border, p.mask_fmax, p.topk, p.contrast = border, 1.0, 4096, 0.5
    sizes = SIZES * copies
    pipe = cd.Pipeline(sizes, params=p, kp_capacity=4096)
    imgs = [synth.image(synth.SEED_RAGGED, i, w, h, nblobs=150) for i, (w, h) in enumerate(SIZES)]
    pipe.upload(imgs * copies)
    pipe.cnn_buffers()
    pipe.pyramid()
    rng = np.random.default_rng(border)
    for o in range(4):
        on = rng.random(pipe.ncells) < 0.5
        a = _records(pipe, np.where(on, 1 << o, 0).astype(np.uint8))
        b = _records(pipe, np.where(on, 0, 1 << o).astype(np.uint8))
        full = _records(pipe, np.full(pipe.ncells, 1 << o, dtype=np.uint8))
        found = 0
        for i in range(pipe.n):
            c0, w4, h4 = pipe.cell_layout(i)
            m = on[c0:c0 + w4 * h4].reshape(h4, w4)
            key = lambda k: sorted(zip(k["iy"].tolist(), k["ix"].tolist(), k["p"].tolist()))  # noqa: E731
            for k, want in ((a[i], True), (b[i], False)):
                assert np.all(k["octave"] == o)
                cy, cx = (k["iy"] << o) >> 2, (k["ix"] << o) >> 2
                assert np.all(m[np.minimum(cy, h4 - 1), np.minimum(cx, w4 - 1)] == want)
            assert key(np.concatenate([a[i], b[i]])) == key(full[i])
            found += len(full[i])
        assert found > 0
