"""Detection's strips are cut by the size of the batch (6, 12, 24 or 48 centre
rows): an image's keypoints are the same in every batch, plain and gated, in
both launch forms, also where a workgroup's strips belong to several images
and where strips are left over."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

KINDS = [(640, 480), (61, 70), (333, 222), (68, 17)]


def _run(imgs, masked, variant):
    pipe = cd.Pipeline([(im.shape[1], im.shape[0]) for im in imgs])
    pipe.upload(imgs)
    pipe.cnn_buffers()
    cd.cdvs_tune_set(pipe.ctx, cd.KERNEL_DETECT, variant)
    # half of the cells of every image, whatever batch it is in
    mask = np.zeros(pipe.ncells, dtype=np.uint8)
    for i in range(pipe.n):
        c0, w4, h4 = pipe.cell_layout(i)
        mask[c0:c0 + w4 * h4] = (np.arange(w4 * h4) * 7 % 13 < 6) * 63
    pipe.d_mask.copy_(torch.from_numpy(mask))
    pipe.pyramid()
    pipe.detect(mask=pipe.d_mask if masked else None)
    torch.cuda.synchronize()
    assert pipe.sync_status() == cd.CDVS_OK
    out = pipe.keypoints()
    for k in out:
        k["image"] = 0
    return out


@pytest.mark.parametrize("masked", [False, True])
def test_keypoints_do_not_depend_on_the_batch(masked):
    imgs = [synth.image(synth.SEED_BATCH, 40 + i, w, h, nblobs=max(5, w * h // 1600)) for i, (w, h) in enumerate(KINDS)]
    want = [_run([im], masked, 0)[0] for im in imgs]          # 6 rows
    assert len(want[0]) > 300
    for n in (33, 160, 460):                                  # 12, 24 and 48 rows
        batch = [imgs[i % 4] for i in range(n)]
        for variant in (0, 1):
            got = _run(batch, masked, variant)
            for i in list(range(4)) + list(range(n - 4, n)) + [n // 2]:
                np.testing.assert_array_equal(got[i], want[i % 4], err_msg=f"image {i} of {n}, variant {variant}")
