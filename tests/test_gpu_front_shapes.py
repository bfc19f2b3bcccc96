"""The front end where its work split changes: factors just above 1 and at
their largest, source widths of every remainder by 4 and around the segment
limits (1272 source columns), 32- and 64-bit sums, and sources of any byte
alignment without row padding.  Every output byte equals the oracle's."""
import numpy as np
import pytest

from oracle import front as F

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

SHAPES = {"small_factors": [(641, 641), (643, 640), (645, 17), (650, 649), (17, 700)],
          "segments": [(1272, 901), (1273, 901), (1279, 1100), (1280, 701), (2544, 300), (2545, 301), (1286, 964)],
          "largest": [(8192, 210), (205, 8191), (8191, 1025), (2901, 2895), (2898, 2897)]}


@pytest.mark.parametrize("shape", list(SHAPES))
def test_shapes_and_alignments(shape):
    rng = np.random.default_rng(len(shape))
    descs, parts, off = [], [], 0
    imgs = [rng.integers(0, 256, size=(h, w)).astype(np.uint8) for w, h in SHAPES[shape]]
    imgs.append(np.full((700, 701), 255, dtype=np.uint8))
    imgs.append(np.zeros((700, 703), dtype=np.uint8))
    for i, im in enumerate(imgs):
        gap = (1, 3, 2, 0)[i % 4]      # rows of exactly the width, at odd addresses
        parts += [np.full(gap, 9, dtype=np.uint8), im.reshape(-1)]
        descs.append(cd.ImageDesc(off + gap, im.shape[1], im.shape[0], im.shape[1], 0))
        off += gap + im.size
    src = torch.from_numpy(np.concatenate(parts)).cuda()
    pipe = cd.Pipeline([cd.cdvs_front_size(im.shape[1], im.shape[0]) for im in imgs])
    pipe.d_images.fill_(7)
    pipe.front_end(src, cd.descs_to_device(descs))
    assert pipe.sync_status() == cd.CDVS_OK
    host = pipe.d_images.cpu().numpy()
    for im, d in zip(imgs, pipe.descs):
        rows = host[d.offset:d.offset + d.pitch * d.height].reshape(d.height, d.pitch)
        np.testing.assert_array_equal(rows[:, :d.width], F.front(im), err_msg=f"source {im.shape}")
        assert (rows[:, d.width:] == 7).all()      # nothing beyond the row
