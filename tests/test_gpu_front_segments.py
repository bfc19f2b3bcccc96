"""The front end at the source widths where the number of column segments
changes.  A segment's source columns have to fit 1024, less eight for
alignment and ends, so an output of 640 columns takes one segment up to 1016
source columns, two up to 2032, three up to 3048, and so on; beside those
widths a segment's columns fill what is staged of them as far as they ever do.
Every output byte equals the oracle's."""
import numpy as np
import pytest

from oracle import front as F

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402


@pytest.mark.parametrize("limit", [1016, 2032, 3048, 4064, 8128])
def test_widths_around_a_segment_limit(limit):
    rng = np.random.default_rng(limit)
    sizes = [(w, h) for w in range(limit - 5, limit + 7) for h in (limit // 36, limit // 9)]   # outputs of 18 rows and more
    sizes += [(211, limit), (211, limit + 1)]            # an output that is 640 rows high and few columns wide
    imgs = [rng.integers(0, 256, size=(h, w)).astype(np.uint8) for w, h in sizes]
    descs, parts, off = [], [], 0
    for i, im in enumerate(imgs):
        gap = i % 4      # rows of exactly the width, at any byte
        parts += [np.full(gap, 9, dtype=np.uint8), im.reshape(-1)]
        descs.append(cd.ImageDesc(off + gap, im.shape[1], im.shape[0], im.shape[1], 0))
        off += gap + im.size
    src = torch.from_numpy(np.concatenate(parts)).cuda()
    pipe = cd.Pipeline([cd.cdvs_front_size(w, h) for w, h in sizes])
    pipe.d_images.fill_(7)
    pipe.front_end(src, cd.descs_to_device(descs))
    assert pipe.sync_status() == cd.CDVS_OK
    host = pipe.d_images.cpu().numpy()
    for im, d in zip(imgs, pipe.descs):
        rows = host[d.offset:d.offset + d.pitch * d.height].reshape(d.height, d.pitch)
        np.testing.assert_array_equal(rows[:, :d.width], F.front(im), err_msg=f"source {im.shape}")
        assert (rows[:, d.width:] == 7).all()
