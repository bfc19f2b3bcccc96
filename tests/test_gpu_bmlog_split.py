"""The frequency-domain scale space where the scales of the blocks left over
from whole rounds are split over several workgroups: an image's planes are the
same bit for bit in batches that split them differently."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

W, H = 417, 290   # 5 x 4 blocks, then 3 x 2, 2 x 1, 1


def _planes(imgs):
    pipe = cd.Pipeline([(W, H)] * len(imgs))
    pipe.upload(imgs)
    pipe.d_pyr.fill_(float("nan"))
    cd.cdvs_pyramid_bmlog(pipe.ctx, pipe.d_images, pipe.d_pyr)
    torch.cuda.synchronize()
    return [np.concatenate([pipe.plane(i, o, k).ravel() for o in range(pipe.num_octaves(i)) for k in range(5)])
            for i in (0, len(imgs) - 1)]


# blocks of the first octaves at 256 units: 20, 6, 2 (split 5, 4, 4); 140, 42,
# 14 (1, 4, 4); 260, 78, 26 (1, 3, 4); 520, 156, 52: 8 left over from a round
# (5, 1, 4); 600, 180, 60 (2, 1, 4)
@pytest.mark.parametrize("n", [7, 13, 26, 30])
def test_split_of_scales_gives_the_same_planes(n):
    img = synth.image(synth.SEED_RAGGED, 3, W, H, nblobs=30)
    one = _planes([img])[0]
    assert np.isfinite(one).all()
    for p in _planes([img] * n):
        np.testing.assert_array_equal(p.view(np.uint32), one.view(np.uint32))
