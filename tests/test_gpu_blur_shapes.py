"""The scale space's tile shapes on batches with enough tiles that each shape
is really taken (octaves of fewer than 256 tiles take the small one): every
shape, and every image alone, gives the same planes bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

SIZES = [(640, 480), (641, 479), (333, 217), (1279, 961), (97, 61), (480, 640), (1000, 750), (129, 33)]


def _planes(pipe, i):
    return [pipe.plane(i, o, k) for o in range(pipe.num_octaves(i)) for k in range(5)]


def test_shapes_and_single_images_give_the_same_planes():
    imgs = [synth.image(synth.SEED_RAGGED, i, w, h, nblobs=30) for i, (w, h) in enumerate(SIZES)]
    pipe = cd.Pipeline(SIZES * 3)     # 3 to 12 times 256 tiles in the first octave, around 256 in the next two
    pipe.upload(imgs * 3)
    want = None
    for v in range(cd.TUNE_VARIANTS):
        cd.cdvs_tune_set(pipe.ctx, cd.KERNEL_SCALES, v)
        pipe.d_pyr.fill_(float("nan"))
        pipe.pyramid()
        torch.cuda.synchronize()
        got = pipe.d_pyr.cpu().numpy().view(np.uint32)
        want = got.copy() if want is None else want
        np.testing.assert_array_equal(got, want, err_msg=f"variant {v}")
    for i, im in enumerate(imgs):
        one = cd.Pipeline([SIZES[i]])
        one.upload([im])
        one.pyramid()
        torch.cuda.synchronize()
        for j in (i, i + 16):
            for a, b in zip(_planes(one, 0), _planes(pipe, j)):
                np.testing.assert_array_equal(a.view(np.uint32), b.view(np.uint32))
