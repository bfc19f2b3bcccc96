"""Contexts of many images: the time to make one grows with the number of
images, not with its square, and its tables (small ones written together,
large ones copied from where they lie) are those of the images' own contexts."""
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402


def _create_ms(n):
    p = cd.default_params()
    p.topk = 100
    descs = [cd.ImageDesc(i * 64 * 32, 32, 32, 64, 0) for i in range(n)]
    best = 1e9
    for _ in range(9):
        t = time.perf_counter()
        ctx = cd.cdvs_ctx_create(p, descs, 100)
        best = min(best, (time.perf_counter() - t) * 1e3)
        cd.cdvs_ctx_destroy(ctx)
    return best


def test_time_grows_with_the_images():
    few, many = _create_ms(512), _create_ms(4096)   # 8 times the images; 64 times where it went by the square
    assert many <= 16 * few, (few, many)


def test_tables_of_many_images():
    sizes = [(40 + 7 * (i % 11), 33 + 5 * (i % 13)) for i in range(900)] + [(640, 480), (500, 641)] * 12
    base = {s: synth.image(7, i, *s, nblobs=12) for i, s in enumerate(sorted(set(sizes)))}
    pipe = cd.Pipeline(sizes)
    pipe.upload([base[s] for s in sizes])
    pipe.run()
    torch.cuda.synchronize()
    assert pipe.sync_status() == cd.CDVS_OK
    kp, ori, desc = pipe.keypoints(), pipe.oriented(), pipe.descriptors()
    fields = [f for f in cd.KP_DTYPE.names if f != "image"]
    for i in (0, 1, 142, 511, 700, 899, 900, 901, 923):
        one = cd.Pipeline([sizes[i]])
        one.upload([base[sizes[i]]])
        one.run()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(kp[i][fields], one.keypoints()[0][fields], err_msg=str(i))
        np.testing.assert_array_equal(ori[i][fields], one.oriented()[0][fields], err_msg=str(i))
        np.testing.assert_array_equal(desc[i], one.descriptors()[0], err_msg=str(i))
