"""Stage C and the canonical order where the finalisation changes its way:
images smaller than a cell, few and many candidates, responses that are all
alike (a period lattice: bins of the counting sort overflow and the sort in
full takes over), more candidates than it holds, and every kind of limit.

With the limit at the capacity, the output is checked against its definition
alone: in canonical order, and no two of adjacent octaves closer than the
duplicate limits.  Any smaller limit must give the same list's beginning."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402


def _lattice(w, h, period):
    y, x = np.mgrid[0:h, 0:w]
    return np.clip(128 + 60 * np.sin(2 * np.pi * x / period) * np.sin(2 * np.pi * y / period), 0, 255).astype(np.uint8)


IMAGES = {
    "tiny": lambda: synth.image(7, 2, 40, 36, nblobs=6),
    "narrow": lambda: synth.image(7, 3, 1500, 33, nblobs=60),
    "scene": lambda: synth.image(synth.SEED_BATCH, 9, 640, 480),
    "lattice": lambda: _lattice(500, 400, 20),
    "flat": lambda: np.full((64, 64), 90, dtype=np.uint8),
    "large": lambda: synth.image(7, 4, 1601, 1203, nblobs=900),
}


def _keypoints(img, topk):
    p = cd.default_params()
    p.topk = topk
    pipe = cd.Pipeline([(img.shape[1], img.shape[0])], params=p, kp_capacity=max(topk, 1))
    pipe.upload([img])
    for _ in range(2):
        pipe.pyramid()
        pipe.detect()
    torch.cuda.synchronize()
    return pipe.keypoints()[0], pipe.sync_status()


@pytest.mark.parametrize("name", list(IMAGES))
def test_canonical_and_free_of_duplicates(name):
    img = IMAGES[name]()
    k, st = _keypoints(img, 8192)
    order = np.lexsort((k["ix"], k["iy"], k["octave"], -np.abs(k["p"])))
    np.testing.assert_array_equal(order, np.arange(len(k)))
    ratio = np.float32(2.0 ** 0.25)
    for o in range(15):
        a, b = k[k["octave"] == o], k[k["octave"] == o + 1]
        if not len(a) or not len(b):
            continue
        dx, dy = a["x"][:, None] - b["x"][None], a["y"][:, None] - b["y"][None]
        s = np.stack(np.broadcast_arrays(a["sigma"][:, None], b["sigma"][None]))
        near = dx * dx + dy * dy <= (2.0 ** (o + 1)) ** 2 * (1 - 1e-6)
        close = s.max(0) <= ratio * s.min(0) * np.float32(1 - 1e-6)
        same = (a["p"][:, None] > 0) == (b["p"][None] > 0)
        assert not (near & close & same).any()
    for topk in (1, 7, 300, 1000):
        short, _ = _keypoints(img, topk)
        np.testing.assert_array_equal(short, k[:topk])
    assert st == cd.CDVS_OK or len(k) == 8192
    if name == "flat":
        assert len(k) == 0
