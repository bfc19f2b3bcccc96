"""Images with more than the 8192 candidates that the finalisation holds: the
cut to the strongest, at counts around the limit, at counts that are no
multiple of four, and with equal responses at the threshold.

The candidates of such an image are found without the cut by gating: a centre
is examined if its cell's bit is set, so masks that split the cells between
them give the same candidates a part at a time.  From all of them the expected
lists follow by the definition of stage C and of the canonical order.  With
dedup_dlog2 = 0 stage C only removes pairs of exactly equal scale."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

HELD = 8192
W, H = 1601, 1203
CW, CH = (W + 3) // 4, (H + 3) // 4


class _Detector:
    def __init__(self, img, topk, dlog2=0.25, contrast=0.4):
        p = cd.default_params()
        p.topk, p.dedup_dlog2, p.contrast, p.mask_fmax = topk, dlog2, contrast, 1.0
        self.pipe = cd.Pipeline([(img.shape[1], img.shape[0])], params=p, kp_capacity=topk)
        self.pipe.upload([img])
        self.pipe.cnn_buffers()
        self.pipe.pyramid()

    def __call__(self, mask=None):
        if mask is not None:
            self.pipe.d_mask.copy_(torch.from_numpy(np.ascontiguousarray(mask, dtype=np.uint8).reshape(-1)))
        self.pipe.detect(mask=None if mask is None else self.pipe.d_mask)
        torch.cuda.synchronize()
        return self.pipe.keypoints()[0].copy(), self.pipe.sync_status()


def _sorted(k):
    return k[np.lexsort((k["ix"], k["iy"], k["octave"], -np.abs(k["p"])))]


def _cells(k):
    o = k["octave"]
    return np.minimum((k["iy"] << o) >> 2, CH - 1) * CW + np.minimum((k["ix"] << o) >> 2, CW - 1)


def _all_candidates(img):
    """Every candidate, a few rows of cells at a time; octaves beyond the mask's bits come with every part."""
    found, parts = _Detector(img, HELD, dlog2=0.0), []
    rows = np.arange(CH)[:, None] * np.ones((1, CW), dtype=int)
    for i in range(6):
        k, st = found(np.where((rows * 6) // CH == i, 0x3F, 0))
        assert st == cd.CDVS_OK and len(k) < HELD
        parts.append(k)
    k = np.concatenate(parts)
    _, first = np.unique(np.stack([k["octave"], k["iy"], k["ix"]]), axis=1, return_index=True)
    return _sorted(k[first])


def _stage_c(k, dlog2):
    """Of two candidates of adjacent octaves within the limits, the weaker one is out (equal: the coarser)."""
    ratio, out = np.float32(2.0 ** dlog2), np.zeros(len(k), dtype=bool)
    for o in range(8):
        a, b = np.flatnonzero(k["octave"] == o), np.flatnonzero(k["octave"] == o + 1)
        for i in a:
            d2 = (k["x"][i] - k["x"][b]) ** 2 + (k["y"][i] - k["y"][b]) ** 2
            hi, lo = np.maximum(k["sigma"][i], k["sigma"][b]), np.minimum(k["sigma"][i], k["sigma"][b])
            lim = np.float32(4.0 ** (o + 1))
            dup = (d2 <= lim) & (hi <= ratio * lo) & ((k["p"][i] > 0) == (k["p"][b] > 0))
            # (no pair so close to a limit that the order of the operations matters)
            edge = (np.abs(d2 / lim - 1) < 1e-6) & (hi <= ratio * lo * 1.001) | (np.abs(hi / (ratio * lo) - 1) < 1e-6) & (d2 <= lim * 1.001)
            assert not edge.any()
            stronger = np.abs(k["p"][b]) > np.abs(k["p"][i])
            out[i] |= bool((dup & stronger).any())
            out[b[dup & ~stronger]] = True
    return k[~out]


@pytest.fixture(scope="module")
def scene():
    img = synth.image(7, 4, W, H, nblobs=2400)
    return img, _all_candidates(img)


def test_far_more_than_it_holds(scene):
    img, cand = scene
    assert HELD + 2000 < len(cand) < W * H // 64
    for dlog2 in (0.0, 0.25):
        want = _stage_c(cand, dlog2)
        for topk in (1, 300, 1000, 4096):
            k, st = _Detector(img, topk, dlog2)()
            assert st == cd.CDVS_OK
            np.testing.assert_array_equal(k, want[:topk], err_msg=f"{dlog2} {topk}")
    # with the limit at what it holds, the weakest of them is among the kept (nothing is out with dlog2 = 0)
    if len(_stage_c(cand[:HELD], 0.0)) == HELD:
        k, st = _Detector(img, HELD, 0.0)()
        assert st == cd.CDVS_ERR_CAPACITY
        np.testing.assert_array_equal(np.abs(k["p"]), np.abs(cand["p"][:HELD]))


@pytest.mark.parametrize("count", [HELD - 1, HELD, HELD + 1, HELD + 2, HELD + 3, HELD + 255, HELD + 1025])
def test_counts_around_the_limit(scene, count):
    img, cand = scene
    cell, gated = _cells(cand), cand["octave"] < 6
    per = np.bincount(cell[gated], minlength=CW * CH)
    order = np.random.default_rng(count).permutation(np.flatnonzero(per))
    on, have = np.zeros(CW * CH, dtype=bool), int((~gated).sum())
    for c in order:   # cells until the count is met exactly
        if have + per[c] <= count:
            on[c] = True
            have += per[c]
    assert have == count
    mask = np.where(on, 0x3F, 0).reshape(CH, CW)
    left = cand[~gated | on[cell]]
    assert len(left) == count
    for dlog2 in (0.0, 0.25):
        want = _stage_c(left, dlog2)
        for topk in (300, 1000):
            k, st = _Detector(img, topk, dlog2)(mask)
            assert st == cd.CDVS_OK
            np.testing.assert_array_equal(k, want[:topk], err_msg=f"{dlog2} {topk}")
    k, st = _Detector(img, HELD, 0.0)(mask)
    want = _stage_c(left, 0.0)
    if count <= HELD:
        assert st == cd.CDVS_OK
        np.testing.assert_array_equal(k, want)
    else:   # what was dropped is at most as strong as the weakest that is left
        assert st == cd.CDVS_ERR_CAPACITY


def test_equal_responses_at_the_threshold():
    """An exact period: a few responses thousands of times each, one of them at the threshold of the cut.  Any of those
    may be held; where the limit reaches down to them the call says so."""
    y, x = np.mgrid[0:20, 0:20]
    tile = np.clip(128 + 60 * np.sin(2 * np.pi * x / 20) * np.sin(2 * np.pi * y / 20), 0, 255).astype(np.uint8)
    img = np.tile(tile, (H // 20 + 1, W // 20 + 1))[:H, :W]
    cand = _all_candidates(img)
    p = np.abs(cand["p"])
    assert HELD < len(cand) < W * H // 64 and p[HELD - 1] == p[HELD]
    for topk in (100, 1000, 5000, HELD):
        k, st = _Detector(img, topk, 0.0)()
        if p[topk - 1] > p[HELD - 1]:
            assert st == cd.CDVS_OK, topk
            np.testing.assert_array_equal(k, cand[:topk], err_msg=str(topk))
        else:
            assert st == cd.CDVS_ERR_CAPACITY, topk
            np.testing.assert_array_equal(k, _sorted(k))
            np.testing.assert_array_equal(np.abs(k["p"]), p[:topk])
