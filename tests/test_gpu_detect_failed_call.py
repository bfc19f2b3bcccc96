"""A detection that fails between its launches leaves nothing behind: the
replay of a captured pass, a capture, and an eager call after it give the
keypoints of an undisturbed pass (candidate, work and active-cell counters
start at zero each time).

The failure is one that the launches report but did not cause: an error that
an unrelated HIP call of the same thread has left."""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402


def _hip():
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    return [ctypes.CDLL(p) for p in sorted(paths)]


def _failing_detect(pipe, mask):
    for lib in _hip():
        assert lib.hipSetDevice(9999) != 0   # refused, and remembered as the thread's last error
    try:
        pipe.detect(mask=mask)
    except cd.CdvsError as e:
        assert e.status == cd.CDVS_ERR_HIP
    else:
        pytest.skip("this runtime's launches do not report an older error")


@pytest.mark.parametrize("variant", ["per_strip", "persistent"])
@pytest.mark.parametrize("gated", [False, True])
def test_pass_after_a_failed_detection(variant, gated):
    imgs = list(synth.fixed_batch(synth.SEED_BATCH, 2))
    p = cd.default_params()
    p.mask_fmax = 0.5   # with every count doubled, octaves with 40% active would fall back to dense
    pipe = cd.Pipeline([(640, 480)] * len(imgs), params=p)
    pipe.upload(imgs)
    pipe.cnn_buffers()
    cd.cdvs_tune_set(pipe.ctx, cd.KERNEL_NAMES.index("detect"), ["per_strip", "persistent"].index(variant))
    mask = None
    if gated:
        rng = np.random.default_rng(8)
        bits = (rng.random((pipe.ncells, 6)) < 0.4).dot(1 << np.arange(6)).astype(np.uint8)
        pipe.d_mask.copy_(torch.from_numpy(bits))
        mask = pipe.d_mask

    def found():
        torch.cuda.synchronize()
        return [k.copy() for k in pipe.keypoints()]

    pipe.pyramid()
    pipe.detect(mask=mask)
    want = found()
    assert all(len(k) > 100 for k in want)

    def check(what):
        for a, b in zip(found(), want):
            np.testing.assert_array_equal(a, b, err_msg=what)
        assert pipe.sync_status() == cd.CDVS_OK, what

    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        pipe.detect(mask=mask)
    check("captured, not run")
    for what in ("replay", "eager", "capture"):
        _failing_detect(pipe, mask)
        pipe.d_count.zero_()
        torch.cuda.synchronize()
        if what == "replay":
            graph.replay()
        elif what == "eager":
            pipe.detect(mask=mask)
        else:   # captured after the failure, and an eager call before its first replay
            again = torch.cuda.CUDAGraph()
            with torch.cuda.graph(again, stream=side):
                pipe.detect(mask=mask)
            pipe.detect(mask=mask)
            check("eager after capture")
            again.replay()
        check(what)
        graph.replay()
        check(what + ", replayed")
    if not gated:
        pipe.run()
        pipe.capture()
        torch.cuda.synchronize()
        _failing_detect(pipe, mask)
        pipe.d_count.zero_()
        pipe.replay()
        check("the context's graph")
