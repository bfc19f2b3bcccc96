"""A context's device memory: its tables and the scratch of the call that
needs most of it (the calls share the region), as include/cdvs.h states it;
and calls that follow one another in that region leave each other's results
alone."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("n,w,h,cap", [(1, 640, 480, 1000), (32, 640, 480, 1000), (256, 640, 480, 1000), (1, 4000, 3000, 2000)])
def test_scratch_is_the_largest_call_s(n, w, h, cap):
    p = cd.default_params()
    p.topk = cap
    torch.cuda.synchronize()
    pitch = (w + 63) // 64 * 64
    descs = [cd.ImageDesc(i * pitch * h, w, h, pitch, 0) for i in range(n)]
    cd.cdvs_ctx_destroy(cd.cdvs_ctx_create(p, descs, cap))   # (the first one loads the library's code too)
    count, free, ctxs = 8, [], []
    free.append(torch.cuda.mem_get_info()[0])
    for _ in range(count):
        ctxs.append(cd.cdvs_ctx_create(p, descs, cap))
    free.append(torch.cuda.mem_get_info()[0])
    for c in ctxs:
        cd.cdvs_ctx_destroy(c)
    used = (free[0] - free[1]) / count
    candidates = -(-max(8192, w * h // 64) // 256) * 256
    detect = n * candidates * (48 if candidates <= 8192 else 52) + (n * 8192 * 4 if candidates > 8192 else 0)
    orient = n * cap * 196
    blocks = n * -(-w // 128) * -(-h // 64)
    backward = 512 * 416 + 4 * 9280 * min(blocks, 512)
    scfv = min(448, n * -(-cap // 32)) * 74752 if n <= 56 else 0
    tables = 2 ** 22 + n * 2 ** 15   # strips, tile owners, images; whole pages
    assert used <= max(detect, orient, backward, scfv) + tables, used / 2 ** 20


def test_calls_share_the_scratch():
    sizes = [(640, 480), (500, 641), (97, 61)]
    imgs = [synth.image(synth.SEED_TRAIN, i, w, h, nblobs=max(4, w * h // 1500)) for i, (w, h) in enumerate(sizes)]
    with np.load(os.path.join(ROOT, "paper_1705_09776_amd", "weights", "scfv_standin.npz")) as z:
        model = dict(z)
    g = torch.Generator(device="cuda").manual_seed(3)
    params = torch.randn(cd.CNN_PARAMS, generator=g, device="cuda") * 0.05

    def make():
        pipe = cd.Pipeline(sizes)
        pipe.upload(imgs)
        pipe.cnn_buffers()
        return pipe

    state = {}

    def detect(pipe):
        pipe.pyramid()
        pipe.detect()
        return [pipe.d_count]

    def orient(pipe):
        pipe.orient()
        pipe.describe()
        return [pipe.d_kp, pipe.d_count_ori]

    def backward(pipe):
        pipe.cnn_forward(params, tau=None, logits=True)
        labels = state.setdefault("labels", torch.randint(0, 64, (pipe.ncells,), generator=g, device="cuda", dtype=torch.int32))
        work = torch.empty(2 * pipe.ncells * cd.CNN_CHANNELS, dtype=torch.int16, device="cuda")
        grad, loss = torch.empty(cd.CNN_PARAMS, device="cuda"), torch.empty(1, device="cuda")
        cd.cdvs_cnn_backward(pipe.ctx, pipe.d_images, params, pipe.d_acts, pipe.d_logits, labels,
                             torch.ones(6, device="cuda"), work, grad, loss)
        return [grad, loss]

    def aggregate(pipe):
        s = cd.Scfv(model, len(sizes))
        cd.cdvs_scfv(pipe.ctx, s, pipe.d_desc, pipe.d_count_ori)
        return [s.gm, s.gv, s.delta, s.order, s.bits]

    def run(pipe, order):
        out = {f.__name__: [t.clone() for t in f(pipe)] for f in order}   # no wait in between
        torch.cuda.synchronize()
        return out

    want = run(make(), [detect, orient, aggregate, backward])
    pipe = make()
    for order in ([detect, backward, orient, aggregate], [backward, detect, orient, backward, aggregate, detect],
                  [aggregate, detect, orient, aggregate, backward]):
        got = run(pipe, order)
        for name, ts in got.items():
            for a, b in zip(ts, want[name]):
                assert torch.equal(a.view(torch.int32), b.view(torch.int32)), (name, [f.__name__ for f in order])
