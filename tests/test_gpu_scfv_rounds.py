"""SCFV of small batches in rounds of tile blocks: images are packed into the
rounds by the descriptors they have, so the same bits have to come out
whatever shares a round with an image, and a batch must not take longer than
one of 81 images (one workgroup per image, whose time does not depend on
their number)."""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MODEL = os.path.join(ROOT, "paper_1705_09776_amd", "weights", "scfv_standin.npz")
WHOLE = 81   # images from which every image has one workgroup


class _Batch:
    def __init__(self, desc, count, cap):
        p = cd.default_params()
        p.topk = cap
        self.pipe = cd.Pipeline([(32, 32)] * desc.shape[0], params=p, kp_capacity=cap)
        with np.load(MODEL) as z:
            self.s = cd.Scfv(dict(z), desc.shape[0])
        self.args = desc.contiguous(), torch.tensor(count, dtype=torch.int32, device="cuda")

    def run(self):
        cd.cdvs_scfv(self.pipe.ctx, self.s, *self.args)

    def bits(self):
        self.run()
        torch.cuda.synchronize()
        return [t.cpu().numpy().view(np.uint32) for t in (self.s.gm, self.s.gv, self.s.delta, self.s.order, self.s.bits)]

    def us(self):
        best = 1e9
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                self.run()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 250.0)
        return best


def _descriptors(n, cap):
    g = torch.Generator(device="cuda").manual_seed(cap)
    d = torch.rand((n, cap, 128), generator=g, device="cuda").pow_(3.0)
    return d / d.norm(dim=2, keepdim=True)


# 448 blocks of 32 descriptors to a round
COUNTS = {
    "full_rounds_then_none": (1000, [1000] * 14 + [0, 1000, 0]),             # 14 x 32 blocks, images without descriptors after
    "one_block_short": (1000, [1000] * 13 + [992, 1000, 1] + [1000] * 12),   # 31 blocks, then one of 32 that no longer fits
    "few_of_many": (4096, [5, 33, 0, 4096, 64, 1, 4096, 4096, 31]),          # 128 blocks each at most, three to a round
    "one_to_a_round": (8192, [8192, 1, 8192, 0, 8000]),                      # 256 blocks each at most
    "more_than_a_wave": (33, [33, 0, 1, 32] * 20),                           # 80 images
}


@pytest.mark.parametrize("which", list(COUNTS))
def test_rounds_equal_one_workgroup_per_image(which):
    cap, count = COUNTS[which]
    n = len(count)
    d = _descriptors(n, cap)
    rest = torch.zeros((WHOLE - n, cap, 128), device="cuda")
    want = _Batch(torch.cat([d, rest]), count + [0] * (WHOLE - n), cap).bits()
    batch = _Batch(d, count, cap)
    for again in range(2):
        got = batch.bits()
        for name, a, b in zip(("gm", "gv", "delta", "order", "bits"), got, want):
            np.testing.assert_array_equal(a, b[:n], err_msg=f"{name}, call {again}")


@pytest.mark.parametrize("cap,n,used", [(8192, 40, 300), (4096, 40, 300), (1000, 80, 300), (1000, 28, 300), (8192, 6, 2730)])
def test_no_slower_than_one_workgroup_per_image(cap, n, used):
    d = _descriptors(n, cap)
    small = _Batch(d, [used] * n, cap)
    whole = _Batch(torch.cat([d, torch.zeros((WHOLE - n, cap, 128), device="cuda")]), [used] * n + [0] * (WHOLE - n), cap)
    t = [(small.us(), whole.us()) for _ in range(2)][-1]
    assert t[0] <= 1.25 * t[1], t
