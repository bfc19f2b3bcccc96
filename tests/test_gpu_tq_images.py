"""Ternary coding where workgroups go by image: capacities around four
workgroups (of 16 descriptors each, or 64 in large batches), a last workgroup that the capacity fills partly, counts at workgroup borders,
none and all; and batches with little in use are not slower than their used
descriptors ask for."""
import numpy as np
import pytest

from oracle import tq

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402
from test_gpu_tq import _encode, model  # noqa: E402,F401


@pytest.mark.parametrize("n,cap", [(5, 63), (5, 64), (5, 65), (3, 1000), (130, 255), (130, 256), (300, 257), (300, 320), (9, 8192)])
def test_counts_at_workgroup_borders(model, n, cap):  # noqa: F811
    rng = np.random.default_rng(cap)
    base = rng.gamma(0.5, 1.0, (499, 128))
    base = (base / np.linalg.norm(base, axis=1, keepdims=True)).astype(np.float32)
    want = tq.encode(base, model, 128)
    edges = [0, 1, 15, 16, 17, 63, 64, 65, cap - 1, cap]
    counts = np.array([min(edges[i % len(edges)], cap) for i in range(n)])
    pick = (np.arange(n)[:, None] * 131 + np.arange(cap)[None, :]) % len(base)
    got = _encode(model, [base[pick[i, :c]] for i, c in enumerate(counts)], counts, cap, 128)
    below = np.arange(cap)[None, :] < counts[:, None]
    np.testing.assert_array_equal(got[below], want[pick[below]])
    assert np.all(got[~below] == 0xFFFFFFFF)


def test_few_descriptors_of_a_large_capacity(model):  # noqa: F811
    """128 images with 100 descriptors each take no longer at capacity 4096 than at capacity 128 (the same work; twice that is allowed)."""
    def us(cap):
        p = cd.default_params()
        p.topk = cap
        pipe = cd.Pipeline([(32, 32)] * 128, params=p, kp_capacity=cap)
        t = cd.Tq(model)
        desc = torch.rand((128, cap, 128), device="cuda")
        count = torch.full((128,), 100, dtype=torch.int32, device="cuda")
        codes = torch.zeros((128, cap, 8), dtype=torch.int32, device="cuda")
        best = 1e9
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                cd.cdvs_encode(pipe.ctx, t, 128, desc, count, codes)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 50.0)
        return best

    small, large = us(128), us(4096)
    assert large <= 2.0 * small, (small, large)
