"""Selection in batches of more images than compute units: images of up to 256
records take the bitonic sort, larger ones the counting passes, side by side
in one batch; the same order as the oracle's from either, and few records cost
less than many (where every image runs the four counting passes they take 0.85
of the time of 300 records, with the few stages of the bitonic sort 0.55)."""
import os

import numpy as np
import pytest

from oracle import relevance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CAP = 1200


def _batch(n, counts):
    with np.load(os.path.join(ROOT, "paper_1705_09776_amd", "weights", "relevance_standin.npz")) as z:
        model = dict(z)
    p = cd.default_params()
    p.topk = CAP
    pipe = cd.Pipeline([(640, 480)] * n if n < 1000 else [(32, 32)] * n, params=p, kp_capacity=CAP)
    rng = np.random.default_rng(n)
    rec = np.zeros((n, CAP), dtype=cd.KP_DTYPE)
    src = rng.integers(0, CAP // 2, (n, CAP))     # many records repeat another's characteristics: ties
    row = np.arange(n)[:, None]
    for f, lo, hi in (("x", 0, 640), ("y", 0, 480), ("sigma", 1, 40), ("p", -60, 60), ("rho", 0, 14), ("p_ss", -20, 20)):
        rec[f] = rng.uniform(lo, hi, (n, CAP)).astype(np.float32)[row, src]
    rec["ix"] = np.arange(CAP)
    pipe.d_kp.copy_(torch.from_numpy(rec.view(np.int32).reshape(n, CAP, 12)))
    pipe.d_count.copy_(torch.tensor(counts, dtype=torch.int32))
    return pipe, rec, model, cd.Relevance(model)


def test_both_sorts_in_one_batch():
    edges = [0, 1, 2, 63, 127, 128, 129, 255, 256, 257, 300, 1023, 1024, 1025, CAP]
    n = 270
    counts = [edges[i % len(edges)] for i in range(n)]
    pipe, rec, model, rel = _batch(n, counts)
    for keep in (CAP, 100):
        pipe.d_kp_ori.fill_(-1)
        cd.cdvs_relevance_select(pipe.ctx, rel, pipe.d_kp, pipe.d_count, keep, pipe.d_kp_ori, pipe.d_count_ori, None)
        torch.cuda.synchronize()
        for i, got in enumerate(pipe.oriented()):
            idx, _ = relevance.select(rec[i, :counts[i]], 640, 480, model, keep)
            np.testing.assert_array_equal(got["ix"], idx, err_msg=f"image {i}, {counts[i]} records, {keep} kept")


def test_few_records_cost_less_than_many():
    pipe, _, _, rel = _batch(1024, [64] * 1024)

    def us(records):
        pipe.d_count.fill_(records)
        best = 1e9
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                cd.cdvs_relevance_select(pipe.ctx, rel, pipe.d_kp, pipe.d_count, 30, pipe.d_kp_ori, pipe.d_count_ori, None)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 50.0)
        return best

    few, many = us(64), us(300)
    assert few <= 0.7 * many, (few, many)
