"""The relevance selection where it sorts in its two ways."""
import numpy as np
import pytest

from oracle import relevance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402
from test_gpu_relevance import CAP, _pipe, model  # noqa: E402, F401


@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 255, 1000, 1023, 1024, 1025, 2049])
def test_sorts_of_either_kind(model, n):  # noqa: F811
    """Up to 1024 records are sorted by counting passes, more by the bitonic
    sort: the same order, ties (about half the records repeat another's
    characteristics) in input order."""
    rng = np.random.default_rng(n)
    pipe = _pipe([(640, 480)])
    rec = np.zeros((1, CAP), dtype=cd.KP_DTYPE)
    src = rng.integers(0, max(1, n // 2 + 1), n)
    for f, lo, hi in (("x", 0, 640), ("y", 0, 480), ("sigma", 1, 40), ("p", -60, 60), ("rho", 0, 14), ("p_ss", -20, 20)):
        rec[f][0, :n] = rng.uniform(lo, hi, n).astype(np.float32)[src] if n else 0
    rec["ix"][0, :n] = np.arange(n)
    pipe.d_kp.copy_(torch.from_numpy(rec.view(np.int32).reshape(1, CAP, 12)))
    pipe.d_count.fill_(n)
    score = torch.zeros((1, CAP), dtype=torch.float32, device="cuda")
    for keep in (CAP, 300):
        cd.cdvs_relevance_select(pipe.ctx, cd.Relevance(model), pipe.d_kp, pipe.d_count, keep, pipe.d_kp_ori,
                                 pipe.d_count_ori, score)
        torch.cuda.synchronize()
        idx, r = relevance.select(rec[0, :n], 640, 480, model, keep)
        got = pipe.oriented()[0]
        assert len(got) == len(idx) == min(n, keep)
        np.testing.assert_array_equal(got["ix"], idx)
        np.testing.assert_array_equal(score.cpu().numpy()[0, :len(idx)].view(np.uint32), r[idx].view(np.uint32))
