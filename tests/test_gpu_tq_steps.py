"""The ternary codes in batches whose waves take several steps."""
import numpy as np
import pytest

from oracle import tq

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_tq import _encode, model  # noqa: E402, F401


@pytest.mark.parametrize("n,cap", [(1, 1), (3, 5), (300, 333), (900, 311)])
def test_waves_of_several_steps(model, n, cap):  # noqa: F811
    """Batches whose waves take one, three and four steps of four descriptors
    (from 65,536 descriptors on), capacities that put several images into one
    step, and counts from none to all: the codes of every descriptor below its
    image's count, and nothing else written."""
    rng = np.random.default_rng(n)
    base = rng.gamma(0.5, 1.0, (997, 128))
    base = (base / np.linalg.norm(base, axis=1, keepdims=True)).astype(np.float32)
    want = tq.encode(base, model, 100)
    counts = rng.integers(0, cap + 1, n)
    counts[0], counts[-1] = cap, cap
    pick = (np.arange(n)[:, None] * 131 + np.arange(cap)[None, :]) % len(base)
    got = _encode(model, [base[pick[i, :c]] for i, c in enumerate(counts)], counts, cap, 100)
    below = np.arange(cap)[None, :] < counts[:, None]
    np.testing.assert_array_equal(got[below], want[pick[below]])
    assert np.all(got[~below] == 0xFFFFFFFF)
