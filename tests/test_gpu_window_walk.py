"""The descriptor's and the orientation's walk over a keypoint's window:
windows from a few pixels to wider than the 64 lanes, cut by every border, on
records placed by hand, against the oracle at the same records."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_1705_09776_amd as cd  # noqa: E402
from parity import oracle_records  # noqa: E402

W, H = 197, 131


@pytest.mark.parametrize("desc_radius,ori_radius", [(6.0, 3.96), (9.7, 8.0), (12.0, 1.1)])
def test_windows_of_all_sizes_and_borders(desc_radius, ori_radius):
    # noise, so that every window has strong gradients: an element's error is
    # then that of the fixed-point shares (half of 2^-12 of a gradient each at
    # the default radius) and of the angle polynomial, far below 1e-3
    img = np.random.default_rng(7).integers(0, 256, (H, W), dtype=np.uint8)
    params = cd.default_params()
    params.desc_radius, params.ori_radius = desc_radius, ori_radius
    pipe = cd.Pipeline([(W, H)], params=params)
    pipe.upload([img])
    pipe.pyramid()
    recs = []
    for o in (0, 1):
        w, h, sc = W >> o, H >> o, float(1 << o)
        for i, s in enumerate((0.4, 0.9, 1.6, 1.93, 2.4, 3.0, 3.2)):
            for fx, fy in ((0.5, 0.5), (0.0, 0.0), (1.0, 1.0), (0.02, 0.6), (0.97, 0.31), (0.43, 0.03), (0.61, 0.98)):
                r = np.zeros(1, dtype=cd.KP_DTYPE)
                r["x"], r["y"] = (fx * (w - 1) + 0.13 * i) * sc, (fy * (h - 1) - 0.07 * i) * sc
                r["sigma"], r["theta"], r["octave"], r["p"] = s * sc, 0.9 * i + 0.1, o, 1.0
                recs.append(r)
    recs = np.concatenate(recs)
    n = len(recs)
    buf = np.zeros((1, pipe.kp_capacity), dtype=cd.KP_DTYPE)
    buf[0, :n] = recs
    dev = torch.from_numpy(buf.view(np.int32).reshape(1, pipe.kp_capacity, 12))
    pipe.d_kp.copy_(dev)
    pipe.d_count.fill_(n)
    pipe.orient()
    torch.cuda.synchronize()
    got_ori = pipe.oriented()[0]
    pipe.d_kp_ori.copy_(dev)
    pipe.d_count_ori.fill_(n)
    pipe.describe()
    torch.cuda.synchronize()
    got = pipe.descriptors()[0][:n]

    O = oracle.Oracle("f32")
    O.P.desc_radius, O.P.ori_radius = desc_radius, ori_radius
    _, flat = O.pyramid(img)
    ref = O.describe(flat, W, H, oracle_records(recs))
    # (the bar of the other descriptor tests: a pixel on the disk's edge may
    # fall either way)
    err = np.abs(got - ref).max(axis=1)
    print(f"max {err.max():.2e}, median {np.median(err):.2e}")
    assert np.mean(err <= 1e-3) >= 0.99
    ref_ori = O.orient(flat, W, H, oracle_records(recs))
    # (a peak at the 80 % bar or a tie may fall either way)
    assert abs(len(got_ori) - len(ref_ori)) <= 0.02 * n
    first = {}
    for r in got_ori:
        first.setdefault((float(r["x"]), float(r["y"]), float(r["sigma"])), r["theta"])
    hits = 0
    want = {}
    for r in ref_ori:
        want.setdefault((float(np.float32(r["x"])), float(np.float32(r["y"])), float(np.float32(r["sigma"]))), r["theta"])
    for k, t in want.items():
        d = abs(first.get(k, 1e9) - t) % (2 * np.pi)
        hits += min(d, 2 * np.pi - d) <= 1e-3
    assert hits >= 0.98 * len(want)
