"""Timed cases of the library: the calls that programs make, over the sizes they make them at.

A case is a dict of plain values; its "kind" is the call:

  extract   keypoints and descriptors of a batch (pyramid, detection, orientation, description)
  gated     the same with detection gated by the learned mask
  stream    many batches with the results handed to the host while the next batch runs
  train     one training step of the mask network: labels, forward, backward, Adam
  scfv      global aggregation of each image's descriptors
  compress  keypoint selection by relevance and ternary coding of the descriptors
  front     larger images brought down to a longer side of 640
  bmlog     the block frequency-domain scale space

listed() names twelve, draw() gives others of the same ranges, prepare() makes the inputs on the GPU from a
seed, run() is one pass, work() what a pass cannot do without, exact() its results in 64 bits.
"""
import math
import os
import random

import numpy as np
import torch

import paper_1705_09776_amd as cd
from paper_1705_09776_amd import surrogate

WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(cd.__file__)), "weights")
ASPECTS = ((4, 3), (3, 2), (16, 9), (1, 1), (3, 4))   # of the ragged batches
BUDGET = 255 * 640 * 480                               # base pixels of the largest drawn case


def listed():
    return [
        # one query image, the lowest latency there is: the captured pass replayed
        dict(name="extract-1x640x480", kind="extract", n=1, w=640, h=480, ragged=False, topk=1000, contrast=1.5, graph=True),
        # the headline workload: a database batch, captured once and replayed
        dict(name="extract-256x640x480", kind="extract", n=256, w=640, h=480, ragged=False, topk=1000, contrast=1.5, graph=True),
        # photographs of mixed aspect ratio, already brought down to 640, called eagerly
        dict(name="extract-48-ragged", kind="extract", n=48, w=640, h=640, ragged=True, topk=1000, contrast=1.5, graph=False),
        # one photograph at full resolution: more candidates than the final stage holds
        dict(name="extract-1x4000x3000", kind="extract", n=1, w=4000, h=3000, ragged=False, topk=1000, contrast=1.5, graph=False),
        # the gated pass as one graph, at the sparse keypoint setting its weights were trained for
        dict(name="gated-128x640x480", kind="gated", n=128, w=640, h=480, ragged=False, topk=1000, contrast=4.0, graph=True),
        # the high-resolution stream: gated batches, keypoints and descriptors handed to the host
        dict(name="stream-4x16x1280x960", kind="stream", n=16, chunks=4, w=1280, h=960, topk=1000),
        # one step of the mask network's training at its own batch size
        dict(name="train-32x640x480", kind="train", n=32, w=640, h=480),
        # the query side of aggregation: one image's descriptors
        dict(name="scfv-1", kind="scfv", n=1, cap=1000, form="context"),
        # the database side: a batch of images
        dict(name="scfv-256", kind="scfv", n=256, cap=1000, form="context"),
        # 300 keypoints selected of every image's, and every descriptor coded in full
        dict(name="compress-256", kind="compress", n=256, cap=1000, keep=300, elements=128),
        # camera images of several sizes brought down to 640
        dict(name="front-64-mixed", kind="front", n=64, w=2048, h=1536, ragged=True),
        # the frequency-domain scale space that the spatial one is compared with
        dict(name="bmlog-32x640x480", kind="bmlog", n=32, w=640, h=480),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("extract", "extract", "extract", "gated", "gated", "stream", "train", "scfv", "scfv", "compress",
                       "front", "bmlog"))
    if kind in ("extract", "gated"):
        ragged = rng.random() < 0.3
        if ragged:
            w = h = _log(rng, 160, 1280)
        elif rng.random() < 0.4:
            w, h = rng.choice(((640, 480), (480, 640), (640, 360), (320, 240), (1280, 960)))
        else:
            w, h = _log(rng, 48, 4000), _log(rng, 48, 3000)
        n = _log(rng, 1, max(1, min(256, BUDGET // (w * h))))
        return dict(kind=kind, n=n, w=w, h=h, ragged=ragged, topk=rng.choice((300, 1000, 1000, 2000)),
                    contrast=rng.choice((1.5, 4.0)), graph=rng.random() < 0.5)
    if kind == "stream":
        w, h = rng.choice(((640, 480), (1280, 960), (1023, 767)))
        chunks = rng.randint(2, 6)
        return dict(kind=kind, n=_log(rng, 2, min(32, BUDGET // (w * h * chunks))), chunks=chunks, w=w, h=h, topk=1000)
    if kind == "train":
        w, h = rng.choice(((640, 480), (1280, 960), (333, 250), (500, 641)))
        return dict(kind=kind, n=_log(rng, 1, max(1, 32 * 640 * 480 // (w * h))), w=w, h=h)
    if kind == "scfv":
        return dict(kind=kind, n=_log(rng, 1, 250), cap=_log(rng, 40, 1000), form=rng.choice(("context", "context", "static")))
    if kind == "compress":
        return dict(kind=kind, n=_log(rng, 1, 250), cap=_log(rng, 100, 1000), keep=rng.choice((100, 300, 650)),
                    elements=rng.choice((128, 100, 64, 20)))
    if kind == "front":
        if rng.random() < 0.5:
            w, h = rng.choice(((1280, 960), (1920, 1080), (800, 600), (3264, 2448)))
            ragged = False
        else:
            w, h = _log(rng, 641, 4000), _log(rng, 400, 3000)
            ragged = rng.random() < 0.5
        return dict(kind=kind, n=_log(rng, 1, max(1, min(128, BUDGET // (2 * w * h)))), w=w, h=h, ragged=ragged)
    w, h = rng.choice(((640, 480), (333, 222), (1280, 960), (97, 61)))
    return dict(kind="bmlog", n=_log(rng, 1, max(1, min(64, 32 * 640 * 480 // (w * h)))), w=w, h=h)


# ---------------------------------------------------------------------------
# Inputs

def _sizes(case):
    """(width, height) of every image: the case's own, or mixed aspect ratios within its w x h."""
    if not case.get("ragged"):
        return [(case["w"], case["h"])] * case["n"]
    rng = random.Random(case["n"] * 7919 + case["w"])
    out = []
    for _ in range(case["n"]):
        a, b = rng.choice(ASPECTS)
        s = min(case["w"] / a, case["h"] / b)
        if case["kind"] == "front":
            s *= rng.uniform(0.55, 1.0)   # a camera's sizes, most of them no multiple of 640
        out.append((max(48, int(a * s)), max(48, int(b * s))))
    return out


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _scenes(n, w, h, g):
    """n u8 images: a ramp, Gaussian blobs and pixel noise (the recipe of the repository's generator, drawn on the GPU)."""
    blobs = int(min(1200, max(8, 200 * w * h / (640 * 480))))
    smax = 40.0 if max(w, h) > 640 else 20.0
    u = torch.rand((4, n, blobs, 1), generator=g, device="cuda")
    s = 2.0 + (smax - 2.0) * u[2]
    x = torch.arange(w, device="cuda", dtype=torch.float32)
    y = torch.arange(h, device="cuda", dtype=torch.float32)
    ax = torch.exp(-((x - u[0] * w) / s).square() * 0.5)
    ay = torch.exp(-((y - u[1] * h) / s).square() * 0.5) * (160.0 * u[3] - 80.0)
    img = (60.0 + 120.0 * x / max(1, w - 1)).expand(n, h, w).contiguous()
    for b in range(blobs):
        img.addcmul_(ay[:, b, :, None], ax[:, b, None, :])
    img += torch.rand((n, h, w), generator=g, device="cuda") * 16.0 - 8.0
    return img.round_().clamp_(0, 255).to(torch.uint8)


def _fill(dst, descs, img):
    """Images (cut from the canvases' top left) into a packed buffer of the given layout."""
    d0 = descs[0]
    if all((d.width, d.height, d.pitch) == (d0.width, d0.height, d0.pitch) for d in descs):
        dst.view(len(descs), d0.height, d0.pitch)[:, :, :d0.width] = img
        return
    for d, im in zip(descs, img):
        dst[d.offset:d.offset + d.pitch * d.height].view(d.height, d.pitch)[:, :d.width] = im[:d.height, :d.width]


def _pipeline(case, sizes, topk):
    p = cd.default_params()
    p.topk = topk
    p.contrast = case.get("contrast", 1.5)
    pipe = cd.Pipeline(sizes, params=p, kp_capacity=topk)
    pipe.d_pyr.zero_()   # (rows are padded: what lies between them is then the same in every run)
    return pipe


def _mask_weights(case):
    """The trained mask network for the image size and contrast, and the threshold stored with it."""
    name, tau = (("surrogate_640x480_t4", 0.02) if case.get("contrast") == 4.0
                 else ("surrogate_640x480", 0.1) if case["w"] <= 640 else ("surrogate_1280x960", 0.02))
    p = np.load(os.path.join(WEIGHTS, name + ".npz"))["params"]
    return torch.from_numpy(np.ascontiguousarray(p, dtype=np.float32)).cuda(), tau


def _model(name):
    with np.load(os.path.join(WEIGHTS, name + ".npz")) as z:
        return {k: z[k] for k in z.files}


def _counts(n, cap, g):
    return (cap - (torch.rand(n, generator=g, device="cuda") * 0.3 * cap).to(torch.int32)).to(torch.int32)


def _descriptors(n, cap, g):
    """Non-negative unit descriptors spread as the aggregation model says (its mixture, brought back to 128 dimensions)."""
    m = {k: torch.from_numpy(np.asarray(v, dtype=np.float32)).cuda() for k, v in _model("scfv_standin").items()}
    i = torch.multinomial(m["weights"], n * cap, replacement=True, generator=g)
    x = m["means"][i] + m["variances"][i].sqrt() * torch.randn((n * cap, 32), generator=g, device="cuda")
    d = m["pca_mean"] + x @ m["pca_matrix"] + 0.02 * torch.randn((n * cap, 128), generator=g, device="cuda")
    d = d.clamp_(0.0, 0.4)
    return (d / d.norm(dim=1, keepdim=True).clamp_min(1e-6)).view(n, cap, 128).contiguous()


def _records(n, cap, w, h, octaves, g):
    """Keypoint records as the detector leaves them, spread over the image and the octaves."""
    r = lambda *s: torch.rand(s, generator=g, device="cuda")   # noqa: E731
    o = (r(n, cap).pow(2.0) * octaves).to(torch.int32).clamp_(0, octaves - 1)
    scale = torch.pow(2.0, o.float())
    kp = torch.zeros((n, cap, 12), dtype=torch.float32, device="cuda")
    kp[..., 0] = r(n, cap) * (w - 1)
    kp[..., 1] = r(n, cap) * (h - 1)
    kp[..., 2] = 1.6 * torch.pow(2.0, r(n, cap)) * scale
    kp[..., 3] = (1.5 + 40.0 * r(n, cap).pow(3.0)) * torch.sign(r(n, cap) - 0.5)
    kp[..., 5] = 4.0 + 8.1 * r(n, cap).pow(2.0)
    kp[..., 6] = torch.randn((n, cap), generator=g, device="cuda") * 3.0
    rec = kp.view(torch.int32)
    rec[..., 8] = torch.arange(n, device="cuda", dtype=torch.int32)[:, None]
    rec[..., 9] = o
    rec[..., 10] = (kp[..., 0] / scale).to(torch.int32)
    rec[..., 11] = (kp[..., 1] / scale).to(torch.int32)
    return rec


class _Consumer:
    """What the host does with a chunk: it keeps the records that count, as an encoder's next stage would."""

    def __init__(self, chunks, n, cap):
        self.count = np.zeros((chunks, n), dtype=np.int32)
        self.kp = np.zeros((chunks, n, cap, 12), dtype=np.float32)
        self.desc = np.zeros((chunks, n, cap, 128), dtype=np.float32)
        self.call = cd.CHUNK_CONSUMER(self.take)

    def take(self, user, chunk, n, cap, counts, kps, descs):
        import ctypes
        view = lambda p, c, s: np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(c)), shape=s)   # noqa: E731
        self.count[chunk] = view(counts, ctypes.c_int32, (n,))
        kp, desc = view(kps, ctypes.c_float, (n, cap, 12)), view(descs, ctypes.c_float, (n, cap, 128))
        for i, m in enumerate(self.count[chunk]):
            self.kp[chunk, i, :m] = kp[i, :m]
            self.desc[chunk, i, :m] = desc[i, :m]
        return 0


# ---------------------------------------------------------------------------
# One pass

def prepare(case, seed):
    g, kind = _generator(seed), case["kind"]
    st = dict(case=case, kind=kind)
    if kind in ("extract", "gated", "bmlog"):
        sizes = _sizes(case)
        pipe = st["pipe"] = _pipeline(case, sizes, case.get("topk", 1000))
        _fill(pipe.d_images, pipe.descs, _scenes(case["n"], max(s[0] for s in sizes), max(s[1] for s in sizes), g))
        if kind == "gated":
            st["params"], st["tau"] = _mask_weights(case)
            if case["graph"]:
                pipe.capture_gated(st["params"], st["tau"])
            else:
                pipe.cnn_buffers()
        elif kind == "extract" and case["graph"]:
            pipe.capture()
    elif kind == "stream":
        pipe = st["pipe"] = _pipeline(case, [(case["w"], case["h"])] * case["n"], case["topk"])
        st["params"], st["tau"] = _mask_weights(case)
        pipe.cnn_buffers()
        st["images"] = torch.zeros(case["chunks"] * pipe.image_bytes, dtype=torch.uint8, device="cuda")
        for c in range(case["chunks"]):
            _fill(st["images"][c * pipe.image_bytes:(c + 1) * pipe.image_bytes], pipe.descs,
                  _scenes(case["n"], case["w"], case["h"], g))
        st["host"] = _Consumer(case["chunks"], case["n"], case["topk"])
    elif kind == "train":
        n, w, h = case["n"], case["w"], case["h"]
        pipe = st["pipe"] = _pipeline(case, [(w, h)] * n, 1000)
        pipe.cnn_buffers()
        _fill(pipe.d_images, pipe.descs, _scenes(n, w, h, g))
        st["octaves"] = min(pipe.num_octaves(0), cd.CNN_HEADS)
        st["kp"], st["count"] = _records(n, 1000, w, h, st["octaves"], g), _counts(n, 1000, g)
        st["params"] = torch.from_numpy(surrogate.init_params(int(seed) % (1 << 31))).cuda()
        for k in ("m", "v", "grad"):
            st[k] = torch.zeros(cd.CNN_PARAMS, dtype=torch.float32, device="cuda")
        st["loss"] = torch.zeros(1, dtype=torch.float32, device="cuda")
        st["pos_weight"] = torch.tensor([10.0, 20.0, 30.0, 40.0, 50.0, 50.0], device="cuda")
        st["labels"] = torch.zeros(pipe.ncells, dtype=torch.int32, device="cuda")
        st["work"] = torch.zeros(2 * pipe.ncells * cd.CNN_CHANNELS, dtype=torch.int16, device="cuda")
        st["step"] = 0
    elif kind == "scfv":
        n, cap = case["n"], case["cap"]
        st["desc"], st["count"] = _descriptors(n, cap, g), _counts(n, cap, g)
        st["scfv"] = cd.Scfv(_model("scfv_standin"), n)
        if case["form"] == "context":
            p = cd.default_params()
            p.topk = cap
            st["pipe"] = cd.Pipeline([(64, 48)] * n, params=p, kp_capacity=cap)
    elif kind == "compress":
        n, cap = case["n"], case["cap"]
        p = cd.default_params()
        p.topk = cap
        st["pipe"] = cd.Pipeline([(640, 480)] * n, params=p, kp_capacity=cap)
        st["kp"], st["count"] = _records(n, cap, 640, 480, 5, g), _counts(n, cap, g)
        st["desc"] = _descriptors(n, cap, g)
        st["rel"], st["tq"] = cd.Relevance(_model("relevance_standin")), cd.Tq(_model("tq_standin"))
        st["kp_out"] = torch.zeros_like(st["kp"])
        st["count_out"] = torch.zeros_like(st["count"])
        st["score"] = torch.zeros((n, cap), dtype=torch.float32, device="cuda")
        st["codes"] = torch.zeros((n, cap, cd.TQ_WORDS), dtype=torch.int32, device="cuda")
    elif kind == "front":
        sizes = _sizes(case)
        descs, off = [], 0
        for w, h in sizes:
            descs.append(cd.ImageDesc(off, w, h, (w + 63) // 64 * 64, 0))
            off += descs[-1].pitch * h
        st["src"], st["descs"] = torch.zeros(off, dtype=torch.uint8, device="cuda"), cd.descs_to_device(descs)
        _fill(st["src"], descs, _scenes(case["n"], max(s[0] for s in sizes), max(s[1] for s in sizes), g))
        st["pipe"] = cd.Pipeline([cd.cdvs_front_size(w, h) for w, h in sizes])
    return st


def _records_out(kp):
    """A record buffer's computed fields and its whole ones."""
    return kp.view(torch.float32)[..., :8], kp[..., 8:]


def run(st):
    kind, case, pipe = st["kind"], st["case"], st.get("pipe")
    if kind in ("extract", "gated"):
        if case["graph"]:
            pipe.replay()
        elif kind == "gated":
            pipe.run_gated(st["params"], st["tau"])
        else:
            pipe.run()
        f, i = _records_out(pipe.d_kp)
        fo, io = _records_out(pipe.d_kp_ori)
        out = dict(count=pipe.d_count, kp=f, kp_at=i, count_ori=pipe.d_count_ori, kp_ori=fo, kp_ori_at=io, desc=pipe.d_desc)
        if kind == "gated":
            out["mask"] = pipe.d_mask
        return out
    if kind == "stream":
        host = st["host"]
        pipe.stream(st["images"], case["chunks"], params=st["params"], tau=st["tau"], consumer=host.call)
        return dict(count=host.count, kp=host.kp[..., :8], kp_at=host.kp.view(np.int32)[..., 8:], desc=host.desc)
    if kind == "train":
        st["step"] += 1
        cd.cdvs_cnn_labels(pipe.ctx, st["kp"], st["count"], st["labels"])
        pipe.cnn_forward(st["params"], tau=None, logits=True)
        cd.cdvs_cnn_backward(pipe.ctx, pipe.d_images, st["params"], pipe.d_acts, pipe.d_logits, st["labels"],
                             st["pos_weight"], st["work"], st["grad"], st["loss"])
        cd.cdvs_cnn_adam(pipe.ctx, st["params"], st["grad"], st["m"], st["v"], st["step"])
        return dict(labels=st["labels"], logits=pipe.d_logits, loss=st["loss"], grad=st["grad"], params=st["params"],
                    m=st["m"], v=st["v"])
    if kind == "scfv":
        s = st["scfv"]
        if case["form"] == "context":
            cd.cdvs_scfv(pipe.ctx, s, st["desc"], st["count"])
        else:
            cd.cdvs_scfv_noalloc(s, st["desc"], st["count"], case["n"], case["cap"])
        return dict(gm=s.gm, gv=s.gv, delta=s.delta, order=s.order, bits=s.bits)
    if kind == "compress":
        cd.cdvs_relevance_select(pipe.ctx, st["rel"], st["kp"], st["count"], case["keep"], st["kp_out"], st["count_out"],
                                 st["score"])
        cd.cdvs_encode(pipe.ctx, st["tq"], case["elements"], st["desc"], st["count"], st["codes"])
        f, i = _records_out(st["kp_out"])
        return dict(count=st["count_out"], kp=f, kp_at=i, score=st["score"], codes=st["codes"])
    if kind == "front":
        pipe.front_end(st["src"], st["descs"])
        return dict(images=pipe.d_images)
    pipe_pyr = pipe.d_pyr
    cd.cdvs_pyramid_bmlog(pipe.ctx, pipe.d_images, pipe_pyr)
    return _planes(pipe_pyr, case)


# ---------------------------------------------------------------------------
# The scale space's layout, sizes and results

def _octaves(w, h):
    out = [(w, h)]
    while min(w, h) >= 32:
        w, h = (w + 1) // 2, (h + 1) // 2
        out.append((w, h))
    return out


def _planes(d_pyr, case):
    """Views of the pyramid buffer, one (image, scale, row, column) block per octave."""
    n, out, off = case["n"], {}, 0
    per = d_pyr.numel() // n
    for o, (w, h) in enumerate(_octaves(case["w"], case["h"])):
        pitch = (w + 31) // 32 * 32
        stride = (pitch * h + 63) // 64 * 64
        out["octave%d" % o] = d_pyr.as_strided((n, 5, h, w), (per, stride, pitch, 1), off)
        off += 5 * stride
    return out


def work(case):
    kind, n = case["kind"], case["n"]
    if kind in ("extract", "gated", "stream", "train", "front", "bmlog"):
        sizes = _sizes(case)
        px = sum(w * h for w, h in sizes) * case.get("chunks", 1)
    cells = lambda: px / 16.0   # noqa: E731
    conv = 2.0 * 4 * 9 * 16 * 16 + 2.0 * 16 * 6     # of the mask network, per cell
    if kind in ("extract", "gated", "stream"):
        octpx = sum(a * b for w, h in sizes for a, b in _octaves(w, h)) * case.get("chunks", 1)
        kp = n * case["topk"] * case.get("chunks", 1) * (0.27 if case.get("contrast") == 4.0 else 1.0)
        # the image in, five planes out and in again, records and descriptors out
        b = px + 40.0 * octpx + kp * (48 + 48 + 512)
        f = 46.0 * px + 263.0 * octpx + 40000.0 * kp
        if kind != "extract":
            b, f = b + cells(), f + conv * cells()
        return dict(bytes=b, flops=f)
    if kind == "train":
        # activations out and in again, the gradients of four layers likewise; three products of the forward's size
        return dict(bytes=px + cells() * (4 * 32 * 2 + 4 * 32 * 2 + 24 * 2 + 8), flops=3 * conv * cells())
    if kind == "scfv":
        d = 0.85 * n * case["cap"]
        return dict(bytes=512.0 * d + n * 512 * (2 * 128 + 4 + 4 + 8) + 4 * (512 * 65 + 33 * 128), flops=139264.0 * d)
    if kind == "compress":
        d = 0.85 * n * case["cap"]
        keep = n * min(case["keep"], 0.85 * case["cap"])
        return dict(bytes=d * (512 + 32 + 28) + keep * (48 + 48 + 4), flops=d * 150.0)
    if kind == "front":
        o = sum(a * b for a, b in (cd.cdvs_front_size(w, h) for w, h in sizes))
        return dict(bytes=float(px + o), flops=4.0 * px)
    octpx = sum(a * b for w, h in sizes for a, b in _octaves(w, h))
    return dict(bytes=px + 20.0 * octpx + 4.0 * (octpx - px), flops=85.0 * 5 * octpx)


def exact(case, seed):
    kind = case["kind"]
    if kind == "scfv":
        return _exact_scfv(prepare(case, seed))
    if kind == "train":
        return _exact_train(prepare(case, seed))
    if kind == "compress":
        return _exact_compress(prepare(case, seed))
    if kind == "bmlog":
        return _exact_bmlog(case, prepare(case, seed)["pipe"])
    # The keypoint path's results hang on comparisons (which pixel is an extremum, which of two responses is the
    # larger), so 64 bits give other records, not nearer ones; the front end's are whole numbers.
    return None


def _exact_scfv(st):
    m = {k: torch.from_numpy(np.asarray(v, dtype=np.float64)).cuda() for k, v in _model("scfv_standin").items()}
    w, M, V = m["weights"], m["means"], m["variances"]
    gm, gv = [], []
    for d, k in zip(st["desc"], st["count"].tolist()):
        x = (d[:k].double() - m["pca_mean"]) @ m["pca_matrix"].T
        x2 = x * x
        logit = w.log() - 0.5 * V.log().sum(1) - 0.5 * (x2 @ (1.0 / V).T - 2.0 * x @ (M / V).T + (M * M / V).sum(1))
        q = torch.softmax(logit, dim=1)
        s0, s1, s2 = q.sum(0)[:, None], q.T @ x, q.T @ x2
        gm.append((s1 - s0 * M) / V.sqrt() / (k * w.sqrt()[:, None]))
        gv.append((s2 - 2.0 * s1 * M + s0 * (M * M - V)) / V / (k * (2.0 * w).sqrt()[:, None]))
    gm, gv = torch.stack(gm), torch.stack(gv)
    return dict(gm=gm, gv=gv, delta=gm.std(dim=2, unbiased=False), order=None, bits=None)


def _exact_train(st):
    n, w, h, pipe = st["case"]["n"], st["case"]["w"], st["case"]["h"], st["pipe"]
    h4, w4, no = (h + 3) // 4, (w + 3) // 4, st["octaves"]
    d = pipe.descs[0]
    img = pipe.d_images.view(n, d.height, d.pitch)[:, :, :w].double() / 255.0
    ys = torch.arange(4 * h4, device="cuda").clamp_max(h - 1)
    xs = torch.arange(4 * w4, device="cuda").clamp_max(w - 1)
    x = img[:, ys][:, :, xs].view(n, h4, 4, w4, 4).permute(0, 1, 3, 2, 4).reshape(n, h4, w4, 16)
    p0 = st["params"].double()
    p = p0.clone().requires_grad_(True)
    at = 0
    for _ in range(4):
        W, b = p[at:at + 2304].view(9, 16, 16), p[at + 2304:at + 2320]
        at += 2320
        z = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
        x = torch.relu(b + sum(z[:, t // 3:t // 3 + h4, t % 3:t % 3 + w4] @ W[t] for t in range(9)))
    z = x @ p[at:at + 96].view(16, 6) + p[at + 96:at + 102]
    y = torch.zeros((n, h4, w4, 6), dtype=torch.float64, device="cuda")
    o, ix, iy = (st["kp"][..., k].long() for k in (9, 10, 11))
    cx, cy = ((ix << o) >> 2).clamp_max(w4 - 1), ((iy << o) >> 2).clamp_max(h4 - 1)
    live = torch.arange(o.shape[1], device="cuda")[None, :] < st["count"][:, None]
    i = torch.arange(n, device="cuda")[:, None].expand_as(o)
    y[i[live], cy[live], cx[live], o[live]] = 1.0
    pw = st["pos_weight"].double()
    sp = torch.nn.functional.softplus
    loss = (pw * y * sp(-z) + (1 - y) * sp(z))[..., :no].mean()
    grad, = torch.autograd.grad(loss, p)
    m, v = 0.1 * grad, 0.001 * grad * grad
    new = p0 - 1e-3 * (m / 0.1) / ((v / 0.001).sqrt() + 1e-8)
    return dict(labels=None, logits=z.detach().reshape(-1, 6), loss=loss.detach().reshape(1), grad=grad, params=new, m=m,
                v=v)


def _exact_compress(st):
    case, k = st["case"], st["kp"].view(torch.float32).double()
    e, val = st["rel"].edges.double(), st["rel"].values.double()
    hx, hy = 319.5, 239.5
    f = (k[..., 2], k[..., 3].abs(), torch.hypot(k[..., 0] - hx, k[..., 1] - hy) / math.hypot(hx, hy), k[..., 5], k[..., 6])
    r = torch.ones_like(f[0])
    for c in range(5):
        r = r * val[c][torch.searchsorted(e[c].contiguous(), f[c].contiguous(), right=True)]
    at = torch.arange(r.shape[1], device="cuda")[None, :]
    r = torch.where(at < st["count"][:, None], r, torch.zeros_like(r)).sort(dim=1, descending=True).values
    r = torch.where(at < st["count"].clamp_max(case["keep"])[:, None], r, torch.zeros_like(r))
    return dict(count=None, kp=None, kp_at=None, score=r, codes=None)


def _exact_bmlog(case, pipe):
    """128 x 128 blocks, 16 pixels shared on every side, filtered in the frequency domain by the taps' transforms."""
    n, d = case["n"], pipe.descs[0]
    base = pipe.d_images.view(n, d.height, d.pitch)[:, :, :d.width].double()
    transfer = []
    for k in range(5):
        s = 1.6 if k == 0 else 1.6 * math.sqrt(2.0 ** (k / 2.0) - 1.0)
        q = torch.arange(-math.ceil(4 * s), math.ceil(4 * s) + 1, device="cuda", dtype=torch.float64)
        t = torch.exp(-q * q / (2 * s * s))
        ring = torch.zeros(128, dtype=torch.float64, device="cuda").index_add_(0, q.long() % 128, t / t.sum())
        transfer.append(torch.fft.fft(ring).real)
    out = {}
    for o, (w, h) in enumerate(_octaves(case["w"], case["h"])):
        planes = torch.empty((n, 5, h, w), dtype=torch.float64, device="cuda")
        if o:
            planes[:, 0] = base
        for y0 in range(0, h, 96):
            ys = torch.arange(y0 - 16, y0 + 112, device="cuda").clamp(0, h - 1)
            for x0 in range(0, w, 96):
                xs = torch.arange(x0 - 16, x0 + 112, device="cuda").clamp(0, w - 1)
                F = torch.fft.fft2(base[:, ys][:, :, xs])
                ny, nx = min(96, h - y0), min(96, w - x0)
                for k in range(1 if o else 0, 5):
                    H = transfer[k] if o or k == 0 else transfer[0] * transfer[k]
                    p = torch.fft.ifft2(F * H[:, None] * H[None, :]).real
                    planes[:, k, y0:y0 + ny, x0:x0 + nx] = p[:, 16:16 + ny, 16:16 + nx]
        out["octave%d" % o] = planes
        base = planes[:, 4, ::2, ::2]
    return out
