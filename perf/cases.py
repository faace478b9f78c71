"""What this framework is timed on: raw uint8 frames in device memory -> patches -> encoder output -> tokens at
the language model's width, for the encoder families and request mixes of `workloads/`, the profiler's request
sweep (images with sides 28*{8..48}, videos of 4..64 frames) and the serving replay (batches of about 16 k tokens,
each with a plan of its own).

A case is a request list given by numbers:
  family     encoder (see FAMILIES)
  images     still images, sides drawn from `sizes` between lo and hi in the family's step
  videos     videos of `frames` frames, `side` pixels square
  text       text requests (no frames)
  resampled  frames arrive at a 16:9 size of their own and are resized to the target
  plan_each  the pass starts with planning the batch, as a server does for requests it has not seen
"""
import functools
import math
import random
import zlib

import torch

import workloads
from paper_2603_26498_amd.runtime import Plan, VisionEncoder

# desc, step of the target sides in pixels, smallest and largest side
FAMILIES = {
    # dynamic resolution, 2x2 merge and projector (the image, video and mixed workloads, profiler and server)
    "dynres": (workloads.qwen_like_desc, 28, 224, 1344),
    # rotary positions, RMSNorm, gated MLP, attention in 8x8-patch windows except in every eighth layer
    "windowed": (workloads.windowed_desc, 28, 224, 1344),
    # images cut into 16x16 patches, no merge, rotary, gated MLP, adapter to 5120
    "varsize": (workloads.plain_rotary_desc, 16, 256, 1024),
    # fixed 336x336 images, 24 layers, d = 1024
    "fixed336": (lambda: workloads.config2(with_frames=False).desc, 336, 336, 336),
    # fixed 378x378 crops, 27 layers, 16 heads of 72, mlp 4304
    "crops378": (lambda: workloads.config9(with_frames=False).desc, 378, 378, 378),
    # fp32 model with a CLS row, images up to 224x224
    "f32": (lambda: workloads.config1(with_frames=False).desc, 16, 64, 224),
}


def _case(name=None, family="dynres", images=0, lo=0, hi=0, sizes=0, videos=0, frames=0, side=0, text=0,
          resampled=False, plan_each=False):
    c = dict(family=family, images=images, lo=lo, hi=hi, sizes=sizes, videos=videos, frames=frames, side=side,
             text=text, resampled=resampled, plan_each=plan_each)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: one image through the small fp32 model (parity and debugging runs)
        _case("f32_image224", "f32", images=1, lo=224, hi=224),
        # an interactive request: one thumbnail-sized image, latency is all that counts
        _case("image224", images=1, lo=224, hi=224),
        # an ordinary chat image that arrives at camera proportions and is planned, resized and encoded on arrival
        _case("image_on_arrival", images=1, lo=392, hi=896, sizes=10, resampled=True, plan_each=True),
        # a short clip: 8 frames at 448x448
        _case("clip8", videos=1, frames=8, side=448),
        # one picture of odd size through the windowed encoder: windows are cut off at the picture's edges
        _case("windowed_image", "windowed", images=1, lo=476, hi=980, sizes=5),
        # one image cut into five crops, the usual input of the fixed-crop encoders
        _case("crops5", "crops378", images=5, lo=378, hi=378),
        # a serving batch: what a 16 k token budget collects from the queues, planned on each pass
        _case("serve_batch", images=12, lo=224, hi=672, sizes=3, videos=1, frames=8, side=448, plan_each=True),
        # throughput on fixed-resolution images
        _case("batch32_336", "fixed336", images=32, lo=336, hi=336),
        # images of any size, no merge
        _case("varsize16", "varsize", images=16, lo=256, hi=1024, sizes=8),
        # a minute of video through the windowed encoder
        _case("windowed_video64", "windowed", videos=1, frames=64, side=448),
        # a minute of video, attention over all 32768 tokens
        _case("video64", videos=1, frames=64, side=448),
        # offline throughput on mixed modalities: two videos, many images, text among them, everything resized
        _case("mixed_batch", images=24, lo=224, hi=1344, sizes=27, videos=2, frames=32, side=448, text=200,
              resampled=True),
    ]


LARGEST_FLOPS = 2.6e14       # about the mixed batch
LARGEST_TOKENS = 102_000


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["image", "image", "clip", "serve", "mixed", "windowed", "windowed", "varsize", "fixed336", "crops378", "f32"])
        sizes = rng.randrange(1 << 20)
        if kind == "image":
            c = _case(images=1, lo=224, hi=1344, sizes=sizes, resampled=rng.random() < 0.5, plan_each=rng.random() < 0.5)
        elif kind == "clip":
            c = _case(videos=1, frames=2 * _log_int(rng, 2, 32), side=28 * rng.randint(8, 16), sizes=sizes,
                      resampled=rng.random() < 0.5)
        elif kind == "serve":
            c = _case(images=_log_int(rng, 2, 32), lo=224, hi=672, sizes=sizes, videos=rng.choice([0, 0, 1]),
                      frames=2 * rng.randint(4, 16), side=448, plan_each=True)
        elif kind == "mixed":
            c = _case(images=_log_int(rng, 2, 40), lo=224, hi=1344, sizes=sizes, videos=rng.randint(0, 2),
                      frames=2 * _log_int(rng, 2, 16), side=28 * rng.randint(8, 16), text=rng.randint(0, 200),
                      resampled=rng.random() < 0.5)
        elif kind == "windowed":
            if rng.random() < 0.5:
                c = _case(family=kind, images=_log_int(rng, 1, 16), lo=224, hi=1344, sizes=sizes, resampled=rng.random() < 0.5)
            else:
                c = _case(family=kind, videos=1, frames=2 * _log_int(rng, 2, 32), side=28 * rng.randint(8, 16), sizes=sizes)
        elif kind == "varsize":
            c = _case(family=kind, images=_log_int(rng, 1, 24), lo=256, hi=1024, sizes=sizes)
        elif kind == "f32":
            c = _case(family=kind, images=_log_int(rng, 1, 16), lo=64, hi=224, sizes=sizes)
        else:
            side = FAMILIES[kind][2]
            c = _case(family=kind, images=_log_int(rng, 1, 48), lo=side, hi=side, sizes=sizes)
        if work(c)["flops"] <= LARGEST_FLOPS and sum(_tokens(c, it) for it in _requests(c)) <= LARGEST_TOKENS:
            return c


def _requests(case):
    """(modality, frames, source height, source width, target height, target width) of every request."""
    step = FAMILIES[case["family"]][1]
    r = random.Random("sizes %d" % case["sizes"])

    def source(h, w):
        if not case["resampled"]:
            return h, w
        sh = r.randint(240, 1080)
        return sh, 2 * round(sh * 8 / 9)

    out = []
    for _ in range(case["videos"]):
        out.append((workloads.VIDEO, case["frames"], *source(case["side"], case["side"]), case["side"], case["side"]))
    for _ in range(case["images"]):
        h = r.randint(-(-case["lo"] // step), case["hi"] // step) * step
        w = r.randint(-(-case["lo"] // step), case["hi"] // step) * step
        out.append((workloads.IMAGE, 1, *source(h, w), h, w))
    out += [(workloads.TEXT, 0, 0, 0, 0, 0)] * case["text"]
    return out


@functools.lru_cache(maxsize=None)
def _desc(family):
    return FAMILIES[family][0]()


def _grid(d, req):
    return 1 if req[1] == 1 else req[1] // d.tpatch, req[4] // d.patch, req[5] // d.patch


def _tokens(case, req):
    if not req[1]:
        return 0
    d = _desc(case["family"])
    t, h, w = _grid(d, req)
    return t * h * w + (1 if d.use_cls else 0)


def work(case):
    d = _desc(case["family"])
    reqs = [q for q in _requests(case) if q[1]]
    seg = [_tokens(case, q) for q in reqs]
    tokens = sum(seg)
    full = float(sum(n * n for n in seg))            # query-key pairs of a full-attention layer
    pairs = full * d.layers
    if d.window:
        win = 0.0
        for q in reqs:
            t, h, w = _grid(d, q)
            rows = [min(d.window, h - i) for i in range(0, h, d.window)]
            cols = [min(d.window, w - i) for i in range(0, w, d.window)]
            win += t * sum((a * b) ** 2 for a in rows for b in cols)
        n_full = d.layers // d.full_every if d.full_every else 0
        pairs = full * n_full + win * (d.layers - n_full)
    mlp = (3 if d.gated else 2) * d.mlp * d.d
    flops = 2.0 * tokens * (d.k * d.d + d.layers * (4 * d.d * d.d + mlp)) + 4.0 * pairs * d.d
    params = d.k * d.d + d.layers * (4 * d.d * d.d + mlp)
    e = 2 if d.dtype == "bf16" else 4
    moved = sum(q[1] * q[2] * q[3] * 3 for q in reqs) + tokens * (d.k * e + d.d * 4)
    if d.out_dim:
        m2 = d.merge * d.merge
        dm = d.d * m2
        flops += 2.0 * (tokens / m2) * dm * (dm + d.out_dim)
        params += dm * (dm + d.out_dim)
        moved += tokens // m2 * d.out_dim * e
    return {"bytes": moved + params * e, "flops": flops}


def tolerance(case):
    """Four times the difference from a float64 evaluation of the same model (patches: none; fp32: 7e-7, largest 4.5e-6
    of the root mean square; bf16 families: 3.8e-3 to 6.5e-3, largest 0.018 to 0.034)."""
    if _desc(case["family"]).dtype == "f32":
        return {"rel": 3e-6, "max": 2e-5}
    return {"rel": 2e-2, "max": 0.12}


@functools.lru_cache(maxsize=None)
def _encoder(family):
    """The encoder with its weights on the GPU, as a serving process keeps it: N(0, 0.02) matrices, gains around 1,
    small biases, the shapes of workloads.make_weights."""
    d = _desc(family)
    g = torch.Generator(device="cuda")
    g.manual_seed(zlib.crc32(family.encode()))

    def rnd(shape, mean, std):
        x = torch.randn(shape, generator=g, device="cuda") * std + mean
        return (x.bfloat16().float() if d.dtype == "bf16" else x).cpu().numpy()

    def mat(o, i):
        return rnd((o, i), 0.0, 0.02)

    w = {"w_pe": mat(d.d, d.k), "b_pe": rnd(d.d, 0.0, 0.02)}
    if d.use_cls:
        w["cls"] = rnd(d.d, 0.0, 0.02)
    if d.pos in ("learned1d", "sep2d"):
        w["pos0"] = mat(d.max_pos, d.d)
    if d.pos == "sep2d":
        w["pos1"] = mat(d.max_pos, d.d)

    def norm(key):
        w[key + "_g"], w[key + "_b"] = rnd(d.d, 1.0, 0.1), rnd(d.d, 0.0, 0.02)

    f1 = (2 if d.gated else 1) * d.mlp
    for l in range(d.layers):
        p = "l%d." % l
        norm(p + "ln1")
        norm(p + "ln2")
        for key, o, i in (("qkv", 3 * d.d, d.d), ("o", d.d, d.d), ("1", f1, d.d), ("2", d.d, d.mlp)):
            w[p + "w_" + key], w[p + "b_" + key] = mat(o, i), rnd(o, 0.0, 0.02)
    if d.final_ln:
        norm("lnf")
    if d.out_dim:
        dm = d.d * d.merge * d.merge
        norm("lnm")
        w["w_m1"], w["b_m1"] = mat(dm, dm), rnd(dm, 0.0, 0.02)
        w["w_m2"], w["b_m2"] = mat(d.out_dim, dm), rnd(d.out_dim, 0.0, 0.02)
    return VisionEncoder(d, w)


def _frames(g, n, h, w):
    """Picture-like frames: a smooth random colour field that drifts from frame to frame, plus sensor noise."""
    coarse = torch.rand((1, 3, h // 24 + 2, w // 24 + 2), generator=g, device="cuda") * 255.0
    field = torch.nn.functional.interpolate(coarse, size=(h, w), mode="bilinear", align_corners=True)[0].permute(1, 2, 0)
    out = torch.empty((n, h, w, 3), dtype=torch.uint8, device="cuda")
    for i in range(n):
        noise = torch.randn((h, w, 3), generator=g, device="cuda") * 6.0
        out[i] = (field.roll((i, 2 * i), (0, 1)) + noise).round_().clamp_(0, 255).to(torch.uint8)
    return out


def _plan(enc, rows, frames):
    return Plan(enc, [(*q, f.data_ptr() if f is not None else None) for q, f in zip(rows, frames)],
                [f for f in frames if f is not None])


def prepare(case, seed):
    enc = _encoder(case["family"])
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rows = _requests(case)
    frames = [_frames(g, *q[1:4]) if q[1] else None for q in rows]
    return {"enc": enc, "rows": rows, "frames": frames, "plan": None if case["plan_each"] else _plan(enc, rows, frames)}


def run(state):
    enc = state["enc"]
    plan = state["plan"] if state["plan"] is not None else _plan(enc, state["rows"], state["frames"])
    patches = enc.preprocess(plan)
    hidden = enc.encode(plan, patches)
    out = {"patches": patches, "hidden": hidden}
    if enc.desc.out_dim:
        out["tokens"] = enc.merge_project(plan, hidden)
    return out
