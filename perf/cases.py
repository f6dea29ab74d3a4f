"""Performance cases of the per-frame hot path: what a program of this framework has it do.

A pass hands frames that already lie in device memory to one or more applications and collects
their results.  Two kinds of passes exist, both through the public calls:

* one frame (or one frame of every stream of a batched application, or one frame of a
  multi-network group): submit, then wait for the result -- the latency a live stream sees;
* a burst: `hs_run_feeds` drives every application of the case back to back over `frames`
  frames (batches), which is how recorded video is processed and how saturation is measured.

Networks, frame sizes, batch sizes and options are those of this repository's own benchmark
and tests; the drawn cases spread over the ranges between them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2402_04466_amd as hs
from paper_2402_04466_amd.harness import AppStream, GroupStream
import synth_inputs as si

DEVICE = "cuda:0"
_LAYERS = {"tiny4": si.TINY4_LAYERS, "resnet18_convlstm": si.RESNET18_CONVLSTM_LAYERS}
_NET = {"tiny4": hs.HS_NET_TINY4, "resnet18_convlstm": hs.HS_NET_RESNET18_CONVLSTM}
_DEFAULTS = dict(net="resnet18_convlstm", frame_w=1920, frame_h=1080, net_w=854, net_h=480, batch=1,
                 apps=1, group=1, frames=1, depth=4, partitions=0, annotate=False,
                 fp32_input=False, threshold=0.5, alpha=0.5)


def _case(name=None, **kw):
    c = dict(_DEFAULTS)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the small network on one small camera stream: nothing but latency, launches, host work
        _case("tiny frame", net="tiny4", frame_w=320, frame_h=240, net_w=128, net_h=128, depth=2,
              fp32_input=True),
        # the small network over a recording with odd frame size, opaque and annotated
        _case("tiny odd annotated burst", net="tiny4", frame_w=322, frame_h=241, net_w=96, net_h=72,
              frames=16, annotate=True, threshold=0.75, alpha=1.0),
        # the big network on a low-resolution live stream
        _case("low-res frame", frame_w=640, frame_h=360, net_w=288, net_h=160),
        # one live full-HD stream: submit-to-result latency
        _case("full-HD frame"),
        # one full-HD recording, back to back (frames overlap in the two lanes)
        _case("full-HD burst", frames=12),
        # a multi-network application: three networks look at every frame, one overlay
        _case("full-HD three networks", group=3),
        # five independent full-HD applications share the device
        _case("full-HD five applications", apps=5, frames=4),
        # six full-HD streams as three applications of two streams, each on its own CU partition
        _case("full-HD partitions", apps=3, batch=2, partitions=3, frames=4),
        # a few streams of an odd frame size batched, annotation layer drawn
        _case("odd-size batch 4", frame_w=1279, frame_h=719, net_w=641, net_h=361, batch=4,
              annotate=True),
        # many low-resolution streams in one batch, no map a multiple of any tile
        _case("low-res batch 16", frame_w=640, frame_h=360, net_w=416, net_h=240, batch=16),
        # twelve full-HD streams batched: latency of one step
        _case("full-HD batch 12", batch=12),
        # the same at saturation: steps back to back
        _case("full-HD batch 12 burst", batch=12, frames=4),
    ]


def _units(c):
    """Frames of the full-size big network a pass amounts to."""
    one = c["net_w"] * c["net_h"] / (854.0 * 480.0)
    if c["net"] == "tiny4":
        one = one / 40.0 + c["frame_w"] * c["frame_h"] / (1920.0 * 1080.0) / 12.0
    return one * c["batch"] * c["apps"] * c["group"] * c["frames"]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        tiny = rng.random() < 0.25
        frame_w = _log_int(rng, 320, 1920)
        frame_h = max(180, int(frame_w * rng.uniform(0.5, 0.75)))
        if tiny:
            net_w = rng.randint(96, 320)
            net_h = int(net_w * rng.uniform(0.6, 1.0))
        else:
            net_w = _log_int(rng, 192, 854)
            net_h = int(net_w * rng.uniform(0.5, 0.6))
        kind = rng.choice(["frame", "frame", "batch", "batch", "burst", "burst", "group", "apps"])
        c = _case(net="tiny4" if tiny else "resnet18_convlstm", frame_w=frame_w, frame_h=frame_h,
                  net_w=net_w, net_h=net_h, annotate=rng.random() < 0.3,
                  fp32_input=tiny and rng.random() < 0.5, depth=rng.choice([2, 4]),
                  threshold=rng.choice([0.3, 0.5, 0.75]), alpha=round(rng.uniform(0.2, 1.0), 2))
        if kind in ("batch", "burst", "apps"):
            c["batch"] = rng.choice([1, 1, 2, 3]) if kind == "apps" else rng.randint(
                2 if kind == "batch" else 1, 16)
        if kind == "burst":
            c["frames"] = rng.randint(3, 16)
        if kind == "group":
            c["group"] = rng.randint(2, 3)
        if kind == "apps":
            c["apps"] = rng.randint(2, 5)
            c["frames"] = rng.randint(2, 6)
            if c["apps"] <= 3 and rng.random() < 0.5:
                c["partitions"] = c["apps"]
        if _units(c) <= 40.0:                     # the largest listed case is 48
            return c


# ---- inputs ---------------------------------------------------------------------------------------
_ctx = None


def _context():
    global _ctx
    if _ctx is None:
        _ctx = hs.hs_init(0)
    return _ctx


def _weights(net, gen):
    """He-normal blob, as synth_inputs.he_normal_blob draws it, made on the GPU."""
    parts = [torch.randn(co * ci * k * k, generator=gen, device=DEVICE) * math.sqrt(2.0 / (ci * k * k))
             for _, co, ci, k in _LAYERS[net]]
    return torch.cat(parts).cpu().numpy()


def _scene(c, pitch, gen):
    """One frame: colour gradient, three grey rectangles (the tools), noise of sigma 10."""
    w, h = c["frame_w"], c["frame_h"]
    x = torch.arange(w, device=DEVICE, dtype=torch.float32)[None, :].expand(h, w)
    y = torch.arange(h, device=DEVICE, dtype=torch.float32)[:, None].expand(h, w)
    img = torch.stack([255 * x / (w - 1), 255 * y / (h - 1), 255 * (x + y) / (w + h - 2)], dim=2)
    u = torch.rand(3, 5, generator=gen, device=DEVICE).cpu().tolist()
    for a, b, e, f, g in u:
        rw, rh = int(w / 16 + a * w * 3 / 16), int(h / 45 + b * h / 15)
        x0, y0 = int(e * (w - rw)), int(f * (h - rh))
        img[y0:y0 + rh, x0:x0 + rw] = 150 + 80 * g
    img = img + 10 * torch.randn(img.shape, generator=gen, device=DEVICE)
    out = torch.zeros((h, pitch), dtype=torch.uint8, device=DEVICE)
    out[:, :3 * w] = img.round_().clamp_(0, 255).to(torch.uint8).reshape(h, 3 * w)
    return out


class _State:
    """The applications a program keeps, with the frames and output buffers it cycles through."""

    def __init__(self, c, seed):
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(int(seed))
        self.case = c
        self.apps, self.owners, self.own_ctx = [], [], None
        if c["partitions"]:
            # a context accounts for the CUs its applications have claimed
            self.own_ctx = hs.hs_init(0)
        ctx = self.own_ctx or _context()
        blob = _weights(c["net"], gen)
        glyphs = si.DEFAULT_GLYPHS if c["annotate"] else None
        for i in range(c["apps"]):
            members = []
            for j in range(c["group"]):
                # every network of a group has its own weights; independent applications are
                # instances of the same model
                w = blob if j == 0 else _weights(c["net"], gen)
                members.append(AppStream(
                    ctx, net=_NET[c["net"]], frame_w=c["frame_w"], frame_h=c["frame_h"],
                    net_w=c["net_w"], net_h=c["net_h"], blob=w, palette=np.roll(si.DEFAULT_PALETTE, j, 0),
                    queue_depth=c["depth"], net_fp32_input=c["fp32_input"], threshold=c["threshold"],
                    alpha=c["alpha"], batch=c["batch"], glyphs=glyphs, device=DEVICE))
            if c["partitions"]:
                per = 256 // c["partitions"] // 8 * 8       # whole groups of eight CUs
                mask = hs.cu_mask_words(range(i * per, (i + 1) * per))
                hs.hs_set_partition(members[0].app, mask, mask)
            self.owners.append(members)
            self.apps.append(GroupStream(ctx, members) if c["group"] > 1 else members[0])
        pitch = self.owners[0][0].frame_pitch
        distinct = min(4, max(2, c["frames"]))
        n_out = c["frames"] if c["frames"] > 1 else c["depth"]
        self.frames = [[[_scene(c, pitch, gen) for _ in range(c["batch"])] for _ in range(distinct)]
                       for _ in self.apps]
        self.outs = [torch.zeros((n_out, c["batch"], c["frame_h"], pitch), dtype=torch.uint8,
                                 device=DEVICE) for _ in self.apps]
        self.out_rows = [[[o[k, j] for j in range(c["batch"])] for k in range(n_out)] for o in self.outs]
        self.feeds = []
        for i, app in enumerate(self.apps):
            f = {"frames": [[t.data_ptr() for t in row] for row in self.frames[i]],
                 "outs": [[t.data_ptr() for t in row] for row in self.out_rows[i]]}
            if c["group"] > 1:
                f.update(group=app.group, results_per_frame=c["group"])
            else:
                f.update(app=app.app, results_per_frame=c["batch"])
            self.feeds.append(f)
        self.views = {}
        self.count = 0

    def view(self, owner, r):
        """Logits, heat map and mask of a result: views of the application's workspace."""
        v = self.views.get(r.d_logits)
        if v is None:
            ws, base = owner.workspace, owner.workspace.data_ptr()
            n = 8 * r.map_w * r.map_h

            def cut(ptr, nbytes, dtype):
                return ws[ptr - base:ptr - base + nbytes].view(dtype).view(8, r.map_h, r.map_w)
            v = (cut(r.d_logits, 4 * n, torch.float32), cut(r.d_heat, 4 * n, torch.float32),
                 cut(r.d_mask, n, torch.uint8))
            self.views[r.d_logits] = v
        return v

    def close(self):
        for a in self.apps:
            a.close()
        self.apps = []
        if self.own_ctx:
            hs.hs_shutdown(self.own_ctx)
            self.own_ctx = None

    def __del__(self):
        self.close()


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    """One pass.  Out come the overlays of every frame, the peaks of every result and, of the
    last frame, logits, heat maps and masks (the earlier ones' device buffers are reused by then).
    The index of a peak jumps between near-equal logits from one correct implementation to
    the next; the value there (`peak`) does not, so that is what comes back of the record."""
    c = state.case
    if c["frames"] == 1 and c["apps"] == 1:
        app, k = state.apps[0], state.count
        state.count += 1
        src = state.frames[0][k % len(state.frames[0])]
        dst = state.out_rows[0][k % len(state.out_rows[0])]
        if c["group"] == 1 and c["batch"] == 1:
            app.submit(src[0], dst[0], k)
            last = [app.wait()]
        else:
            app.submit_batch(src, dst, k)
            last = app.wait_batch()
        overlay = [state.outs[0][k % len(state.out_rows[0])]]
        per_app, peaks = [last], [list(r.peak) for r in last]
    else:
        results = hs.hs_run_feeds(state.feeds, 0.0, c["frames"])[0]
        overlay = state.outs
        per_app = [res[-1] for res in results]
        peaks = [list(r.peak) for res in results for frame in res for r in frame]
    maps = []
    for members, last in zip(state.owners, per_app):
        for j, r in enumerate(last):
            maps.append(state.view(members[j] if c["group"] > 1 else members[0], r))
    return {"overlay": overlay, "peak": np.array(peaks, dtype=np.float32), "maps": maps}


# ---- what a pass cannot do without ------------------------------------------------------------------
def _conv_flops(net, net_w, net_h):
    """Multiply-adds x 2 of one frame's convolutions."""
    def half(n):
        return (n + 1) // 2
    total, h, w = 0.0, net_h, net_w
    if net == "tiny4":
        for (_, co, ci, k), s in zip(_LAYERS[net], (2, 2, 1, 1)):
            if s == 2:
                h, w = half(h), half(w)
            total += 2.0 * h * w * co * ci * k * k
        return total, (h, w)
    for name, co, ci, k in _LAYERS[net]:
        if name == "stem":
            h, w = half(h), half(w)
        elif name.endswith(".b0.a") and not name.startswith("l1"):
            h, w = half(h), half(w)
        total += 2.0 * h * w * co * ci * k * k
        if name == "stem":
            h, w = half(h), half(w)                 # max-pool behind the stem
    return total, (h, w)


def work(case):
    """Frames read, overlays and maps written and weights read once (fp16, per application: each
    holds its own copy), the recurrent state read and written; flops of the convolutions."""
    c = case
    flops, (mh, mw) = _conv_flops(c["net"], c["net_w"], c["net_h"])
    frames = c["apps"] * c["frames"] * c["batch"]
    passes = frames * c["group"]
    weights = 2.0 * si.blob_num_floats(_LAYERS[c["net"]]) * c["apps"] * c["group"]
    nbytes = frames * 6.0 * c["frame_w"] * c["frame_h"] + weights + passes * 72.0 * mh * mw
    if c["fp32_input"]:
        nbytes += passes * 12.0 * c["net_w"] * c["net_h"]
    if c["net"] != "tiny4":
        nbytes += c["apps"] * c["group"] * c["batch"] * 2 * 6.0 * 256 * mh * mw
    return {"bytes": nbytes, "flops": passes * flops}


def tolerance(case):
    """Activations are stored in fp16 between the layers (20 of them in the big network): two
    correct implementations differ by their roundings, a few 1e-3 of the result's norm.  A mask
    cell whose logit lies within that of the threshold may flip, and its overlay pixels with it."""
    return {"rel": 1e-2, "max": 0.2, "differ": 0.01}
