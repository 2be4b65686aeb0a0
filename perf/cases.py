"""The work a user of this package has it do, as cases that can be timed and compared.

Each case goes through the public entry points (``Segmenter``, ``Batch`` and the ``gmm_*`` calls of
``_abi``) over the sizes, state types and options that the package's workloads use: one stream per
launch (160x120 up to 1920x1080, paired, colour only, depth only, pitched, four-channel), batches of
streams of uneven sizes, the serving executor on host frames, a checkpoint taken and resumed, and
the evaluation of masks. Frames are synthetic scenes of the kind ``synth`` describes (a static
background, moving boxes, sensor noise, depth holes, optionally a drifting colour gain), drawn from
the case's seed on the GPU. A model has been running for a while before its first measured frame,
except where the case says it is fresh.
"""
import math

import numpy as np
import torch

import paper_2110_14934_amd as gmm
from paper_2110_14934_amd import _abi, quality

DEV = "cuda"
MODES = {"rgbd": _abi.GMM_RGB | _abi.GMM_DEPTH, "rgb": _abi.GMM_RGB, "depth": _abi.GMM_DEPTH}
ALPHA, K, T, W_INIT = 0.01, 2.5, 0.7, 0.01
SIGMA0, VAR_MIN = (30.0, 50.0), (9.0, 25.0)

# sizes of the Kinect-class sensors (v1: 320x240, 640x480; v2: 512x424 depth, 1920x1080 colour)
MIX_64 = "16*320x240+32*640x480+8*512x424depth+8*1920x1080rgb"
MIX_16 = "4*320x240+8*640x480+2*512x424depth+2*1920x1080rgb"


def listed():
    return [
        # one small camera, the lowest latency: the smallest call
        stream("stream-160x120", 160, 120, M=3, hole=0.02),
        # the ordinary single camera: one VGA colour + depth stream, fused masks, every frame
        stream("stream-640x480", 640, 480),
        # a camera switched on (or its scene cut): a fresh model's first frames, where every pixel
        # makes a new component; a snapshot of the fresh model is put back first, as a user who
        # rolls a stream back does
        stream("fresh-640x480", 640, 480, fresh=True),
        # a large colour-only camera with half-size state, as the serving mix holds it
        stream("colour-1920x1080-f16", 1920, 1080, modalities="rgb", state="f16"),
        # a crop of larger images (rows with a pitch, an odd size), mixtures and fusion called
        # apart, bf16 state, the light drifting
        stream("pitched-641x479-bf16", 641, 479, M=4, state="bf16", pitched=True, calls="split", gain=True),
        # the four-channel variant (one mixture over colour and depth byte)
        stream("augmented-640x480", 640, 480, calls="augmented"),
        # many cameras of uneven sizes in one launch, frame slots prepared in advance
        {"name": "batch-64", "kind": "batch", "streams": MIX_64, "M": 5, "state": "f32", "calls": "slots", "frames": 8},
        # many equal cameras, half-size state, new frame buffers in every call
        {"name": "batch-32x640x480-f16", "kind": "batch", "streams": "32*640x480", "M": 5, "state": "f16",
         "calls": "apply", "frames": 8},
        # the batched call that allocates nothing, small cameras
        {"name": "static-24-small", "kind": "batch", "streams": "16*160x120+8*320x240", "M": 3, "state": "f32",
         "calls": "static", "frames": 8},
        # a serving tick: host frames in, host masks out
        {"name": "tick-16-f16", "kind": "tick", "streams": MIX_16, "M": 5, "state": "f16", "frames": 8},
        # a checkpoint put back, one frame, a checkpoint taken (state in the canonical layout)
        {"name": "resume-320x240", "kind": "resume", "streams": "1*320x240", "M": 5, "state": "f32", "calls": "frame"},
        # evaluation of the three masks of a colour + depth frame against the truth
        {"name": "evaluate-640x480", "kind": "evaluate", "width": 640, "height": 480, "masks": 3},
    ]


def stream(name, width, height, modalities="rgbd", M=5, state="f32", calls="fused", pitched=False, gain=False,
           fresh=False, hole=0.05, rho="alpha"):
    case = {"kind": "stream", "width": width, "height": height, "modalities": modalities, "M": M, "state": state,
            "calls": calls if modalities == "rgbd" else "single", "pitched": pitched, "gain": gain, "fresh": fresh,
            "hole": hole, "rho": rho}
    if name:
        case["name"] = name
    return case


def draw(rng):
    kind = rng.choices(("stream", "batch", "tick", "resume", "evaluate"), (8, 4, 2, 2, 1))[0]
    state = rng.choice(("f32", "f32", "f16", "bf16"))
    M = rng.choice((3, 4, 5, 5))
    if kind == "stream":
        w, h = _size(rng, 64 * 48, 1920 * 1080)
        modalities = rng.choice(("rgbd", "rgbd", "rgbd", "rgb", "depth"))
        return stream(None, w, h, modalities, M, state, rng.choice(("fused", "fused", "split", "augmented")),
                      rng.random() < 0.25, rng.random() < 0.3, rng.random() < 0.2, rng.choice((0.0, 0.02, 0.05)),
                      rng.choice(("alpha", "alpha", "alpha", "density")))
    if kind == "batch":
        n = int(round(math.exp(rng.uniform(math.log(2), math.log(64)))))
        return {"kind": "batch", "streams": _streams(rng, n, 640 * 480), "M": M, "state": state,
                "calls": rng.choice(("slots", "apply", "static")), "frames": 8}
    if kind == "tick":
        n = int(round(math.exp(rng.uniform(0, math.log(16)))))
        return {"kind": "tick", "streams": _streams(rng, n, 640 * 480), "M": M, "state": state, "frames": 8}
    if kind == "resume":
        w, h = _size(rng, 64 * 48, 240 * 160)
        calls = rng.choice(("frame", "frame", "batch", "static", "augmented"))
        mode = "" if calls == "augmented" else rng.choice(("", "", "rgb", "depth"))
        return {"kind": "resume", "streams": "%d*%dx%d%s" % (rng.choice((1, 1, 2)), w, h, mode), "M": M, "state": state,
                "calls": calls}
    w, h = _size(rng, 64 * 48, 1920 * 1080)
    return {"kind": "evaluate", "width": w, "height": h, "masks": rng.choice((1, 2, 3, 8))}


def _size(rng, least, most):
    """A width and height with least <= width * height <= most, mostly odd, about 4:3."""
    area = math.exp(rng.uniform(math.log(least), math.log(most)))
    w = max(1, int(math.sqrt(area * rng.uniform(1.0, 1.8))))
    return w, max(1, int(area / w))


def _streams(rng, n, most):
    """n streams in up to three groups of equal ones."""
    parts, left = [], n
    while left:
        k = left if len(parts) == 2 else rng.randint(1, left)
        parts.append("%d*%dx%d%s" % ((k,) + _size(rng, 64 * 48, most) + (rng.choice(("", "", "rgb", "depth")),)))
        left -= k
    return "+".join(parts)


def _groups(text):
    """"4*320x240+2*512x424depth" -> [(320, 240, "rgbd"), ...], one entry per stream."""
    got = []
    for part in text.split("+"):
        n, rest = part.split("*")
        mode = next((m for m in ("rgb", "depth") if rest.endswith(m)), "rgbd")
        w, h = rest[:len(rest) - len(mode)].split("x") if mode != "rgbd" else rest.split("x")
        got += [(int(w), int(h), mode)] * int(n)
    return got


# ---- inputs ------------------------------------------------------------------------------------

class Scene:
    """Frames of one synthetic stream, on the GPU."""

    def __init__(self, width, height, modalities, gen, frames, hole=0.05, gain=False, pitched=False):
        H, W = height, width
        self.rgb, self.depth, self.boxes = [], [], []
        small = min(H, W)
        boxes = []
        for _ in range(3):
            s = max(1, int(small * (0.08 + 0.17 * _unit(gen))))
            boxes.append((s, _unit(gen), _unit(gen), 1 + int(4 * _unit(gen)), 1 + int(4 * _unit(gen))))
        bg = torch.randint(0, 256, (H, W, 3), generator=gen, device=DEV).float() if "rgb" in modalities else None
        for t in range(frames):
            at = []
            for s, u, v, dx, dy in boxes:
                x, y = int(u * (W - s)) + dx * t, int(v * (H - s)) + dy * t
                at.append((min(max(x, 0), W - s), min(max(y, 0), H - s), s))
            self.boxes.append(at)
            if bg is not None:
                f = bg.clone()
                for x, y, s in at:
                    f[y:y + s, x:x + s] = 200.0
                f = f * (0.8 + 0.012 * t) if gain else f
                f += 2.0 * torch.randn(H, W, 3, generator=gen, device=DEV)
                self.rgb.append(_rows(f.round_().clamp_(0, 255).to(torch.uint8), pitched))
            if "d" in modalities:
                f = torch.full((H, W), 2000.0, device=DEV)
                for x, y, s in at:
                    f[y:y + s, x:x + s] = 1200.0
                f += math.sqrt(10.0) * torch.randn(H, W, generator=gen, device=DEV)
                f = f.round_().clamp_(1, 65535)
                if hole:
                    f.mul_((torch.rand(H, W, generator=gen, device=DEV) >= hole).float())
                self.depth.append(_rows(f.to(torch.int32).to(torch.uint16), pitched))

    def frame(self, i):
        return (self.rgb[i] if self.rgb else None), (self.depth[i] if self.depth else None)


def _unit(gen):
    return float(torch.rand(1, generator=gen, device=DEV))


def _rows(frame, pitched):
    """The frame as it is, or as a window of a wider buffer (rows with a pitch)."""
    if not pitched:
        return frame
    H, W = frame.shape[:2]
    wide = torch.zeros((H, W + 23) + tuple(frame.shape[2:]), dtype=frame.dtype, device=DEV)
    wide[:, 7:7 + W] = frame
    return wide[:, 7:7 + W]


class Clip:
    """Plays frame indices forwards, then backwards, so that the scene never jumps."""

    def __init__(self, n):
        self.order = list(range(n)) + list(range(n - 2, 0, -1))
        self.at = 0

    def next(self):
        i = self.order[self.at]
        self.at = (self.at + 1) % len(self.order)
        return i


class State:
    pass


def prepare(case, seed):
    s = State()
    s.kind = case["kind"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    {"stream": _prepare_stream, "batch": _prepare_batch, "tick": _prepare_tick, "resume": _prepare_resume,
     "evaluate": _prepare_evaluate}[s.kind](s, case, gen)
    return s


def run(s):
    return s.run()


def _segmenter(w, h, mode, M, state, **more):
    return gmm.Segmenter(w, h, MODES[mode], M, state_dtype=state, **more)


# ---- one stream per launch -----------------------------------------------------------------------

def _prepare_stream(s, case, gen):
    w, h, mode, calls = case["width"], case["height"], case["modalities"], case["calls"]
    n = 4 if case["fresh"] else 8
    s.scene = Scene(w, h, mode, gen, n, case["hole"], case["gain"], case["pitched"])
    s.seg = _segmenter(w, h, mode, case["M"], case["state"], rho=case["rho"], augmented=calls == "augmented")
    s.clip = Clip(n)

    def one():
        rgb, depth = s.scene.frame(s.clip.next())
        if calls == "fused":
            return s.seg.apply_fused(rgb, depth)
        if calls == "augmented":
            return s.seg.apply_augmented(rgb, depth)
        fg_rgb, fg_depth = s.seg.apply(rgb, depth)
        if calls == "split":
            return fg_rgb, fg_depth, s.seg.fuse(fg_rgb, fg_depth)
        return fg_rgb, fg_depth

    if case["fresh"]:
        s.snapshot = torch.empty(s.seg.state_bytes(), dtype=torch.uint8, device=DEV)
        s.seg.save_state(s.snapshot)

        def fresh():
            s.seg.restore_state(s.snapshot)
            s.clip.at = 0
            for _ in range(n):
                out = one()
            return out

        s.run = fresh
        return
    s.run = one
    for _ in range(40):
        one()


# ---- many streams in one launch ------------------------------------------------------------------

def _prepare_batch(s, case, gen):
    groups, n = _groups(case["streams"]), case["frames"]
    s.scenes = [Scene(w, h, mode, gen, n) for w, h, mode in groups]
    s.segs = [_segmenter(w, h, mode, case["M"], case["state"]) for w, h, mode in groups]
    # every mask of the batch in one buffer
    sizes = [gmm.mask_words(w * h) * (3 if mode == "rgbd" else 1) for w, h, mode in groups]
    s.masks = torch.zeros(sum(sizes), dtype=torch.int64, device=DEV)
    for seg, part in zip(s.segs, torch.split(s.masks, sizes)):
        words = gmm.mask_words(seg.npix)
        names = [k for k in ("fg_rgb", "fg_depth", "fused") if getattr(seg, k) is not None]
        for k, name in enumerate(names):
            setattr(seg, name, part[k * words:(k + 1) * words])
    s.clip = Clip(n)
    frames = [[sc.frame(i) for sc in s.scenes] for i in range(n)]
    calls = case["calls"]
    s.batch = gmm.Batch(s.segs, n_slots=n)
    if calls == "slots":
        for i in range(n):
            s.batch.set_frames(i, frames[i])

        def one():
            s.batch.run(s.clip.next())
            return s.masks
    elif calls == "apply":
        def one():
            s.batch.apply(frames[s.clip.next()])
            return s.masks
    else:
        handles = [seg.handle for seg in s.segs]
        ios = [s.batch.ios(f) for f in frames]

        def one():
            gmm._abi.gmm_batch_apply_static(handles, ios[s.clip.next()])
            return s.masks
    s.run = one
    for _ in range(24):
        one()


# ---- the serving executor ------------------------------------------------------------------------

class Executor:
    """An executor with its streams in one device arena, and their host buffers."""

    def __init__(self, groups, M, state):
        self.x = _abi.gmm_exec_create(0, 4)
        cfgs = [_abi.gmm_config_default(w, h, MODES[mode], M, state_dtype=_abi.DTYPES[state]) for w, h, mode in groups]
        needs = [(_abi.gmm_exec_stream_bytes(c) + 255) // 256 * 256 for c in cfgs]
        self.arena = torch.empty(sum(needs) + 256, dtype=torch.uint8, device=DEV)
        at = (self.arena.data_ptr() + 255) // 256 * 256
        self.handles = []
        for c, need in zip(cfgs, needs):
            self.handles.append(_abi.gmm_exec_create_stream(self.x, c, at, need))
            at += need

    def __del__(self):
        for h in self.handles:
            _abi.gmm_exec_destroy_stream(self.x, h)
        _abi.gmm_exec_destroy(self.x)


def _prepare_tick(s, case, gen):
    groups, n = _groups(case["streams"]), case["frames"]
    torch.cuda.synchronize()
    s.exec = Executor(groups, case["M"], case["state"])
    sizes = [gmm.mask_words(w * h) * (3 if mode == "rgbd" else 1) for w, h, mode in groups]
    s.masks = torch.zeros(sum(sizes), dtype=torch.int64, pin_memory=True)
    s.host, ticks = [], [[] for _ in range(n)]
    for (w, h, mode), handle, part in zip(groups, s.exec.handles, torch.split(s.masks, sizes)):
        scene, words = Scene(w, h, mode, gen, n), gmm.mask_words(w * h)
        for i in range(n):
            bufs = []
            for f in scene.frame(i):
                b = None
                if f is not None:
                    b = torch.empty(f.shape, dtype=f.dtype, pin_memory=True)
                    b.copy_(f)
                bufs.append(b)
            s.host.append(bufs)
            it = _abi.gmm_exec_item()
            it.handle = handle
            it.host_rgb = bufs[0].data_ptr() if bufs[0] is not None else None
            it.host_depth = bufs[1].data_ptr() if bufs[1] is not None else None
            p = part.data_ptr()
            if mode == "depth":
                it.host_fg_depth = p
            else:
                it.host_fg_rgb = p
            if mode == "rgbd":
                it.host_fg_depth, it.host_fused = p + 8 * words, p + 16 * words
            ticks[i].append(it)
    s.clip = Clip(n)

    def one():
        _abi.gmm_exec_launch(s.exec.x, ticks[s.clip.next()])
        _abi.gmm_exec_drain(s.exec.x)
        _abi.gmm_exec_poll(s.exec.x)
        return s.masks

    s.run = one
    for _ in range(24):
        one()


# ---- checkpoint and resume -----------------------------------------------------------------------

def _checkpoint(case, seed):
    """Per stream: its canonical state ([param][rank][pixel] blocks, float64) as an earlier
    gmm_read_state gave it, every value representable in the storage type, and its next frame."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    M, store = case["M"], {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[case["state"]]

    def rounded(t):
        return t.to(store).double()

    got = []
    for w, h, mode in _groups(case["streams"]):
        n = w * h
        scene = Scene(w, h, mode, gen, 1)
        rgb, depth = scene.frame(0)
        blocks = []
        for x, mod in _inputs(rgb, depth, case["calls"]):
            v = x.double().reshape(n, -1).t()                                    # (C, n)
            C = v.shape[0]
            span = 255.0 if C > 1 else 4000.0
            mu = torch.rand((M, C, n), generator=gen, device=DEV).double() * span
            noise = torch.randn((M, C, n), generator=gen, device=DEV).double()
            mu[0] = v + 2.0 * noise[0]
            if M > 1:  # a tenth of the pixels stand on their second component
                second = torch.rand(n, generator=gen, device=DEV) < 0.1
                mu[1] = torch.where(second, mu[0], mu[1])
                mu[0] = torch.where(second, span - mu[0], mu[0])
            var = VAR_MIN[mod] * (1.0 + 3.0 * torch.rand((M, n), generator=gen, device=DEV).double())
            wt = torch.rand((M, n), generator=gen, device=DEV).double().pow(2) * 0.3 ** torch.arange(M, device=DEV).double()[:, None]
            wt[0] += 1.0
            live = torch.randint(2, M + 1, (n,), generator=gen, device=DEV) if M > 1 else torch.ones(n, device=DEV)
            empty = torch.arange(M, device=DEV)[:, None] >= live[None, :]
            wt = torch.where(empty, torch.zeros_like(wt), wt)
            wt = rounded(wt / wt.sum(0))
            var = rounded(torch.where(empty, torch.full_like(var, SIGMA0[mod] ** 2), var))
            mu = rounded(torch.where(empty[:, None, :], torch.zeros_like(mu), mu))
            order = torch.argsort(wt / var.sqrt(), dim=0, descending=True, stable=True)
            mu = torch.gather(mu, 0, order[:, None, :].expand_as(mu))
            var, wt = torch.gather(var, 0, order), torch.gather(wt, 0, order)
            blocks.append((mu.cpu().numpy(), var.cpu().numpy(), wt.cpu().numpy()))
        fuse = None
        if mode == "rgbd" and case["calls"] != "augmented":
            fuse = (torch.randint(0, 2, (n,), generator=gen, device=DEV).double().cpu().numpy(),
                    torch.randint(-3, 4, (n,), generator=gen, device=DEV).double().cpu().numpy())
        got.append((w, h, mode, blocks, fuse, rgb, depth))
    return got


def _inputs(rgb, depth, calls):
    """What each mixture of a stream sees, int32 (H, W, C), and whose constants it has (0 colour, 1 depth)."""
    if calls == "augmented":  # colour and the depth in 16 mm steps
        d8 = (depth.to(torch.int32) >> 4).clamp(max=255)
        return [(torch.cat([rgb.to(torch.int32), d8[..., None]], -1), 0)]
    return [(x.to(torch.int32), mod) for x, mod in ((rgb, 0), (depth, 1)) if x is not None]


def _canonical(blocks, fuse):
    """(mu (M, C, n), var (M, n), w (M, n)) blocks and (I, cpt) in the order gmm_read_state uses."""
    flat = []
    for mu, var, wt in blocks:
        flat += [mu.transpose(1, 0, 2).reshape(-1), var.reshape(-1), wt.reshape(-1)]
    if fuse is not None:
        flat += list(fuse)
    return np.concatenate(flat)


def _prepare_resume(s, case, gen):
    s.streams, calls = _checkpoint(case, gen.initial_seed()), case["calls"]
    s.segs = [_segmenter(w, h, mode, case["M"], case["state"], augmented=calls == "augmented")
              for w, h, mode, *_ in s.streams]
    s.saved = [_canonical(blocks, fuse) for _, _, _, blocks, fuse, _, _ in s.streams]
    frames = [(rgb, depth) for *_, rgb, depth in s.streams]
    s.batch = gmm.Batch(s.segs) if calls == "batch" else None
    handles = [seg.handle for seg in s.segs]

    def one():
        for seg, saved in zip(s.segs, s.saved):
            seg.write_state(saved)
        if calls == "batch":
            s.batch.apply(frames)
        elif calls == "static":
            _abi.gmm_batch_apply_static(handles, [
                _abi.stream_io(rgb, depth, seg.fg_rgb, seg.fg_depth, seg.fused) for seg, (rgb, depth) in zip(s.segs, frames)])
        else:
            for seg, (rgb, depth) in zip(s.segs, frames):
                if calls == "augmented":
                    seg.apply_augmented(rgb, depth)
                elif seg.fused is not None:
                    seg.apply_fused(rgb, depth)
                else:
                    seg.apply(rgb, depth)
        out = []
        for seg in s.segs:
            masks = [seg.fg] if calls == "augmented" else [seg.fg_rgb, seg.fg_depth, seg.fused]
            out.append({"masks": [m for m in masks if m is not None], "state": seg.read_state()})
        return out

    s.run = one


def exact(case, seed):
    """The resumed state after its frame, in 64 bits; the other cases return masks or counts alone."""
    if case["kind"] != "resume":
        return None
    out = []
    for w, h, mode, blocks, fuse, rgb, depth in _checkpoint(case, seed):
        after, fgs = [], []
        for (mu, var, wt), (x, mod) in zip(blocks, _inputs(rgb, depth, case["calls"])):
            v = x.cpu().numpy().astype(np.float64).reshape(w * h, -1).T
            hole = None if mod == 0 and case["calls"] != "augmented" else depth.cpu().numpy().reshape(-1) == 0
            new, fg = _mixture_step(mu, var, wt, v, mod, hole)
            after.append(new)
            fgs.append(fg)
        state = _canonical(after, _list1(fuse, fgs[0], fgs[1]) if fuse is not None else None)
        out.append({"masks": [None] * (3 if fuse is not None else 1), "state": state})
    return out


def _mixture_step(mu, var, wt, x, mod, hole):
    """One frame of the adaptive mixture of every pixel: x (C, n) into mu (M, C, n), var, wt (M, n);
    a pixel without a reading (hole) keeps its state."""
    M, n = var.shape
    a, pix = float(np.float32(ALPHA)), np.arange(n)
    d2 = ((x[None] - mu) ** 2).sum(1)
    hits = (wt > 0) & (d2 < K * K * var)
    matched = hits.any(0)
    t = np.where(matched, hits.argmax(0), M - 1)       # the first match, or the last rank replaced
    m0, v0, w0 = mu[t, :, pix].T, var[t, pix], wt[t, pix]
    m1 = np.where(matched, (1 - a) * m0 + a * x, x)
    r2 = ((x - m1) ** 2).sum(0)
    v1 = np.where(matched, np.maximum(VAR_MIN[mod], (1 - a) * v0 + a * r2), SIGMA0[mod] ** 2)
    w1 = np.where(matched, (1 - a) * w0 + a, float(np.float32(W_INIT)))
    nm, nv, nw = mu.copy(), var.copy(), (1 - a) * wt
    nm[t, :, pix], nv[t, pix], nw[t, pix] = m1.T, v1, w1
    nw /= nw.sum(0)
    order = np.argsort(-nw / np.sqrt(nv), axis=0, kind="stable")
    nm = np.take_along_axis(nm, order[:, None, :], 0)
    nv, nw = np.take_along_axis(nv, order, 0), np.take_along_axis(nw, order, 0)
    q = (order == t[None]).argmax(0)
    over = np.cumsum(nw, 0) > float(np.float32(T))
    B = np.where(over.any(0), over.argmax(0) + 1, M)
    fg = ~matched | (q >= B)
    if hole is not None:
        nm, nv, nw = np.where(hole, mu, nm), np.where(hole, var, nv), np.where(hole, wt, nw)
        fg &= ~hole
    return (nm, nv, nw), fg


def _list1(fuse, r, d):
    """The fused bit and counter after one step of the fusion rule."""
    I, c = fuse[0].astype(bool), fuse[1]
    same, top, low = r == d, c == 3, c == -3
    I1 = np.where(same, d, np.where(top, r, np.where(low, d, I)))
    c1 = np.where(same | top | low, 0.0, c + np.where(I == r, 1.0, -1.0))
    return I1.astype(np.float64), c1


# ---- evaluation ----------------------------------------------------------------------------------

def _prepare_evaluate(s, case, gen):
    w, h = case["width"], case["height"]
    s.npix, s.pairs = w * h, []
    for _ in range(case["masks"]):
        scene = Scene(w, h, "", gen, 1)
        truth = torch.zeros((h, w), dtype=torch.bool, device=DEV)
        for x, y, side in scene.boxes[0]:
            truth[y:y + side, x:x + side] = True
        wrong = torch.rand((h, w), generator=gen, device=DEV) < 0.03
        s.pairs.append((quality.pack_mask(truth ^ wrong), quality.pack_mask(truth)))
    s.counts = torch.zeros((case["masks"], 4), dtype=torch.int64, device=DEV)

    def one():
        for (pred, truth), counts in zip(s.pairs, s.counts):
            _abi.gmm_mask_confusion(pred, truth, s.npix, counts)
        return s.counts

    s.run = one


# ---- what a pass cannot do without ---------------------------------------------------------------

def _model_work(w, h, mode, M, state, augmented=False, fused=True):
    """(bytes, flops) of one frame of one stream: the frame read, the masks written, and of the state
    what a frame that keeps every pixel on its first component reads and writes (that component, the
    key that confirms its rank, and in 16 bits every weight); a fresh model writes its components."""
    n, size = w * h, 4 if state == "f32" else 2
    total = flops = 0.0
    channels = [4] if augmented else [C for C, m in ((3, "rgb"), (1, "d")) if m in mode]
    for C in channels:
        weights = 1 if state == "f32" else M
        total += n * size * (2 * (C + 1 + weights) + (1 if M > 1 else 0)) + n * (C if C == 3 else 2 if C == 1 else 5) + n / 8
        flops += n * (10 * C + 15)
    if mode == "rgbd" and fused and not augmented:
        total += n * (2 + 1 / 8)
        flops += 4 * n
    return total, flops


def work(case):
    kind = case["kind"]
    if kind == "evaluate":
        words = gmm.mask_words(case["width"] * case["height"])
        return {"bytes": case["masks"] * (16.0 * words + 32), "flops": case["masks"] * 12.0 * words}
    if kind == "stream":
        b, f = _model_work(case["width"], case["height"], case["modalities"], case["M"], case["state"],
                           case["calls"] == "augmented", case["calls"] in ("fused", "split"))
        return {"bytes": b * (4 if case["fresh"] else 1), "flops": f * (4 if case["fresh"] else 1)}
    b = f = 0.0
    for w, h, mode in _groups(case["streams"]):
        augmented = case["calls"] == "augmented" if kind == "resume" else False
        x, y = _model_work(w, h, mode, case["M"], case["state"], augmented)
        b, f = b + x, f + y
        if kind == "resume":  # the canonical state in and out
            values = 6 * case["M"] if augmented else ((5 * case["M"] if "rgb" in mode else 0) + (3 * case["M"] if "d" in mode else 0)
                                                      + (2 if mode == "rgbd" else 0))
            b += 16.0 * w * h * values
    return {"bytes": b, "flops": f}
