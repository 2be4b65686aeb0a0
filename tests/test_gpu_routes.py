"""Every entry point on every route it can take gives what one launch per stream gives, bit for bit:
rows streamed past the caches or kept in them, descriptors in kernel arguments or in tables that are
used again, blocks that walk tiles, host buffers used in place or copied, and the mixes of these.
Which route a call takes is checked without a GPU (tests/routes_check.cpp)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2110_14934_amd import GMM_DEPTH, GMM_RGB, Batch, Segmenter, _abi

pytestmark = pytest.mark.gpu
BOTH = GMM_RGB | GMM_DEPTH
SIZES = [(160, 120, BOTH), (97, 61, GMM_RGB), (64, 48, GMM_DEPTH), (333, 77, BOTH), (1, 1, BOTH), (130, 1, BOTH)]
MASKS = ("fg_rgb", "fg_depth", "fused")


def scene(w, h, m, frames, seed):
    """A static background with sensor noise, missing depth and pixels that jump: every path of the
    per-pixel body."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rnd = lambda *s: torch.rand(s, generator=gen, device="cuda")
    bg, bd = rnd(h, w, 3) * 255, 500 + 3000 * rnd(h, w)
    out = []
    for _ in range(frames):
        jump = rnd(h, w) < 0.1
        rgb = torch.where(jump[..., None], 255 - bg, bg) + 4 * rnd(h, w, 3) - 2
        dep = torch.where(jump, bd / 2, bd) + 6 * rnd(h, w)
        dep = torch.where(rnd(h, w) < 0.05, torch.zeros_like(dep), dep)
        out.append((rgb.round().clamp(0, 255).to(torch.uint8) if m & GMM_RGB else None,
                    dep.round().to(torch.int32).to(torch.uint16) if m & GMM_DEPTH else None))
    return out


def segmenters(sizes, dtype, alphas=(0.05,), M=5, **more):
    return [Segmenter(w, h, m, M, state_dtype=dtype, alpha=alphas[i % len(alphas)], **more) for i, (w, h, m) in enumerate(sizes)]


def step(seg, rgb, depth, how="fused"):
    if how == "augmented":
        return [seg.apply_augmented(rgb, depth).clone()]
    if how == "fused" and seg.fused is not None:
        seg.apply_fused(rgb, depth)
    else:
        seg.apply(rgb, depth)
        if how == "split" and seg.fused is not None:
            seg.fuse(seg.fg_rgb, seg.fg_depth)
    return [getattr(seg, k).clone() if getattr(seg, k) is not None else None for k in MASKS]


def reference(sizes, frames, dtype, how="fused", **more):
    """Masks of every frame set and the final states, one stream after the other, one launch a frame."""
    masks, states = [], []
    for seg, sc in zip(segmenters(sizes, dtype, **more), frames):
        masks.append([step(seg, rgb, depth, how) for rgb, depth in sc])
        states.append(seg.read_state())
        seg.close()
    return masks, states


def same(got, want):
    for a, b in zip(got, want):
        assert (a is None) == (b is None)
        if a is not None:
            assert torch.equal(a.cpu(), b.cpu())


class Ticks:
    """An executor over the handles of some segmenters, with host buffers of chosen kinds."""

    def __init__(self, segs, ring=3, tuning=None):
        self.x = _abi.gmm_exec_create(0, ring)
        if tuning:
            _abi.gmm_exec_set_tuning(self.x, *tuning)
        self.segs = segs
        for s in segs:
            _abi.gmm_exec_attach(self.x, s.handle)

    def prepare(self, frames, kinds=("pinned",), wanted=lambda i, k: True, turn=0):
        """A tick's items; kinds[(stream + buffer + turn) % n] says where each host buffer lies. Returns
        them, the buffers to keep and the masks per stream."""
        items, keep, masks = [], [], []
        for i, (s, (rgb, depth)) in enumerate(zip(self.segs, frames)):
            kind = lambda b: kinds[(i + b + turn) % len(kinds)]
            r = host(rgb, kind(0)) if rgb is not None else None
            d = host(depth, kind(1)) if depth is not None else None
            o = [host(torch.zeros_like(getattr(s, k)), kind(2 + j)) if getattr(s, k) is not None and wanted(i, j) else None
                 for j, k in enumerate(MASKS)]
            it = _abi.gmm_exec_item()
            it.handle = s.handle
            it.host_rgb = r.data_ptr() if r is not None else None
            it.host_depth = d.data_ptr() if d is not None else None
            for name, b in zip(("host_fg_rgb", "host_fg_depth", "host_fused"), o):
                setattr(it, name, b.data_ptr() if b is not None else None)
            items.append(it)
            keep.append((r, d, o))
            masks.append(o)
        return items, keep, masks

    def launch(self, items):
        _abi.gmm_exec_launch(self.x, items)

    def drain(self):
        _abi.gmm_exec_drain(self.x)
        return _abi.gmm_exec_poll(self.x)

    def close(self):
        self.drain()
        for s in self.segs:
            _abi.gmm_exec_detach(self.x, s.handle)
        _abi.gmm_exec_destroy(self.x)


_hip, _allocated = None, []


def host(t, kind):
    """The tensor in host memory: pageable, page-locked ("pinned"), page-locked but not aligned for the
    kernel ("odd"), or page-locked with flags that leave its coherence open or deny it."""
    t = t.cpu().contiguous()
    if kind == "pageable":
        return t.clone()
    if kind == "pinned":
        return t.pin_memory()
    if kind == "odd":
        buf = torch.zeros(t.numel() * t.element_size() + 16, dtype=torch.uint8).pin_memory()
        v = buf[1:1 + t.numel() * t.element_size()]
        v.copy_(t.reshape(-1).view(torch.uint8))
        return v
    global _hip
    _hip = _hip or ctypes.CDLL("libamdhip64.so")
    n = t.numel() * t.element_size()
    p = ctypes.c_void_p()
    flags = {"portable": 0x1, "noncoherent": 0x80000000}[kind]
    assert _hip.hipHostMalloc(ctypes.byref(p), ctypes.c_size_t(n), ctypes.c_uint(flags)) == 0
    _allocated.append(p)
    v = torch.frombuffer((ctypes.c_uint8 * n).from_address(p.value), dtype=torch.uint8)
    v.copy_(t.reshape(-1).view(torch.uint8))
    return v


@pytest.fixture(autouse=True)
def give_back():
    yield
    torch.cuda.synchronize()
    while _allocated:
        _hip.hipHostFree(_allocated.pop())


def as_words(b):
    return None if b is None else b if b.dtype == torch.int64 else b.clone().view(torch.int64)


@pytest.fixture(scope="module")
def spacer():
    """A stream whose frame alone passes more bytes than the last-level cache holds: a frame of it
    between two frames of another stream makes that one's rows stream."""
    seg = Segmenter(3072, 2048, BOTH, 5)
    rgb = torch.zeros((2048, 3072, 3), dtype=torch.uint8, device="cuda")
    depth = torch.ones((2048, 3072), dtype=torch.int32, device="cuda").to(torch.uint16)
    yield lambda: seg.apply(rgb, depth)
    seg.close()


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("entry", ["fused", "split", "augmented", "batch", "static", "exec", "exec-copied", "batch-40",
                                   "static-40", "exec-40"])
def test_streamed_rows_equal_kept_rows(entry, dtype, spacer):
    T = 5
    sizes = SIZES if not entry.endswith("-40") else [(65 + i, 3, (BOTH, GMM_RGB, GMM_DEPTH)[i % 3]) for i in range(40)]
    if entry == "augmented":
        sizes = [(w, h, BOTH) for w, h, _ in sizes]
    frames = [scene(w, h, m, T, i) for i, (w, h, m) in enumerate(sizes)]
    how = entry if entry in ("split", "augmented") else "fused"
    more = {"augmented": True} if entry == "augmented" else {}
    want, states = reference(sizes, frames, dtype, how, **more)
    segs = segmenters(sizes, dtype, **more)
    batch = Batch(segs) if entry.startswith("batch") else None
    ticks = Ticks(segs) if entry.startswith("exec") else None
    try:
        for t in range(T):
            spacer()
            fs = [sc[t] for sc in frames]
            if batch is not None:
                batch.apply(fs)
            elif entry.startswith("static"):
                ios = [_abi.stream_io(r, d, s.fg_rgb, s.fg_depth, s.fused) for s, (r, d) in zip(segs, fs)]
                _abi.gmm_batch_apply_static([s.handle for s in segs], ios)
            elif ticks is not None:
                items, keep, got = ticks.prepare(fs, ("pageable",) if entry.endswith("copied") else ("pinned",))
                ticks.launch(items)
                ticks.drain()
            else:
                got = [step(s, r, d, how) for s, (r, d) in zip(segs, fs)]
            for i, s in enumerate(segs):
                g = got[i] if ticks is not None or entry in ("fused", "split", "augmented") else [getattr(s, k) for k in MASKS]
                same(g, want[i][t])
        for s, st in zip(segs, states):
            assert np.array_equal(s.read_state(), st)
    finally:
        if batch is not None:
            batch.close()
        if ticks is not None:
            ticks.close()
        for s in segs:
            s.close()


# 40 streams take a table, 5 and 32 equal ones the kernel's arguments, mixed constants a table also
# below 33; each call finds the tables as another left them
@pytest.mark.parametrize("alphas", [(0.05,), (0.05, 0.02)])
def test_static_tables_used_again(alphas):
    sizes = [(65 + i, 3, (BOTH, GMM_RGB, GMM_DEPTH)[i % 3]) for i in range(40)]
    sets = [list(range(40)), list(range(34)), [39, 3, 17, 0, 21], list(range(8, 40)), list(range(39, -1, -1)), list(range(33))]
    T = [sum(i in s for s in sets) for i in range(40)]
    frames = [scene(w, h, m, T[i], i) for i, (w, h, m) in enumerate(sizes)]
    want, states = reference(sizes, frames, "f32", alphas=alphas)
    segs = segmenters(sizes, "f32", alphas)
    at = [0] * 40
    for s in sets:  # back to back: no synchronisation between the calls
        ios = [_abi.stream_io(*frames[i][at[i]], segs[i].fg_rgb, segs[i].fg_depth, segs[i].fused) for i in s]
        _abi.gmm_batch_apply_static([segs[i].handle for i in s], ios)
        for i in s:
            same([getattr(segs[i], k) for k in MASKS], want[i][at[i]])
            at[i] += 1
    for s, st in zip(segs, states):
        assert np.array_equal(s.read_state(), st)
        s.close()


@pytest.mark.parametrize("tuning", [(256, 256, 1), (512, 512, 1), (256, 1024, 2)])
@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_blocks_that_walk_many_tiles(tuning, dtype):
    sizes = [(1280, 720, BOTH), (641, 479, GMM_RGB), (160, 120, GMM_DEPTH), (512, 424, BOTH)]  # 1.4 M pixels, 256 CUs
    frames = [scene(w, h, m, 3, i) for i, (w, h, m) in enumerate(sizes)]
    want, states = reference(sizes, frames, dtype)
    segs = segmenters(sizes, dtype)
    batch = Batch(segs)
    batch.set_tuning(*tuning)
    for t in range(3):
        batch.apply([sc[t] for sc in frames])
        for s, w in zip(segs, want):
            same([getattr(s, k) for k in MASKS], w[t])
    batch.close()
    for s, st in zip(segs, states):
        assert np.array_equal(s.read_state(), st)
        s.close()


KINDS = {"pageable": ("pageable",), "odd": ("odd",), "open": ("portable", "noncoherent"),
         "mixed": ("pinned", "pageable", "odd", "pinned", "noncoherent")}


# two ticks in flight, some masks not wanted (the fused one always: it runs List 1), every kind of
# buffer in turn at every frame and mask; 6 streams with their descriptors in the kernel's arguments,
# 40 and mixed constants with a table; launch shapes of the caller's
@pytest.mark.parametrize("kinds", sorted(KINDS))
@pytest.mark.parametrize("n,alphas,tuning", [(6, (0.05,), None), (6, (0.05, 0.02), (256, 1024, 1)), (40, (0.05,), None),
                                             (40, (0.05,), (512, 512, 2))])
def test_ticks_of_every_kind_of_buffer(kinds, n, alphas, tuning):
    T = 6
    sizes = (SIZES * 7)[:n]
    frames = [scene(w, h, m, T, i) for i, (w, h, m) in enumerate(sizes)]
    want, states = reference(sizes, frames, "f16", alphas=alphas)
    segs = segmenters(sizes, "f16", alphas)
    ticks = Ticks(segs, tuning=tuning)
    made = [ticks.prepare([sc[t] for sc in frames], KINDS[kinds], lambda i, j: j == 2 or (i + j + t) % 5 != 0, t)
            for t in range(T)]
    got, done = [m for _, _, m in made], []
    for t in range(T):
        while len(done) < t - 1:  # at most two in flight
            done += _abi.gmm_exec_poll(ticks.x)
        ticks.launch(made[t][0])
    done += ticks.drain()
    assert [d[0] for d in done] == list(range(1, T + 1))
    for t in range(T):
        for i in range(n):
            for j in range(3):
                if got[t][i][j] is not None:
                    assert torch.equal(as_words(got[t][i][j]), want[i][t][j].cpu()), (t, i, j)
    ticks.close()
    for s, st in zip(segs, states):
        assert np.array_equal(s.read_state(), st)
        s.close()


def test_masks_over_frames_and_over_each_other():
    """A mask may lie in the memory of the frame it comes from, or share memory with another mask: the
    frame counts as it was before the tick, and of masks in one place the last one's words stay."""
    sizes, T = [(160, 120, BOTH), (333, 77, BOTH)], 4
    frames = [scene(w, h, m, T, i) for i, (w, h, m) in enumerate(sizes)]
    want, states = reference(sizes, frames, "f32")
    segs = segmenters(sizes, "f32")
    ticks = Ticks(segs)
    for t in range(T):
        items, bufs = [], []
        shared = torch.zeros(segs[1].fg_rgb.numel(), dtype=torch.int64).pin_memory()
        for s, sc in zip(segs, frames):
            rgb, depth = host(sc[t][0], "pinned"), host(sc[t][1], "pinned")
            it = _abi.gmm_exec_item()
            it.handle, it.host_rgb, it.host_depth = s.handle, rgb.data_ptr(), depth.data_ptr()
            it.host_fg_rgb, it.host_fg_depth, it.host_fused = rgb.data_ptr() + 64, depth.data_ptr(), shared.data_ptr()
            items.append(it)
            bufs.append((rgb, depth))
        ticks.launch(items)
        ticks.drain()
        for (rgb, depth), s, w in zip(bufs, segs, want):
            n = s.fg_rgb.numel() * 8
            assert torch.equal(rgb.reshape(-1)[64:64 + n].clone().view(torch.int64), w[t][0].cpu())
            assert torch.equal(depth.reshape(-1).view(torch.uint8)[:n].clone().view(torch.int64), w[t][1].cpu())
        assert torch.equal(shared, want[1][t][2].cpu())
    ticks.close()
    for s, st in zip(segs, states):
        assert np.array_equal(s.read_state(), st)
        s.close()
