"""The batched launch's own choices: which stream a block's piece belongs to (the search over the
streams' first tiles) and how the default shape cuts tiles, bit for bit against one launch per stream."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2110_14934_amd import GMM_DEPTH, GMM_RGB, Batch, Segmenter, _abi

pytestmark = pytest.mark.gpu
MODS = (GMM_RGB | GMM_DEPTH, GMM_RGB, GMM_DEPTH)


def _streams(sizes, dtype, alphas):
    return [Segmenter(w, h, MODS[i % 3], 2, state_dtype=dtype, alpha=alphas[i % len(alphas)])
            for i, (w, h) in enumerate(sizes)]


def _frames(sizes, gen):
    out = []
    for i, (w, h) in enumerate(sizes):
        rgb = torch.randint(0, 256, (h, w, 3), generator=gen, device="cuda").to(torch.uint8)
        depth = (torch.randint(0, 3, (h, w), generator=gen, device="cuda") * 900).to(torch.int32).to(torch.uint16)
        m = MODS[i % 3]
        out.append((rgb if m & GMM_RGB else None, depth if m & GMM_DEPTH else None))
    return out


def _check(sizes, call, dtype, sets=3, alphas=(0.05,)):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(sizes))
    one, many = _streams(sizes, dtype, alphas), _streams(sizes, dtype, alphas)
    batch = Batch(many) if call == "apply" else None
    for _ in range(sets):
        frames = _frames(sizes, gen)
        for seg, (rgb, depth) in zip(one, frames):
            seg.apply_fused(rgb, depth) if seg.fused is not None else seg.apply(rgb, depth)
        ios = [_abi.stream_io(rgb, depth, s.fg_rgb, s.fg_depth, s.fused) for s, (rgb, depth) in zip(many, frames)]
        if call == "apply":
            _abi.gmm_batch_apply(batch.handle, ios)
        else:
            _abi.gmm_batch_apply_static([s.handle for s in many], ios)
        for a, b in zip(one, many):
            for name in ("fg_rgb", "fg_depth", "fused"):
                if getattr(a, name) is not None:
                    assert torch.equal(getattr(a, name), getattr(b, name))
    for i in {0, 1, len(sizes) // 2, len(sizes) - 1} & set(range(len(sizes))):
        assert np.array_equal(one[i].read_state(), many[i].read_state())


# one stream, powers of two and their neighbours
@pytest.mark.parametrize("n,call", [(1, "apply"), (63, "static"), (64, "apply"), (65, "static"), (130, "apply"),
                                    (1024, "static"), (4097, "apply")])
def test_every_piece_finds_its_stream(n, call):
    sizes = [((1, 1), (300, 1), (33, 40), (1025, 1))[(i * 7 + i // 5) % 4] for i in range(n)]
    _check(sizes, call, "f32", sets=2)


# widths around the pieces' and tiles' ends; few pixels in all (pieces of 256) and many (of 512)
@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("extra", [[], [(1920, 1093)]])
def test_default_pieces_cover_every_pixel(extra, dtype):
    sizes = [(w, 1) for w in (1, 63, 255, 256, 257, 511, 512, 513, 767, 769, 1023, 1024, 1025, 2049)]
    _check(sizes + extra, "apply", dtype)


# descriptors travel as kernel arguments, the model constants once per run of equal ones: none alike,
# short and long runs, runs that end inside and at the end of a launch's 32 (16) streams, and the
# largest batch that goes this way with its neighbours
@pytest.mark.parametrize("call", ["apply", "static"])
@pytest.mark.parametrize("n,alphas", [(40, (0.05, 0.02)), (70, (0.05,) * 32 + (0.02,) * 5), (33, (0.05,) * 32 + (0.1,)),
                                      (17, (0.05,) * 3 + (0.1,)), (32, (0.05,)), (63, (0.05,)), (64, (0.05,)),
                                      (65, (0.05,)), (64, (0.05,) * 20 + (0.1,) * 12)])
def test_streams_keep_their_own_descriptors(n, alphas, call):
    _check([(65 + i, 3) for i in range(n)], call, "f16", alphas=alphas)
