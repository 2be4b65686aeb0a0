"""State I/O on the device: every canonical value is rounded once to the storage type and comes
back exactly, at the edges of the layout and of the conversion buffer."""
from __future__ import annotations

import numpy as np
import pytest

from oracle.mixture import round_to_storage
from paper_2110_14934_amd import GMM_DEPTH, GMM_RGB, Segmenter

pytestmark = pytest.mark.gpu

RGBD = GMM_RGB | GMM_DEPTH
# one pixel; a ragged tile; a canonical block that ends inside a buffer's length and one whose
# planes straddle several; more pixels than half a buffer (2^19) holds, for the List 1 elements
SHAPES = [(1, 1, RGBD, 5), (65, 3, RGBD, 3), (161, 121, GMM_RGB, 4), (161, 121, GMM_DEPTH, 2), (512, 424, RGBD, 5),
          (725, 724, RGBD, 1)]


def rounded(v, dtype):
    """The value stored: one rounding to nearest even, past the largest finite value to infinity."""
    if dtype == "f16":
        with np.errstate(over="ignore"):
            return v.astype(np.float16).astype(np.float64)
    return round_to_storage(v, dtype)


def values(n, dtype, rng):
    """Doubles that need rounding: spread over the type's range, halfway cases, subnormals, zeros."""
    lo, p = {"f32": (-149, 24), "f16": (-24, 11), "bf16": (-133, 8)}[dtype]
    hi = 15 if dtype == "f16" else 127
    v = np.ldexp(1.0 + rng.random(n), rng.integers(lo - 2, hi, n))
    ties = np.ldexp(rng.integers(2 ** (p - 1), 2 ** p, n) + 0.5, rng.integers(lo, hi - p, n))
    v = np.where(rng.random(n) < 0.3, ties, v) * rng.choice([-1.0, 1.0], n)
    return np.where(rng.random(n) < 0.05, 0.0, v)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("w,h,modalities,M", SHAPES)
def test_write_rounds_once_and_read_is_exact(w, h, modalities, M, dtype):
    rng = np.random.default_rng([w, h, M])
    n, both = w * h, modalities == RGBD
    seg = Segmenter(w, h, modalities, M, state_dtype=dtype)
    params = M * n * ((5 if modalities & GMM_RGB else 0) + (3 if modalities & GMM_DEPTH else 0))
    state = values(params, dtype, rng)
    expect = rounded(state, dtype)
    if both:
        fuse = np.concatenate([rng.integers(0, 2, n), rng.integers(-3, 4, n)]).astype(np.float64)
        state, expect = np.concatenate([state, fuse]), np.concatenate([expect, fuse])
    seg.write_state(state)
    got = seg.read_state()
    assert np.array_equal(got, expect)
    seg.write_state(got)  # what was read is representable: it goes back unchanged
    assert np.array_equal(seg.read_state(), expect)


@pytest.mark.parametrize("dtype,largest", [("f16", 65504.0), ("bf16", 3.3895313892515355e38)])
def test_overflow_rounds_to_infinity(dtype, largest):
    seg = Segmenter(4, 1, GMM_DEPTH, 1, state_dtype=dtype)
    half = largest * (2.0 ** (-12 if dtype == "f16" else -9))  # under half an ulp
    v = np.array([largest, largest + half, largest * 1.01, -np.inf] + [1.0] * 8)
    seg.write_state(v)
    assert seg.read_state()[:4].tolist() == [largest, largest, np.inf, -np.inf]


def test_four_channel_state_round_trips():
    rng = np.random.default_rng(4)
    seg = Segmenter(67, 5, RGBD, 5, augmented=True)
    v = rng.random(6 * 5 * 67 * 5)
    seg.write_state(v)
    assert np.array_equal(seg.read_state(), v.astype(np.float32).astype(np.float64))
