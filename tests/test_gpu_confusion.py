"""gmm_mask_confusion at the ends of its ranges: one lane's words, one block's, several blocks', the
last word's valid bits, and pad bits that must not count."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2110_14934_amd import _abi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npix", [1, 63, 64, 65, 64 * 1024, 64 * 1024 + 1, 64 * 4096 + 17, 64 * 16384, 64 * 16384 + 1,
                                  64 * 20480 - 5, 64 * 70001 + 3])
def test_counts_match_popcounts(npix):
    rng = np.random.default_rng(npix)
    words = (npix + 63) // 64
    p, t = (rng.integers(0, 1 << 64, words, dtype=np.uint64) for _ in range(2))  # pad bits set at random
    pad = words * 64 - npix
    pb, tb = (np.unpackbits(x.view(np.uint8), bitorder="little")[:words * 64 - pad].astype(bool) for x in (p, t))
    counts = torch.full((4,), -7, dtype=torch.int64, device="cuda")
    dev = [torch.from_numpy(x.view(np.int64)).cuda() for x in (p, t)]
    for _ in range(2):  # overwritten, not added to
        _abi.gmm_mask_confusion(dev[0], dev[1], npix, counts)
    assert counts.tolist() == [int((pb & tb).sum()), int((pb & ~tb).sum()), int((~pb & ~tb).sum()), int((~pb & tb).sum())]
