"""Chunk sums folded from the partial sums that the main kernels store (whole
chunks, which fold nothing, are switched off): every number of slices a chunk
can have in the folds' ranges (one, up to 8, 16 and more slices per whole
chunk), one slice more or less, and tiles that begin with other chunks, against
the CPU oracle (all outputs bit for bit, with a corrupted wire).  The folds of
more than 16,384 chunks of many slices run in the full-size tests."""
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2509_03047_amd import flashrestore as F  # noqa: E402
from paper_2509_03047_amd import workloads as W  # noqa: E402
from tests.test_gpu_parity_small import _check_against_oracle  # noqa: E402


def _table(C, rng, align):
    """Derived pairs and plain entries whose sizes lie around whole chunks and
    whole 4 KiB and 16 KiB slices, at offsets that are multiples of `align`."""
    sizes = sorted({b + d for b in (16, 4096, 16384, C, C + 4096, 2 * C, 2 * C + 16384, 3 * C - 4096)
                    for d in (-4, 0, 4) if b + d > 0})
    rows, so, do = [], 0, 0
    up = lambda x: -(-x // align) * align  # noqa: E731
    for k, nb in enumerate(sizes):
        n = nb // 4
        if k % 3 == 0:  # a bf16 image of 2 n bytes and its master of 4 n
            i = len(rows)
            rows.append([so, do, n, W.BF16, i + 1])
            so, do = up(so + 2 * n), up(do + 2 * n + 32)
        rows.append([so, do, n, W.F32, -1])
        so, do = up(so + 4 * n + 16 * (k % 2)), up(do + 4 * n)
    return np.array([tuple(r) for r in rows], dtype=W.TABLE_DTYPE), so, do


@pytest.mark.parametrize("align", [16, 128])
@pytest.mark.parametrize("C", [16, 1 << 12, 1 << 13, 1 << 14, 1 << 15, 1 << 16, 1 << 17, 1 << 18, 1 << 20])
def test_partial_sums_fold_to_the_oracle(C, align, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for k in [k for k in os.environ if k.startswith("FLASHRESTORE_")]:
        monkeypatch.delenv(k)
    monkeypatch.setenv("FLASHRESTORE_SMALL", "0")
    rng = np.random.default_rng(C + align)
    t, sb, db = _table(C, rng, align)
    src = W.random_tiny_state(t, sb, rng)
    info = F.Plan(t, C, sb, db).info
    assert 5 not in (info["pack_walk"], info["unpack_walk"])
    _check_against_oracle(t, C, src, sb, db, corrupt_rng=rng, tag=f"fold C={C} align={align}")


@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("n", [32768, 32769, 33000])
def test_sums_of_chunks_of_one_slice(n, swap, monkeypatch):
    """Chunks of one slice each: stored as they are up to 32,768 of them, above
    that at the slots' places, found by the chunk's id where the slots are in
    chunk order and through the table of places where they are not (the compare
    of a table that lists its tensors out of arena order)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for k in [k for k in os.environ if k.startswith("FLASHRESTORE_")]:
        monkeypatch.delenv(k)
    monkeypatch.setenv("FLASHRESTORE_SMALL", "0")
    C, rng = 256, np.random.default_rng(n)
    a, b = n // 3, n - n // 3  # chunks of the two entries, the last one ragged
    off = (0, a * C) if not swap else (b * C, 0)
    t = np.array([(off[0], 0, a * C // 4, W.F32, -1), (off[1], a * C, b * C // 4 - 3, W.F32, -1)], dtype=W.TABLE_DTYPE)
    src = W.random_tiny_state(t, n * C, rng)
    _check_against_oracle(t, C, src, n * C, n * C, corrupt_rng=rng, tag=f"n={n} swap={swap}")
