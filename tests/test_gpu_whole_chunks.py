"""One whole chunk per workgroup (small states) against the CPU oracle: every
workgroup size, chunks at and around its vectors, capped grids (a workgroup
then takes several chunks), payload gaps, and the same tables with the path
switched off."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2509_03047_amd import workloads as W  # noqa: E402
from tests.test_gpu_parity_small import _check_against_oracle  # noqa: E402


@pytest.mark.parametrize("grid", ["0", "3"])
@pytest.mark.parametrize("limit", ["0", "4000000000"])
@pytest.mark.parametrize("C", [16, 64, 1024, 2048, 4096, 8192, 16384, 32768, 65536])
def test_whole_chunks_match_oracle(C, limit, grid, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("FLASHRESTORE_SMALL", limit)
    monkeypatch.setenv("FLASHRESTORE_MAX_GRID", grid)
    rng = np.random.default_rng(C + int(grid))
    for it, seg in enumerate((16, 16, 4096)):
        # sizes in bytes around none, one and two chunks: parameter images (2 n)
        # with their masters (4 n), plain fp32 and bf16 entries, empty ones
        rows, so, do = [], 0, 0
        for k, nb in enumerate([0, 4, 12, C - 4, C, C + 4, 2 * C - 8, 2 * C, 2 * C + 4, 3 * C + 12]):
            n = max(nb, 0) // 4
            if (k + it) % 2 == 0:
                rows.append([so, do, n, W.BF16, len(rows) + 1])
                so, do = so + -(-2 * n // 16) * 16 + 16 * it, do + -(-2 * n // 16) * 16
            rows.append([so, do, n, W.F32, -1])
            so, do = so + 4 * -(-n // 4) * 4, do + 4 * -(-n // 4) * 4 + 48 * it
            rows.append([so, do, 2 * n + 1, W.BF16, -1])
            so, do = so + -(-(4 * n + 2) // 16) * 16, do + -(-(4 * n + 2) // 16) * 16
        t = np.array([tuple(r) for r in rows], dtype=W.TABLE_DTYPE)
        src = W.random_tiny_state(t, so, rng)
        _check_against_oracle(t, C, src, so, do, corrupt_rng=rng, tag=f"C={C} seg={seg} it={it}", seg=seg)


def test_states_around_the_size_rule_match_oracle():
    """States just below and above the sizes at which operations change from
    whole chunks to walks (64 MiB with whole 64 KiB chunks)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(7)
    for extra in (-4, 0, 4):
        n = (64 << 20) // 4 + extra
        t = np.array([(0, 0, n, W.F32, -1)], dtype=W.TABLE_DTYPE)
        nb = -(-4 * n // 16) * 16
        src = W.random_tiny_state(t, nb, rng)
        _check_against_oracle(t, 1 << 16, src, nb, nb, corrupt_rng=rng, tag=f"64 MiB {extra:+d}")


@pytest.mark.parametrize("C,mb,align,seg,pack,unpack", [
    (4096, 2000, 16, 16, True, False), (4096, 900, 16, 16, True, True), (4096, 900, 256, 16, True, False),
    (2048, 2000, 16, 4096, True, False), (2048, 120, 16, 16, True, True), (2048, 200, 16, 16, True, False),
    (1024, 600, 16, 16, True, False), (1024, 600, 16, 4096, False, False), (1024, 500, 16, 4096, True, False),
    (1 << 15, 300, 256, 16, True, False), (1 << 15, 400, 256, 16, False, False), (1 << 14, 400, 256, 16, True, False),
    (1 << 16, 60, 256, 16, True, True), (1 << 16, 80, 256, 16, True, False), (1 << 16, 600, 256, 16, False, False),
])
def test_which_states_take_whole_chunks(C, mb, align, seg, pack, unpack, monkeypatch):
    """The sizes at which pack and unpack change from whole chunks to walks, by
    chunk size and alignment of the side written (plan info: 5 is whole
    chunks).  Plans only: no state is built."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_03047_amd import flashrestore as F

    monkeypatch.delenv("FLASHRESTORE_SMALL", raising=False)
    per = (mb * 1_000_000 // 4 // 16 // 4096 * 4096) + (4 if align == 16 else 0)  # four entries
    step = 16 * per + (0 if align == 16 else -16 * per % align)
    t = np.array([(k * step, k * step, 4 * per, W.F32, -1) for k in range(4)], dtype=W.TABLE_DTYPE)
    info = F.Plan(t, C, 4 * step, 4 * step, segment_align=seg).info
    assert ((info["pack_walk"] == 5), (info["unpack_walk"] == 5)) == (pack, unpack), info
