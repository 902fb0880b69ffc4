"""Bitmaps and counts written by the last workgroup to arrive: chunk counts
around one bitmap word, one group of words and the size from which a finalize
launch takes over, several calls in a row on one plan (each has to leave the
arrival words as it found them), none, some and all chunks set."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2509_03047_amd import flashrestore as F  # noqa: E402
from paper_2509_03047_amd import workloads as W  # noqa: E402

C = 64


@pytest.mark.parametrize("n", [1, 31, 32, 33, 2048, 2049, 4097, 8192, 8193])
def test_bits_and_counts_over_calls_in_a_row(n, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("FLASHRESTORE_SMALL", str(1 << 30))
    # a parameter image with its master (three chunks to a workgroup) and a plain entry
    p = 16 * ((n - 1) // 6)  # p parameters: p / 32 + p / 16 chunks
    used = -(-2 * p // C) + -(-4 * p // C)
    rows = [(0, 0, p, W.BF16, 1), (2 * p, 2 * p, p, W.F32, -1), (6 * p, 6 * p, (n - used) * C // 4, W.F32, -1)]
    t = np.array(rows, dtype=W.TABLE_DTYPE)
    nb = 6 * p + (n - used) * C
    plan = F.Plan(t, C, nb, nb)
    assert plan.n_chunks == n
    rng = np.random.default_rng(n)
    src = torch.zeros(nb, dtype=torch.uint8, device="cuda")
    src[6 * p:] = torch.from_numpy(rng.integers(0, 256, size=nb - 6 * p, dtype=np.uint8)).cuda()
    payload, sums, dst = plan.empty_payload(), plan.empty_sums(), torch.zeros_like(src)
    bits, count = plan.empty_bitmap().fill_(-1), plan.empty_counter().fill_(-1)
    plan.pack(src, payload, sums)

    def check(want, what):
        got = F.bitmap_indices(bits, n)
        assert int(count.item()) == len(want), what
        assert np.array_equal(got, want), what
        bits.fill_(-1), count.fill_(-1)

    for k, share in enumerate((0.0, 0.1, 1.0, 0.0, 0.5)):
        bad = np.flatnonzero(rng.random(n) < share)
        sent = sums.clone()
        sent[torch.from_numpy(bad).cuda(), k % 2] ^= 1 << (k * 13)
        plan.unpack(payload, sent, dst, bits, count)
        check(bad, f"unpack {share}")
        assert torch.equal(dst, src)
        plan.compare_sums(sums, sent, bits, count)
        check(bad, f"sums {share}")
        other = src.clone()
        at = np.concatenate([[0], np.cumsum([-(-2 * p // C), -(-4 * p // C)])])  # first chunk of each entry
        e = np.searchsorted(at, bad, side="right") - 1
        e = np.where((p == 0) & (e < 2), 2, e)
        byte = np.array([r[0] for r in rows])[e] + (bad - at[e]) * C
        other[torch.from_numpy(byte).cuda()] ^= 0x40
        for with_sums in (False, True):
            a, b = (plan.empty_sums(), plan.empty_sums()) if with_sums else (None, None)
            plan.verify_replicas(src, other, bits, count, a, b)
            check(bad, f"compare {share} {with_sums}")
        # the differing chunks as a list, repaired
        plan.compare_sums(sums, sent, bits, count)
        flagged = bits.clone()
        pay, ls, cnt = plan.empty_delta_payload(), plan.empty_sums(), torch.zeros(2, dtype=torch.int64, device="cuda")
        plan.pack_flagged(src, flagged, pay, ls, cnt)
        assert int(cnt[0]) == len(bad)
        wrong = np.flatnonzero(rng.random(len(bad)) < 0.3)
        ls[torch.from_numpy(wrong).cuda(), 0] ^= 1
        plan.unpack_flagged(pay, ls, flagged, other, bits, count)
        check(wrong, f"list {share}")
        if p == 0 or share in (0.0, 1.0):
            assert torch.equal(other, src)


def test_calls_after_overlapping_ones_are_right(monkeypatch):
    """Whole-state calls of one plan on two streams without ordering (against
    the rule: their own bits and counts are undefined, their bytes are not)
    leave nothing behind for the calls after them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("FLASHRESTORE_SMALL", str(1 << 30))
    n = 4097
    t = np.array([(0, 0, n * C // 4, W.F32, -1)], dtype=W.TABLE_DTYPE)
    plan = F.Plan(t, C, n * C, n * C)
    rng = np.random.default_rng(9)
    src = torch.from_numpy(rng.integers(0, 256, size=n * C, dtype=np.uint8)).cuda()
    payload, sums, dst = plan.empty_payload(), plan.empty_sums(), torch.zeros_like(src)
    plan.pack(src, payload, sums)
    other = src.clone()
    want = np.flatnonzero(rng.random(n) < 0.2)
    other[torch.from_numpy(want * C).cuda()] ^= 1
    mine = [(plan.empty_bitmap(), plan.empty_counter(), torch.cuda.Stream()) for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(50):
        (b0, c0, s0), (b1, c1, s1) = mine
        plan.verify_replicas(src, other, b0, c0, stream=s0)
        plan.unpack(payload, sums, dst, b1, c1, stream=s1)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)
    for bits, count, _ in mine:
        plan.verify_replicas(src, other, bits.fill_(-1), count.fill_(-1))
        assert int(count.item()) == want.size and np.array_equal(F.bitmap_indices(bits, n), want)
        plan.unpack(payload, sums, dst, bits.fill_(-1), count.fill_(-1))
        assert int(count.item()) == 0 and F.bitmap_indices(bits, n).size == 0
