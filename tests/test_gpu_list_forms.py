"""Delta lists in every form the builder distinguishes, against the CPU
oracle: consecutive ids (no upload), scattered and dense ones (uploaded,
turned into a bitmap), plans of one block of chunk ids up to more than the
blocks fold themselves, chunks that a workgroup holds whole and larger ones,
and whole chunks switched off."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2509_03047_amd import workloads as W  # noqa: E402
from tests.test_gpu_delta import _one  # noqa: E402


def _table(n_bytes, rng):
    """Two parameter images with their masters and plain entries, ragged ends,
    about n_bytes in all, sender and receiver alike with gaps."""
    rows, off = [], 0
    for k, share in enumerate((0.3, 0.1, 0.25, 0.05, 0.3)):
        n = max(3, int(n_bytes * share) // 6 * 1 + int(rng.integers(0, 7)))
        if k % 2 == 0:
            rows.append([off, off, n, W.BF16, len(rows) + 1])
            off += -(-2 * n // 16) * 16 + 16 * k
        rows.append([off, off, n, W.F32, -1])
        off += -(-4 * n // 16) * 16
    return np.array([tuple(r) for r in rows], dtype=W.TABLE_DTYPE), off


@pytest.mark.parametrize("small", [None, "0"])
@pytest.mark.parametrize("C,n_bytes", [
    (1 << 16, 1 << 20),    # a few chunks: one block
    (1 << 12, 2 << 20),    # about 600 chunks: every block builds the others' maps
    (1 << 10, 4 << 20),    # about 4,700 chunks: blocks fold the others' maps
    (1 << 4, 9 << 20),     # more than 524,288 chunks: the scan of its own
    (1 << 17, 9 << 20),    # chunks larger than a workgroup holds
])
def test_list_forms_match_oracle(C, n_bytes, small, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if small is not None:
        monkeypatch.setenv("FLASHRESTORE_SMALL", small)
    rng = np.random.default_rng(C)
    t, nb = _table(n_bytes, rng)
    src = W.random_tiny_state(t, nb, rng)
    recv = rng.integers(0, 256, size=nb, dtype=np.uint8)
    sizes = t["numel"].astype(np.int64) * np.where(t["dtype"] == W.F32, 4, 2)
    n = int((-(-sizes // C)).sum())
    first = np.concatenate([[0], np.cumsum(-(-sizes // C))])  # of each entry
    lists = [np.arange(n), np.array([0]), np.array([n - 1]),
             np.arange(first[1], first[2] + 1), np.arange(n // 3, max(n // 3 + 1, 2 * n // 3))]
    lists.append(np.unique(rng.integers(0, n, size=max(1, n // 3))))         # dense
    lists.append(np.unique(rng.integers(0, n, size=min(n, 40))))             # scattered
    lists.append(np.unique(np.concatenate([first[:-1], first[1:] - 1])))     # ends of entries
    for k in (256 * C, 256 * C + 1):  # longer lists of small chunks are unpacked by slices
        if k + 7 <= n:
            lists += [np.arange(k) + 7, np.delete(np.arange(n), 9)[:k]]
    if n > 2:
        lists.append(np.delete(np.arange(n), n // 2))                        # all but one
    for k, ids in enumerate(lists):
        for seg in (None, 4096) if k % 3 == 0 and n < 10000 else (None,):
            _one(t, C, src, recv, ids.astype(np.uint32), rng, f"C={C} list {k} seg={seg}", seg=seg)


@pytest.mark.parametrize("C", [1 << 14, 1 << 15, 1 << 16])
def test_long_host_lists_write_every_bit_and_the_count(C):
    """Host lists around the length from which lists of large chunks take a
    finalize launch (8,192; below 32 KiB chunks the last workgroup to arrive
    writes bits and count at any length): consecutive and scattered ids, none,
    some and all chunks bad."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_03047_amd import flashrestore as F

    rng = np.random.default_rng(C + 1)
    rows, off = [], 0
    for n in [C // 4 + 9] + [int(x) for x in rng.integers(1, 9, size=9000)]:  # one entry of two chunks
        rows.append((off, off, n, W.F32, -1))
        off += -(-4 * n // 16) * 16
    t = np.array(rows, dtype=W.TABLE_DTYPE)
    plan = F.Plan(t, C, off, off)
    n = plan.n_chunks
    assert n == 9002
    src = torch.from_numpy(rng.integers(0, 256, size=off, dtype=np.uint8)).to("cuda")
    for ids in (np.arange(8192), np.arange(8193), np.arange(3, n), np.delete(np.arange(n), 5)[:8192],
                np.delete(np.arange(n), [5, 8000])):
        ids = ids.astype(np.uint32)
        payload = torch.empty(plan.delta_layout(ids), dtype=torch.uint8, device="cuda")
        sums = torch.empty(len(ids), 2, dtype=torch.int64, device="cuda")
        plan.pack_chunks(src, ids, payload, sums)
        for share in (0.0, 0.2, 1.0):
            want = np.flatnonzero(rng.random(len(ids)) < share)
            sent = sums.clone()
            sent[torch.from_numpy(want).to("cuda"), 1] ^= 2
            dst = torch.zeros_like(src)
            bad = torch.full(((len(ids) + 31) // 32,), -1, dtype=torch.int32, device="cuda")
            n_bad = plan.empty_counter().fill_(-1)
            plan.unpack_chunks(payload, sent, ids, dst, bad, n_bad)
            assert int(n_bad.item()) == len(want), (len(ids), share)
            words = bad.cpu().numpy().view(np.uint32)
            got = np.flatnonzero(np.unpackbits(words.view(np.uint8), bitorder="little"))  # past the list: clear
            assert np.array_equal(got, want), (len(ids), share)
