"""Device memory of a plan: the second set of partial sums is only there for
walks that keep two sums a slot (the compare with sums, unpack's derived
groups)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2509_03047_amd import flashrestore as F  # noqa: E402
from paper_2509_03047_amd import workloads as W  # noqa: E402


def test_second_set_of_partial_sums_only_where_it_is_used(monkeypatch):
    """20,000 tensors at 16-byte offsets, none derived, in 16 KiB chunks: the
    compare with sums takes whole chunks, so one set is enough (522 bytes a
    chunk in all; 671 with two).  With whole chunks switched off the compare
    walks, and has both."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = W.stress_workload(2, 20000, 256, 1 << 20, 1 << 14)
    torch.zeros(1, device="cuda")

    def bytes_per_chunk():
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        plan = F.Plan(w.table, 1 << 14, w.src_arena_bytes, w.dst_arena_bytes)
        used = before - torch.cuda.mem_get_info()[0]
        return used / plan.n_chunks

    monkeypatch.delenv("FLASHRESTORE_SMALL", raising=False)
    one = bytes_per_chunk()
    monkeypatch.setenv("FLASHRESTORE_SMALL", "0")
    two = bytes_per_chunk()
    assert one < 580 and two > one + 60, (one, two)
