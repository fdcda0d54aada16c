"""The workspace of batched secAccess calls where memory is short."""
import pytest
import torch

from paper_2209_03526_amd import fss


@pytest.mark.parametrize("free,calls,want", [(10_000, 64, 10_000 // 1000), (64_000, 64, 64), (1_500, 64, 1), (1_000, 1, 1),
                                             (3_999, 9, 2)])
def test_as_many_calls_as_memory_is_free_for(monkeypatch, free, calls, want):
    """An allocation that fails is tried again with half the calls, down to one call's workspace."""
    empty = torch.empty

    def some(n, **k):
        if n > free:
            raise torch.OutOfMemoryError("no memory")
        return empty(n, **k)
    monkeypatch.setattr(torch, "empty", some)
    got = fss._side_by_side(1000, calls, "cpu").numel() // 1000
    assert min(want, calls) / 2 < got <= min(want, calls)


def test_not_even_one(monkeypatch):
    def none(n, **k):
        raise torch.OutOfMemoryError("no memory")
    monkeypatch.setattr(torch, "empty", none)
    with pytest.raises(torch.OutOfMemoryError):
        fss._side_by_side(1000, 8, "cpu")


def test_the_batch_call_falls_back(monkeypatch):
    """rss_sec_access_batch itself asks for less when 64 calls' workspace does not fit."""
    asked, empty = [], torch.empty

    def some(n, **k):
        asked.append(n)
        if len(asked) < 3:
            raise torch.OutOfMemoryError("no memory")
        return empty(n, **k)
    t = empty(1, dtype=torch.int32)
    monkeypatch.setattr(torch, "empty", some)
    monkeypatch.setattr(fss, "_stream", lambda s: 0)
    monkeypatch.setattr(fss.LIB, "rss_sec_access_batch", lambda *a: fss.OK)
    fss.rss_sec_access_batch(10, 64, [0] * 24, t, 5, [t] * 3, 1, [t] * 3, (1, 2, 3), [0] * 8, [0] * 24, [t] * 3, [t] * 3, t, t)
    single = int(fss.LIB.rss_sec_access_workspace_bytes(5, 64, 1))
    assert asked == [single * 8, single * 4, single * 2]
