"""Bins.copy_*: which streams wait for which, with streams and device memory that only write down what is asked of them."""
import pytest
import torch

from paper_2511_04283_amd import binding as B


class Stream:
    def __init__(self, name, calls):
        self.name, self.calls = name, calls

    def wait_stream(self, other):
        self.calls.append((self.name, "waits for", other.name))


class Memory:
    def __init__(self, calls):
        self.calls = calls

    def clone(self):
        self.calls.append("copy")
        return torch.zeros(8, dtype=torch.int32)


@pytest.mark.parametrize("copy", ["copy_keys", "copy_gauss", "copy_ranges", "copy_order"])
@pytest.mark.parametrize("own", [True, False])
def test_copies_are_ordered_with_the_context(monkeypatch, own, copy):
    """fs_bin_sort returns when it has its totals, with ranges, order, keys and indices still being written on the context's
    stream: a copy on another stream waits for that one, and that one waits for the copy."""
    calls = []
    ctx_stream, current = Stream("context", calls), Stream("current", calls)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: current if own else ctx_stream)
    monkeypatch.setattr(torch, "as_tensor", lambda raw, device=None: Memory(calls))
    bins = B.Bins(8, B.fs_bins(keys_sorted=64, gauss_sorted=64, tile_ranges=64, tile_order=64), 4, torch.device("cuda:0"), ctx_stream)
    getattr(bins, copy)()
    assert calls == ([("current", "waits for", "context"), "copy", ("context", "waits for", "current")] if own else ["copy"])
