"""binding.py's native half: the addresses of a call's tensors, and that it takes and refuses what a look at each of them in Python does."""
import ctypes

import pytest
import torch

from paper_2511_04283_amd import binding as B


def names(k):
    return tuple(f"array {j}" for j in range(k))


def test_nothing_is_written_beyond_the_structure():
    from paper_2511_04283_amd import _marshal
    room = (ctypes.c_uint64 * 4)(*[7] * 4)
    one = (torch.zeros(3),)
    assert _marshal.fill(room, 0, one, 0, ((3,),)) == 0 and list(room) == [7] * 4   # (not on the GPU)
    assert _marshal.fill(room, 32, (), 0, ()) == 0
    for offset, tensors in ((25, one), (32, one), (-8, one), (8, one * 4), (1 << 62, one)):
        with pytest.raises(ValueError):
            _marshal.fill(room, offset, tensors, 0, ((3,),) * len(tensors))
    for args in ((room, 0, one, 0, ()), (room, 0, list(one), 0, ((3,),)), (room, 0, one, 0), (bytes(32), 0, one, 0, ((3,),)),
                 (room, "0", one, 0, ((3,),)), (room, 0, one, -1, ((3,),))):
        with pytest.raises((TypeError, BufferError, OverflowError)):
            _marshal.fill(*args)
    assert list(room) == [7] * 4


class Sub(torch.Tensor):
    pass


@pytest.mark.gpu
def test_what_is_taken_and_refused():
    dev = "cuda:0"
    f = lambda *s: torch.zeros(s, device=dev)
    good = [f(6, 3), f(6, 2, 3), f(6), torch.zeros(6, dtype=torch.int32, device=dev), f(0, 3)]
    shapes = ((6, 3), (6, 2, 3), (6,), (6,), (0, 3))
    dtypes = [torch.int32 if k == 3 else torch.float32 for k in range(5)]

    def addresses(tensors):
        room = (ctypes.c_uint64 * 7)(*[7] * 7)
        B._addresses(room, 8, tuple(tensors), shapes, names(5), 1 << 3)
        assert room[0] == room[6] == 7
        return list(room)[1:6]

    assert addresses(good) == [t.data_ptr() for t in good]
    wide = f(6, 8)
    others = [f(6, 3).double(), f(6, 4), f(5, 3), f(18), wide[:, :3], f(3, 6).t(), torch.zeros(6, 3), None, [1.0], 3, torch.nn.Parameter(f(6, 3)),
              f(6, 3).as_subclass(Sub), wide.view(-1)[:18].view(6, 3), wide.view(-1)[1:19].view(6, 3), f(1, 3).expand(6, 3),
              torch.zeros((6, 3), device="meta"), f(6, 3).to_sparse(), f(6, 3).requires_grad_(), f(6, 3).half(), f(6, 3, 1)]
    refused = 0
    for other in others:
        tensors = [other, *good[1:]]
        try:   # (the look in Python)
            want = [B._chk(t, d, s, "").data_ptr() for t, d, s in zip(tensors, dtypes, shapes)]
        except Exception as e:
            refused += 1
            with pytest.raises(type(e)) as got:
                addresses(tensors)
            assert not isinstance(e, ValueError) or "array 0" in str(got.value)
        else:
            assert addresses(tensors) == want
    assert refused == 15
    with pytest.raises(ValueError, match="array 3"):
        addresses([*good[:3], f(6), good[4]])
    with pytest.raises(ValueError, match="array 2"):
        addresses([*good[:2], good[3], *good[3:]])
