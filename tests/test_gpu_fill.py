"""launch_fill_u32, which clears counters, record flags and the dense records of a backward pass with the Compact Box."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("count", [0, 1, 2, 3, 4, 5, 1023, 1025, 4 * 2048 * 256 - 1, 4 * 2048 * 256, 4 * 2048 * 256 + 5, 5000003])
def test_every_word_of_the_range_and_no_other(count, offset):
    """Stores of one word and of four, a rest of each, and more words than the launch has threads for at a time."""
    import torch
    from paper_2511_04283_amd import binding as B
    fill = B.load_library()._ZN2fs15launch_fill_u32EP12ihipStream_tPjjl
    fill.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_int64]
    words = torch.full((count + 16,), 7, dtype=torch.int32, device="cuda:0")
    assert words.data_ptr() % 16 == 0
    assert fill(torch.cuda.current_stream().cuda_stream, words.data_ptr() + 4 * offset, 9, count) == 0
    assert bool((words[offset:offset + count] == 9).all()) and bool((words[:offset] == 7).all()) and bool((words[offset + count:] == 7).all())
