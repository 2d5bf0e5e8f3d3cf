"""What a context's bookkeeping says after a call that failed half way, how its calls wait for the GPU's words and which placement
they choose, on the CPU:
abi.hip's host code on a stub of the GPU (host_abi_stub.cpp) whose launches and allocations fail, and whose words come late or
never, on request."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if not os.path.exists(HIPCC) or not shutil.which("objcopy"):
        pytest.skip("no hipcc / objcopy")
    out = str(tmp_path_factory.mktemp("stub"))
    csrc = os.path.join(ROOT, "paper_2511_04283_amd", "csrc")
    flags = ["-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-w", "-I", csrc, "-I",
             os.path.join(ROOT, "include")]
    for name, src in (("abi", os.path.join(csrc, "abi.hip")), ("stub", os.path.join(ROOT, "tests", "host_abi_stub.cpp"))):
        subprocess.run([HIPCC, *flags, "-c", src, "-o", f"{out}/{name}.o"], check=True)
    # (launchers that no test here reaches, and the device code, stay undefined: weak, so that the library loads without them)
    subprocess.run(["objcopy", "--wildcard", "--weaken-symbol=_ZN2fs*", "--weaken-symbol=__hip_fatbin*", f"{out}/abi.o"], check=True)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-o", f"{out}/libstub.so", f"{out}/abi.o", f"{out}/stub.o"], check=True)
    return ctypes.CDLL(f"{out}/libstub.so")


class Ctx:
    """A context on the stub and the arguments of its calls (arrays nobody reads)."""

    def __init__(self, lib, pairs, n=1):
        from paper_2511_04283_amd import binding as B
        self.B, self.lib, self.h, self.n = B, lib, ctypes.c_void_p(), n
        lib.fs_last_error.restype = ctypes.c_char_p
        assert lib.fs_create(ctypes.byref(self.h), 0, None, None) == B.FS_OK
        self.room = ctypes.create_string_buffer(1 << 16)
        some = (ctypes.addressof(self.room) + 15) // 16 * 16
        fill = lambda s, names: [setattr(s, k, some) for k in names] and s
        self.cam = B.fs_camera(width=32, height=16, fx=16.0, fy=16.0)
        self.g = fill(B.fs_gaussians(n=n, sh_degree=0), ("means", "scales", "quats", "opacities", "sh"))
        self.proj = fill(B.fs_projected(), [f for f, _ in B.fs_projected._fields_])
        self.grads = fill(B.fs_grads(), ("dmeans", "dscales", "dquats", "dopacities", "dsh", "dmean2d"))
        five = (ctypes.c_void_p * 5)(*[some] * 5)
        self.state = B.fs_train_state(n, 0, five, five, five, five, some, some, some)
        self.some = ctypes.c_void_p(some)
        self.pairs(pairs)

    def pairs(self, n):
        ctypes.c_int64.in_dll(self.lib, "stub_pairs").value = n

    def backward(self, mode):
        """fs_bin_sort and fs_render_bwd; the flags that were set when its first kernel was launched, or the status."""
        b = self.B.fs_bins()
        r = ctypes.byref
        self.lib.fs_set_record_mode(self.h, mode)
        rc = self.lib.fs_bin_sort(self.h, r(self.proj), r(self.cam), ctypes.c_int64(self.n), r(b))
        if rc == self.B.FS_OK:
            rc = self.lib.fs_render_bwd(self.h, r(self.g), r(self.cam), r(self.proj), r(b), self.some, self.some, self.some,
                                        r(self.grads))
        self.rc = rc
        return rc or ctypes.c_int64.in_dll(self.lib, "stub_stale_flags").value

    def train(self, mode):
        prm = self.B.fs_train_params(0.2, (ctypes.c_float * 5)(), 0.9, 0.999, 1e-15, 1, 0, 1)
        self.out3 = out3 = (ctypes.c_double * 3)()
        r = ctypes.byref
        self.lib.fs_set_record_mode(self.h, mode)
        rc = self.lib.fs_train_step(self.h, r(self.state), r(self.cam), self.some, r(prm), out3)
        self.rc = rc
        return rc or ctypes.c_int64.in_dll(self.lib, "stub_stale_flags").value


@pytest.mark.parametrize("call", ["backward", "train"])
def test_flags_left_by_a_failed_backward_outlive_a_dense_one(stub, call):
    """A sparse backward pass that fails behind its first kernel leaves flags; a dense one in between does not touch them, so
    the next sparse one has to clear them."""
    c = Ctx(stub, pairs=100)
    step, B = getattr(c, call), c.B
    assert step(B.FS_RECORDS_SPARSE) == 0
    ctypes.c_int.in_dll(stub, "stub_fail_preprocess_bwd").value = 1
    assert step(B.FS_RECORDS_SPARSE) == -3   # FS_EHIP
    step(B.FS_RECORDS_DENSE)
    assert step(B.FS_RECORDS_SPARSE) == 0    # not 100
    stub.fs_destroy(c.h)


@pytest.mark.parametrize("call", ["backward", "train"])
def test_flags_after_their_array_failed_to_grow(stub, call):
    """The array of flags is given back before a larger one is asked for; where that fails, the next one may have the old
    one's size, and holds anything."""
    c = Ctx(stub, pairs=100)
    step, B = getattr(c, call), c.B
    assert step(B.FS_RECORDS_SPARSE) == 0
    c.pairs(30_000)
    step(B.FS_RECORDS_DENSE)                 # (every other array grows here)
    fail = ctypes.c_size_t.in_dll(stub, "stub_fail_malloc_of")
    fail.value = 32768
    assert step(B.FS_RECORDS_SPARSE) == -2   # FS_ENOMEM
    fail.value = 0
    assert b"record flags" in stub.fs_last_error(c.h)
    c.pairs(100)
    assert step(B.FS_RECORDS_SPARSE) == 0    # not 100
    stub.fs_destroy(c.h)


def set_int(stub, name, value):
    ctypes.c_int.in_dll(stub, name).value = value


# (the ordering in one launch, and in several)
FRAMES = [1, 20000]


@pytest.mark.parametrize("n", FRAMES)
@pytest.mark.parametrize("call", ["backward", "train"])
def test_words_behind_a_long_queue_are_all_that_is_waited_for(stub, call, n):
    """Totals and loss that come later than the host looks for without a pause: the call goes on with them, not when the stream
    has nothing left to do."""
    c = Ctx(stub, pairs=100, n=n)
    syncs = ctypes.c_int.in_dll(stub, "stub_syncs")
    getattr(c, call)(c.B.FS_RECORDS_DENSE)   # (arrays that grow wait for the stream)
    before = syncs.value
    set_int(stub, "stub_queue", 3)
    try:
        for _ in range(2):
            getattr(c, call)(c.B.FS_RECORDS_DENSE)
            assert c.rc == c.B.FS_OK and syncs.value == before
            if call == "train":
                assert list(c.out3) == [0.25, 0.5, 0.75]
    finally:
        set_int(stub, "stub_queue", 0)
    stub.fs_destroy(c.h)


@pytest.mark.parametrize("n", FRAMES)
@pytest.mark.parametrize("words, call, message", [(1, "backward", b"totals"), (1, "train", b"totals"), (2, "train", b"loss")])
def test_words_that_never_come(stub, words, call, message, n):
    """... are an error in every call that waits for them, and the next call does not set them anew before the stream is done."""
    c = Ctx(stub, pairs=100, n=n)
    step, B = getattr(c, call), c.B
    step(B.FS_RECORDS_DENSE)
    set_int(stub, "stub_never", words)
    try:
        step(B.FS_RECORDS_DENSE)
        assert c.rc == -3   # FS_EHIP
    finally:
        set_int(stub, "stub_never", 0)
    assert message in stub.fs_last_error(c.h)
    syncs = ctypes.c_int.in_dll(stub, "stub_syncs")
    for waits in (1, 0):
        before = syncs.value
        step(B.FS_RECORDS_DENSE)
        assert c.rc == B.FS_OK and syncs.value - before == waits
        if call == "train":
            assert list(c.out3) == [0.25, 0.5, 0.75]
    stub.fs_destroy(c.h)


def test_placement_is_chosen_by_the_ordering_before(stub):
    """From a million Gaussians on, placement by bands where the ordering before had the candidates that make it worth while (with
    fewer it is the slower way), in a context's first ordering in any case; count, placement and split of an ordering agree."""
    c = Ctx(stub, pairs=0)
    c.cam.width, c.cam.height = 1920, 1080
    bands = (ctypes.c_int * 3).in_dll(stub, "stub_bands")

    def by_bands(n, pairs):
        c.pairs(pairs)
        before = list(bands)
        b = c.B.fs_bins()
        assert stub.fs_bin_sort(c.h, ctypes.byref(c.proj), ctypes.byref(c.cam), ctypes.c_int64(n), ctypes.byref(b)) == c.B.FS_OK
        count, place, split = (x - y for x, y in zip(bands, before))
        assert count in (0, 1) and place == split and (place > 0) == (count == 1)
        return count == 1

    M = 1000000
    assert by_bands(M, 3 * M)            # (the first: by the number of Gaussians)
    assert by_bands(M, 100000)           # 3 M before
    assert not by_bands(M, 100000)
    assert not by_bands(3 * M, 2850000 - 1)
    assert not by_bands(3 * M, 2850000)
    assert by_bands(3 * M, 4 * M)
    assert not by_bands(M - 1, 4 * M)
    assert by_bands(M, 0)
    assert not by_bands(M, 3 * M)
    c.cam.width = c.cam.height = 128     # 64 tiles
    assert not by_bands(M, 3 * M)
    c.cam.width = 129
    assert by_bands(M, 3 * M)
    stub.fs_destroy(c.h)


def test_one_launch_is_chosen_by_gaussians_and_tiles(stub):
    """The whole ordering in one launch up to the sizes where several are the faster way, further in a training step; a second launch
    only where the buffers were too small (a new context's hold four tiles a Gaussian and more)."""
    launches = (ctypes.c_int * 2).in_dll(stub, "stub_small")
    for training, most, tests in ((False, 10000, 4000000), (True, 16384, 12000000)):
        for n, tiles in ((1, 1), (most, 1), (most + 1, 1), (1000, 1024), (1000, 1025), (tests // 1000, 1000), (tests // 1000 + 1, 1000)):
            c = Ctx(stub, pairs=4 * n, n=n)
            c.cam.width = 16 * tiles
            for call in range(3):
                if call == 1:
                    c.pairs(100 * max(n, 1000))
                before = list(launches)
                c.train(c.B.FS_RECORDS_DENSE) if training else c.backward(c.B.FS_RECORDS_DENSE)
                assert c.rc == c.B.FS_OK
                small = n <= most and tiles <= 1024 and n * tiles <= tests
                assert [x - y for x, y in zip(launches, before)] == [small, small and call == 1], (training, n, tiles)
            stub.fs_destroy(c.h)


@pytest.mark.parametrize("call", ["backward", "train"])
def test_one_launch_that_waited_too_long_for_itself(stub, call):
    """Where the totals of an ordering in one launch never come, because its workgroups have given up waiting for each other, the general
    launches order the frame; the next call takes one launch again."""
    launches, counts = (ctypes.c_int * 2).in_dll(stub, "stub_small"), ctypes.c_int.in_dll(stub, "stub_counts")
    c = Ctx(stub, pairs=100)
    step, B = getattr(c, call), c.B
    for never in (0, 3, 3, 0):
        before = [*launches, counts.value]
        set_int(stub, "stub_never", never)
        try:
            step(B.FS_RECORDS_SPARSE)
        finally:
            set_int(stub, "stub_never", 0)
        assert c.rc == B.FS_OK and stub.fs_last_error(c.h) == b""
        assert [x - y for x, y in zip([*launches, counts.value], before)] == [1, 0, never != 0]
        if call == "train":
            assert list(c.out3) == [0.25, 0.5, 0.75]
    stub.fs_destroy(c.h)


@pytest.mark.parametrize("call", ["fs_render_fwd", "fs_render_fwd_loss", "fs_render_bwd", "fs_score_accumulate"])
def test_bins_are_of_one_grid_of_tiles(stub, call):
    """A camera of another grid than the one that the bins were ordered for is refused before anything is launched: its tiles have other
    numbers.  Another size of the same grid is not."""
    c = Ctx(stub, pairs=100)
    B, r, some = c.B, ctypes.byref, c.some
    bins = B.fs_bins()
    assert stub.fs_bin_sort(c.h, r(c.proj), r(c.cam), ctypes.c_int64(1), r(bins)) == B.FS_OK
    args = {"fs_render_fwd": lambda: (r(c.proj), r(bins), r(c.cam), some, some, some),
            "fs_render_fwd_loss": lambda: (r(c.proj), r(bins), r(c.cam), some, some, some, some, some, some),
            "fs_render_bwd": lambda: (r(c.g), r(c.cam), r(c.proj), r(bins), some, some, some, r(c.grads)),
            "fs_score_accumulate": lambda: (r(c.proj), r(bins), r(c.cam), some, some, some, some)}[call]
    for width, height in ((16, 16), (16, 32), (48, 16), (33, 16), (32, 17)):
        c.cam.width, c.cam.height = width, height
        assert getattr(stub, call)(c.h, *args()) == -1   # FS_EINVAL
        assert b"another grid" in stub.fs_last_error(c.h)
    if call in ("fs_render_fwd", "fs_render_bwd"):
        c.cam.width, c.cam.height = 17, 3
        assert getattr(stub, call)(c.h, *args()) == B.FS_OK
    stub.fs_destroy(c.h)


@pytest.mark.parametrize("longest, record", [(1, 1), (16384, 1), (16385, 0), (70000, 0)])
def test_a_record_of_blended_pairs_only_for_lists_sorted_per_tile(stub, longest, record):
    """Longer lists are ordered by the radix sort, which may leave the keys where the record would lie, and have places beyond its 16
    bits."""
    blends = (ctypes.c_int * 2).in_dll(stub, "stub_blends")
    ctypes.c_int64.in_dll(stub, "stub_longest").value = longest
    try:
        for n in FRAMES:
            c = Ctx(stub, pairs=100, n=n)
            before = list(blends)
            c.train(c.B.FS_RECORDS_SPARSE)
            assert c.rc == c.B.FS_OK and [x - y for x, y in zip(blends, before)] == [record, record]
            stub.fs_destroy(c.h)
    finally:
        ctypes.c_int64.in_dll(stub, "stub_longest").value = 1


@pytest.mark.parametrize("n", FRAMES)
def test_arrays_that_grow_together_take_one_allocation(stub, n):
    """A new context's first ordering and backward pass: ranges, the scan's sums, what there is for each Gaussian, for each pair, the
    records and their flags.  More pairs: the last three again; as many: none."""
    mallocs = ctypes.c_int.in_dll(stub, "stub_mallocs")
    c = Ctx(stub, pairs=100, n=n)
    for pairs, allocations in ((100, 6), (100, 0), (400_000, 3), (100, 0), (400_000, 0)):
        c.pairs(pairs)
        before = mallocs.value
        assert c.backward(c.B.FS_RECORDS_SPARSE) == 0
        assert mallocs.value - before == allocations, pairs
    stub.fs_destroy(c.h)


def test_after_an_allocation_for_several_arrays_failed(stub):
    """None of them is there then; the next call that needs no more than before allocates anew."""
    c = Ctx(stub, pairs=100, n=20000)
    fail = ctypes.c_size_t.in_dll(stub, "stub_fail_malloc_of")
    assert c.backward(c.B.FS_RECORDS_SPARSE) == 0
    c.pairs(400_000)
    fail.value = 20 << 19
    assert c.backward(c.B.FS_RECORDS_SPARSE) == -2   # FS_ENOMEM
    fail.value = 0
    assert b"pairs" in stub.fs_last_error(c.h)
    c.pairs(100)
    assert c.backward(c.B.FS_RECORDS_SPARSE) == 0
    stub.fs_destroy(c.h)
