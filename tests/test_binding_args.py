"""Argument marshalling of the Python bindings: the bytes a C call sees are
those numpy's conversion gives, over the forms an argument may take."""

import ctypes as C

import numpy as np
import pytest

from paper_2606_23087_amd import flowpool as fp


def seen(arg, ptype, n):
    """The first n elements as the C side reads them."""
    f = C.CFUNCTYPE(C.c_int32, ptype)
    got = []
    f(lambda p: got.append([p[i] for i in range(n)] if p else None) or 0)(arg)
    return got[0]


def read_only(a):
    a.flags.writeable = False
    return a


ARRAYS = [
    np.arange(7, dtype=np.int32),
    np.arange(7, dtype=np.int64) * -3,
    np.arange(20, dtype=np.int32)[::3],
    np.arange(12, dtype=np.int32).reshape(3, 4).T[1],
    np.arange(5, dtype=">i4"),
    read_only(np.arange(7, dtype=np.int32)),
    read_only(np.zeros(0, np.int32)),
    [1, 2, 3], (4,), [], range(3), np.int64(9), np.zeros((2, 0), np.int32), [True, False],
]


@pytest.mark.parametrize("a", ARRAYS, ids=[str(i) for i in range(len(ARRAYS))])
def test_array_arguments(a):
    want = np.ascontiguousarray(a, np.int32)
    arr, arg = fp._arr(a, np.int32, fp._i32p)
    assert arr.shape == want.shape
    assert seen(arg, fp._i32p, want.size) == want.ravel().tolist()      # never null, also when empty
    assert fp._arr(None, np.int32, fp._i32p) == (None, None)


@pytest.mark.parametrize("ids", [[1, 2, 3], (7,), [], [2**64 - 1], [np.uint64(5), np.int32(6)], [True], np.arange(4),
                                 np.arange(9, dtype=np.uint64)[::2], read_only(np.arange(3, dtype=np.uint64))])
def test_sample_ids(ids):
    want = np.ascontiguousarray(ids, np.uint64)
    arr, arg = fp._ids(ids)
    assert len(arr) == len(want)
    assert seen(arg, fp._u64p, len(want)) == want.tolist()


def test_sample_ids_that_are_no_uint64_go_numpys_way():
    arr, arg = fp._ids([1.0, 2.0])
    assert seen(arg, fp._u64p, 2) == [1, 2]
    with pytest.raises(OverflowError):
        fp._ids([-1])
    with pytest.raises((TypeError, ValueError)):
        fp._ids(["x"])


@pytest.mark.parametrize("ids", [[-1], [2**64 + 5], (np.int64(-7),), []])
def test_pack_ids_wrap_as_ctypes_integers_do(ids):
    def entry(pool, idp, n, *rest):
        assert seen(idp, fp._u64p, n) == [int(i) % 2**64 for i in ids] and n == len(ids)
        return fp.FP_OK

    assert fp.pack_microbatch(0, ids, None, 0, None, 0, stream=0, _entry=entry) == (0, 0)
    with pytest.raises(TypeError):
        fp.pack_microbatch(0, [1.0], None, 0, None, 0, stream=0, _entry=entry)


@pytest.mark.parametrize("n", [0, 1, 64, 65, 3000])
def test_row_sums(n):
    a = np.full(n, 2**31 - 1, np.int32)
    assert fp._rows(a) == n * (2**31 - 1)
    assert fp._rows(np.ones((2, 3), np.int32)) == 6


@pytest.mark.gpu
def test_default_stream_is_torchs_current_one():
    import torch
    torch.cuda.init()
    side = torch.cuda.Stream()
    assert fp._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert fp._stream(None) == side.cuda_stream == fp._stream(side)
