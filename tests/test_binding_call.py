"""The binding's extension module against the ctypes route it stands beside:
length arrays in every accepted form, values outside int32, and the workspace
sizes of the same arguments (CPU only; host arithmetic)."""
import ctypes

import numpy as np
import pytest

from paper_2609_39819_amd import kvt

FORMS = [[3, 5, 2 ** 31 - 1], (3, 5, 7), np.array([3, 5, 7], dtype=np.int32), np.array([3, 5, 7], dtype=np.int64),
         np.array([3, 5, 7], dtype=np.uint8), np.array([[3, 5], [7, 9]], dtype=np.int32),
         np.arange(20, dtype=np.int32)[::2], (np.int64(7), 8), [True, 2], list(range(300)), []]


@pytest.mark.parametrize("form", range(len(FORMS)))
def test_pack_takes_what_the_ctypes_arrays_take(form):
    x = FORMS[form]
    want = list(kvt._i32_array(x))
    packed, n, tokens = kvt._native().pack(x, x, kvt._i32_array)
    assert n == len(want) and tokens == sum(want)
    assert np.frombuffer(packed, dtype=np.int32).tolist() == want + want
    packed, n, tokens = kvt._native().pack(x, None, kvt._i32_array)
    assert n == tokens == len(want)
    assert np.frombuffer(packed, dtype=np.int32).tolist() == want + [1] * len(want)


def test_pack_never_wraps():
    for bad in ([2 ** 31], [-2 ** 31 - 1], [1, 2 ** 70], np.array([2 ** 33], dtype=np.int64),
                np.array([2 ** 32], dtype=np.uint64)):
        for args in ((bad, None), ([1] * len(bad), bad)):
            with pytest.raises((OverflowError, ValueError)):
                kvt._native().pack(*args, kvt._i32_array)
    with pytest.raises(ValueError):
        kvt._native().pack([1, 2], [1], kvt._i32_array)         # a sequence without a suffix length


def test_workspace_matches_the_ctypes_call():
    L = kvt.lib()
    pool = (0x10000000, 0x20000000000, 1 << 20, 8, 128, kvt.KVT_DTYPE_BF16)
    for P, S, hq in (([8192], [512], 32), ([30011], [67], 32), ([65535, 40000], [1, 1], 96)):
        raw, rs = kvt.raw_pool(*pool), kvt.RawSeqs(P, S, 0x30000000000, 5000)
        packed, n, _ = kvt._native().pack(P, S, kvt._i32_array)
        for entry in ("kvt_extend_workspace_bytes", "kvt_decode_workspace_bytes"):
            want = getattr(L, entry)(ctypes.byref(raw), ctypes.byref(rs.struct), hq)
            assert kvt._native().workspace(L.address[entry], *pool, packed, n, 0x30000000000, 5000, None, hq) == want
        want = L.kvt_cascade_workspace_bytes_ex(ctypes.byref(raw), ctypes.byref(rs.struct), 4096,
                                                kvt.CASCADE_SHARED_PASS, hq)
        assert kvt._native().workspace(L.address["kvt_cascade_workspace_bytes_ex"], *pool, packed, n, 0x30000000000,
                                       5000, None, hq, 4096, kvt.CASCADE_SHARED_PASS) == want


def test_a_host_table_smaller_than_the_call_is_refused():
    pool = (0x10000000, 0x20000000000, 64, 1, 64, kvt.KVT_DTYPE_BF16)
    packed, n, _ = kvt._native().pack([16, 16], [4, 4], kvt._i32_array)
    table = np.zeros((1, 3), dtype=np.int32)
    with pytest.raises(ValueError):
        kvt._native().workspace(kvt.lib().address["kvt_extend_workspace_bytes"], *pool, packed, n, 0x30000000000, 3,
                                table, 4)


class Converted:
    """Lengths that only numpy can read; reading them runs `then`."""

    def __init__(self, values, then):
        self.values, self.then = values, then

    def __array__(self, dtype=None, copy=None):
        self.then()
        return np.array(self.values, dtype=np.int64)


@pytest.mark.parametrize("form", ["list", "int32 array", "tuple"])
@pytest.mark.parametrize("change", ["clear", "shrink", "objects", "other"])
def test_pack_keeps_the_lengths_it_took(form, change):
    """Reading the suffix lengths may run Python code (a conversion here) that
    changes the prefix lengths: the call goes on with the values as taken."""
    n = 4000
    prefix = list(range(n))
    if form == "int32 array":
        prefix = np.arange(n, dtype=np.int32)

    def then():
        if form == "int32 array":
            prefix[:] = -1
        elif form == "list":
            if change == "clear":
                prefix.clear()
            elif change == "shrink":
                del prefix[1:]
            else:
                prefix[:] = [None if change == "objects" else -7] * n

    x = tuple(prefix) if form == "tuple" else prefix
    packed, count, tokens = kvt._native().pack(x, Converted([1] * n, then), kvt._i32_array)
    assert count == tokens == n
    assert np.frombuffer(packed, dtype=np.int32).tolist() == list(range(n)) + [1] * n


def test_pack_passes_a_failed_conversion_on():
    def fail():
        raise KeyError("no lengths")
    with pytest.raises(KeyError):
        kvt._native().pack([1, 2], Converted([1, 1], fail), kvt._i32_array)
    with pytest.raises(TypeError):
        kvt._native().pack([1, 2], object(), lambda x: "neither")
