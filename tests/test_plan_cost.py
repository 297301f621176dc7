"""The split plans of extend, cascade and decode calls (CPU only; host
arithmetic): how many partial sets each gives, and what a plan costs the host.
"""
import ctypes
import time

import pytest

from paper_2609_39819_amd import kvt

# Hq, Hkv, D, dtype, P, S, shared, partial sets of (extend, cascade, its shared pass), whether it runs the shared pass
PLANS = [
    (4, 1, 64, "f32", [4096 + 37 * i for i in range(16)], [128 - i for i in range(16)], 4096, (8, 5, 5), 1),
    (4, 1, 64, "f32", [32768 + 40 * i for i in range(24)], [32] * 24, 32768, (10, 17, 17), 1),
    (32, 8, 128, "bf16", [4096, 4200, 4100], [9, 16, 3], 4096, (10, 32, 32), 1),
    (24, 2, 128, "bf16", [4500] * 9, [11] * 9, 4096, (13, 28, 28), 1),
    (96, 8, 128, "bf16", [32768 + 64 * i for i in range(16)], [16] * 16, 32768, (2, 10, 10), 1),
    # private parts of unlike lengths
    (96, 8, 128, "bf16", [2048, 2900, 7000, 12000, 30000, 60000, 90000, 100000], [100, 77, 32, 90, 64, 128, 50, 99],
     2048, (2, 5, 5), 1),
    (64, 64, 128, "f32", [20000, 21000], [70, 300], 16384, (2, 6, 6), 1),
    # private parts of more than one round of a kv-head's CUs
    (32, 8, 128, "bf16", [8192 + 83 * i for i in range(24)], [200 - 2 * i for i in range(24)], 8192, (8, 9, 9), 1),
    (32, 8, 128, "bf16", [4096 + 5 * i for i in range(100)], [20] * 100, 4096, (4, 2, 2), 1),
    # the plain extend
    (16, 1, 64, "bf16", [600, 40000, 1000], [300, 20, 700], 512, (16, 16, 17), 0),
]


def call(hq, hkv, D, dtype, P, S):
    pool = kvt.raw_pool(0x10000000, 0x20000000000, 1 << 24, hkv, D,
                        kvt.KVT_DTYPE_BF16 if dtype == "bf16" else kvt.KVT_DTYPE_F32)
    return pool, kvt.RawSeqs(P, S, 0x30000000000, 1 << 16)


def part_bytes(sets, rows, D):
    return -(-sets * rows * D * 4 // 256) * 256 + sets * rows * 8


@pytest.mark.parametrize("case", range(len(PLANS)))
def test_partial_sets(case):
    hq, hkv, D, dtype, P, S, shared, sets, uses = PLANS[case]
    L = kvt.lib()
    pool, s = call(hq, hkv, D, dtype, P, S)
    p, q = ctypes.byref(pool), ctypes.byref(s.struct)
    ws = L.kvt_cascade_workspace_bytes_ex
    got = (L.kvt_extend_workspace_bytes(p, q, hq), ws(p, q, shared, kvt.CASCADE_AUTO, hq),
           ws(p, q, shared, kvt.CASCADE_SHARED_PASS, hq))
    assert got == tuple(part_bytes(n, sum(S) * hq, D) for n in sets)
    assert ws(p, q, shared, kvt.CASCADE_PLAIN, hq) == got[0]
    assert L.kvt_cascade_uses_shared_pass(p, q, shared, hq) == uses


@pytest.mark.parametrize("case", [0, 1, 5, 7])
def test_a_cascade_is_planned_in_microseconds(case):
    """A plan is paid for twice per call.  Against a query that returns at its
    first check, the least of many runs of each in turn, it takes 5 to 7 of
    its times (27 to 42 when every unit goes through a heap of the CUs, both
    routes are planned in full and a second split count is always tried)."""
    hq, hkv, D, dtype, P, S, shared, _, _ = PLANS[case]
    pool, s = call(hq, hkv, D, dtype, P, S)
    p, q, ws = ctypes.byref(pool), ctypes.byref(s.struct), kvt.lib().kvt_cascade_workspace_bytes_ex

    def run(pool):
        t = time.perf_counter()
        for _ in range(20):
            ws(pool, q, shared, kvt.CASCADE_AUTO, hq)
        return time.perf_counter() - t
    both = [(run(None), run(p)) for _ in range(80)]
    checks, plan = (min(x) for x in zip(*both))
    print(f"case {case}: {plan / 20 * 1e6:.1f} us, {plan / checks:.1f} times the bare query")
    assert plan < 16 * checks


@pytest.mark.parametrize("P,dtype,sets", [
    ([8191] * 64, "bf16", 1),       # two workgroups for each CU: whole rounds already
    ([8191] * 70, "bf16", 2),       # 48 more than that
    ([8191] * 80, "bf16", 1),       # half a round more
    ([16383] * 34, "bf16", 4),      # 2 at 1024 keys each leave 32 workgroups for the last round
    ([16383] * 40, "bf16", 2),
    ([32767] * 8 + [2047] * 40, "bf16", 3),          # the longest decide
    ([32767] * 40 + [14000] * 8, "bf16", 2),         # they do not
    ([2047 + 400 * i for i in range(36)], "bf16", 2),
    ([2047 + 400 * i for i in range(36)], "f32", 3),   # one workgroup fits a CU: more and shorter rounds
])
def test_partial_sets_of_large_decode_batches(P, dtype, sets):
    """96/8 heads of 128, at least one unit per CU."""
    L = kvt.lib()
    pool, s = call(96, 8, 128, dtype, P, [1] * len(P))
    got = L.kvt_decode_workspace_bytes(ctypes.byref(pool), ctypes.byref(s.struct), 96)
    assert got == (part_bytes(sets, 96 * len(P), 128) if sets > 1 else 0)
