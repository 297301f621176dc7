"""Decoding steps at the edges of their split rules: small batches, whose keys
split over the CUs down to 128 keys per split where the merge is worth it (one
split and two, 64 splits, the tail split holding few keys or none), and batches of at least one unit
per CU, where the longest context decides; against the oracle and the unsplit
step, and with a workspace that only fits the base split count.
"""
import numpy as np
import pytest

from oracle import oracle_append, oracle_extend
from paper_2609_39819_amd import kvt
from paper_2609_39819_amd.workloads import build_workload

from gpu_common import compare, say, stage, to_f64

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # (P, Hq, Hkv, D, dtype, splits)
    ([255], 8, 2, 64, "f32", 1),              # 256 keys in two splits would take longer than in one
    ([638], 8, 2, 64, "f32", 1),              # 639 keys: four splits take 479 of them from a workgroup
    ([639], 8, 2, 64, "f32", 5),              # 640 keys: five splits take 512
    ([798] * 16, 8, 8, 128, "bf16", 1),       # 799 keys, room for two splits: they take 399
    ([799] * 16, 8, 8, 128, "bf16", 2),       # 400
    ([1999] * 16, 8, 8, 64, "f32", 1),        # two splits in fp32
    ([8320], 12, 1, 128, "bf16", 64),         # 8321 keys of one kv-head: 64 splits of 5 tiles, the last 11 empty
    ([8191, 8191], 32, 1, 128, "bf16", 64),   # 8192 keys: 64 splits of exactly 4 tiles
    ([3001, 1502, 2222], 16, 4, 128, "bf16", 11),   # like contexts: 1503 keys of the shortest
    ([3006, 1502], 16, 4, 128, "bf16", 1),    # 3007 keys, the longest more than twice the shortest: the larger batches' rule
    ([8191] + [20 + 60 * i for i in range(31)], 8, 8, 64, "bf16", 2),    # 256 units, 8192 keys of the longest
    ([8190] + [20 + 60 * i for i in range(31)], 8, 8, 64, "bf16", 1),    # one key less
    ([8200] + [17 + 31 * i for i in range(31)], 8, 8, 128, "f32", 2),
]


def parts(need, rows, D):
    return next(n for n in range(0, 129) if (-(-n * rows * D * 4 // 256) * 256 + n * rows * 8 if n > 1 else 0) >= need)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("case", range(len(CASES)))
def test_small_batch_decode_matches_the_oracle(case):
    P, Hq, Hkv, D, dtype, splits = CASES[case]
    B = len(P)
    w = build_workload(name=f"decode-small{case}", seed=5200 + case, prefix_len=P, suffix_len=[1] * B,
                       num_q_heads=Hq, num_kv_heads=Hkv, head_dim=D, dtype=dtype)
    d = stage(w)
    kvt.append_kv(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, d["k_new"], d["v_new"])
    args = (d["q"], d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.scale)
    need = kvt.decode_workspace_bytes(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, Hq)
    assert max(1, parts(need, B * Hq, D)) == splits
    out, lse = kvt.decode_attention(*args, return_lse=True)
    whole, whole_lse = kvt.decode_attention(*args, return_lse=True, use_workspace=False)
    torch.cuda.synchronize()
    kp, vp = oracle_append(w.k_pool_c, w.v_pool_c, w.compact_table, w.prefix_len, w.suffix_len, w.k_new, w.v_new)
    ref, ref_lse = oracle_extend(w.q, kp, vp, w.compact_table, w.prefix_len, w.suffix_len, Hkv, w.scale)
    compare(to_f64(out, dtype), ref, "small batch vs oracle")
    compare(to_f64(out, dtype), to_f64(whole, dtype), "split vs unsplit")
    # row sums of bf16-rounded probabilities: one lse errs by at most 2^-9
    # relative to the sum, plus, for fp32 storage, the rounding of the logits
    assert np.abs(lse.cpu().numpy() - ref_lse).max() <= (2 ** -9 if dtype == "bf16" else 1e-2)
    assert float((lse - whole_lse).abs().max()) <= 2 ** -8


@pytest.mark.timeout(300)
def test_a_workspace_for_fewer_splits_is_accepted():
    """A workspace of 16 partial sets (all that any single context asked for
    before small batches split further) still runs the call, on 16 splits."""
    P, Hq, Hkv, D = [20000], 32, 8, 128
    w = build_workload(name="decode-old-ws", seed=5300, prefix_len=P, suffix_len=[1], num_q_heads=Hq,
                       num_kv_heads=Hkv, head_dim=D, dtype="bf16")
    d = stage(w)
    kvt.append_kv(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, d["k_new"], d["v_new"])
    args = (d["q"], d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.scale)
    need = kvt.decode_workspace_bytes(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, Hq)
    sixteen = 16 * Hq * (D + 2) * 4
    assert need == 32 * Hq * (D + 2) * 4
    full = kvt.decode_attention(*args)
    ws = torch.full((sixteen,), 0xFF, dtype=torch.uint8, device="cuda")
    few = kvt.decode_attention(*args, workspace=ws)
    with pytest.raises(kvt.KvtError) as e:
        kvt.decode_attention(*args, workspace=ws[:sixteen - 16])
    assert e.value.status == kvt.KVT_ERR_WORKSPACE
    torch.cuda.synchronize()
    say("16 splits vs 32 splits")
    compare(to_f64(few, "bf16"), to_f64(full, "bf16"), "16 splits vs 32")


PER_CU = [
    # (contexts, shortest, longest, Hq, Hkv, D, dtype): how many workgroups share a CU
    (70, 500, 6000, 24, 4, 128, "bf16"),      # unlike contexts: one
    (200, 900, 2600, 8, 8, 64, "bf16"),       # many of them: two of the four that fit
    (300, 900, 2600, 4, 4, 64, "f32"),        # two of three
    (90, 1500, 2900, 32, 8, 128, "bf16"),     # like contexts, a last round of 208 units: one
    (112, 1500, 2900, 16, 8, 64, "bf16"),     # 896 units: two of four
    (90, 300, 590, 8, 8, 64, "f32"),          # short ones: as many as fit
]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("case", range(len(PER_CU)))
def test_a_batch_gives_the_bits_of_its_steps_alone(case):
    """However many workgroups share a CU, and in whatever order they run, an
    unsplit step of a batch gives what each context's own unsplit step (fewer
    units than CUs) gives.  Pages are shared at random to keep the pool small."""
    n, lo, hi, Hq, Hkv, D, dtype = PER_CU[case]
    rng = np.random.default_rng(5400 + case)
    P = np.exp(rng.uniform(np.log(lo), np.log(hi), n)).astype(int).tolist()
    P[0], P[1] = lo, hi
    tt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(case)
    kp, vp = (torch.randn(300, Hkv, 16, D, generator=g, device="cuda", dtype=tt) for _ in range(2))
    q = torch.randn(n, Hq, D, generator=g, device="cuda", dtype=tt)
    table = torch.randint(0, 300, (n, hi // 16 + 1), generator=g, device="cuda", dtype=torch.int32)
    say(f"{n} contexts of {lo}..{hi} keys, {Hq}/{Hkv} heads of {D}, {dtype}")
    out, lse = kvt.decode_attention(q, kp, vp, table, P, return_lse=True, use_workspace=False)
    for b in range(n):
        one, one_lse = kvt.decode_attention(q[b:b + 1], kp, vp, table[b:b + 1], P[b:b + 1], return_lse=True,
                                            use_workspace=False)
        assert torch.equal(one, out[b:b + 1]) and torch.equal(one_lse, lse[b:b + 1]), b
