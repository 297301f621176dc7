"""The shared pass of a cascade on few row tiles, whose shared part splits as a
short message does, against the oracle and the plain extend, and the
workspaces its calls asked for before (fewer splits) still accepted.
"""
import numpy as np
import pytest

from oracle import oracle_append, oracle_extend
from paper_2609_39819_amd import kvt
from paper_2609_39819_amd.workloads import build_workload

from gpu_common import compare, gather_rows, sample_rows, say, stage, to_f64

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # (P, S, shared, Hq, Hkv, D, dtype, partial sets)
    ([4096, 4200, 4100], [9, 16, 3], 4096, 32, 8, 128, "bf16", 32),     # 112 rows per kv-head, one row tile
    ([4500] * 9, [11] * 9, 4096, 24, 2, 128, "bf16", 28),               # 1188 rows: 4 full tiles and 5 waves of a fifth
    ([2100, 2080], [5, 6], 2064, 4, 1, 64, "f32", 33),                  # shared not a multiple of 64
    ([8300] * 5, [16] * 5, 8192, 8, 1, 64, "bf16", 49),                 # one kv-head, 640 rows
]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("case", range(len(CASES)))
def test_shared_pass_on_few_row_tiles(case):
    P, S, shared, Hq, Hkv, D, dtype, sets = CASES[case]
    w = build_workload(name=f"casc-split{case}", seed=7100 + case, prefix_len=P, suffix_len=S, num_q_heads=Hq,
                       num_kv_heads=Hkv, head_dim=D, dtype=dtype, shared_prefix_blocks=shared // 16)
    d = stage(w)
    kvt.append_kv(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, d["k_new"], d["v_new"])
    args = (d["q"], d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len)
    need = kvt.cascade_workspace_bytes(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, shared,
                                       Hq, kvt.CASCADE_SHARED_PASS)
    one = w.total_tokens * Hq * (D + 2) * 4
    say(f"cascade case {case}: {need / one:.1f} partial sets")
    rows = w.total_tokens * Hq
    assert need == -(-sets * rows * D * 4 // 256) * 256 + sets * rows * 8
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    out, lse = kvt.cascade_extend_attention(*args, shared, w.scale, return_lse=True, workspace=ws,
                                            mode=kvt.CASCADE_SHARED_PASS)
    plain, plain_lse = kvt.extend_attention(*args, w.scale, return_lse=True, use_workspace=False)
    torch.cuda.synchronize()
    compare(to_f64(out, dtype), to_f64(plain, dtype), "cascade vs plain")
    assert float((lse - plain_lse).abs().max()) <= 2 ** -8     # sums of bf16-rounded probabilities
    kp, vp = oracle_append(w.k_pool_c, w.v_pool_c, w.compact_table, w.prefix_len, w.suffix_len, w.k_new, w.v_new)
    picked = sample_rows(w, 8, seed=case)
    ref, _ = oracle_extend(w.q, kp, vp, w.compact_table, w.prefix_len, w.suffix_len, Hkv, w.scale, rows=picked)
    compare(gather_rows(to_f64(out, dtype), w, picked), ref, "cascade vs oracle")


@pytest.mark.timeout(300)
@pytest.mark.parametrize("mode", [kvt.CASCADE_SHARED_PASS, kvt.CASCADE_PLAIN])
def test_a_workspace_for_the_base_splits_is_accepted(mode):
    """4096 shared keys give 4 splits at 1024 keys each and one private set, the
    plain extend 4 splits; a workspace of that size still runs the call, and
    a smaller one is refused."""
    P, S, shared, Hq, Hkv, D = [4096, 4200, 4100], [9, 16, 3], 4096, 32, 8, 128
    w = build_workload(name="casc-old-ws", seed=7200, prefix_len=P, suffix_len=S, num_q_heads=Hq, num_kv_heads=Hkv,
                       head_dim=D, dtype="bf16", shared_prefix_blocks=shared // 16)
    d = stage(w)
    kvt.append_kv(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, d["k_new"], d["v_new"])
    args = (d["q"], d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, shared)
    need = kvt.cascade_workspace_bytes(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, shared,
                                       Hq, mode)
    one = w.total_tokens * Hq * (D + 2) * 4
    base = (4 + 1) * one if mode == kvt.CASCADE_SHARED_PASS else 4 * one
    assert need > base
    full = kvt.cascade_extend_attention(*args, mode=mode)
    ws = torch.full((base,), 0xFF, dtype=torch.uint8, device="cuda")
    few = kvt.cascade_extend_attention(*args, mode=mode, workspace=ws)
    with pytest.raises(kvt.KvtError) as e:
        kvt.cascade_extend_attention(*args, mode=mode, workspace=ws[:one])
    assert e.value.status == kvt.KVT_ERR_WORKSPACE
    torch.cuda.synchronize()
    compare(to_f64(few, "bf16"), to_f64(full, "bf16"), "base splits vs the plan's")
