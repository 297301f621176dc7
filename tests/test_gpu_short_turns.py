"""Short messages, whose key ranges split until the chip is filled and whose
last (partly filled) row tile takes fewer splits than the full ones: at the
edges of row tiles, waves and split counts, against the oracle and the
unsplit call, with the workspace's bytes all NaN beforehand (a set that holds
no keys for a row is never read).
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
    # (P, S, Hq, Hkv, D, dtype, partial sets, key splits of the last row tile)
    ([4000], [67], 32, 8, 128, "bf16", 16, 10),   # 268 rows: a full tile and one of 12 rows
    ([4001], [96], 32, 8, 128, "bf16", 18, 12),   # 384 rows: four waves in the last tile
    ([4001], [97], 32, 8, 128, "bf16", 15, 14),   # 388 rows: five
    ([4001], [128], 32, 8, 128, "bf16", 15, 15),   # 512 rows: the last tile is full
    ([3999], [1], 16, 8, 64, "f32", 32, 32),   # 2 rows in all
    ([5000], [33], 8, 1, 64, "bf16", 64, 42),   # 264 rows of one kv-head: many splits, two tiles
    ([2500, 3100, 4200], [70, 9, 40], 24, 2, 128, "bf16", 19, 18),   # like contexts, last tiles of each weight
    ([3000], [40], 32, 8, 128, "f32", 16, 16),   # 160 rows
    ([2300], [300], 20, 5, 128, "bf16", 9, 9),   # kv-heads that do not divide the CUs
    # so many rows that the other merge kernel runs
    ([12011], [614], 64, 8, 128, "bf16", 3, 2),    # 4912 rows: 19 full tiles and one of 48 rows
    ([14146], [475], 96, 8, 64, "f32", 4, 3),      # 5700 rows: 22 and one of 68
]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("case", range(len(CASES)))
def test_short_turn_matches_the_oracle_and_the_unsplit_call(case):
    P, S, Hq, Hkv, D, dtype, sets, last = CASES[case]
    w = build_workload(name=f"short{case}", seed=6100 + case, prefix_len=P, suffix_len=S, num_q_heads=Hq,
                       num_kv_heads=Hkv, head_dim=D, dtype=dtype)
    d = stage(w)
    kvt.append_kv(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, d["k_new"], d["v_new"])
    args = (d["q"], d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, w.scale)
    need = kvt.extend_workspace_bytes(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, Hq)
    rows = w.total_tokens * Hq
    say(f"short turn {case}: {need / (rows * (D + 2) * 4):.1f} partial sets")
    assert need == -(-sets * rows * D * 4 // 256) * 256 + sets * rows * 8
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")      # NaN in fp32
    out, lse = kvt.extend_attention(*args, return_lse=True, workspace=ws)
    again = kvt.extend_attention(*args, workspace=ws)
    whole, whole_lse = kvt.extend_attention(*args, return_lse=True, use_workspace=False)
    torch.cuda.synchronize()
    assert torch.equal(out, again), "run to run"
    # the last row's part of every set: written by the splits that its tile has, and only by them
    o = ws.view(torch.float32)[:sets * rows * D].view(sets, rows, D)[:, rows - 1]
    assert torch.isnan(o).all(dim=1).tolist() == [False] * last + [True] * (sets - last)
    compare(to_f64(out, dtype), to_f64(whole, dtype), "split vs unsplit")
    # both sums add probabilities rounded to bf16 (2^-9 relative at most)
    assert float((lse - whole_lse).abs().max()) <= 2 ** -8
    kp, vp = oracle_append(w.k_pool_c, w.v_pool_c, w.compact_table, w.prefix_len, w.suffix_len, w.k_new, w.v_new)
    picked = sample_rows(w, 32, seed=case)
    ref, ref_lse = oracle_extend(w.q, kp, vp, w.compact_table, w.prefix_len, w.suffix_len, Hkv, w.scale, rows=picked)
    compare(gather_rows(to_f64(out, dtype), w, picked), ref, "short turn vs oracle")
    err = float(np.abs(gather_rows(lse.cpu().numpy().astype(np.float64), w, picked) - ref_lse).max())
    assert err <= (2 ** -9 if dtype == "bf16" else 1e-2), "lse vs oracle"


@pytest.mark.timeout(300)
def test_a_workspace_for_fewer_splits_is_accepted():
    """7000 keys, 32 new tokens: at 1024 keys per split 6 partial sets were
    asked for; that workspace still runs the call, and one of less than that
    is refused."""
    P, S, Hq, Hkv, D = [7000], [32], 32, 8, 128
    w = build_workload(name="short-old-ws", seed=6200, prefix_len=P, suffix_len=S, num_q_heads=Hq, num_kv_heads=Hkv,
                       head_dim=D, dtype="bf16")
    d = stage(w)
    kvt.append_kv(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, d["k_new"], d["v_new"])
    args = (d["q"], d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, w.scale)
    need = kvt.extend_workspace_bytes(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, Hq)
    six = 6 * 32 * Hq * (D + 2) * 4
    assert need > six
    full = kvt.extend_attention(*args)
    ws = torch.full((six,), 0xFF, dtype=torch.uint8, device="cuda")
    few = kvt.extend_attention(*args, workspace=ws)
    with pytest.raises(kvt.KvtError) as e:
        kvt.extend_attention(*args, workspace=ws[:six - 16])
    assert e.value.status == kvt.KVT_ERR_WORKSPACE
    torch.cuda.synchronize()
    compare(to_f64(few, "bf16"), to_f64(full, "bf16"), "6 splits vs the plan's")


@pytest.mark.timeout(300)
@pytest.mark.parametrize("op", ["extend", "decode"])
def test_an_unaligned_workspace_runs_unsplit_where_the_base_plan_does(op):
    """1900 keys give one split at 1024 keys each: the call took any workspace
    argument before short messages split further, and still does."""
    S = 37 if op == "extend" else 1
    w = build_workload(name="short-unaligned", seed=6300, prefix_len=[1900], suffix_len=[S], num_q_heads=32,
                       num_kv_heads=8, head_dim=128, dtype="bf16")
    d = stage(w)
    kvt.append_kv(d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len, d["k_new"], d["v_new"])
    if op == "extend":
        call, need = kvt.extend_attention, kvt.extend_workspace_bytes
        args = (d["q"], d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len, w.suffix_len)
    else:
        call, need = kvt.decode_attention, kvt.decode_workspace_bytes
        args = (d["q"], d["k_pool"], d["v_pool"], d["block_table"], w.prefix_len)
    size = need(*args[1:], 32)
    assert size > 0
    ws = torch.full((size + 16,), 0xFF, dtype=torch.uint8, device="cuda")
    out = call(*args, w.scale, workspace=ws[1:])
    whole = call(*args, w.scale, use_workspace=False)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), whole.view(torch.int16))
    assert bool((ws == 0xFF).all()), "the workspace is not touched"
