"""Contexts whose keys of one kv-head span more than 2^32 bytes (2^23 to 2^25
positions), through block tables that repeat a few pages so that the pool
stays tiny.

One page holds sixteen needles: its key row r is a multiple of unit vector
e_r, and query head h asks for e_h with a logit of 50 over the zeros
elsewhere, so that out[h] = V[row h of that page] to within 2^25 * e^-50 of the
values.  The page lies where the bytes from its first row to the end of the
context are 2^32 and a few rows: an offset formed in 32 bits from that distance
takes one row of the page for several.
"""
import numpy as np
import pytest

from paper_2609_39819_amd import kvt

from gpu_common import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

HEADS = 16
PAGE = 16
TYPES = [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)]


@pytest.mark.timeout(120)
@pytest.mark.parametrize("op", ["extend", "cascade"])
@pytest.mark.parametrize("dtype,D", TYPES)
def test_rows_2_to_the_32_bytes_before_the_end(dtype, D, op):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    span = (1 << 32) // (D * (2 if dtype == "bf16" else 4))   # positions of one kv-head in 2^32 bytes
    S, seqs = 3, 2                             # two sequences of the same pages, but for their last one
    P = span + 104 - S
    needle_at = 6 * PAGE                       # 2^32 bytes and 7 rows before the last position
    g = torch.Generator(device="cuda").manual_seed(5 + D)
    pool = (7, 1, PAGE, D)
    k_pool = torch.zeros(pool, dtype=dt, device="cuda")
    v_pool = torch.randn(pool, generator=g, device="cuda").to(torch.bfloat16).to(dt)   # exact in either type
    eye = torch.eye(HEADS, D, device="cuda")
    k_pool[4, 0] = (20 * eye).to(dt)
    q = (20 * eye).to(dt).expand(S * seqs, HEADS, D).contiguous()
    new = torch.zeros((S * seqs, 1, D), dtype=dt, device="cuda")
    ids = np.random.default_rng(31 + D).integers(0, 4, -(-(P + S) // PAGE)).astype(np.int32)
    ids[needle_at // PAGE] = 4
    bt = torch.from_numpy(np.stack([ids] * seqs)).cuda()
    bt[:, -1] = torch.tensor([5, 6], dtype=torch.int32)
    assert P // PAGE == (P + S - 1) // PAGE == len(ids) - 1, "the new tokens go into the last page"
    want = v_pool[4, 0].float()
    say(f"{op} {dtype} D={D}: {P} + {S} tokens, needles at {needle_at}")
    args = (k_pool, v_pool, bt, [P] * seqs, [S] * seqs)
    kvt.append_kv(*args, new, new)
    if op == "extend":
        out = kvt.extend_attention(q, *args, 50.0 / 400.0)
    else:                                      # one shared page; the private parts hold the needles
        out = kvt.cascade_extend_attention(q, *args, PAGE, 50.0 / 400.0, mode=kvt.CASCADE_SHARED_PASS)
    torch.cuda.synchronize()
    # p and l carry the same bf16 probability, so the one rounding left is the output's
    err = ((out.float() - want).abs() / want.abs().clamp_min(2 ** -6)).amax(dim=(0, 2))
    say("largest relative error per needle", [f"{e:.1e}" for e in err.tolist()])
    assert float(err.max()) <= 2 ** -8
