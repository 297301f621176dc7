"""Calls of the paged-KV attention library at the sizes its users make them.

Each case is one pass that a serving engine makes for one layer: the new
tokens' K/V go into their pages (``kvt.append_kv``) and the new tokens attend
over prefix + suffix (``kvt.extend_attention``, ``kvt.decode_attention`` or
``kvt.cascade_extend_attention``).  The pass returns the attention output, the
log-sum-exp where the caller asks for it, and the two page pools it updated.

Inputs are N(0, 1) in the storage type, drawn on the GPU from the seed: random
tensors at the recorded lengths stand in for traces, and scale 1/sqrt(D) gives
logits of unit variance.  The pool has a quarter more pages than the batch
uses, and the block tables are random permutations of them.
"""
import math

import torch

from paper_2609_39819_amd import kvt

PAGE = 16
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, op, seqs, hq, hkv, d, dtype="bf16", lse=False, shared=0, lo=0, hi=0, new_lo=1, new_hi=1):
    """``seqs`` sequences whose reused lengths lie in lo..hi (log-uniform; for
    a shared prefix uniform, on top of it) and whose new tokens in
    new_lo..new_hi (uniform)."""
    return dict(name=name, op=op, seqs=seqs, hq=hq, hkv=hkv, d=d, dtype=dtype, lse=lse, shared=shared, lo=lo, hi=hi,
                new_lo=new_lo, new_hi=new_hi)


def listed():
    return [
        # the smallest turn of the package's own workloads: fp32 storage, a
        # few pages, where launches and the call itself are the cost
        _case("tiny_turn_f32", "extend", 1, 4, 1, 64, "f32", lo=240, hi=240, new_lo=16, new_hi=16),
        # an agent's short tool result over a long context, odd lengths; the
        # caller keeps the lse (to merge with another GPU's key range)
        _case("short_turn", "extend", 1, 32, 8, 128, lse=True, lo=30011, hi=30011, new_lo=67, new_hi=67),
        # the ordinary turn: 8K reused, 512 new tokens, 32/8 heads
        _case("gqa_8k_turn", "extend", 1, 32, 8, 128, lo=8192, hi=8192, new_lo=512, new_hi=512),
        # the same turn of a small model kept in fp32 (head_dim 64)
        _case("turn_8k_f32", "extend", 1, 32, 8, 64, "f32", lse=True, lo=8192, hi=8192, new_lo=512, new_hi=512),
        # the headline turn: 128K reused, 2048 new tokens, 96/8 heads ...
        _case("react_128k", "extend", 1, 96, 8, 128, lo=131072, hi=131072, new_lo=2048, new_hi=2048),
        # ... and one GPU's share of it under 4-way head parallelism
        _case("react_128k_tp4", "extend", 1, 24, 2, 128, lo=131072, hi=131072, new_lo=2048, new_hi=2048),
        # agents at different depths of their loops in one call (ragged)
        _case("ragged_agents", "extend", 8, 96, 8, 128, lo=2048, hi=131072, new_lo=32, new_hi=128),
        # forked sub-agents adding a short message over their parent's context
        _case("forked_short", "cascade", 16, 96, 8, 128, shared=32768, lo=0, hi=1023, new_lo=16, new_hi=16),
        # one decoding step of a single agent deep in its context ...
        _case("decode_1_128k", "decode", 1, 96, 8, 128, lo=131072, hi=131072),
        # ... of a batch of 32 agents ...
        _case("decode_batch_32", "decode", 32, 96, 8, 128, lo=2048, hi=32768),
        # ... and of a large serving batch with shorter contexts
        _case("decode_batch_256", "decode", 256, 96, 8, 128, lo=1024, hi=8192),
        # the largest call: an early message of a 258K context was replaced
        # and everything after it is recomputed
        _case("mutation_258k", "extend", 1, 96, 8, 128, lo=204800, hi=204800, new_lo=57344, new_hi=57344),
    ]


def draw(rng):
    """One more call of the same ranges: turns from a few tokens to thousands
    over no, short or long contexts, ragged batches, forked batches and
    decoding steps, with the listed cases' head layouts and types."""

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["extend", "extend", "extend", "cascade", "decode", "decode"])
    hq, hkv, d, dtype = rng.choice([(4, 1, 64, "f32"), (32, 8, 64, "f32"), (32, 8, 128, "bf16"), (32, 8, 128, "bf16"),
                                    (32, 8, 64, "bf16"), (24, 2, 128, "bf16"), (96, 8, 128, "bf16"),
                                    (96, 8, 128, "bf16")])
    lse = rng.random() < 0.3
    if op == "decode":
        seqs = log(1, 256)
        hi = log(256, min(131072, 2000000 // seqs))
        return _case("", op, seqs, hq, hkv, d, dtype, lse, lo=max(64, hi // rng.choice([1, 2, 16])), hi=max(64, hi))
    if op == "cascade":
        seqs = rng.randint(2, 24)
        new = log(8, 256)
        return _case("", op, seqs, hq, hkv, d, dtype, lse, shared=PAGE * log(64, 2048), lo=0, hi=log(64, 4096),
                     new_lo=max(1, new // 2), new_hi=new)
    seqs = rng.choice([1, 1, 1, rng.randint(2, 12)])
    hi = 0 if rng.random() < 0.15 else log(200, 131072)   # 0: a context seen for the first time
    new = log(8, 4096 if seqs == 1 else 512)
    return _case("", op, seqs, hq, hkv, d, dtype, lse, lo=hi if seqs == 1 else hi // rng.choice([1, 4, 32]), hi=hi,
                 new_lo=new if seqs == 1 else max(1, new // 3), new_hi=new)


def _lengths(case):
    """Reused and new lengths per sequence.  They belong to the case, not to
    the seed of the inputs, so that every seed's pass does the same work."""
    g = torch.Generator().manual_seed(case["seqs"] * 1000003 + case["hi"] * 31 + case["new_hi"])
    n = case["seqs"]
    u, w = torch.rand(n, generator=g, dtype=torch.float64), torch.rand(n, generator=g, dtype=torch.float64)
    lo, hi = case["lo"], case["hi"]
    if case["shared"] or lo == 0:
        prefix = case["shared"] + lo + (u * (hi - lo + 1)).floor()
    else:
        prefix = (math.log(lo) + u * (math.log(hi) - math.log(lo))).exp().round()
    suffix = case["new_lo"] + (w * (case["new_hi"] - case["new_lo"] + 1)).floor()
    return prefix.to(torch.int64).tolist(), suffix.to(torch.int64).tolist()


def _used_pages(case, prefix, suffix):
    pages = [-(-(p + s) // PAGE) for p, s in zip(prefix, suffix)]
    shared = case["shared"] // PAGE
    return pages, shared, shared + sum(n - shared for n in pages)


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(seed)
    dtype = DTYPES[case["dtype"]]
    prefix, suffix = _lengths(case)
    pages, shared, used = _used_pages(case, prefix, suffix)
    total = used + used // 4 + 1

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=dtype)

    order = torch.randperm(total, generator=g, device=dev).to(torch.int32)
    table = torch.zeros((len(pages), max(pages)), dtype=torch.int32, device=dev)
    at = shared
    for b, n in enumerate(pages):
        table[b, :shared] = order[:shared]
        table[b, shared:n] = order[at:at + n - shared]
        at += n - shared
    tokens = sum(suffix)
    pool = (total, case["hkv"], PAGE, case["d"])
    return dict(case=case, prefix=prefix, suffix=suffix, table=table, k_pool=normal(*pool), v_pool=normal(*pool),
                q=normal(tokens, case["hq"], case["d"]), k_new=normal(tokens, case["hkv"], case["d"]),
                v_new=normal(tokens, case["hkv"], case["d"]))


def run(s):
    case = s["case"]
    kvt.append_kv(s["k_pool"], s["v_pool"], s["table"], s["prefix"], s["suffix"], s["k_new"], s["v_new"])
    if case["op"] == "decode":
        r = kvt.decode_attention(s["q"], s["k_pool"], s["v_pool"], s["table"], s["prefix"], return_lse=case["lse"])
    elif case["op"] == "cascade":
        r = kvt.cascade_extend_attention(s["q"], s["k_pool"], s["v_pool"], s["table"], s["prefix"], s["suffix"],
                                         case["shared"], return_lse=case["lse"])
    else:
        r = kvt.extend_attention(s["q"], s["k_pool"], s["v_pool"], s["table"], s["prefix"], s["suffix"],
                                 return_lse=case["lse"])
    out, lse = r if case["lse"] else (r, None)
    return {"out": out, "lse": lse, "k_pool": s["k_pool"], "v_pool": s["v_pool"]}


def work(case):
    """Every cached token's K and V read once (a shared prefix once for the
    batch), the new tokens' K/V read and written, q read, out (and lse)
    written; 4 * D flops per query head and visible key."""
    prefix, suffix = _lengths(case)
    size = 2 if case["dtype"] == "bf16" else 4
    shared, d, hq, hkv = case["shared"], case["d"], case["hq"], case["hkv"]
    tokens = sum(suffix)
    cached = shared + sum(p - shared for p in prefix) + tokens
    moved = (2 * cached + 4 * tokens) * hkv * d * size + 2 * tokens * hq * d * size
    if case["lse"]:
        moved += tokens * hq * 4
    pairs = sum(s * p + s * (s + 1) // 2 for p, s in zip(prefix, suffix))
    return {"bytes": moved, "flops": 4 * d * hq * pairs}


def tolerance(case):
    # the probabilities are rounded to bf16 for the value product (as are q,
    # K and V in fp32 storage) and the bf16 output once more; the same call
    # with and without key splits (sums in another order, probabilities
    # rounded against another reference) differs by up to 3.2e-3, an element
    # by up to 2.4e-2: about three and four times that
    return {"rel": 1e-2, "max": 0.1}


def exact(case, seed):
    """The same pass in float64: gathered logical K and V, full scores, masked
    softmax, weighted values."""
    if work(case)["flops"] > 4e13:      # minutes in float64
        return None
    s = prepare(case, seed)
    d, hq, hkv = case["d"], case["hq"], case["hkv"]
    group = hq // hkv
    k_pool, v_pool = s["k_pool"], s["v_pool"]
    dev = k_pool.device
    tokens = sum(s["suffix"])
    out = torch.empty((tokens, hq, d), dtype=torch.float64, device=dev)
    lse = torch.empty((tokens, hq), dtype=torch.float64, device=dev)
    at = 0
    for b, (p, n) in enumerate(zip(s["prefix"], s["suffix"])):
        pos = torch.arange(p, p + n, device=dev)
        page, slot = s["table"][b].long()[pos // PAGE], pos % PAGE
        k_pool[page, :, slot] = s["k_new"][at:at + n]
        v_pool[page, :, slot] = s["v_new"][at:at + n]
        at += n
    at = 0
    for b, (p, n) in enumerate(zip(s["prefix"], s["suffix"])):
        length = p + n
        page = s["table"][b, :-(-length // PAGE)].long()
        seen = torch.arange(length, device=dev)
        step = max(1, int(2 ** 28 // (length * group)))
        for h in range(hkv):
            k = k_pool[page, h].reshape(-1, d)[:length].double()
            v = v_pool[page, h].reshape(-1, d)[:length].double()
            kt = k.t().contiguous()
            for t in range(0, n, step):
                m = min(step, n - t)
                rows = slice(at + t, at + t + m)
                heads = slice(h * group, (h + 1) * group)
                q = s["q"][rows, heads].double().reshape(m * group, d)
                x = torch.mm(q, kt).mul_(1.0 / math.sqrt(d)).view(m, group, length)
                last = torch.arange(p + t, p + t + m, device=dev)
                x.masked_fill_((seen[None, :] > last[:, None])[:, None, :], -math.inf)
                top = x.amax(dim=-1, keepdim=True)
                x = x.sub_(top).exp_()
                total = x.sum(dim=-1, keepdim=True)
                lse[rows, heads] = (top + total.log())[..., 0]
                out[rows, heads] = torch.mm(x.view(m * group, length), v).view(m, group, d) / total
        at += n
    return {"out": out, "lse": lse if case["lse"] else None, "k_pool": None, "v_pool": None}
