"""The work a user has this library do, as measurable cases: whole ring schedules, single block steps with
their Update, attention of a short Query chunk to long cached K/V chunks, and merges of partial results.

A case is a dict of plain values; "path" names the entry points it goes through:
  ring    tr_ring_attn without a workspace: Algorithm 1's schedule on one GPU
  sched   tr_ring_attn_sched: the zigzag, Ring Attention and hybrid orders
  blocks  tr_ring_attn_blocks: the two-kernel form, the block result stored as bf16 or fp32 in between
  steps   one device's loop over K/V chunks written by the caller: the first block goes straight into the fp32
          accumulators (tr_block_attn), every later one is a tr_block_attn followed by tr_merge
  fold    the same loop with tr_block_attn_merge for the later blocks
  at      tr_block_attn_causal_at: a Query chunk at its position behind cached keys
  merge   tr_merge of n partial results in turn, from an empty accumulator
  nary    tr_merge_n of n partial results
Lengths are per sequence; "layout" is "bhsd" (dense [B,H,S,D]) or "token" ([B,S,H,D] handed over through the
strides, the layout in which a model's projections leave Q, K and V).
"""
import math

import torch

import paper_2412_20501_amd as tr

SCHEDULES = {"ring": tr.TR_SCHED_RING_ATTENTION, "zigzag": tr.TR_SCHED_ZIGZAG, "hybrid": tr.TR_SCHED_HYBRID}
DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}


def listed():
    return [
        # the four-device walk-through at its smallest: a schedule whose cost is launches and host calls
        {"name": "ring_small", "path": "ring", "B": 1, "Hq": 2, "Hkv": 2, "S": 256, "D": 64, "n": 4, "causal": False, "layout": "bhsd"},
        # causal prefill of a 32K prompt, 8 devices replayed (32 heads of 128: the 7B head shape)
        {"name": "ring_causal_32k", "path": "ring", "B": 1, "Hq": 32, "Hkv": 32, "S": 32768, "D": 128, "n": 8, "causal": True, "layout": "bhsd"},
        # long-context prefill with grouped-query heads, 16 devices: the largest
        {"name": "ring_gqa_128k", "path": "ring", "B": 1, "Hq": 32, "Hkv": 8, "S": 131072, "D": 128, "n": 16, "causal": True, "layout": "bhsd"},
        # a diffusion transformer's full attention: head dim 64, batch 2, four devices
        {"name": "ring_dit_16k", "path": "ring", "B": 2, "Hq": 24, "Hkv": 24, "S": 16384, "D": 64, "n": 4, "causal": False, "layout": "bhsd"},
        # a moderate prompt under the zigzag partition, grouped-query heads, the model's token-major layout
        {"name": "zigzag_token_8k", "path": "sched", "order": "zigzag", "inner": 1, "B": 1, "Hq": 32, "Hkv": 8, "S": 8192, "D": 128, "n": 4,
         "causal": True, "layout": "token"},
        # bf16 transport of the block results between Attention and Update, chunks that are no whole tiles
        {"name": "blocks_bf16_ragged", "path": "blocks", "block": "bf16", "B": 1, "Hq": 16, "Hkv": 4, "S": 6008, "D": 128, "n": 4,
         "causal": True, "layout": "bhsd"},
        # the block step the benchmark quotes: a Query chunk of 4096 against two K/V chunks of 4096, bf16 block_out merged
        {"name": "steps_4k", "path": "steps", "B": 1, "Hq": 32, "Hkv": 32, "Sq": 4096, "Sk": 4096, "D": 128, "n": 2, "diag": False,
         "block": "bf16", "layout": "bhsd"},
        # a diagonal chunk and one before it, head dim 64, odd length, fp32 blocks
        {"name": "steps_diag_odd", "path": "steps", "B": 2, "Hq": 12, "Hkv": 12, "Sq": 1777, "Sk": 1777, "D": 64, "n": 2, "diag": True,
         "block": "fp32", "layout": "bhsd"},
        # chunked prefill: 500 new tokens behind a cache of 12000 (keys 12500), grouped-query heads
        {"name": "prefill_at_12k", "path": "at", "B": 1, "Hq": 32, "Hkv": 8, "Sq": 500, "Sk": 12500, "D": 128, "q0": 12000, "k0": 0,
         "block": "bf16", "layout": "token"},
        # decode: one new token for each of 4 sequences against four devices' K/V chunks of 8192
        {"name": "decode_32k", "path": "fold", "B": 4, "Hq": 32, "Hkv": 8, "Sq": 1, "Sk": 8192, "D": 128, "n": 4, "diag": False, "layout": "bhsd"},
        # the merge-only workload: eight fp32 partial results of a 32K sequence in ring order
        {"name": "merge_8x32k", "path": "merge", "B": 1, "H": 32, "S": 32768, "D": 128, "n": 8, "block": "fp32"},
        # everything that arrived meanwhile folded at once: six bf16 partials, odd length
        {"name": "nary_6_odd", "path": "nary", "B": 2, "H": 16, "S": 5003, "D": 128, "n": 6, "block": "bf16", "acc": False},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def _heads(rng, most):
    hkv = rng.choice([h for h in (1, 2, 3, 4, 8, 12, 16, 32) if h <= most])
    group = rng.choice([g for g in (1, 1, 2, 3, 4, 8) if g * hkv <= most])
    return hkv * group, hkv


def draw(rng):
    path = rng.choice(["ring", "ring", "sched", "blocks", "steps", "fold", "at", "merge", "nary"])
    if path in ("merge", "nary"):
        case = {"path": path, "B": rng.choice([1, 1, 2, 4]), "H": rng.choice([2, 3, 8, 12, 16, 32]), "S": _log_int(rng, 64, 16384),
                "D": rng.choice([64, 128]), "n": _log_int(rng, 2, 12), "block": rng.choice(["fp32", "bf16"])}
        if path == "nary":
            case["acc"] = rng.random() < 0.5
        return case
    hq, hkv = _heads(rng, 32)
    case = {"path": path, "B": rng.choice([1, 1, 2, 4]), "Hq": hq, "Hkv": hkv, "D": rng.choice([64, 128, 128]),
            "layout": rng.choice(["bhsd", "bhsd", "token"])}
    if path in ("ring", "sched", "blocks"):
        n = rng.choice([2, 3, 4, 8])
        causal, parts = rng.random() < 0.5, n
        if path == "sched":
            case["order"] = rng.choice(["ring", "zigzag", "hybrid"])
            case["inner"] = 1
            if case["order"] == "zigzag":
                causal, parts = True, 2 * n
            elif case["order"] == "hybrid":
                case["inner"] = rng.choice([d for d in (1, 2, 3, 4) if n % d == 0])
        length = _log_int(rng, 256, 32768)
        whole = rng.choice([1, 1, 64, 128])              # chunks of any length, or of whole tiles
        chunk = max(whole, length // parts // whole * whole)
        case.update(S=chunk * parts, n=n, causal=causal)
        if path == "blocks":
            case["block"] = rng.choice(["bf16", "fp32"])
    elif path == "steps":
        sq = _log_int(rng, 64, 8192)
        diag = rng.random() < 0.5
        case.update(Sq=sq, Sk=sq if diag else _log_int(rng, 64, 8192), n=rng.choice([1, 2, 4]), diag=diag, block=rng.choice(["bf16", "fp32"]))
    elif path == "fold":
        case.update(Sq=_log_int(rng, 1, 128), Sk=_log_int(rng, 512, 16384), n=rng.choice([1, 2, 4, 8]), diag=False)
    else:
        sq, past = _log_int(rng, 16, 4096), _log_int(rng, 64, 28000)
        case.update(Sq=sq, Sk=past + sq, q0=past, k0=0, block=rng.choice(["bf16", "fp32"]))
    return case


def _qkv(gen, B, H, S, D, layout):
    """N(0,1) values in bf16: what the attention of a normalised model sees, and what every workload here is drawn from."""
    if layout == "token":
        return torch.randn((B, S, H, D), device="cuda", dtype=torch.bfloat16, generator=gen).permute(0, 2, 1, 3)
    return torch.randn((B, H, S, D), device="cuda", dtype=torch.bfloat16, generator=gen)


def _empty(B, H, S, D, layout, dtype):
    if layout == "token":
        return torch.empty((B, S, H, D), device="cuda", dtype=dtype).permute(0, 2, 1, 3)
    return torch.empty((B, H, S, D), device="cuda", dtype=dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    st = dict(case)
    path = case["path"]
    if path in ("merge", "nary"):
        B, H, S, D, n = case["B"], case["H"], case["S"], case["D"], case["n"]
        dtype = DTYPES[case["block"]]
        # partial results as the merge workload has them: values N(0,1), log-sum-exps U(-5, 15)
        st["outs"] = [torch.randn((B, H, S, D), device="cuda", dtype=dtype, generator=gen) for _ in range(n)]
        st["lses"] = [torch.rand((B, H, S), device="cuda", generator=gen) * 20 - 5 for _ in range(n)]
        st["out"] = torch.empty((B, H, S, D), device="cuda")
        st["lse"] = torch.empty((B, H, S), device="cuda")
        if path == "nary" and case["acc"]:
            st["seen"] = torch.rand((B, H, S), device="cuda", generator=gen) * 20 - 5
            st["held"] = torch.randn((B, H, S, D), device="cuda", generator=gen)
        return st
    B, Hq, Hkv, D, layout = case["B"], case["Hq"], case["Hkv"], case["D"], case["layout"]
    st["scale"] = 1.0 / math.sqrt(D)
    if path in ("ring", "sched", "blocks"):
        S = case["S"]
        st["q"], st["k"], st["v"] = _qkv(gen, B, Hq, S, D, layout), _qkv(gen, B, Hkv, S, D, layout), _qkv(gen, B, Hkv, S, D, layout)
        st["out"], st["lse"] = _empty(B, Hq, S, D, layout, torch.float32), torch.empty((B, Hq, S), device="cuda")
        if path == "blocks":
            dt = tr.TR_BF16 if case["block"] == "bf16" else tr.TR_F32
            st["block_dtype"] = dt
            st["ws"] = torch.empty(tr.tr_ring_attn_blocks_workspace_bytes(st["q"], case["n"], dt), dtype=torch.uint8, device="cuda")
        return st
    Sq, Sk = case["Sq"], case["Sk"]
    st["q"] = _qkv(gen, B, Hq, Sq, D, layout)
    if path == "at":
        st["k"], st["v"] = _qkv(gen, B, Hkv, Sk, D, layout), _qkv(gen, B, Hkv, Sk, D, layout)
        st["out"] = _empty(B, Hq, Sq, D, layout, DTYPES[case["block"]])
    else:
        st["kv"] = [(_qkv(gen, B, Hkv, Sk, D, layout), _qkv(gen, B, Hkv, Sk, D, layout)) for _ in range(case["n"])]
        st["out"] = _empty(B, Hq, Sq, D, layout, torch.float32)
        if path == "steps" and case["n"] > 1:
            st["blk_out"], st["blk_lse"] = _empty(B, Hq, Sq, D, layout, DTYPES[case["block"]]), torch.empty((B, Hq, Sq), device="cuda")
    st["lse"] = torch.empty((B, Hq, Sq), device="cuda")
    return st


def run(st):
    path, out, lse = st["path"], st["out"], st["lse"]
    if path == "ring":
        tr.tr_ring_attn(st["q"], st["k"], st["v"], st["n"], st["causal"], out, lse, st["scale"])
    elif path == "sched":
        tr.tr_ring_attn_sched(st["q"], st["k"], st["v"], st["n"], st["causal"], SCHEDULES[st["order"]], out, lse, st["scale"], st["inner"])
    elif path == "blocks":
        tr.tr_ring_attn_blocks(st["q"], st["k"], st["v"], st["n"], st["causal"], out, lse, st["block_dtype"], st["ws"], st["scale"])
    elif path == "steps":
        mask = tr.TR_MASK_CAUSAL_DIAG if st["diag"] else tr.TR_MASK_NONE       # the device's own chunk comes first
        k, v = st["kv"][0]
        tr.tr_block_attn(st["q"], k, v, mask, st["scale"], out, lse)
        for k, v in st["kv"][1:]:
            tr.tr_block_attn(st["q"], k, v, tr.TR_MASK_NONE, st["scale"], st["blk_out"], st["blk_lse"])
            tr.tr_merge(out, lse, st["blk_out"], st["blk_lse"])
    elif path == "fold":
        k, v = st["kv"][0]
        tr.tr_block_attn(st["q"], k, v, tr.TR_MASK_NONE, st["scale"], out, lse)
        for k, v in st["kv"][1:]:
            tr.tr_block_attn_merge(st["q"], k, v, tr.TR_MASK_NONE, st["scale"], out, lse)
    elif path == "at":
        tr.tr_block_attn_causal_at(st["q"], st["k"], st["v"], st["q0"], st["k0"], st["scale"], out, lse)
    elif path == "merge":
        lse.fill_(float("-inf"))                       # an empty accumulator: its out is not read as a result
        for bo, bl in zip(st["outs"], st["lses"]):
            tr.tr_merge(out, lse, bo, bl)
    else:
        if st["acc"]:
            out.copy_(st["held"])
            lse.copy_(st["seen"])
        tr.tr_merge_n(out, lse, st["outs"], st["lses"], st["acc"])
    return out, lse


def work(case):
    path = case["path"]
    if path in ("merge", "nary"):
        rows = case["B"] * case["H"] * case["S"]
        block = 2 if case["block"] == "bf16" else 4
        partial = rows * (case["D"] * block + 4)
        held = rows * (case["D"] + 1) * 4
        reads = case["n"] * partial + (held if case.get("acc") else 0)
        return {"bytes": reads + held, "flops": 2.0 * rows * case["D"] * case["n"]}
    B, Hq, Hkv, D = case["B"], case["Hq"], case["Hkv"], case["D"]
    if path in ("ring", "sched", "blocks"):
        Sq, Sk = case["S"], case["S"]
        pairs = Sq * (Sq + 1) / 2 if case["causal"] else Sq * Sk
        out_bytes = 4
    elif path == "at":
        Sq, Sk = case["Sq"], case["Sk"]
        first = case["q0"] - case["k0"] + 1              # keys the first Query row sees; every row sees them all up to itself
        pairs = Sq * first + Sq * (Sq - 1) / 2
        out_bytes = 2 if case["block"] == "bf16" else 4
    else:
        Sq, Sk = case["Sq"], case["Sk"] * case["n"]
        pairs = Sq * Sk - (Sq * (Sq - 1) / 2 if case["diag"] else 0)
        out_bytes = 4
    return {"bytes": B * (Hq * Sq * (D * (2 + out_bytes) + 4) + 2 * Hkv * Sk * D * 2), "flops": 4.0 * B * Hq * D * pairs}


def tolerance(case):
    """About four times the distance from the same operation in 64 bits: out 1.0e-3 .. 1.7e-3 (rounding the weights to bf16),
    2.4e-3 where blocks are bf16 too, largest element 6.5e-2 of the root mean square (a causal sequence's first rows, which
    single values dominate) and 1.8e-2 elsewhere; the merges 3.5e-7 and 3.9e-6."""
    if case["path"] in ("merge", "nary"):
        return {"rel": 1.5e-6, "max": 1.6e-5}
    causal = case.get("causal") or case.get("diag") or case["path"] == "at"
    return {"rel": 9e-3 if case.get("block") == "bf16" else 6.5e-3, "max": 0.4 if causal else 8e-2}


def exact(case, seed):
    """out and lse in 64 bits from the definitions: attention over every key a row sees, and partial results weighted by
    exp(lse_i - lse).  Row blocks keep the score matrix near a gigabyte."""
    st = prepare(case, seed)
    if case["path"] in ("merge", "nary"):
        outs, lses = list(st["outs"]), list(st["lses"])
        if case.get("acc"):
            outs, lses = outs + [st["held"]], lses + [st["seen"]]
        lse = torch.logsumexp(torch.stack([x.double() for x in lses]), 0)
        out = torch.zeros(st["out"].shape, dtype=torch.float64, device="cuda")
        for o, x in zip(outs, lses):
            out += torch.exp(x.double() - lse)[..., None] * o.double()
        return out, lse
    B, Hq, Hkv, D, scale = case["B"], case["Hq"], case["Hkv"], case["D"], st["scale"]
    kv = st["kv"] if "kv" in st else [(st["k"], st["v"])]
    Sq = st["q"].shape[2]
    out = torch.empty((B, Hq, Sq, D), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, Hq, Sq), dtype=torch.float64, device="cuda")
    causal = case.get("causal") or case.get("diag") or case["path"] == "at"
    first = case.get("q0", 0) - case.get("k0", 0)          # Query row r sees the keys up to r + first of the chunk that holds the diagonal
    own = kv[0][0].shape[2]                                # keys of that chunk; those behind it are seen by every row
    rows = torch.arange(Sq, device="cuda")
    for b in range(B):
        for g in range(Hkv):
            k = torch.cat([x[b, g].double() for x, _ in kv])
            v = torch.cat([x[b, g].double() for _, x in kv])
            step = max(64, min(Sq, (1 << 27) // k.shape[0]))
            for h in range(g * (Hq // Hkv), (g + 1) * (Hq // Hkv)):
                for r0 in range(0, Sq, step):
                    r1 = min(Sq, r0 + step)
                    n = min(k.shape[0], r1 + first) if causal and len(kv) == 1 else k.shape[0]
                    s = (st["q"][b, h, r0:r1].double() * scale) @ k[:n].t()
                    if causal:
                        m = min(n, own)
                        s[:, :m].masked_fill_(torch.arange(m, device="cuda")[None, :] > rows[r0:r1, None] + first, float("-inf"))
                    top = s.amax(1, keepdim=True)
                    s.sub_(top).exp_()
                    total = s.sum(1)
                    out[b, h, r0:r1] = (s @ v[:n]) / total[:, None]
                    lse[b, h, r0:r1] = top[:, 0] + total.log()
    return out, lse
