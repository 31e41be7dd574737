"""The work that is timed on an MI355X: calls of the package's entry points over the shapes that a serving loop gives them.

A case is one dict of plain values; `prepare` makes what a serving loop has in hand (paged pools, block table, queries, index
lists, outputs, workspace), `run` makes the calls of one pass, `exact` is the same in float64 with plain torch.

Values.  The queries of one group (the k+1 positions and the heads that share a KV head) have a direction in common, as
adjacent decoding steps of one request have, and each (request, KV head) has as many *pillar* tokens as its budget allows:
keys that lean towards that direction, the first positions (attention sinks) among them, the rest anywhere.  They carry
most of the attention mass, which is what the method lives on, and few other tokens come near them, so the selected set does
not hang on the last bits of a score.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2512_01278_amd as pa

DEVICE = "cuda:0"
SINKS = 4                  # attention sinks: the first positions of every context
SHARED = 0.7               # weight of the direction that the queries of a group share
GAIN = (9.0, 11.0)         # how far a pillar key leans towards it (ordinary keys are standard normal)

QWEN = dict(hq=32, hkv=8, dim=128, page=16, k=4, q="bf16", kv="bf16")       # attention layer of an 8B model, four drafts


def listed():
    return [
        # the smallest round there is: two short contexts in fp32, the three stages as three calls, on the kernels for any shape
        dict(name="round_f32_b2", op="three_calls", batch=2, hq=4, hkv=1, dim=64, page=16, k=3, q="f32", kv="f32", lens="uniform",
             lo=300, hi=512, budget=64),
        # one user at a prompt: one request, verification with selection and a draft step; launches and latency are what counts
        dict(QWEN, name="round_b1_2k", op="round", batch=1, lens="uniform", lo=2100, hi=2100, budget=128),
        # a small server: 32 requests of one length, verification with selection and a draft step
        dict(QWEN, name="round_b32_4k", op="round", batch=32, lens="uniform", lo=4096, hi=4096, budget=256),
        # the batch the benchmark reports: 128 reasoning requests of 1 to 8 K tokens, 5 % of them kept: verification with selection,
        dict(QWEN, name="verify_select_b128_8k", op="verify_select", batch=128, lens="uniform", lo=1024, hi=8192, budget=0),
        # one draft step of the same batch on its lists,
        dict(QWEN, name="draft_b128_8k", op="draft", batch=128, lens="uniform", lo=1024, hi=8192, budget=0),
        # and one iteration of it as a unified batch: every fifth request verifies, the others draft
        dict(QWEN, name="mixed_b128_8k", op="mixed", batch=128, lens="uniform", lo=1024, hi=8192, budget=0),
        # long reasoning: few requests, 24 to 32 K tokens, pages of 64, eight drafts, 2048 tokens kept
        dict(QWEN, name="verify_select_b16_32k", op="verify_select", batch=16, page=64, k=8, lens="uniform", lo=24576, hi=32768,
             budget=2048),
        dict(QWEN, name="draft_b16_32k", op="draft", batch=16, page=64, k=8, lens="uniform", lo=24576, hi=32768, budget=2048),
        # a larger model with an fp8 cache: 64 requests of very unequal length
        dict(QWEN, name="verify_select_fp8_b64", op="verify_select", batch=64, hq=64, kv="fp8_e4m3", lens="lognormal", lo=512, hi=32768,
             budget=512),
        dict(QWEN, name="draft_fp8_b64", op="draft", batch=64, hq=64, kv="fp8_e4m3", lens="lognormal", lo=512, hi=32768, budget=512),
        # the static drafts the method is compared with: verification without the statistic, sinks + window lists, a draft step
        dict(QWEN, name="window_round_b32", op="window_round", batch=32, lens="uniform", lo=700, hi=4500, budget=256),
        # requests that speculate different numbers of tokens, contexts of any length, lists wanted but no scores
        dict(QWEN, name="hetero_b24_ragged", op="hetero", batch=24, hq=16, hkv=4, lens="log", lo=5, hi=3000, budget=64),
    ]


def draw(rng):
    """One more case: any operation, 1 to 128 requests, contexts of tens of tokens to 32 K, 1 to 64 query rows per KV head."""
    op = rng.choice(["round", "verify_select", "draft", "mixed", "verify_select", "draft", "window_round", "hetero", "three_calls"])
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    c = dict(op=op, dim=128, page=rng.choice([16, 16, 32, 64]), q="bf16", kv=rng.choice(["bf16", "bf16", "fp8_e4m3"]))
    c["hkv"] = rng.choice([1, 2, 4, 8, 8])
    group = rng.choice([1, 2, 4, 4, 8])
    c["hq"] = c["hkv"] * group
    c["k"] = min(rng.randint(0, 8), 64 // group - 1)
    c["batch"] = log(1, 128)
    c["hi"] = log(64, 32768)
    c["lo"] = max(c["k"] + 1, int(c["hi"] * rng.uniform(0.1, 1.0)))
    c["lens"] = rng.choice(["uniform", "log"])
    c["budget"] = rng.choice([0, 0, log(32, 2048)])
    if op == "three_calls" and rng.random() < 0.5:       # the kernels for any shape: small sizes only
        c.update(dim=64, q="f32", kv="f32", hkv=min(c["hkv"], 2), batch=min(c["batch"], 4), hi=min(c["hi"], 2048))
        c.update(hq=c["hkv"] * min(group, 4), k=min(c["k"], 4))
        c["lo"] = min(c["lo"], c["hi"])
    rows = (c["k"] + 1) * c["hq"] // c["hkv"]
    most = 3.2e9 / (c["hkv"] * (512 + 16 * rows))        # tokens of all contexts: a drawn case costs no more than the largest listed one
    c["batch"] = max(1, min(c["batch"], int(most / c["hi"])))
    return c


# ---------------------------------------------------------------- sizes ----
def _lengths(case):
    rng = random.Random(251201278 + case["batch"])
    lo, hi, least = case["lo"], case["hi"], case["k"] + 1
    one = {
        "uniform": lambda: rng.randint(lo, hi),
        "log": lambda: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))),
        "lognormal": lambda: min(hi, max(lo, int(round(math.exp(math.log(8192.0) + 0.6 * rng.gauss(0.0, 1.0)))))),
    }[case["lens"]]
    return [max(least, one()) for _ in range(case["batch"])]


def _budgets(case, lens):
    """A fixed number of tokens, or (0) 5 % of the context in whole blocks of 64."""
    return [min(n, case["budget"] or 64 * math.ceil(0.05 * n / 64)) for n in lens]


def _spec_lens(case):
    rng = random.Random(1278 + case["batch"])
    return [rng.randint(0, case["k"]) for _ in range(case["batch"])]


def _split(case):
    """The requests of a unified batch that verify, and those that draft: rounds of k drafts and one verification."""
    every = range(case["batch"])
    return [b for b in every if b % (case["k"] + 1) == 0], [b for b in every if b % (case["k"] + 1)]


def work(case):
    lens = _lengths(case)
    buds = _budgets(case, lens)
    size = {"f32": 4, "bf16": 2, "fp8_e4m3": 1}
    kv, qo = size[case["kv"]], size[case["q"]]
    hq, hkv, d, nq = case["hq"], case["hkv"], case["dim"], case["k"] + 1
    spec = [s + 1 for s in _spec_lens(case)] if case["op"] == "hetero" else [nq] * case["batch"]
    scores = 4 if case["op"] in ("verify_select", "round", "mixed", "three_calls") else 0
    total = {"bytes": 0, "flops": 0}

    def verify(b, select=True):
        total["bytes"] += lens[b] * hkv * (2 * d * kv + scores) + 2 * spec[b] * hq * d * qo + 4 * spec[b] * hq
        total["bytes"] += buds[b] * hkv * 4 if select else 0
        total["bytes"] += -(-lens[b] // case["page"]) * hkv * 8 if case["kv"] == "fp8_e4m3" else 0
        total["flops"] += 4 * lens[b] * spec[b] * hq * d

    def draft(b):
        total["bytes"] += buds[b] * hkv * (2 * d * kv + 4) + 2 * hq * d * qo + 4 * hq
        total["flops"] += 4 * buds[b] * hq * d

    every = range(case["batch"])
    ver, dra = _split(case) if case["op"] == "mixed" else ([] if case["op"] == "draft" else every, [] if case["op"] in ("verify_select", "hetero") else every)
    for b in ver:
        verify(b, select=case["op"] != "window_round")
    for b in dra:
        draft(b)
    return total


def tolerance(case):
    """Measured against `exact`, the worst output of a case and of eight drawn ones: relative 2.4e-3 and at most 0.021 for outputs in
    bf16 (the results and the probabilities that the matrix cores take are rounded to it; lse and scores are closer), 1.3e-6 and
    5.7e-6 in fp32; four times that.  No entry of an index list differed; a tie on the budget's edge may move some."""
    if case["q"] == "f32":
        return {"rel": 5e-6, "max": 2.5e-5, "differ": 0.002}
    return {"rel": 1e-2, "max": 0.08, "differ": 0.002}


# --------------------------------------------------------------- inputs ----
_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    lens, nq = _lengths(case), case["k"] + 1
    buds = _budgets(case, lens)
    B, hq, hkv, d, page = case["batch"], case["hq"], case["hkv"], case["dim"], case["page"]
    group, widest, most = hq // hkv, max(lens), max(buds)
    qt = _DTYPE[case["q"]]
    randn = lambda *shape: torch.randn(*shape, generator=gen, device=DEVICE)

    # the pool holds a quarter more pages than the batch needs, in no order
    per = [-(-n // page) for n in lens]
    pages = sum(per) + -(-sum(per) // 4)
    order = torch.randperm(pages, generator=gen, device=DEVICE).to(torch.int32)
    table = torch.zeros(B, max(per), dtype=torch.int32, device=DEVICE)
    at = 0
    for b in range(B):
        table[b, :per[b]] = order[at:at + per[b]]
        at += per[b]

    base = randn(B, hkv, d)
    lean = SHARED * base[:, None, :, None, :]
    q = (lean + math.sqrt(1 - SHARED ** 2) * randn(B, nq, hkv, group, d)).reshape(B, nq, hq, d).to(qt)
    q_draft = (lean[:, 0] + math.sqrt(1 - SHARED ** 2) * randn(B, hkv, group, d)).reshape(B, hq, d).to(qt)

    wide = torch.bfloat16 if case["kv"] == "bf16" else torch.float32
    k_pool = torch.randn(pages, hkv, page, d, generator=gen, device=DEVICE, dtype=wide)
    v_pool = torch.randn(pages, hkv, page, d, generator=gen, device=DEVICE, dtype=wide)
    lists = torch.full((B, hkv, most), -1, dtype=torch.int32, device=DEVICE)
    heads = torch.arange(hkv, device=DEVICE)[:, None]
    for b in range(B):
        place = torch.rand(hkv, lens[b], generator=gen, device=DEVICE)
        place[:, :SINKS] = 2.0
        pos = place.topk(buds[b], dim=1).indices.sort(dim=1).values            # [hkv, budget]
        lists[b, :, :buds[b]] = pos.to(torch.int32)
        gain = GAIN[0] + (GAIN[1] - GAIN[0]) * torch.rand(hkv, buds[b], 1, generator=gen, device=DEVICE)
        where = (table[b].long()[pos // page], heads.expand_as(pos), pos % page)
        k_pool[where] = (k_pool[where].float() + gain * base[b][:, None, :] / math.sqrt(d)).to(wide)

    k_scale = v_scale = None
    if case["kv"] == "fp8_e4m3":                         # one scale per page and KV head
        def quantise(pool):
            scale = pool.abs().amax(dim=(2, 3)) / 448.0
            return (pool / scale[:, :, None, None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8), scale
        k_pool, k_scale = quantise(k_pool)
        v_pool, v_scale = quantise(v_pool)

    as_int = lambda v: torch.tensor(v, dtype=torch.int32, device=DEVICE)
    s = dict(op=case["op"], k=case["k"], hkv=hkv, widest=widest, most=most, lens=lens, buds=buds)
    s["kv"] = pa.KvCache(k_pool=k_pool, v_pool=v_pool, block_table=table, seq_lens=as_int(lens), num_q_heads=hq, q_dtype=case["q"],
                         kv_dtype=case["kv"], sm_scale=1.0 / math.sqrt(d), max_seq_len=widest, k_scale=k_scale, v_scale=v_scale)
    s["q"], s["q_draft"], s["budgets"], s["lists"] = q, q_draft, as_int(buds), lists
    s["out"] = torch.zeros(B, nq, hq, d, dtype=qt, device=DEVICE)
    s["lse"] = torch.zeros(B, nq, hq, device=DEVICE)
    s["scores"] = torch.zeros(B, hkv, -(-widest // 64) * 64, device=DEVICE)
    s["indices"] = lists.clone()                         # of the last verification: what a draft step reads
    s["counts"] = as_int(buds)
    s["d_out"] = torch.zeros(B, hq, d, dtype=qt, device=DEVICE)
    s["d_lse"] = torch.zeros(B, hq, device=DEVICE)
    s["spec_lens"] = as_int(_spec_lens(case))
    s["verifying"], s["drafting"] = (as_int(ids) if ids else None for ids in _split(case))
    s["workspace"] = torch.empty(pa.pillar_workspace_bytes(s["kv"], case["k"], most), dtype=torch.uint8, device=DEVICE)
    return s


# ------------------------------------------------------------- one pass ----
def run(s):
    kv, op = s["kv"], s["op"]

    def draft():
        pa.pillar_sparse_decode(kv, s["q_draft"], s["indices"], s["counts"], s["most"], s["d_out"], s["d_lse"], s["workspace"])

    if op in ("verify_select", "round"):
        pa.pillar_verify_select(kv, s["q"], s["k"], s["out"], s["lse"], s["scores"], s["budgets"], s["most"], s["indices"], s["counts"],
                                s["workspace"])
        if op == "round":
            draft()
    elif op == "three_calls":
        pa.pillar_verify_attn(kv, s["q"], s["k"], s["out"], s["lse"], s["scores"], s["workspace"])
        pa.pillar_select_topk(s["scores"], kv.seq_lens, s["budgets"], s["widest"], s["most"], s["indices"], s["counts"], s["workspace"])
        draft()
    elif op == "draft":
        draft()
    elif op == "window_round":
        pa.pillar_verify_attn(kv, s["q"], s["k"], s["out"], s["lse"], None, s["workspace"])
        pa.pillar_window_indices(kv.seq_lens, s["budgets"], s["hkv"], SINKS, s["most"], s["indices"], s["counts"])
        draft()
    elif op == "hetero":
        pa.pillar_verify_hetero(kv, s["q"], s["k"], s["spec_lens"], s["out"], s["lse"], None, s["workspace"], budgets=s["budgets"],
                                max_budget=s["most"], indices=s["indices"], counts=s["counts"])
    elif op == "mixed":
        pa.pillar_mixed_step(kv, s["verifying"], s["drafting"], s["q"], s["k"], s["out"], s["lse"], s["scores"], s["budgets"], s["most"],
                             s["indices"], s["counts"], s["q_draft"], s["d_out"], s["d_lse"], s["workspace"])
    return {name: s[name] for name in _OUTPUTS[op]}


_VERIFIED = ("out", "lse", "scores", "indices", "counts")
_DRAFTED = ("d_out", "d_lse")
_OUTPUTS = {
    "verify_select": _VERIFIED,
    "round": _VERIFIED + _DRAFTED,
    "three_calls": _VERIFIED + _DRAFTED,
    "mixed": _VERIFIED + _DRAFTED,
    "draft": _DRAFTED,
    "window_round": ("out", "lse", "indices", "counts") + _DRAFTED,
    "hetero": ("out", "lse", "indices", "counts"),
}


# ----------------------------------------------------- the same in 64 bits ----
def exact(case, seed):
    s = prepare(case, seed)
    op, kv, nq, page = s["op"], s["kv"], case["k"] + 1, case["page"]
    hkv, d = case["hkv"], case["dim"]
    group = case["hq"] // hkv
    f64 = dict(dtype=torch.float64, device=DEVICE)
    r = {name: torch.zeros(s[name].shape, **f64) if s[name].is_floating_point() else s[name].clone() for name in _OUTPUTS[op]}

    def rows(pool, scale, b):
        ids = kv.block_table[b, :-(-s["lens"][b] // page)].long()
        x = (pool.view(torch.float8_e4m3fn) if scale is not None else pool)[ids].double()
        if scale is not None:
            x = x * scale[ids].double()[:, :, None, None]
        return x.transpose(0, 1).reshape(hkv, -1, d)[:, :s["lens"][b]]

    def verify(b, n_q):
        n = s["lens"][b]
        k, v = rows(kv.k_pool, kv.k_scale, b), rows(kv.v_pool, kv.v_scale, b)
        q = s["q"][b, :n_q].double().reshape(n_q, hkv, group, d).permute(1, 0, 2, 3).reshape(hkv, n_q * group, d)
        logits = torch.matmul(q, k.transpose(1, 2).contiguous()) * kv.sm_scale
        last = n - n_q + torch.arange(n_q, device=DEVICE).repeat_interleave(group)
        logits.masked_fill_(torch.arange(n, device=DEVICE)[None, :] > last[:, None], -math.inf)
        lse = torch.logsumexp(logits, dim=2)
        p = torch.exp(logits - lse[:, :, None])
        spread = lambda x: x.reshape(hkv, n_q, group, -1).permute(1, 0, 2, 3).reshape(n_q, hkv * group, -1)
        r["out"][b, :n_q] = spread(torch.matmul(p, v))
        r["lse"][b, :n_q] = spread(lse[:, :, None])[:, :, 0]
        mean = p.mean(dim=1)
        if "scores" in r:
            r["scores"][b, :, :n] = mean
        if op != "window_round":
            best = torch.sort(mean, dim=1, descending=True, stable=True).indices[:, :s["buds"][b]].sort(dim=1).values
            r["indices"][b].fill_(-1)
            r["indices"][b, :, :s["buds"][b]] = best.to(torch.int32)

    def draft(b, lists):
        k, v = rows(kv.k_pool, kv.k_scale, b), rows(kv.v_pool, kv.v_scale, b)
        pos = lists[b, :, :s["buds"][b]].long()[:, :, None].expand(-1, -1, d)
        q = s["q_draft"][b].double().reshape(hkv, group, d)
        logits = torch.matmul(q, k.gather(1, pos).transpose(1, 2).contiguous()) * kv.sm_scale
        r["d_lse"][b] = torch.logsumexp(logits, dim=2).reshape(-1)
        r["d_out"][b] = torch.matmul(torch.softmax(logits, dim=2), v.gather(1, pos)).reshape(-1, d)

    every = range(case["batch"])
    if op == "window_round":                             # sinks, then the most recent tokens
        for b in every:
            budget, first = s["buds"][b], min(SINKS, s["buds"][b])
            entry = torch.arange(budget, device=DEVICE)
            r["indices"][b].fill_(-1)
            r["indices"][b, :, :budget] = torch.where(entry < first, entry, s["lens"][b] - budget + entry).to(torch.int32)
    ver, dra = _split(case) if op == "mixed" else (every, every)
    spec = _spec_lens(case)
    if "out" in r:
        for b in ver:
            verify(b, spec[b] + 1 if op == "hetero" else nq)
    if "d_out" in r:
        for b in dra:
            draft(b, s["lists"] if op in ("draft", "mixed") else r["indices"])
    return r
