"""The work this framework is used for, as cases that can be timed and checked.

A serving program fills a paged cache once per prompt and then, for every
token, calls one of the decode paths: one launch for a GQA level, estimate +
scan + combine for the others, the front + gated scan over a two-plane INT8
cache (with the step's token appended), both levels of a shared-prefix cascade,
or a verification of draft columns.  The listed cases are those calls at the
sizes of the benchmark's workloads and of the published evaluation (ragged
batches of 8-16K keys, head dims 64 and 128, GQA groups of 1 to 16);
``draw`` spreads over the same ranges.

Inputs are the benchmark's: N(0, 1) queries, keys and values rounded to BF16,
a fixed share of "spike" keys moved along their group's query direction, a few
sink keys, physical pages in random order.  Everything is made on the GPU from
the seed.  ``exact`` evaluates the same rule in 64 bits with plain torch: the
sampled reference, the depth rule, the two-plane codes and their gates.
"""

import math

import torch

import paper_2609_33410_amd as F

LOG2E = 1.4426950408889634
DEV = "cuda:0"
INF = math.inf
V8_EXP = -6          # E4M3 scale 2^-6: covers |v| <= 7
KAPPA = -4.0         # refine thresholds, the binding's defaults


# --------------------------------------------------------------- the cases --

def _base(name, kind, **kw):
    c = {"name": name, "kind": kind, "batch": 1, "heads": 32, "kv_heads": 8, "dim": 128,
         "len_lo": 1024, "len_hi": 1024, "page": 16, "splits": 1, "T": 0.0, "spike_share": 0.01,
         "sinks": 4, "model": "none", "out": "f32", "values8": False, "prefix": 0, "drafts": 0}
    c.update(kw)
    return c


def listed():
    return [
        # smallest call: one short MHA request on a contiguous cache (a unit
        # of a toy or draft model): latency and launches
        _base("tiny_mha_contiguous_512", "levels", heads=4, kv_heads=4, dim=64, len_lo=512,
              len_hi=512, page=0, spike_share=0.016, sinks=0),
        # one interactive user's short, odd-length context, GQA, BF16 out
        _base("gqa_one_user_1003_T16", "fused", len_lo=1003, len_hi=1003, splits=8, T=16.0,
              out="bf16"),
        # ordinary serving batch, dense decode
        _base("gqa_16x8192_dense", "fused", batch=16, len_lo=8192, len_hi=8192, splits=4,
              out="bf16"),
        # long contexts at a finite depth
        _base("gqa_8x32768_T16", "fused", batch=8, len_lo=32768, len_hi=32768, splits=16, T=16.0),
        # the largest call: MHA, ragged 64K-128K contexts, dense
        _base("mha_4x64k_128k_dense", "levels", batch=4, heads=32, kv_heads=32, len_lo=72212,
              len_hi=118806, splits=32, spike_share=0.005, sinks=0),
        # shared system prompt with short private suffixes, both levels in one scan
        _base("cascade_64x_16384_1024", "cascade", batch=64, heads=8, kv_heads=1, prefix=16384,
              len_lo=1024, len_hi=1024, splits=32, spike_share=0.0, sinks=0),
        # a token's step over the two-plane cache, BF16 values: ragged 8-16K,
        # GQA groups of 8
        _base("q8_step_32x8k_16k_g8_T16", "q8", batch=32, kv_heads=4, len_lo=8192, len_hi=16384,
              splits=8, T=16.0),
        # the same with 8-bit values, head dim 64, dense
        _base("q8v8_step_32x8k_16k_d64_dense", "q8", batch=32, heads=64, dim=64, len_lo=8192,
              len_hi=16384, splits=4, values8=True),
        # GQA groups of 16 over the two-plane cache
        _base("q8_step_32x8k_16k_g16_T16", "q8", batch=32, kv_heads=2, len_lo=8192, len_hi=16384,
              splits=16, T=16.0),
        # verification of four-token draft chains
        _base("drafts_4_32x4096_dense", "drafts", batch=32, len_lo=4096, len_hi=4096, splits=4,
              drafts=4),
        # a prompt's cache written in both 8-bit formats
        _base("prompt_q8v8_4x8192", "prompt_q8", batch=4, len_lo=8192, len_hi=8192),
        # a prompt's BF16 cache and the value means of the cut-key model
        _base("prompt_bf16_mean_4x8192", "prompt_bf16", batch=4, len_lo=8192, len_hi=8192,
              model="mean"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fused", "fused", "levels", "levels", "cascade", "q8", "q8", "q8", "drafts",
                       "prompt_q8", "prompt_bf16"])
    dim = rng.choice([64, 128])
    page = rng.choice([16, 16, 16, 32, 64])
    depth = rng.choice([0.0, 0.0, 24.0, 16.0, 14.0, 12.0])
    c = _base(None, kind, dim=dim, page=page, T=depth, sinks=rng.choice([0, 1, 4]),
              spike_share=rng.choice([0.002, 0.005, 0.01, 0.02]), out=rng.choice(["f32", "bf16"]))
    del c["name"]
    if kind == "cascade":
        group = rng.choice([4, 8])
        c.update(kv_heads=rng.choice([1, 2]), batch=rng.randint(9, 64) if group == 4 else
                 rng.randint(5, 64), prefix=16 * _log_int(rng, 32, 1024), spike_share=0.0, sinks=0,
                 page=16, len_lo=rng.randint(1, 512))
        c["heads"] = group * c["kv_heads"]
        c["len_hi"] = c["len_lo"] + rng.randint(0, 512)
        tiles = (c["prefix"] + 63) // 64
        riding = (64 // group + 1) * ((c["len_hi"] + 63) // 64)
        c["splits"] = max(1, min(32, (tiles + 7) // 8), (riding + tiles + 47) // 48)
        return c
    if kind == "fused":
        group = rng.choice([2, 4, 8])
    elif kind == "levels":
        group = rng.choice([1, 1, 1, 4, 8, 16])
    elif kind == "q8":
        group = rng.choice([1, 4, 8, 16])
        c["values8"] = rng.random() < 0.5
    else:
        group = rng.choice([4, 8])
    if kind == "levels" and c["T"]:
        c["model"] = rng.choice(["none", "mean", "block"])
    if kind == "prompt_bf16":
        c["model"] = rng.choice(["mean", "block"])
    c["kv_heads"] = rng.choice([1, 2, 4, 8]) if group > 1 else rng.choice([4, 8, 32])
    c["heads"] = group * c["kv_heads"]
    # at most 1.5 GB of BF16 keys and values (a prompt: a quarter of it), at
    # least one short request
    most = 1.5e9 / (c["kv_heads"] * dim * 4)
    if kind.startswith("prompt"):
        most /= 4
    total = _log_int(rng, 200, int(most))
    c["batch"] = min(_log_int(rng, 1, 64), max(1, total // 64))
    hi = max(17, min(total // c["batch"], 131072))
    c["len_hi"] = hi
    c["len_lo"] = rng.randint(max(1, hi // 2), hi)
    if kind == "drafts":
        c["drafts"] = rng.choice([2, 4])
    tiles = (hi + 63) // 64
    c["splits"] = max(1, min(64, tiles, -(-1024 // (c["batch"] * c["kv_heads"]))))
    return c


def _lens(c):
    """Ragged lengths between len_lo and len_hi, in an order that mixes short and long."""
    b, lo, hi = c["batch"], c["len_lo"], c["len_hi"]
    even = [hi - (hi - lo) * i // max(1, b - 1) for i in range(b)]
    return [even[(i * 5 + 2) % b] if b % 5 else even[(i * 7 + 2) % b if b % 7 else i]
            for i in range(b)]


def _depth(c):
    return c["T"] if c["T"] else INF


def work(c):
    lens, hkv, h, d, b = _lens(c), c["kv_heads"], c["heads"], c["dim"], c["batch"]
    keys = sum(lens)
    if c["kind"] == "prompt_q8":      # BF16 rows in; two planes each and the scales out
        n = keys * hkv
        return {"bytes": n * (8 * d + 2), "flops": n * d * math.log2(d)}
    if c["kind"] == "prompt_bf16":    # K and V rows copied; V summed
        n = keys * hkv
        return {"bytes": n * 8 * d, "flops": n * d}
    cols = b * max(1, c["drafts"])
    small = 2 * cols * h * d + (2 if c["out"] == "bf16" and c["kind"] == "fused" else 4) * \
        cols * h * d + 8 * cols * h
    if c["kind"] == "cascade":
        rows = (c["prefix"] + keys) * hkv
        flops = 4.0 * d * h * (b * c["prefix"] + keys)
    else:
        rows = keys * hkv
        flops = 4.0 * d * h * keys * max(1, c["drafts"])
    # every key row is read; value rows (and second planes) of a finite depth
    # or of unrefined keys depend on the data and are not counted
    key_bytes = d + 2 if c["kind"] == "q8" else 2 * d
    val_bytes = (d if c["values8"] else 2 * d) if not c["T"] else 0
    return {"bytes": rows * (key_bytes + val_bytes) + small, "flops": flops}


def tolerance(c):
    """About four times what the path shows against ``exact``."""
    if c["kind"] == "prompt_q8":
        return "exact"                # integer codes
    if c["kind"] == "prompt_bf16":
        return {"rel": 1e-6}          # copies, and FP32 sums: 6e-8 seen
    if c["kind"] == "fused" and c["out"] == "bf16":
        return {"rel": 8e-3}          # one rounding to BF16: 1.7e-3 seen
    if not c["T"]:
        return {"rel": 2e-5}          # 5e-6 seen
    # a key whose weight is 2^-T of the reference may fall on either side of
    # the depth's threshold: 9e-5 seen
    return {"rel": 4e-4}


# --------------------------------------------------------------- the inputs --

def _rng(seed):
    return torch.Generator(device=DEV).manual_seed(1 + seed)


def _inputs(c, seed):
    """The pool (BF16 pages, spikes and sinks in place), tables and queries."""
    g = _rng(seed)
    b, h, hkv, d, page = c["batch"], c["heads"], c["kv_heads"], c["dim"], c["page"]
    lens = _lens(c)
    m = c["drafts"]
    q = torch.randn(b, h, d, generator=g, device=DEV).to(torch.bfloat16)
    u = q.float().view(b, hkv, h // hkv, d).sum(2)
    u = u / u.norm(dim=-1, keepdim=True)
    s = {"q": q, "lens": lens}
    n_max = max(lens) + m
    if page == 0:
        k = torch.randn(b, hkv, n_max, d, generator=g, device=DEV, dtype=torch.bfloat16)
        v = torch.randn(b, hkv, n_max, d, generator=g, device=DEV, dtype=torch.bfloat16)
        bt = None
    else:
        pages = [(n + m + page - 1) // page for n in lens]
        pre = (c["prefix"] + page - 1) // page
        spare = b * m
        total = pre + sum(pages)
        k = torch.randn(total + spare, hkv, page, d, generator=g, device=DEV, dtype=torch.bfloat16)
        v = torch.randn(total + spare, hkv, page, d, generator=g, device=DEV, dtype=torch.bfloat16)
        perm = torch.randperm(total, generator=g, device=DEV).to(torch.int32)
        bt = torch.zeros(b, max(pages), dtype=torch.int32, device=DEV)
        first = pre
        for r, n in enumerate(pages):
            bt[r, :n] = perm[first:first + n]
            first += n
        s["prefix_bt"] = perm[:pre].view(1, -1).contiguous()
        s["spare"] = (total + torch.arange(spare, dtype=torch.int32, device=DEV)).view(spare, 1)
    for r, n in enumerate(lens):
        spikes = int(c["spike_share"] * n)
        for alpha, j in ((3.0 if n > 600 else 4.0,
                          torch.randint(0, n, (hkv, spikes), generator=g, device=DEV)),
                         (6.0, torch.arange(min(n, c["sinks"]), device=DEV).expand(hkv, -1))):
            if j.shape[1] == 0:
                continue
            heads = torch.arange(hkv, device=DEV)[:, None].expand_as(j)
            at = (r, heads, j) if page == 0 else (bt[r][j // page].long(), heads, j % page)
            k[at] = (k[at].float() + alpha * math.sqrt(d) * u[r][:, None, :]).to(torch.bfloat16)
    s.update(k=k, v=v, bt=bt, seq_lens=torch.tensor(lens, dtype=torch.int32, device=DEV),
             scale=1.0 / math.sqrt(d))
    if m:  # a column's query: its request's query and noise
        noise = torch.randn(b, m, h, d, generator=g, device=DEV) / 3.0
        s["q"] = (q.float()[:, None] + noise).to(torch.bfloat16).view(b * m, h, d)
    if c["kind"] == "q8":
        s["app_k"] = torch.randn(b, hkv, d, generator=g, device=DEV).to(torch.bfloat16)
        s["app_v"] = torch.randn(b, hkv, d, generator=g, device=DEV).to(torch.bfloat16)
    return s


def _view(s, c, **kw):
    return F.kv_view(s["k"], s["v"], s["seq_lens"], num_kv_heads=c["kv_heads"],
                     max_seq_len=max(s["lens"]), block_table=s["bt"], **kw)


def _tokens(c, lens):
    """Token lists of whole prompts: sequence and position of every token."""
    seq = torch.repeat_interleave(torch.arange(len(lens), device=DEV),
                                  torch.tensor(lens, device=DEV)).to(torch.int32)
    pos = torch.cat([torch.arange(n, device=DEV) for n in lens]).to(torch.int32)
    return seq, pos


def _prompt_inputs(c, seed):
    g = _rng(seed)
    b, hkv, d, page = c["batch"], c["kv_heads"], c["dim"], c["page"]
    lens = _lens(c)
    n = sum(lens)
    k = torch.randn(n, hkv, d, generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn(n, hkv, d, generator=g, device=DEV).to(torch.bfloat16)
    pages = [(x + page - 1) // page for x in lens]
    perm = torch.randperm(sum(pages), generator=g, device=DEV).to(torch.int32)
    bt = torch.zeros(b, max(pages), dtype=torch.int32, device=DEV)
    first = 0
    for r, p in enumerate(pages):
        bt[r, :p] = perm[first:first + p]
        first += p
    seq, pos = _tokens(c, lens)
    return {"k_src": k, "v_src": v, "bt": bt, "seq": seq, "pos": pos, "lens": lens,
            "pool": (sum(pages), hkv, page, d),
            "seq_lens": torch.tensor(lens, dtype=torch.int32, device=DEV)}


def prepare(c, seed):
    kind, b, h, hkv, d = c["kind"], c["batch"], c["heads"], c["kv_heads"], c["dim"]
    if kind.startswith("prompt"):
        s = _prompt_inputs(c, seed)
        k = torch.zeros(s["pool"], dtype=torch.bfloat16, device=DEV)
        kw = dict(num_kv_heads=hkv, max_seq_len=max(s["lens"]), block_table=s["bt"])
        if kind == "prompt_q8":
            s["keys"] = F.q8_empty_keys(k)
            s["vals"] = F.v8_empty_values(k, V8_EXP)
            for t in (s["keys"].plane_a, s["keys"].plane_b, s["keys"].scale, s["vals"].plane_p,
                      s["vals"].plane_r):
                t.zero_()
            s["kv"] = F.kv_view(s["keys"].plane_a, None, s["seq_lens"], k_is_layout_only=True,
                                **kw)
        else:
            s["k"], s["v"] = k, torch.zeros_like(k)
            s["kv"] = F.kv_view(s["k"], s["v"], s["seq_lens"], **kw)
            s["mean"] = torch.empty(b, hkv, d, device=DEV) if c["model"] == "mean" else \
                torch.empty(b, hkv, F.block_count(max(s["lens"])), d, device=DEV)
        s["case"] = dict(c)
        return s
    s = _inputs(c, seed)
    s["case"] = dict(c)
    rows = int(s["q"].shape[0])
    s["z"] = torch.empty(rows, h, device=DEV)
    s["qv"] = F.q_view(s["q"])
    if kind == "fused":
        s["kv"] = _view(s, c)
        s["part_A"] = torch.empty(c["splits"], b, h, d, device=DEV)
        s["part_L"] = torch.empty(c["splits"], b, h, device=DEV)
        s["arrivals"] = torch.zeros(b, hkv, dtype=torch.int32, device=DEV)
        s["o"] = torch.empty(b, h, d, device=DEV, dtype=torch.bfloat16 if c["out"] == "bf16"
                             else torch.float32)
        s["lse"] = torch.empty(b, h, device=DEV)
    elif kind == "levels":
        s["kv"] = _view(s, c)
        s["mean"] = s["bm"] = None
        if c["model"] == "mean":
            s["mean"] = F.fold_value_mean(s["kv"], torch.empty(b, hkv, d, device=DEV))
        elif c["model"] == "block":
            s["bm"] = [F.fold_value_block_mean(s["kv"], torch.empty(
                b, hkv, F.block_count(max(s["lens"])), d, device=DEV))]
    elif kind == "cascade":
        pre, page = c["prefix"], c["page"]
        s["suffix"] = _view(s, c)
        s["prefix"] = F.kv_view(
            s["k"], s["v"], torch.tensor([pre], dtype=torch.int32, device=DEV), num_kv_heads=hkv,
            max_seq_len=pre, block_table=s["prefix_bt"],
            row_indptr=torch.tensor([0, b], dtype=torch.int32, device=DEV),
            row_req=torch.arange(b, dtype=torch.int32, device=DEV), max_reqs_per_seq=b)
        flat = torch.cat([s["prefix_bt"].expand(b, -1), s["bt"]], dim=1).contiguous()
        s["flat"] = F.kv_view(s["k"], None, s["seq_lens"] + pre, num_kv_heads=hkv,
                              max_seq_len=pre + max(s["lens"]), block_table=flat)
        s["part_A"] = torch.empty(c["splits"], b, h, d, device=DEV)
        s["part_L"] = torch.empty(c["splits"], b, h, device=DEV)
        s["o"] = torch.empty(b, h, d, device=DEV)
        s["lse"] = torch.empty(b, h, device=DEV)
    elif kind == "q8":
        _encode(c, s)
        s["part_A"] = torch.empty(c["splits"], b, h, d, device=DEV)
        s["part_L"] = torch.empty(c["splits"], b, h, device=DEV)
        s["o"] = torch.empty(b, h, d, device=DEV)
        s["lse"] = torch.empty(b, h, device=DEV)
    elif kind == "drafts":
        m = c["drafts"]
        parent = ([-1] + list(range(m - 1))) * b
        s["views"] = F.fold_draft_views(s["k"], s["v"], s["bt"], [n + m for n in s["lens"]],
                                        list(range(0, b * m + 1, m)), parent, s["spare"],
                                        num_kv_heads=hkv)
    return s


def _encode(c, s):
    """A prompt's two-plane cache (and 8-bit values) from the BF16 pool."""
    n_pool, hkv, page, d = s["k"].shape
    pool = F.kv_view(s["k"], None, torch.full((n_pool,), page, dtype=torch.int32, device=DEV),
                     num_kv_heads=hkv, max_seq_len=page)
    seq = torch.arange(n_pool, dtype=torch.int32, device=DEV).repeat_interleave(page)
    pos = torch.arange(page, dtype=torch.int32, device=DEV).repeat(n_pool)

    def rows(t):
        return t.permute(0, 2, 1, 3).reshape(n_pool * page, hkv, d).contiguous()

    s["keys"] = F.q8_empty_keys(s["k"])
    F.fold_q8_write_keys(pool, rows(s["k"]), seq, pos, s["keys"])
    s["vals"] = None
    if c["values8"]:
        s["vals"] = F.v8_empty_values(s["v"], V8_EXP)
        F.fold_v8_write_values(pool, rows(s["v"]), seq, pos, s["vals"])
        s["v"] = None
    del s["k"]
    s["kv"] = F.kv_view(s["keys"].plane_a, s["v"], s["seq_lens"], num_kv_heads=hkv,
                        max_seq_len=max(s["lens"]), block_table=s["bt"], k_is_layout_only=True)
    s["code"] = F.q8_empty_query(s["q"])
    s["seq"] = torch.arange(c["batch"], dtype=torch.int32, device=DEV)
    s["pos"] = s["seq_lens"] - 1


# ------------------------------------------------------------------ one pass --

def run(s):
    c = s["case"]
    kind, T = c["kind"], _depth(c)
    if kind == "fused":
        F.fold_decode_fused(s["kv"], s["qv"], s["scale"], T, c["splits"], s["part_A"], s["part_L"],
                            s["arrivals"], s["z"], s["o"], lse_out=s["lse"])
        return {"o": s["o"], "lse": s["lse"], "z": s["z"]}
    if kind == "levels":
        F.fold_ref_estimate(s["kv"], s["qv"], s["scale"], s["z"])
        o, _, _, lse, _ = F.fold_decode([s["kv"]], s["q"], s["z"], T, [c["splits"]], s["scale"],
                                        lse=True, value_mean=s["mean"], block_means=s["bm"])
        return {"o": o, "lse": lse, "z": s["z"]}
    if kind == "cascade":
        F.fold_ref_estimate(s["flat"], s["qv"], s["scale"], s["z"])
        F.fold_decode_cascade(s["prefix"], s["suffix"], s["qv"], s["scale"], s["z"], T,
                              c["splits"], 0, s["part_A"], s["part_L"])
        F.fold_combine(s["part_A"], s["part_L"], s["o"], z=s["z"], lse_out=s["lse"])
        return {"o": s["o"], "lse": s["lse"], "z": s["z"]}
    if kind == "q8":
        F.fold_q8_write_keys(s["kv"], s["app_k"], s["seq"], s["pos"], s["keys"])
        if s["vals"] is None:
            F.fold_append_kv(s["kv"], None, s["app_v"], s["seq"], s["pos"], None, s["v"])
        else:
            F.fold_v8_write_values(s["kv"], s["app_v"], s["seq"], s["pos"], s["vals"])
        F.fold_q8_front(s["kv"], s["keys"], s["q"], s["scale"], s["code"], s["z"],
                        req_lens=s["seq_lens"], kappa=KAPPA, kappa_v=KAPPA)
        F.fold_q8_decode_split(s["kv"], s["keys"], s["code"], s["z"], T, c["splits"], 0,
                               s["part_A"], s["part_L"], values=s["vals"])
        F.fold_combine(s["part_A"], s["part_L"], s["o"], z=s["z"], lse_out=s["lse"])
        return {"o": s["o"], "lse": s["lse"], "z": s["z"]}
    if kind == "drafts":
        dv = s["views"]
        F.fold_ref_estimate(dv.estimate, s["qv"], s["scale"], s["z"])
        o, _, _, lse, _ = F.fold_decode([dv.committed, dv.ancestors], s["q"], s["z"], T,
                                        [c["splits"], 1], s["scale"], lse=True)
        return {"o": o, "lse": lse, "z": s["z"]}
    if kind == "prompt_q8":
        keys, vals = s["keys"], s["vals"]
        F.fold_q8_write_keys(s["kv"], s["k_src"], s["seq"], s["pos"], keys)
        F.fold_v8_write_values(s["kv"], s["v_src"], s["seq"], s["pos"], vals)
        return {"a": keys.plane_a, "b": keys.plane_b, "scale": keys.scale, "p": vals.plane_p,
                "r": vals.plane_r}
    F.fold_append_kv(s["kv"], s["k_src"], s["v_src"], s["seq"], s["pos"], s["k"], s["v"])
    if c["model"] == "mean":
        F.fold_value_mean(s["kv"], s["mean"])
    else:
        F.fold_value_block_mean(s["kv"], s["mean"])
    return {"k": s["k"], "v": s["v"], "mean": s["mean"]}


# --------------------------------------------------------- the same in 64 bits --

def _reference(samples_of, n):
    """log2 of the trimmed stratified estimate; samples_of(idx) -> [G, len(idx)]
    base-2 scores."""
    if n <= 192:
        return torch.logsumexp(samples_of(torch.arange(n, device=DEV)) / LOG2E, 1) * LOG2E
    r = n - 64
    bnd = 1 + (torch.arange(129, device=DEV) * r) // 128
    mid = (bnd[:-1] + bnd[1:] - 1) // 2
    near = torch.cat([torch.zeros(1, dtype=torch.long, device=DEV),
                      torch.arange(n - 63, n, device=DEV)])
    se, sm = samples_of(near), samples_of(mid)
    top = torch.maximum(se.amax(1), sm.amax(1))[:, None]
    kept = torch.sort(torch.exp2(sm - top), dim=1).values[:, 8:-8]
    return top[:, 0] + torch.log2(torch.exp2(se - top).sum(1) + (r / 112.0) * kept.sum(1))


def _gather(pool, table, kvh, n, page):
    """Logical rows 0..n-1 of one kv head, in 64 bits."""
    t = pool[table[:(n + page - 1) // page].long(), kvh]
    return t.reshape(-1, *t.shape[2:])[:n].double()


def _fold(s, v, z, T, mean=None, block=False):
    """(o, lse) of base-2 scores s [G, n] and values v [n, d] at depth T."""
    x = s - z[:, None]
    w = torch.exp2(x)
    total = w.sum(1, keepdim=True)
    live = x >= -T
    a = (w * live) @ v
    cut = w * ~live
    if mean is not None:
        a += cut.sum(1, keepdim=True) * mean
    if block:
        n, d = v.shape
        t = (n + 63) // 64
        pad = torch.zeros(t * 64 - n, d, dtype=v.dtype, device=DEV)
        size = torch.full((t, 1), 64.0, dtype=v.dtype, device=DEV)
        size[-1] = n - 64 * (t - 1)
        mu = torch.cat([v, pad]).view(t, 64, d).sum(1) / size
        cp = torch.cat([cut, pad.new_zeros(cut.shape[0], pad.shape[0])], 1)
        a += cp.view(-1, t, 64).sum(2) @ mu
    return a / total, z + torch.log2(total[:, 0])


def _hadamard(d):
    h = torch.ones(1, 1, dtype=torch.float64, device=DEV)
    while h.shape[0] < d:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)])
    return h


def _planes(x, s):
    """Planes a, b of rotated rows x under per-row scales s (0: a zero row)."""
    y = torch.where(s > 0, x / torch.where(s > 0, s, 1.0), 0.0)
    a = torch.round(y)
    return a, torch.clamp(torch.round(256.0 * (y - a)), -128, 127)


def _key_codes(k):
    """(a, b, e) of keys [..., d] in 64 bits; e a BF16 value rounded up."""
    x = k.double() @ _hadamard(k.shape[-1])
    m = x.abs().amax(-1, keepdim=True)
    e = m / 127.0
    low = (1 << 45) - 1
    e = ((e.view(torch.int64) + low) & ~low).view(torch.float64)
    e = torch.where(m >= 127.0 * 2.0 ** -126, e, 0.0)
    a, b = _planes(x, e)
    return a, b, e


def _value_codes(v):
    """(p, r) codes of 8-bit values as uint8."""
    y = v.float() * 2.0 ** -V8_EXP
    p = y.to(torch.float8_e4m3fn)
    r = (16.0 * (y - p.float())).to(torch.float8_e4m3fn)

    def code(t):
        u = t.view(torch.uint8)
        return torch.where(u == 0x80, torch.zeros_like(u), u)

    return code(p), code(r)


def _exact_prompt(c, seed):
    s = _prompt_inputs(c, seed)
    page = c["page"]
    phys = s["bt"][s["seq"].long(), s["pos"].long() // page].long()
    slot = s["pos"].long() % page

    def place(x, dtype):
        out = torch.zeros(s["pool"][:3] + tuple(x.shape[2:]), dtype=dtype, device=DEV)
        out[phys, :, slot] = x.to(dtype)
        return out

    if c["kind"] == "prompt_q8":
        a, b, e = _key_codes(s["k_src"])
        p, r = _value_codes(s["v_src"])
        bits = (e[..., 0].float().view(torch.int32) >> 16).to(torch.int16)
        return {"a": place(a, torch.int8), "b": place(b, torch.int8),
                "scale": place(bits, torch.int16), "p": place(p, torch.uint8),
                "r": place(r, torch.uint8)}
    means = []
    for v in torch.split(s["v_src"], s["lens"]):
        v = v.double().transpose(0, 1)
        if c["model"] == "mean":
            means.append(v.mean(1))
        else:
            t = F.block_count(max(s["lens"]))
            mu = v.new_zeros(v.shape[0], t, v.shape[2])
            for i, blk in enumerate(torch.split(v, 64, dim=1)):
                mu[:, i] = blk.mean(1)
            means.append(mu)
    return {"k": place(s["k_src"], torch.bfloat16), "v": place(s["v_src"], torch.bfloat16),
            "mean": torch.stack(means)}


def _exact_q8(c, s, r, kvh, q):
    n, page, d = s["lens"][r], c["page"], c["dim"]
    k = _gather(s["k"], s["bt"][r], kvh, n, page)
    v = _gather(s["v"], s["bt"][r], kvh, n, page)
    k[n - 1], v[n - 1] = s["app_k"][r, kvh].double(), s["app_v"][r, kvh].double()
    ka, kb, e = _key_codes(k)
    x = q.double() @ _hadamard(d)
    f = x.abs().amax(-1, keepdim=True) / 127.0
    qa, qb = _planes(x, f)
    qh = (qa + qb / 256.0).T
    eta = (LOG2E * s["scale"] * f / d).float().double()

    def score(a):
        return eta * (e * (a @ qh)).T

    z = _reference(lambda i: score(ka)[:, i], n)
    T = _depth(c)
    coarse = score(ka)
    xc = coarse - z[:, None]
    tau = KAPPA + math.ceil(math.log2(n)) if n > 1 else KAPPA
    live = (xc >= -T).any(0)
    refine = live & (xc >= -tau).any(0)
    sc = coarse + refine * score(kb) / 256.0
    if c["values8"]:
        p, rr = _value_codes(v.to(torch.bfloat16))
        p, rr = (t.view(torch.float8_e4m3fn).double() for t in (p, rr))
        v = 2.0 ** V8_EXP * (p + refine[:, None] * rr / 16.0)
    o, lse = _fold(sc, v, z, T)
    return o, lse, z


def exact(c, seed):
    if c["kind"].startswith("prompt"):
        return _exact_prompt(c, seed)
    s = _inputs(c, seed)
    b, hkv, page = c["batch"], c["kv_heads"], c["page"]
    rows, h, d = s["q"].shape
    group, m, T = h // hkv, max(1, c["drafts"]), _depth(c)
    o = torch.empty(rows, h, d, dtype=torch.float64, device=DEV)
    lse = torch.empty(rows, h, dtype=torch.float64, device=DEV)
    z = torch.empty_like(lse)
    pre = c["prefix"]
    for r in range(b):
        n = s["lens"][r]
        for kvh in range(hkv):
            hs = slice(kvh * group, (kvh + 1) * group)
            if c["kind"] == "q8":
                o[r, hs], lse[r, hs], z[r, hs] = _exact_q8(c, s, r, kvh, s["q"][r, hs])
                continue
            if page == 0:
                k, v = s["k"][r, kvh, :n].double(), s["v"][r, kvh, :n].double()
            else:
                nn = n + c["drafts"]
                k = _gather(s["k"], s["bt"][r], kvh, nn, page)
                v = _gather(s["v"], s["bt"][r], kvh, nn, page)
            if pre:
                k = torch.cat([_gather(s["k"], s["prefix_bt"][0], kvh, pre, page), k])
                v = torch.cat([_gather(s["v"], s["prefix_bt"][0], kvh, pre, page), v])
            for col in range(r * m, (r + 1) * m):
                sc = (s["q"][col, hs].double() @ k.T) * (LOG2E * s["scale"])
                zz = _reference(lambda i: sc[:, i], n + pre)
                if c["drafts"]:  # a chain: committed keys and the drafts up to this column
                    seen = n + col - r * m + 1
                    oo, ll = _fold(sc[:, :seen], v[:seen], zz, T)
                else:
                    oo, ll = _fold(sc, v, zz, T, v.mean(0) if c["model"] == "mean" else None,
                                   c["model"] == "block")
                o[col, hs], lse[col, hs], z[col, hs] = oo, ll, zz
    return {"o": o, "lse": lse, "z": z}
