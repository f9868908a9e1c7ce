"""The work a user of this library has it do, as cases that can be timed and checked.

Three kinds, each through the public entry points of paper_2509_04377_amd:

  decode  one page period of a decode loop at its budget: `page` consecutive decode steps (each appends one token
          per sequence and attends to everything cached), in which every sequence fills exactly one page, has its
          pages scored and drops the lowest one.  After a period the cache is as long as before, so a pass can be
          repeated for ever, as the loop of a long generation is.  Either one layer (`PagedCache`) or all layers of a
          model, in layer order (`LayeredCache`).
  attend  one call of the paged attention over a cache of ragged lengths (a budget that is never reached: full
          attention).
  prune   one layer's prompt pruned to the budget and split into pages.

A case is a dict of plain values: `kind`; `dtype`, `layout`, `seqs`, `kv_heads`, `q_heads`, `head_dim`, `page`
everywhere; `driver`, `layers`, `budget`, `stagger`, `mode` for decode; `min_len`, `max_len` for attend and prune;
`budget` for prune.
"""
import math
import random

import torch

from paper_2509_04377_amd import binding as pe
from paper_2509_04377_amd import synth
from paper_2509_04377_amd.engine import LayeredCache, PagedCache

DEVICE = "cuda"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _decode(name, dtype, seqs, kv_heads, q_heads, head_dim, page, budget, layers, driver="layers", layout="per_head",
            stagger=False, mode="plain"):
    return {"name": name, "kind": "decode", "dtype": dtype, "layout": layout, "seqs": seqs, "kv_heads": kv_heads,
            "q_heads": q_heads, "head_dim": head_dim, "page": page, "budget": budget, "layers": layers, "driver": driver,
            "stagger": stagger, "mode": mode}


def _prompt(name, kind, dtype, seqs, kv_heads, q_heads, head_dim, page, min_len, max_len, budget=0, layout="per_head"):
    return {"name": name, "kind": kind, "dtype": dtype, "layout": layout, "seqs": seqs, "kv_heads": kv_heads,
            "q_heads": q_heads, "head_dim": head_dim, "page": page, "min_len": min_len, "max_len": max_len,
            "budget": budget}


def listed():
    return [
        # the smallest call there is: one sequence, one layer, fp32 (launches and host work are all of it)
        _decode("decode_tiny_f32", "f32", 1, 4, 8, 64, 16, 256, 1, driver="cache"),
        # one layer of the 1B shape stepped on its own, as a model whose forward calls the cache layer by layer does
        _decode("decode_1b_layer", "bf16", 8, 8, 32, 64, 16, 2048, 1, driver="cache"),
        # all 16 layers of the 1B shape at the middle of its three budgets: a small batch, little traffic per launch
        _decode("decode_1b_model", "bf16", 8, 8, 32, 64, 16, 1024, 16),
        # the 3B shape (three query heads to a KV head); sequences reach their page boundaries at different steps, as
        # in a serving batch, so every step scores and evicts a few of them
        _decode("decode_3b_stagger", "bf16", 16, 8, 24, 128, 16, 1024, 28, stagger=True),
        # the 8B shape at full batch: the largest of the decode loops, bound by memory
        _decode("decode_8b_model", "bf16", 32, 8, 32, 128, 16, 2048, 32),
        # few sequences with a long cache each: rows are split over the chip
        _decode("decode_8b_long", "bf16", 4, 8, 32, 128, 16, 4096, 32),
        # the layout of a stock paged cache (one table row per sequence), page scores kept from step to step
        _decode("decode_8b_shared", "bf16", 32, 8, 32, 128, 16, 2048, 8, layout="shared", mode="cached"),
        # attention alone, eight query heads to a KV head, ragged lengths, larger pages
        _prompt("attend_ragged_g8", "attend", "bf16", 24, 8, 64, 128, 32, 37, 8191),
        # prompts of the 1B shape: one layer, launch-bound
        _prompt("prune_1b", "prune", "bf16", 8, 8, 32, 64, 16, 4096, 4096, 1024),
        # prompts of the 3B shape: ragged lengths
        _prompt("prune_3b_ragged", "prune", "bf16", 16, 8, 24, 128, 16, 2048, 16384, 1024),
        # prompts of the 8B shape at full batch: the largest prune
        _prompt("prune_8b", "prune", "bf16", 32, 8, 32, 128, 16, 16384, 16384, 2048),
        # a few very long prompts
        _prompt("prune_8b_long", "prune", "bf16", 4, 8, 32, 128, 16, 65536, 65536, 4096),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of the ranges above: any supported type, head size, page size, group size and layout, sizes spread over
    their logarithm, none larger than the listed ones."""
    kind = rng.choice(("decode", "decode", "attend", "prune"))
    dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
    elem = 2 if dtype == "bf16" else 4
    group = rng.choice((1, 2, 3, 4, 4, 5, 7, 8))
    kv_heads = rng.choice((1, 2, 3, 4, 8, 8))
    head_dim = rng.choice((64, 128, 128))
    page = rng.choice((16, 16, 32, 64, 128))
    layout = rng.choice(("per_head", "per_head", "shared"))
    seqs = _log_int(rng, 1, 48)
    row = seqs * kv_heads * head_dim * elem * 2   # bytes of K and V per token of every sequence
    common = {"kind": kind, "dtype": dtype, "layout": layout, "seqs": seqs, "kv_heads": kv_heads,
              "q_heads": group * kv_heads, "head_dim": head_dim, "page": page}
    if kind == "decode":
        budget = page * _log_int(rng, max(2, 256 // page), 8192 // page)
        while budget > 2 * page and row * budget * max(4, group) > (1 << 30):
            budget = budget // (2 * page) * page
        # a pass is `page` steps: no more launches, and no more traffic, than the largest listed case has
        layers = max(1, min(_log_int(rng, 1, 32), 512 // page, (1 << 32) // (row * budget), (1 << 36) // (row * budget * page)))
        modes = ("plain", "plain", "cached") + (("one_pass",) if layout == "per_head" else ())
        driver = "cache" if layers == 1 else "layers"
        return dict(common, budget=budget, layers=layers, driver=driver, stagger=rng.random() < 0.5, mode=rng.choice(modes))
    if kind == "attend":
        max_len = _log_int(rng, 64, 32768)
        while max_len > 64 and row * max_len > (1 << 31):
            max_len = max_len // 2 + 1
        return dict(common, min_len=rng.randint(1, max_len), max_len=max_len, budget=0)
    max_len = _log_int(rng, 512, 131072)
    while max_len > 512 and row * max_len > (1 << 31):
        max_len = max_len // 2 + 1
    budget = page * _log_int(rng, max(1, 256 // page), max(2, min(8192, max_len) // page))
    return dict(common, min_len=rng.randint(max(1, max_len // 8), max_len), max_len=max_len, budget=budget)


# ---- inputs ------------------------------------------------------------------------------------------------------
def _workload(case, budget):
    return synth.Workload("perf", 0, case["dtype"], max(1, case.get("layers", 1)), case["kv_heads"], case["q_heads"],
                          case["head_dim"], case["page"], case["seqs"], (1,), budget, case["page"], "lognormal", True)


def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _rows(shape, g, dtype):
    """Rows of D elements ~ N(0,1) with a lognormal scale per row (token, head)."""
    x = torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float32)
    x *= torch.exp(0.5 * torch.randn(shape[:-1] + (1,), generator=g, device=DEVICE, dtype=torch.float32))
    return x.to(dtype)


def _fill(pool, g):
    step = max(1, (1 << 26) // pool[0].numel())
    for i in range(0, pool.shape[0], step):
        part = pool[i:i + step]
        part.copy_(_rows(tuple(part.shape), g, pool.dtype))


def _lens(case, seed):
    if case["kind"] == "decode":
        if case["stagger"]:
            return [case["budget"] - (5 * s) % case["page"] for s in range(case["seqs"])]
        return [case["budget"]] * case["seqs"]
    r = random.Random(int(seed) * 7919 + 17)
    lens = [r.randint(case["min_len"], case["max_len"]) for _ in range(case["seqs"])]
    lens[0] = case["max_len"]
    return lens


def prepare(case, seed):
    return {"decode": _prepare_decode, "attend": _prepare_attend, "prune": _prepare_prune}[case["kind"]](case, seed)


def _prepare_decode(case, seed):
    g, dtype = _gen(seed), DTYPES[case["dtype"]]
    shared, layers, lens = case["layout"] == "shared", case["layers"], _lens(case, seed)
    wl = _workload(case, case["budget"])
    layout = synth.page_layout(wl, lens * layers, seed, shared=shared)
    dims = (case["kv_heads"], case["q_heads"], case["head_dim"], case["page"])
    if case["driver"] == "cache":
        cache = PagedCache.create(dtype, case["seqs"], *dims, layout, case["budget"], device=DEVICE, shared=shared)
        folded = cache
    else:
        cache = LayeredCache(dtype, layers, case["seqs"], *dims, layout, case["budget"], device=DEVICE, shared=shared)
        folded = cache.folded
    folded.cached_scores = case["mode"] == "cached"
    folded.fused_evict = case["mode"] == "one_pass"
    _fill(folded.k_pool, g)
    _fill(folded.v_pool, g)
    folded.seq_lens.copy_(torch.tensor(lens * layers, dtype=torch.int32, device=DEVICE))
    cache.set_host_lens(lens)
    lead = (case["page"],) + ((layers,) if case["driver"] == "layers" else ()) + (case["seqs"],)
    kv, qo = lead + (case["kv_heads"], case["head_dim"]), lead + (case["q_heads"], case["head_dim"])
    q = torch.randn(qo, generator=g, device=DEVICE, dtype=torch.float32).to(dtype)
    return {"kind": "decode", "cache": cache, "folded": folded, "new_k": _rows(kv, g, dtype), "new_v": _rows(kv, g, dtype),
            "q": q, "out": torch.empty_like(q)}


def _tables(case, lens, seed):
    """Block table of every row: ceil(len / page) pages each, physical ids a random permutation of the pool."""
    rows = 1 if case["layout"] == "shared" else case["kv_heads"]
    B = case["page"]
    need = torch.tensor([(n + B - 1) // B for n in lens], dtype=torch.int64)
    cols = torch.arange(int(need.max()))
    used = (cols[None, None, :] < need[:, None, None]).expand(-1, rows, -1)
    g = torch.Generator()
    g.manual_seed(int(seed) + 1)
    pages = int(used.sum())
    table = torch.full(used.shape, -1, dtype=torch.int32)
    table[used] = torch.randperm(pages, generator=g).to(torch.int32)
    return (table[:, 0] if case["layout"] == "shared" else table).contiguous().to(DEVICE), pages


def _pool_shape(case, pages):
    per_token = (case["kv_heads"], case["head_dim"]) if case["layout"] == "shared" else (case["head_dim"],)
    return (pages, case["page"]) + per_token


def _desc(case, table, pages):
    return pe.make_desc(DTYPES[case["dtype"]], case["seqs"], case["kv_heads"], case["q_heads"], case["head_dim"],
                        case["page"], table.shape[-1], pages,
                        pe.PE_LAYOUT_SHARED if case["layout"] == "shared" else pe.PE_LAYOUT_PER_HEAD)


def _prepare_attend(case, seed):
    g, dtype, lens = _gen(seed), DTYPES[case["dtype"]], _lens(case, seed)
    table, pages = _tables(case, lens, seed)
    k = torch.empty(_pool_shape(case, pages), dtype=dtype, device=DEVICE)
    v = torch.empty_like(k)
    _fill(k, g)
    _fill(v, g)
    desc = _desc(case, table, pages)
    q = torch.randn((case["seqs"], case["q_heads"], case["head_dim"]), generator=g, device=DEVICE).to(dtype)
    return {"kind": "attend", "desc": desc, "k_pool": k, "v_pool": v, "table": table, "q": q, "out": torch.empty_like(q),
            "seq_lens": torch.tensor(lens, dtype=torch.int32, device=DEVICE),
            "workspace": pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc, device=DEVICE)}


def _prepare_prune(case, seed):
    g, dtype, lens = _gen(seed), DTYPES[case["dtype"]], _lens(case, seed)
    table, pages = _tables(case, [min(n, case["budget"]) for n in lens], seed)
    total = sum(lens)
    shape = (total, case["kv_heads"], case["head_dim"])
    k = torch.empty(shape, dtype=dtype, device=DEVICE)
    v = torch.empty_like(k)
    _fill(k, g)
    _fill(v, g)
    cu = torch.tensor([sum(lens[:i]) for i in range(len(lens) + 1)], dtype=torch.int32)
    desc = _desc(case, table, pages)
    kept = (case["seqs"],) + (() if case["layout"] == "shared" else (case["kv_heads"],)) + (case["budget"],)
    return {"kind": "prune", "desc": desc, "k": k, "v": v, "cu": cu.to(DEVICE), "max_len": max(lens), "budget": case["budget"],
            "table": table, "k_pool": torch.zeros(_pool_shape(case, pages), dtype=dtype, device=DEVICE),
            "v_pool": torch.zeros(_pool_shape(case, pages), dtype=dtype, device=DEVICE),
            "seq_lens": torch.zeros(case["seqs"], dtype=torch.int32, device=DEVICE),
            "kept": torch.full(kept, -1, dtype=torch.int32, device=DEVICE),
            "workspace": pe.alloc_workspace(pe.PE_OP_PREFILL_PRUNE, desc, total, device=DEVICE)}


# ---- one pass ----------------------------------------------------------------------------------------------------
def run(state):
    s = state
    if s["kind"] == "decode":
        cache, f = s["cache"], s["folded"]
        for new_k, new_v, q, out in zip(s["new_k"], s["new_v"], s["q"], s["out"]):
            cache.decode_step(new_k, new_v, q, out)
        return {"out": s["out"], "block_table": f.block_table, "seq_lens": f.seq_lens, "k_pool": f.k_pool,
                "v_pool": f.v_pool}
    if s["kind"] == "attend":
        pe.pe_paged_decode(s["desc"], s["q"], s["k_pool"], s["v_pool"], s["table"], s["seq_lens"],
                           s["desc"].head_dim ** -0.5, s["out"], s["workspace"])
        return {"out": s["out"]}
    pe.pe_prefill_prune(s["desc"], s["k"], s["v"], s["cu"], s["k"].shape[0], s["max_len"], s["budget"], s["k_pool"],
                        s["v_pool"], s["table"], s["seq_lens"], s["kept"], s["workspace"])
    return {"k_pool": s["k_pool"], "v_pool": s["v_pool"], "seq_lens": s["seq_lens"], "kept": s["kept"]}


# ---- what a pass cannot do without ---------------------------------------------------------------------------------
def work(case):
    elem = 2 if case["dtype"] == "bf16" else 4
    S, Hk, Hq, D, B = case["seqs"], case["kv_heads"], case["q_heads"], case["head_dim"], case["page"]
    rows_per_seq = 1 if case["layout"] == "shared" else Hk
    kv = Hk * D * elem * 2   # K and V of one token
    if case["kind"] == "decode":
        L, C = case["layers"], case["budget"]
        nbytes = flops = 0
        for start in _lens(case, 0):
            n = start
            for _ in range(B):
                if n % B == 0 and n >= C:
                    scored = B if case["mode"] == "cached" else n   # pages read to decide which one goes
                    nbytes += scored * kv + 2 * rows_per_seq * (n // B) * 4
                    flops += 4 * scored * Hk * D
                    n -= B
                n += 1
                nbytes += n * kv + kv + 2 * Hq * D * elem + rows_per_seq * ((n + B - 1) // B) * 4
                flops += 4 * n * Hq * D
        return {"bytes": L * nbytes, "flops": L * flops}
    lens = _lens(case, 0)
    if case["kind"] == "attend":
        tokens = sum(lens)
        return {"bytes": tokens * kv + 2 * S * Hq * D * elem + rows_per_seq * tokens // B * 4,
                "flops": 4 * tokens * Hq * D}
    kept = sum(min(n, case["budget"]) for n in lens)
    # the whole prompt is read once, the kept tokens are written (a single reading of the prompt is the least)
    return {"bytes": sum(lens) * kv + kept * kv + rows_per_seq * kept * 4, "flops": 4 * sum(lens) * Hk * D}


def tolerance(case):
    if case["kind"] == "prune":
        return "exact"   # copies of the prompt's rows, and integers
    # attention: fp32 accumulation.  bf16 results carry their rounding (1.6e-3 in the 2-norm, measured); fp32 ones the
    # accumulated rounding of their sums (2.2e-7 over 256 tokens, more over some thousand).  Tables and lengths are the same, bit for bit.
    return {"rel": 6.5e-3, "max": 0.03} if case["dtype"] == "bf16" else {"rel": 2e-6, "max": 5e-5}


# ---- the same in 64 bits, in plain torch -------------------------------------------------------------------------------
def exact(case, seed):
    state = prepare(case, seed)
    return {"decode": _exact_decode, "attend": _exact_attend, "prune": _exact_prune}[case["kind"]](case, seed, state)


def _token_scores(k, v):
    """||V|| / ||K|| over the last axis in fp64, rounded once to fp32."""
    nk = k.double().square().sum(-1).sqrt()
    nv = v.double().square().sum(-1).sqrt()
    return torch.where(nv == 0, torch.zeros_like(nv), nv / nk)


def _attention(q, k, v, lens):
    """q [S, Hq, D], k and v [S, T, Hk, D], lens [S] -> [S, Hq, D] in fp64."""
    S, Hq, D = q.shape
    Hk = k.shape[2]
    kd = k.double().permute(0, 2, 1, 3).contiguous().view(S * Hk, -1, D)
    logits = torch.bmm(q.double().view(S * Hk, Hq // Hk, D), kd.transpose(1, 2).contiguous()) * D ** -0.5
    dead = torch.arange(k.shape[1], device=DEVICE)[None, :] >= lens[:, None]
    dead = dead[:, None, None, :].expand(S, Hk, 1, -1).reshape(S * Hk, 1, -1)
    p = torch.softmax(logits.masked_fill(dead, float("-inf")), dim=-1)
    vd = v.double().permute(0, 2, 1, 3).contiguous().view(S * Hk, -1, D)
    return torch.bmm(p, vd).view(S, Hq, D)


def _gather(pool, table, shared):
    """[S, T, Hk, D] view of the pages of `table` ([S, Hk, n], shared: [S, n]); unused entries read page 0."""
    pages = pool[table.clamp(min=0).long()]
    if shared:
        return pages.flatten(1, 2)
    return pages.flatten(2, 3).transpose(1, 2)


def _exact_attend(case, seed, s):
    shared, out = case["layout"] == "shared", []
    lens = s["seq_lens"].tolist()
    for i, n in enumerate(lens):
        nb = (n + case["page"] - 1) // case["page"]
        table = s["table"][i:i + 1, ..., :nb]
        out.append(_attention(s["q"][i:i + 1], _gather(s["k_pool"], table, shared), _gather(s["v_pool"], table, shared),
                              s["seq_lens"][i:i + 1]))
    return {"out": torch.cat(out)}


def _exact_prune(case, seed, s):
    shared, B = case["layout"] == "shared", case["page"]
    k_pool, v_pool, kept, seq_lens = (torch.zeros_like(s["k_pool"]), torch.zeros_like(s["v_pool"]),
                                      torch.full_like(s["kept"], -1), torch.zeros_like(s["seq_lens"]))
    cu = s["cu"].tolist()
    for i in range(case["seqs"]):
        k, v = s["k"][cu[i]:cu[i + 1]], s["v"][cu[i]:cu[i + 1]]
        n = min(k.shape[0], case["budget"])
        score = _token_scores(k, v).float()   # [L, Hk]
        if shared:
            score = score.double().mean(1, keepdim=True).float()
        order = torch.sort(score, dim=0, stable=True).indices   # ties: the lower index goes first
        stay = torch.sort(order[k.shape[0] - n:], dim=0).values.t().contiguous()   # [Hk or 1, n]
        seq_lens[i] = n
        at = torch.arange(n, device=DEVICE)
        if shared:
            kept[i, :n] = stay[0].int()
            page = s["table"][i].long()[at // B]
            k_pool[page, at % B], v_pool[page, at % B] = k[stay[0]], v[stay[0]]
        else:
            kept[i, :, :n] = stay.int()
            page = s["table"][i].long()[:, at // B]
            heads = torch.arange(k.shape[1], device=DEVICE)[:, None]
            k_pool[page, at[None] % B], v_pool[page, at[None] % B] = k[stay, heads], v[stay, heads]
    return {"k_pool": k_pool, "v_pool": v_pool, "seq_lens": seq_lens, "kept": kept}


def _exact_decode(case, seed, s):
    shared, B, S, L = case["layout"] == "shared", case["page"], case["seqs"], case["layers"]
    f = s["folded"]
    if f.k_pool.numel() * B > (1 << 36):
        return None
    layered = case["driver"] == "layers"
    k_pool, v_pool, spare = f.k_pool, f.v_pool, f.spare
    table = f.block_table.clone()          # [L * S, Hk, n] or [L * S, n]
    heads = table.shape[1:-1]
    freed, used = f.freed_phys.clone(), f.spare_used.clone().long()
    lens, out = _lens(case, seed), []
    Hk = case["kv_heads"]

    def page_scores(pages):
        sc = torch.cat([_token_scores(k_pool[p], v_pool[p]).mean(1).float() for p in pages.reshape(-1).split(1 << 14)])
        if shared:   # one decision per sequence: the mean over its heads
            sc = sc.double().mean(-1).float()
        return sc.view(pages.shape)

    for step in range(B):
        new_k, new_v, q = s["new_k"][step], s["new_v"][step], s["q"][step]
        if not layered:
            new_k, new_v, q = new_k[None], new_v[None], q[None]
        for i in range(S):
            n, rows = lens[i], torch.arange(L, device=DEVICE) * S + i
            if n > 0 and n % B == 0 and n >= case["budget"]:
                nb = n // B
                row = table[rows][..., :nb]
                sc = page_scores(row.long())
                first = (sc == sc.amin(-1, keepdim=True)).int().cumsum(-1)
                at = (first == 0).sum(-1, keepdim=True)   # entries before the first lowest one
                freed[rows] = row.gather(-1, at)[..., 0]
                cols = torch.arange(nb, device=DEVICE).expand(row.shape)
                src = (cols + (cols >= at)).clamp(max=nb - 1)
                row = row.gather(-1, src)
                row[..., nb - 1] = -1
                whole = table[rows]
                whole[..., :nb] = row
                table[rows] = whole
                n -= B
            jb, slot = n // B, n % B
            if slot == 0:
                fr, us = freed[rows], used[rows]
                page = torch.where(fr >= 0, fr, spare[rows].gather(-1, us[..., None])[..., 0])
                used[rows] = us + (fr < 0)
                freed[rows] = -1
                whole = table[rows]
                whole[..., jb] = page
                table[rows] = whole
            page = table[rows][..., jb].long()
            k_pool[page, slot], v_pool[page, slot] = new_k[:, i], new_v[:, i]
            lens[i] = n + 1
        nb = (max(lens) + B - 1) // B
        dev_lens = torch.tensor(lens, device=DEVICE)
        rows_out = []
        for l in range(L):
            t = table[l * S:(l + 1) * S, ..., :nb]
            rows_out.append(_attention(q[l], _gather(k_pool, t, shared), _gather(v_pool, t, shared), dev_lens))
        out.append(torch.stack(rows_out) if layered else rows_out[0])
    return {"out": torch.stack(out), "block_table": table, "seq_lens": torch.tensor(lens * L, dtype=torch.int32, device=DEVICE),
            "k_pool": None, "v_pool": None}
