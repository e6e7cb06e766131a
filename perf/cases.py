"""Performance cases of the fork-aware attention library: what a serving program has it do at a
fork, with the sizes it meets there.

A case is one of three kinds of work, all through the public binding:

* ``step``: one fused append + decode step (``Plan.step`` / ``Plan.step_paged``) of every attention
  layer of a model, each layer with K/V of its own, so that a layer's cache comes from HBM as it does
  in a whole model.  The suffix lengths are set back first, so that a pass can be repeated.
* ``decode``: a decode over K/V that is already in place (``Plan.decode``, ``Plan.decode_paged`` or
  ``decode_noalloc``), where the program's own projection kernels write the cache.
* ``prefill``: the branches' instruction (or, with one sequence, harvested text) over the shared
  prefix (``Plan.prefill`` / ``Plan.prefill_paged``).

Values follow the library's synthetic workloads: N(0, 1) queries, keys and values, keys scaled per
(KV head, channel) by a LogNormal(0, 0.5) factor, in bf16.  Lengths come from the case (``len_seed``),
values from the seed.
"""
import math
import random

import torch

from paper_2608_13667_amd import forkattn as fa

PAGE = 16
CHUNK_ROWS = 256  # query rows that exact() scores at once


def _case(name, kind, hq, hkv, d, prefix, suffix, *, branches=5, tasks=1, paged=False, noalloc=False, layers=1, tokens=0,
          main=(0, 0), value_scale=1.0, key_scale=True, len_seed=1):
    c = dict(kind=kind, hq=hq, hkv=hkv, d=d, branches=branches, tasks=tasks, paged=paged, noalloc=noalloc, layers=layers,
             tokens=tokens, prefix_lo=prefix[0], prefix_hi=prefix[1], suffix_lo=suffix[0], suffix_hi=suffix[1],
             main_lo=main[0], main_hi=main[1], value_scale=value_scale, key_scale=key_scale, len_seed=len_seed)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest fork: a small model (head dim 64) over a short context; launches and latency
        _case("tiny-step", "step", 8, 2, 64, (512, 512), (0, 64), layers=8, value_scale=0.125, key_scale=False),
        # an agent's early turns: 8k context, 32 query / 8 KV heads
        _case("mid-step", "step", 32, 8, 128, (8192, 8192), (256, 1024), layers=8),
        # the library's headline: 32k context, 40 query / 8 KV heads
        _case("long-step", "step", 40, 8, 128, (32768, 32768), (512, 2048), layers=4),
        # one task on the page pool at an odd context length
        _case("paged-step", "step", 40, 8, 128, (23017, 23017), (100, 900), paged=True, layers=4),
        # the longest context, 64 query heads
        _case("very-long-decode", "decode", 64, 8, 128, (131072, 131072), (1024, 4096)),
        # fork at turn onset: the main thread's suffix is the whole Thought; a harness that may not allocate
        _case("onset-noalloc", "decode", 40, 8, 128, (32768, 32768), (0, 512), main=(4096, 8192), noalloc=True),
        # a server's batch: 16 tasks of five sequences, contexts of 4k to 64k, on one page pool
        _case("tasks-decode", "decode", 32, 8, 128, (4096, 65536), (0, 2048), tasks=16, paged=True),
        # a branch instruction of a few words
        _case("prefill-4", "prefill", 40, 8, 128, (32768, 32768), (0, 0), tokens=4),
        # a one-line instruction, on the page pool, at an odd context length
        _case("prefill-16-paged", "prefill", 40, 8, 128, (23017, 23017), (0, 40), tokens=16, paged=True),
        # a full instruction paragraph at the headline's context
        _case("prefill-64", "prefill", 40, 8, 128, (32768, 32768), (0, 40), tokens=64),
        # the harvested thoughts appended to the main context
        _case("harvest-paged", "prefill", 40, 8, 128, (33827, 33827), (0, 0), branches=1, tokens=256, paged=True),
        # instructions in a model of head dim 64
        _case("prefill-32-d64", "prefill", 32, 8, 64, (8192, 8192), (0, 40), tokens=32),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "decode", "decode", "prefill", "prefill", "prefill"])
    d = rng.choice([64, 128, 128, 128])
    hkv = rng.choice([2, 4, 8, 8, 8])
    group = rng.choice([4, 5, 5, 7, 8])
    branches = rng.randint(2, min(8, 64 // group))
    paged = rng.random() < 0.5
    seed = rng.randrange(1 << 20)
    if kind == "prefill":
        if rng.random() < 0.25:
            branches = 1
        tokens = _log_uniform(rng, 1, min(256 if branches == 1 else 64, 512 // branches))
        # at most the listed cases' work: 2e11 flops
        most = 200_000_000_000 // (4 * d * hkv * group * branches * tokens)
        prefix = _log_uniform(rng, 512, min(32768, most))
        return _case(None, kind, hkv * group, hkv, d, (prefix, prefix), (0, rng.choice([0, 40, 300])), branches=branches,
                     tokens=tokens, paged=paged, len_seed=seed)
    suffix = (rng.randint(0, 256), rng.randint(256, 2048))
    if kind == "step":
        prefix = _log_uniform(rng, 512, 32768)
        return _case(None, kind, hkv * group, hkv, d, (prefix, prefix), suffix, branches=branches, paged=paged,
                     layers=4, len_seed=seed)
    tasks = rng.choice([1, 2, 5, 11]) if paged else 1
    prefix = _log_uniform(rng, 512, 131072 if tasks == 1 else 32768)
    return _case(None, kind, hkv * group, hkv, d, (prefix // 4 if tasks > 1 else prefix, prefix), suffix,
                 branches=branches, tasks=tasks, paged=paged, noalloc=not paged and prefix <= 32768 and rng.random() < 0.3,
                 main=(2048, 8192) if rng.random() < 0.25 else (0, 0), len_seed=seed)


def _lengths(c):
    """Prefix length of each task, suffix length of each sequence (before a step's or instruction's tokens)."""
    r = random.Random(c["len_seed"])
    prefix = [r.randint(c["prefix_lo"], c["prefix_hi"]) for _ in range(c["tasks"])]
    suffix = []
    for _ in range(c["tasks"]):
        own = [r.randint(c["suffix_lo"], c["suffix_hi"]) for _ in range(c["branches"])]
        if c["main_hi"]:
            own[0] = r.randint(c["main_lo"], c["main_hi"])
        suffix += own
    return prefix, suffix


def _new_tokens(c):
    return 1 if c["kind"] == "step" else c["tokens"]


def _pages(n):
    return (n + PAGE - 1) // PAGE


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    hq, hkv, d, n_seq = c["hq"], c["hkv"], c["d"], c["tasks"] * c["branches"]
    prefix, suffix = _lengths(c)
    new = _new_tokens(c)
    cap = max(1, max(suffix) + new)

    def values(*shape):
        x = torch.randn(*shape, generator=gen, device="cuda", dtype=torch.bfloat16)
        return x.mul_(c["value_scale"]) if c["value_scale"] != 1.0 else x

    def keys(scale, *shape):
        x = values(*shape)
        return x.mul_(scale) if c["key_scale"] else x

    q_shape = (c["branches"], c["tokens"], hq, d) if c["kind"] == "prefill" else (n_seq, hq, d)
    lens0 = torch.tensor([suffix] * c["layers"], dtype=torch.int32, device="cuda")
    state = {"case": c, "lens0": lens0, "lens": lens0.clone(), "layers": []}
    out = torch.empty(c["layers"], *q_shape, device="cuda")
    lse = torch.empty(c["layers"], *q_shape[:-1], device="cuda")
    state["out"], state["lse"] = out, lse

    if c["paged"]:
        n_pre, n_suf = [_pages(n) for n in prefix], [_pages(n + new) for n in suffix]
        n_pages, width = sum(n_pre) + sum(n_suf), max(n_pre) + max(n_suf)
        table = torch.full((n_seq, width), -1, dtype=torch.int32)
        ids = torch.randperm(n_pages, generator=torch.Generator().manual_seed(seed)).to(torch.int32)
        at = 0
        for t in range(c["tasks"]):
            own = ids[at:at + n_pre[t]]
            at += n_pre[t]
            for s in range(t * c["branches"], (t + 1) * c["branches"]):
                table[s, :n_pre[t]] = own
                table[s, n_pre[t]:n_pre[t] + n_suf[s]] = ids[at:at + n_suf[s]]
                at += n_suf[s]
        table = table.cuda()
        if c["kind"] == "prefill":
            state["plan"] = fa.Plan.prefill_paged_plan(hq, hkv, d, c["branches"], c["tokens"], prefix[0], width, n_pages, cap)
        else:
            starts = [t * c["branches"] for t in range(c["tasks"] + 1)]
            state["plan"] = fa.Plan.paged_plan(hq, hkv, d, starts, prefix, width, n_pages, cap)
    elif c["kind"] == "prefill":
        state["plan"] = fa.Plan.prefill_plan(hq, hkv, d, c["branches"], c["tokens"], prefix[0], cap, cap)
    elif not c["noalloc"]:
        state["plan"] = fa.Plan.contig(hq, hkv, d, n_seq, prefix[0], cap, cap)
    state["cap"], state["prefix"], state["suffix"] = cap, prefix, suffix

    for i in range(c["layers"]):
        scale = torch.empty(hkv, 1, d, device="cuda").log_normal_(0.0, 0.5, generator=gen).to(torch.bfloat16)
        s = {"q": values(*q_shape), "lens": state["lens"][i], "out": out[i], "lse": lse[i]}
        if c["paged"]:
            s["k_pool"], s["v_pool"], s["table"] = keys(scale, n_pages, hkv, PAGE, d), values(n_pages, hkv, PAGE, d), table
        else:
            s["prefix_k"], s["prefix_v"] = keys(scale, hkv, prefix[0], d), values(hkv, prefix[0], d)
            s["suffix_k"], s["suffix_v"] = keys(scale, n_seq, hkv, cap, d), values(n_seq, hkv, cap, d)
        if c["kind"] == "step":
            s["k_new"], s["v_new"] = keys(scale[:, 0], n_seq, hkv, d), values(n_seq, hkv, d)
        state["layers"].append(s)
    return state


def run(state):
    c, plan = state["case"], state.get("plan")
    result = {"out": state["out"], "lse": state["lse"]}
    if c["kind"] == "step":
        state["lens"].copy_(state["lens0"])
        for s in state["layers"]:
            if c["paged"]:
                plan.step_paged(s["q"], s["k_new"], s["v_new"], s["k_pool"], s["v_pool"], s["table"], s["lens"], s["out"],
                                s["lse"])
            else:
                plan.step(s["q"], s["k_new"], s["v_new"], s["prefix_k"], s["prefix_v"], s["suffix_k"], s["suffix_v"],
                          s["lens"], s["out"], s["lse"])
        result["lens"] = state["lens"]
        result["cache"] = [[s["k_pool"], s["v_pool"]] if c["paged"] else [s["suffix_k"], s["suffix_v"]]
                           for s in state["layers"]]
        return result
    for s in state["layers"]:
        if c["paged"]:
            call = plan.prefill_paged if c["kind"] == "prefill" else plan.decode_paged
            call(s["q"], s["k_pool"], s["v_pool"], s["table"], s["lens"], s["out"], s["lse"])
        elif c["noalloc"]:
            fa.decode_noalloc(c["hq"], c["hkv"], c["d"], state["prefix"][0], state["cap"], state["cap"], s["q"], s["prefix_k"],
                              s["prefix_v"], s["suffix_k"], s["suffix_v"], s["lens"], s["out"], s["lse"])
        else:
            call = plan.prefill if c["kind"] == "prefill" else plan.decode
            call(s["q"], s["prefix_k"], s["prefix_v"], s["suffix_k"], s["suffix_v"], s["lens"], s["out"], s["lse"])
    return result


def work(case):
    """One pass: every layer's prefix and suffix K/V once, q in and the fp32 output and lse out (a
    step's new token in and into the cache); 4 d flops per query row and key it sees."""
    c = case
    prefix, suffix = _lengths(c)
    token = 2 * 2 * c["hkv"] * c["d"]  # K and V of one position
    group_rows = c["hq"] * max(1, c["tokens"])
    rows = c["tasks"] * c["branches"] * group_rows
    read = (sum(prefix) + sum(suffix)) * token
    io = rows * (c["d"] * (2 + 4) + 4)
    pairs = 0  # (query row, key) pairs
    for i, n in enumerate(suffix):
        seen = prefix[i // c["branches"]] + n
        if c["kind"] == "prefill":
            pairs += c["hq"] * (c["tokens"] * seen + c["tokens"] * (c["tokens"] + 1) // 2)
        else:
            pairs += c["hq"] * (seen + (1 if c["kind"] == "step" else 0))
    if c["kind"] == "prefill":
        read += c["branches"] * c["tokens"] * token
    elif c["kind"] == "step":
        io += 2 * len(suffix) * token
    return {"bytes": c["layers"] * (read + io), "flops": c["layers"] * 4 * c["d"] * pairs}


def tolerance(case):
    # fp32 sums of products with p carried as two bf16 terms (16 bits): 5e-6 from 64 bits at every
    # size, so two such results are up to 7e-6 apart; four times that
    return {"rel": 3e-5, "max": 1e-3}


def _attend(q, k, v, limit):
    """Attention of rows q [R][d] over keys k, v [L][d] (float64), row r seeing keys [0, limit[r]); (out, lse)."""
    outs, lses = [], []
    key = torch.arange(k.shape[0], device=k.device)
    for r in range(0, q.shape[0], CHUNK_ROWS):
        s = (q[r:r + CHUNK_ROWS] @ k.T) / math.sqrt(q.shape[1])
        s.masked_fill_(key[None, :] >= limit[r:r + CHUNK_ROWS, None], -math.inf)
        lse = torch.logsumexp(s, 1)
        outs.append(torch.exp(s - lse[:, None]) @ v)
        lses.append(lse)
    return torch.cat(outs), torch.cat(lses)


def _context(c, state, s, seq, length):
    """K and V [Hkv][prefix + length][d] of a sequence in float64."""
    n_pre = state["prefix"][seq // c["branches"]]
    if not c["paged"]:
        return [torch.cat([s["prefix_" + x], s["suffix_" + x][seq, :, :length]], 1).double() for x in "kv"]
    row, got = s["table"][seq].long(), []
    for x in "kv":
        pre = s[x + "_pool"][row[:_pages(n_pre)]].transpose(0, 1).reshape(c["hkv"], -1, c["d"])[:, :n_pre]
        suf = s[x + "_pool"][row[_pages(n_pre):_pages(n_pre) + _pages(length)]].transpose(0, 1)
        got.append(torch.cat([pre, suf.reshape(c["hkv"], -1, c["d"])[:, :length]], 1).double())
    return got


def exact(case, seed):
    c, state = case, prepare(case, seed)
    group, new = c["hq"] // c["hkv"], _new_tokens(c)
    result = {"out": torch.empty_like(state["out"], dtype=torch.float64),
              "lse": torch.empty_like(state["lse"], dtype=torch.float64)}
    for i, s in enumerate(state["layers"]):
        for seq in range(len(state["suffix"])):
            n, n_pre = state["suffix"][seq], state["prefix"][seq // c["branches"]]
            if c["kind"] == "step":  # the appended token is in the cache when the row is read
                if c["paged"]:
                    page = int(s["table"][seq, _pages(n_pre) + n // PAGE])
                    s["k_pool"][page, :, n % PAGE], s["v_pool"][page, :, n % PAGE] = s["k_new"][seq], s["v_new"][seq]
                else:
                    s["suffix_k"][seq, :, n], s["suffix_v"][seq, :, n] = s["k_new"][seq], s["v_new"][seq]
            k, v = _context(c, state, s, seq, n + new)
            q = s["q"][seq].reshape(-1, c["hkv"], group, c["d"]).double()  # [tokens][Hkv][G][d]
            last = torch.arange(q.shape[0], device="cuda") + n_pre + n + (1 if new else 0)
            limit = last.repeat_interleave(group)
            for g in range(c["hkv"]):
                o, l = _attend(q[:, g].reshape(-1, c["d"]), k[g], v[g], limit)
                heads = slice(g * group, (g + 1) * group)
                result["out"][i][seq][..., heads, :] = o.reshape(*s["out"][seq].shape[:-2], group, c["d"])
                result["lse"][i][seq][..., heads] = l.reshape(*s["lse"][seq].shape[:-1], group)
    if c["kind"] == "step":
        result["lens"] = state["lens"] + 1
        result["cache"] = [[s["k_pool"], s["v_pool"]] if c["paged"] else [s["suffix_k"], s["suffix_v"]]
                           for s in state["layers"]]
    return result
