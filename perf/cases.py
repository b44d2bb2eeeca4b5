"""Performance cases of the token-importance path: what a serving program has this library do per request.

A pass is what such a program enqueues between the draft model's forward passes and the base model's prefill:
score the prompt tokens against the draft's K cache, select the chunks to keep, gather ids, positions and (where
the base model takes embeddings) rows.  A case is one of three kinds:

  "step"    Scorer.run, Selector.run, Gatherer.run -- the three calls of the path
  "one"     score_pool_select and Gatherer.run -- the single-launch entry point for one short prompt
  "select"  Selector.run and Gatherer.run on scores that are there already (kept sets of several rates are
            drawn from one scoring, and single tokens are kept: the paper's variant without chunks)

The shapes are those of the repository's workloads (drafts shaped like Llama-3.x 1B and 8B, prompts of 1K to 128K
tokens, batches of 64 ragged prompts, one query without look-ahead or up to eight with it) and odd sizes between.
"""
import math
import random

import torch

from paper_2502_02789_amd import binding as sp
from paper_2502_02789_amd import device as spd

#: layers, query heads, KV heads, head dim of the draft models
MODELS = {"tiny": (2, 8, 2, 64), "1b": (16, 32, 8, 64), "8b": (32, 32, 8, 128)}
VOCAB = 128256
#: keys read by the largest listed case: 64 prompts of 1K to 4K tokens of the 8B-shaped draft
MOST_KEY_BYTES = 11.0e9


def listed():
    return [
        # the smallest request: a short question, last prompt token only, one launch for scores and kept set
        _case("one prompt 1000 tiny", kind="one", model="tiny", lo=1000, hi=1000, n=1, keep=0.25),
        # one chat-sized prompt, last prompt token only, on a GPU that other streams use as well
        _case("one prompt 2K last token", model="8b", lo=2048, hi=2048, n=1, exclusive=False, keep=0.3),
        # one chat-sized prompt of odd length with eight look-ahead queries
        _case("one prompt 3001 look-ahead", model="8b", lo=3001, hi=3001, n=8),
        # a small draft on a medium prompt, eight look-ahead queries
        _case("one prompt 8K look-ahead 1b", model="1b", lo=8192, hi=8192, n=8),
        # the headline: a long document, eight look-ahead queries, idle GPU
        _case("one prompt 32K look-ahead", model="8b", lo=32768, hi=32768, n=8),
        # the same class of request with the other reading of the layer reduction, odd length
        _case("one prompt 30011 mean", model="8b", lo=30011, hi=30011, n=8, mean=True),
        # the same class with the draft's cache stored in 8 bits
        _case("one prompt 32K 8-bit", model="8b", lo=32768, hi=32768, n=8, bits=8),
        # the same class while other streams use the GPU (no promise of an idle device), odd length
        _case("one prompt 24577 shared", model="8b", lo=24577, hi=24577, n=8, exclusive=False),
        # the longest prompts, kept embedding rows gathered for the base model
        _case("one prompt 128K gather", model="8b", lo=131072, hi=131072, n=8, chunk=64, keep=0.05, embed=8192),
        # a full batch of ragged prompts without look-ahead: the most keys in one call
        _case("batch 64 last token", model="8b", b=64, lo=1024, hi=4096, n=1, keep=0.3),
        # a batch of ragged prompts with look-ahead (some rows end early) out of a paged cache
        _case("batch 16 look-ahead paged", model="8b", b=16, lo=300, hi=3000, n=8, page=16, valid=True),
        # a batch keeping single tokens from given scores, embedding rows gathered
        _case("select tokens batch 8", kind="select", b=8, lo=2000, hi=16000, chunk=1, window=1, embed=4096),
    ]


def _case(name=None, **kw):
    c = dict(kind="step", model="8b", b=1, lo=0, hi=0, n=8, mean=False, bits=16, page=0, valid=False, exclusive=True,
             chunk=32, window=13, keep=0.1, embed=0)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: kinds as in the list, lengths over the whole range (mostly odd), the options independent."""
    r = rng.random()
    keep = rng.choice([0.05, 0.1, 0.2, 0.3])
    if r < 0.1:
        n = _log_int(rng, 100, 2048)
        return _case(kind="one", model="tiny", lo=n, hi=n, n=1, keep=keep)
    if r < 0.2:
        lo = _log_int(rng, 200, 4000)
        return _case(kind="select", b=_log_int(rng, 1, 32), lo=lo, hi=min(16000, 4 * lo + rng.randrange(100)),
                     chunk=rng.choice([1, 1, 16, 32]), window=rng.choice([1, 5, 13]), keep=keep,
                     embed=rng.choice([0, 4096, 8192]))
    opt = dict(keep=keep, chunk=rng.choice([16, 32, 64]), mean=rng.random() < 0.2, bits=8 if rng.random() < 0.2 else 16,
               page=rng.choice([0, 0, 0, 16, 64]), exclusive=rng.random() < 0.75)
    model = rng.choice(["1b", "8b", "8b"])
    if r < 0.65:  # one prompt; where the GPU is shared or the cache is 8-bit not the longest ones
        top = 131072 if opt["exclusive"] and opt["bits"] == 16 else 32768
        n = _log_int(rng, 500, top)
        return _case(model=model, lo=n, hi=n, n=rng.choice([1, 2, 4, 5, 8, 8, 8]), embed=rng.choice([0, 0, 4096]), **opt)
    n = rng.choice([1, 1, 1, 2, 4, 8, 8])
    hi = _log_int(rng, 600, 4096)
    lo = max(200, int(hi * rng.uniform(0.1, 0.9)))
    b = _log_int(rng, 2, 64)
    while b > 2 and b * (lo + hi) / 2 * _key_bytes_per_token(model, 16) > (MOST_KEY_BYTES if n == 1 else MOST_KEY_BYTES / 4):
        b -= 1
    return _case(model=model, b=b, lo=lo, hi=hi, n=n, valid=n > 1 and rng.random() < 0.5, **opt)


def _key_bytes_per_token(model, bits):
    L, _, H_kv, d = MODELS[model]
    return L * H_kv * d * bits // 8


def _lens(c):
    """Prompt lengths of the batch: part of the case, the same for every seed."""
    r = random.Random("%d %d %d" % (c["b"], c["lo"], c["hi"]))
    return [r.randint(c["lo"], c["hi"]) for _ in range(c["b"])]


def _kept(c):
    return int(sp.sp_keep_upper_bound(_lens(c), c["chunk"], c["keep"]))


def _inputs(c, seed):
    """What the draft model leaves behind, made on the GPU from the seed: stored queries, K cache (already rotated, as
    serving caches are), the lengths, token ids.  One percent of the prompt, in runs of up to 64 tokens, has keys
    aligned with the last token's query, as salient passages do; the rest is noise of unit variance."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    lens = _lens(c)
    T, B = sum(lens), len(lens)
    x = {"lens": lens, "T": T}
    x["cu"] = torch.tensor([0] + lens, dtype=torch.int64).cumsum(0).to(torch.int32).to(dev)
    x["ids"] = torch.randint(0, VOCAB, (T,), generator=g, device=dev, dtype=torch.int32)
    if c["kind"] == "select":
        # probabilities: heavy-tailed, all positive
        x["scores"] = torch.exp(2.0 * torch.randn(T, generator=g, device=dev)) / 16000.0
        return x
    L, H, H_kv, d = MODELS[c["model"]]
    N = c["n"]
    x["q"] = torch.randn((L, B, N, H, d), generator=g, device=dev).to(torch.bfloat16)
    r = random.Random(seed)
    salient, owner, start = [], [], 0
    for b, m in enumerate(lens):
        run = min(64, m)
        for _ in range(max(1, round(0.01 * m / run))):
            at = r.randrange(m - run + 1)
            salient += range(start + at, start + at + run)
            owner += [b] * run
        start += m
    pairs = sorted(dict(zip(salient, owner)).items())
    tok = torch.tensor([t for t, _ in pairs], device=dev)
    own = torch.tensor([b for _, b in pairs], device=dev)
    row = tok
    if c["page"]:
        # pages of all sequences shuffled over one pool per layer, one page to spare
        page, need = c["page"], [-(-m // c["page"]) for m in lens]
        perm = torch.randperm(sum(need) + 1, generator=g, device=dev)
        table = torch.zeros((B, max(need)), dtype=torch.int32, device=dev)
        used, rows = 0, []
        for b, m in enumerate(lens):
            table[b, : need[b]] = perm[used : used + need[b]].to(torch.int32)
            i = torch.arange(m, device=dev)
            rows.append(perm[used + i // page] * page + i % page)
            used += need[b]
        x["table"], x["row"] = table, torch.cat(rows)
        row = x["row"][tok]
        n_rows = (used + 1) * page
    else:
        n_rows = T
    ks, scales = [], []
    for l in range(L):
        k = torch.randn((n_rows, H_kv, d), generator=g, device=dev, dtype=torch.bfloat16)
        lead = x["q"][l, :, 0, :: H // H_kv, :]  # the first head of every group
        k[row] = (k[row].float() + 3.0 * lead[own].float()).to(torch.bfloat16)
        if c["bits"] == 8:
            sc = k.abs().amax(dim=(0, 2)).float() / 448.0
            k = (k.float() / sc[None, :, None]).to(torch.float8_e4m3fn).view(torch.uint8)
            scales.append(sc)
        ks.append(k.view(-1, c["page"], H_kv, d) if c["page"] else k)
    x["k"] = ks
    x["k_scale"] = torch.stack(scales).contiguous() if scales else None
    x["n_valid"] = torch.randint(1, N + 1, (B,), generator=g, device=dev, dtype=torch.int32) if c["valid"] else None
    return x


_tables = {}


def _embedding(width):
    """The base model's embedding table: weights, laid out once per process."""
    if width not in _tables:
        g = torch.Generator(device="cuda")
        g.manual_seed(width)
        _tables[width] = torch.randn((VOCAB, width), generator=g, device="cuda", dtype=torch.bfloat16) * 0.02
    return _tables[width]


def prepare(case, seed):
    c = _case(**case)
    x = _inputs(c, seed)
    s = {"kind": c["kind"], "inputs": x}
    if c["kind"] == "select":
        scores = x["scores"]
    else:
        paged = dict(block_table=x["table"], page_size=c["page"], total_tokens=x["T"]) if c["page"] else {}
        s["scorer"] = spd.Scorer(x["q"], x["k"], x["cu"], H_kv=MODELS[c["model"]][2],
                                 scale=1.0 / math.sqrt(MODELS[c["model"]][3]),
                                 layer_reduce=sp.SP_LAYER_MEAN if c["mean"] else sp.SP_LAYER_MAX, n_valid=x["n_valid"],
                                 exclusive_device=c["exclusive"], keep_workspace=c["exclusive"],
                                 max_seqlen=max(x["lens"]) if c["b"] > 1 else 0, k_scale=x["k_scale"], **paged)
        scores = s["scorer"].scores
    s["selector"] = spd.Selector(scores, x["cu"], chunk=c["chunk"], pool_window=c["window"], keep_rate=c["keep"],
                                 capacity=_kept(c))
    s["gatherer"] = spd.Gatherer(s["selector"], token_ids=x["ids"], embed=_embedding(c["embed"]) if c["embed"] else None)
    return s


def run(state):
    out = {}
    if state["kind"] == "one":
        out["scores"] = spd.score_pool_select(state["scorer"], state["selector"])[0]
    else:
        if state["kind"] == "step":
            out["scores"] = state["scorer"].run()
        state["selector"].run()
    ids, pos, decode, rows = state["gatherer"].run()
    out.update(kept_idx=state["selector"].kept_idx, cu_keep=state["selector"].cu_keep, kept_ids=ids, kept_pos=pos,
               decode_pos=decode)
    if rows is not None:
        out["rows"] = rows
    return out


def work(case):
    c = _case(**case)
    T, B, kept = sum(_lens(c)), c["b"], _kept(c)
    out = 12 * kept + 8 * B  # indices, ids, positions; offsets, decode positions
    small = 4 * B + 4 * kept + out + 2 * kept * c["embed"] * 2  # lengths, token ids of kept tokens, rows in and out
    if c["kind"] == "select":
        return {"bytes": 4 * T + small, "flops": T * c["window"]}
    L, H, H_kv, d = MODELS[c["model"]]
    q = L * B * c["n"] * H * d * 2
    return {"bytes": T * _key_bytes_per_token(c["model"], c["bits"]) + q + 4 * T + small,
            "flops": 2 * L * H * c["n"] * d * T}


def tolerance(case):
    # Kept sets follow from given scores by exact comparisons.  Scores are fp32: products of bf16 or 8-bit values
    # (exact) summed over the head dim in fp32, fp32 exponentials and sums; against 64 bits they are off by 1e-6 to
    # 2e-6 (2-norm).  A chunk whose score ties with the k-th to that accuracy may change places with it.
    if case["kind"] == "select":
        return "exact"
    return {"rel": 8e-6, "max": 8e-5, "differ": 0.01}


def exact(case, seed):
    """The scores in 64 bits: softmax of every row over the prompt's keys, maximum over heads, maximum or mean over
    layers, mean over the valid queries."""
    c = _case(**case)
    if c["kind"] == "select":
        return None  # whole numbers and copied rows only
    x = _inputs(c, seed)
    none = dict.fromkeys(("kept_idx", "cu_keep", "kept_ids", "kept_pos", "decode_pos"))
    if c["embed"]:
        none["rows"] = None  # copies of the table's
    L, H, H_kv, d = MODELS[c["model"]]
    N, G = c["n"], H // H_kv
    scores, start = [], 0
    for b, m in enumerate(x["lens"]):
        rows = x["row"][start : start + m] if c["page"] else slice(start, start + m)
        total = None
        for l in range(L):
            k = x["k"][l].reshape(-1, H_kv, d)[rows]
            if c["bits"] == 8:
                k = k.view(torch.float8_e4m3fn).float().double() * x["k_scale"][l].double()[None, :, None]
            k = k.double().permute(1, 2, 0).contiguous()                                    # [H_kv, d, m]
            q = x["q"][l, b].double().view(N, H_kv, G, d).permute(1, 0, 2, 3).reshape(H_kv, N * G, d).contiguous()
            s = torch.matmul(q, k) / math.sqrt(d)
            a = torch.softmax(s, dim=-1).view(H_kv, N, G, m).amax(dim=(0, 2))               # [N, m]
            total = a if total is None else total + a if c["mean"] else torch.maximum(total, a)
        if c["mean"]:
            total = total / L
        nv = N if x["n_valid"] is None else int(x["n_valid"][b])
        scores.append(total[:nv].mean(dim=0))
        start += m
    return dict(none, scores=torch.cat(scores))
