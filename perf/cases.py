"""The work whose speed is measured: the calls a serving loop of this library
makes, over the range of batches it serves.

A case names one kind of call and its sizes:

  step       attention, then both logit passes: one whole fused draft-verify step
  attention  draft_verify_attention
  overlap    multibranch_attention, correction and continuation branches
  quadratic  multibranch_attention, one draft block per accepted length
  round      verify_and_confidence, both logit passes of a step
  verify     verify_accept
  draft      draft_confidence
  decide     plan_branches, match_branches and plan_block_sizes of one round

The ragged structure of a batch (context lengths, block sizes, page table)
follows from the case (its ``layout`` number), the tensors' values from the
seed.  Attention inputs are unit normal, so the scaled scores have unit
spread; logits are drawn as the library's benchmark draws them.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2609_34388_amd import binding
from paper_2609_34388_amd import workloads as W

DELTA = 0.15  # draft margin below which a position is risky


def _attn(name, kind, requests, ctx, verify, draft, layout, heads=(32, 8, 128), vocab=128256):
    return dict(name=name, kind=kind, requests=requests, q_heads=heads[0], kv_heads=heads[1], head_dim=heads[2],
                ctx_min=ctx[0], ctx_max=ctx[1], verify=verify, draft=draft, vocab=vocab, layout=layout)


def _rows(name, kind, requests, verify, draft, vocab, pad, bonus, layout, noalloc=False):
    return dict(name=name, kind=kind, requests=requests, verify=verify, draft=draft, vocab=vocab, pad=pad,
                bonus=bonus, noalloc=noalloc, layout=layout)


def listed():
    return [
        # One user, the whole step: a chain of small launches where latency counts.
        _attn("step_one_request", "step", 1, (4096, 4096), "16", "16", 0),
        # A small server's batch: 16 requests of 1k to 8k tokens, every block size.
        _attn("attention_16", "attention", 16, (1024, 8192), "4,8,16,32", "4,8,16,32", 0),
        # Full concurrency, short contexts, small blocks.
        _attn("attention_128", "attention", 128, (512, 4096), "2,2,2,2,4,4,4,8,8,16", "2,2,2,2,4,4,4,8,8,16", 0),
        # Long documents: 64 requests of 16k to 32k tokens, the largest case.
        _attn("attention_long", "attention", 64, (16384, 32768), "4,8,16,32", "4,8,16,32", 0),
        # A smaller backbone (head size 64, four query heads per KV head), odd lengths and blocks.
        _attn("attention_d64", "attention", 48, (257, 6001), "1,3,7,13", "3,5,11,16", 1, heads=(16, 4, 64)),
        # An overlap round at full concurrency: three branches per request.
        _attn("overlap_128", "overlap", 128, (512, 4096), "2,2,2,2,4,4,4,8,8,16", "2,2,2,2,4,4,4,8,8,16", 0),
        # The quadratic layout, one draft block per accepted length: many rows per key.
        _attn("quadratic_16", "quadratic", 16, (1024, 8192), "4,8,16", "4,8,16", 0),
        # Logits of a small server's step.
        _rows("round_16", "round", 16, "4,8,16,32", "4,8,16,32", 128256, 0, False, 0),
        # Logits of 64 requests with large blocks: the largest logit pass.
        _rows("round_64", "round", 64, "4,8,16,32", "4,8,16,32", 128256, 0, False, 0),
        # Verification alone with bonus rows over an odd vocabulary: rows start at any 2-byte place.
        _rows("verify_odd_vocab", "verify", 40, "2,4,8,16", "0", 65537, 0, True, 0),
        # Draft confidence alone over a vocabulary that is no whole number of chunks.
        _rows("draft_151936", "draft", 12, "0", "4,8,16", 151936, 0, False, 0),
        # A round's decisions for the requests of a whole server group.
        dict(name="decide_1024", kind="decide", requests=1024, bins=8, layout=0),
    ]


# ---------------------------------------------------------------------------
# Structure of a case
def _values(text):
    return tuple(int(x) for x in text.split(","))


def _layout(case, seed=0):
    attn = "ctx_min" in case
    spec = W.WorkloadSpec("case", 17, case["requests"], case["q_heads"] if attn else 1, case["kv_heads"] if attn else 1,
                          case["head_dim"] if attn else 64, case["vocab"],
                          ("uniform", case["ctx_min"], case["ctx_max"]) if attn else ("fixed", 0),
                          ("choice", _values(case["verify"]), None), ("choice", _values(case["draft"]), None),
                          ("uniform", 0.5, 2.0), 1.0)
    lay = W.make_layout(spec, seed=case["layout"], bonus_rows=bool(case.get("bonus", False)))
    return dataclasses.replace(lay, seed=seed)


def _branches(case, lay):
    fixed = dataclasses.replace(lay, seed=case["layout"])  # the branches belong to the structure
    return W.overlap_branches(fixed) if case["kind"] == "overlap" else W.quadratic_branches(fixed)


def _structure(case, seed=0):
    """Layout, and the branch lists of a branched case (else None)."""
    lay = _layout(case, seed)
    if case["kind"] not in ("overlap", "quadratic"):
        return lay, None
    br = _branches(case, lay)
    return dataclasses.replace(W.make_overlap_layout(dataclasses.replace(lay, seed=case["layout"]), br), seed=seed), br


def _visible(lay, br):
    """Visible (query row, key) pairs of the batch."""
    total = 0
    for r in range(lay.num_requests):
        L, V, n = int(lay.ctx_len[r]), int(lay.n_verify[r]), int(lay.q_len[r])
        total += V * L + V * (V + 1) // 2
        for prefix, lead, rows in (br[r] if br else [(V, 0, n - V)]):
            total += rows * (L + prefix) + lead * (lead + 1) // 2 + (rows - lead) * rows
    return total


def _attn_work(case):
    lay, br = _structure(case)
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    keys, rows = int(lay.kv_len.sum()), lay.total_q
    return (keys * hkv * d * 4 + rows * hq * (d * 4 + 4) + int(lay.page_indptr[-1]) * 4,
            4 * d * hq * _visible(lay, br))


def _rows_work(case):
    lay = _layout(case)
    v, d, R = lay.total_verify_rows, lay.total_draft_rows, lay.num_requests
    if case["kind"] == "verify":
        d = 0
    if case["kind"] == "draft":
        v = 0
    # per entry: maximum, difference, exponential, two sums
    return ((v + d) * case["vocab"] * 2 + v * 12 + d * 24 + (R * 16 if v else 0), (v + d) * case["vocab"] * 6)


def _decide_rows(case):
    rng = np.random.default_rng([case["layout"], case["requests"]])
    return rng.choice(np.asarray(W.BLOCK_CANDIDATES), size=case["requests"])


def work(case):
    if case["kind"] == "decide":
        R, rows = case["requests"], int(_decide_rows(case).sum())
        nb = len(W.BLOCK_CANDIDATES)
        return dict(bytes=rows * 4 + R * 88 + nb * nb * case["bins"] * 8, flops=rows + R * (case["bins"] + 4 * nb))
    bytes_, flops = 0, 0
    if "ctx_min" in case:
        bytes_, flops = _attn_work(case)
    if case["kind"] in ("step", "round", "verify", "draft"):
        b, f = _rows_work(case)
        bytes_, flops = bytes_ + b, flops + f
    return dict(bytes=bytes_, flops=flops)


# ---------------------------------------------------------------------------
# Inputs
def _dev():
    return torch.device("cuda")


def _i32(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.int32, device=_dev())


def _logit_inputs(case, lay):
    """Verify logits, judged tokens and draft logits, rows ``pad`` entries apart beyond the vocabulary."""
    inp = W.make_logit_inputs(lay, _dev())
    pad = case.get("pad", 0)
    if pad:
        for k in ("verify_logits", "draft_logits"):
            wide = torch.zeros(inp[k].shape[0], case["vocab"] + pad, dtype=torch.bfloat16, device=_dev())
            wide[:, :case["vocab"]] = inp[k]
            inp[k] = wide[:, :case["vocab"]]
    return inp


def _decide_inputs(case, seed):
    R = case["requests"]
    block = _decide_rows(case)
    indptr = np.concatenate([[0], np.cumsum(block)]).astype(np.int32)
    rng = np.random.default_rng([seed, R, 5])
    d = W.make_block_policy_inputs(seed=seed, num_requests=R, num_s_bins=case["bins"])
    accept = np.minimum(d["accept_len"], block)
    full = rng.random(R) < 0.3
    accept[full] = block[full]
    rows = int(indptr[-1])
    return dict(margin=rng.beta(1.0, 1.5, rows).astype(np.float32), top2=rng.integers(0, 128256, rows),
                row_indptr=indptr, accept_len=accept, next_token=rng.integers(0, 128256, R), block_len=block,
                cont_first=rng.integers(0, 128256, R), accept_entropy=d["accept_entropy"],
                entropy_hist=d["entropy_hist"], policy=d)


def prepare(case, seed):
    kind = case["kind"]
    st = dict(kind=kind)
    if kind == "decide":
        d = _decide_inputs(case, seed)
        p = d["policy"]
        R, dev = case["requests"], _dev()
        cost = [1.0, 1.3, 2.0]  # a step's cost by block size, relative to the smallest
        st["policy"] = binding.make_block_policy(p["candidates"], p["s_edges"], cost, 4.0,
                                                 torch.as_tensor(p["value"], device=dev))
        for k in ("top2", "row_indptr", "accept_len", "next_token", "block_len", "cont_first"):
            st[k] = _i32(d[k])
        for k in ("margin", "accept_entropy", "entropy_hist"):
            st[k] = torch.as_tensor(d[k], dtype=torch.float32, device=dev)
        e = lambda *s: torch.empty(*s, dtype=torch.int32, device=dev)
        st["plan"] = dict(n_risky=e(R), n_corr=e(R), corr_pos=e(R, 2), corr_tok=e(R, 2), continuation=e(R))
        st["reused"] = e(R)
        st["sizes"] = dict(next_block=e(R), order=e(R), bucket_offsets=e(len(W.BLOCK_CANDIDATES) + 1))
        return st
    lay, br = _structure(case, seed)
    if "ctx_min" in case:
        st.update(W.make_attention_inputs(lay, _dev()))
        st["layout"] = binding.make_layout(st["q"], st["k_cache"], lay.q_indptr, lay.n_verify, lay.ctx_len,
                                           lay.page_indptr, _i32(lay.page_indices))
        if br is not None:
            flat = [b for one in br for b in one]
            st["branches"] = binding.make_branches(np.concatenate([[0], np.cumsum([len(one) for one in br])]),
                                                   *([b[i] for b in flat] for i in range(3)))
            need = binding.multibranch_workspace_bytes(st["layout"], st["branches"])
        else:
            need = binding.attention_workspace_bytes(st["layout"])
        st["workspace"] = binding.new_workspace(need, _dev()) if need else None
        st["out"] = torch.empty_like(st["q"])
        st["lse"] = torch.empty(st["q"].shape[:2], dtype=torch.float32, device=_dev())
    if kind in ("step", "round", "verify", "draft"):
        inp = _logit_inputs(case, lay)
        st.update(inp)
        st["row_indptr"] = _i32(lay.row_indptr)
        v, d, R, vocab = lay.total_verify_rows, lay.total_draft_rows, lay.num_requests, case["vocab"]
        st["noalloc"] = bool(case.get("noalloc", False))
        need = (binding.verify_accept_workspace_bytes(R, v, vocab) if kind == "verify" else
                binding.draft_confidence_workspace_bytes(d, vocab) if kind == "draft" else
                binding.verify_and_confidence_workspace_bytes(R, v, d, vocab))
        st["row_workspace"] = binding.new_workspace(need, _dev())
        e = lambda n, t: torch.empty(n, dtype=t, device=_dev())
        i, f = torch.int32, torch.float32
        st["verified"] = dict(row_argmax=e(v, i), accept_len=e(R, i), next_token=e(R, i), row_entropy=e(v, f),
                              accept_entropy=e(R, f))
        st["drafted"] = dict(top1=e(d, i), top2=e(d, i), p1=e(d, f), p2=e(d, f), margin=e(d, f), entropy=e(d, f))
    return st


# ---------------------------------------------------------------------------
# One pass
def _run_attention(st):
    if "branches" in st:
        out, lse = binding.multibranch_attention(st["q"], st["k_cache"], st["v_cache"], st["layout"], st["branches"],
                                                 out=st["out"], lse=st["lse"], workspace=st["workspace"])
    else:
        out, lse = binding.draft_verify_attention(st["q"], st["k_cache"], st["v_cache"], None, None, None, None, None,
                                                  layout=st["layout"], out=st["out"], lse=st["lse"],
                                                  workspace=st["workspace"])
    return dict(out=out, lse=lse)


def run(state):
    st, kind = state, state["kind"]
    if kind == "decide":
        plan = binding.plan_branches(st["margin"], st["top2"], st["row_indptr"], DELTA, out=st["plan"])
        reused = binding.match_branches(st["accept_len"], st["next_token"], st["block_len"], plan, st["cont_first"],
                                        out=st["reused"])
        sizes = binding.plan_block_sizes(st["policy"], st["accept_len"], st["accept_entropy"], st["block_len"],
                                         st["entropy_hist"], out=st["sizes"])
        return dict(plan=plan, reused=reused, sizes=sizes, entropy_hist=st["entropy_hist"])
    res = {}
    if "q" in st:
        res.update(_run_attention(st))
    if kind in ("step", "round"):
        v, d = binding.verify_and_confidence(st["verify_logits"], st["row_indptr"], st["draft_tokens"],
                                             st["draft_logits"], workspace=st["row_workspace"],
                                             out_verify=st["verified"], out_draft=st["drafted"],
                                             noalloc=st["noalloc"])
        res.update(verified=v, drafted=d)
    elif kind == "verify":
        res["verified"] = binding.verify_accept(st["verify_logits"], st["row_indptr"], st["draft_tokens"],
                                                workspace=st["row_workspace"], out=st["verified"])
    elif kind == "draft":
        res["drafted"] = binding.draft_confidence(st["draft_logits"], workspace=st["row_workspace"],
                                                  out=st["drafted"])
    return res


# ---------------------------------------------------------------------------
# The same outputs in 64 bits
def _exact_attention(case, lay, br, inp):
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    g, dev = hq // hkv, inp["q"].device
    scale = 1.0 / math.sqrt(d)
    out = torch.empty(inp["q"].shape, dtype=torch.float64, device=dev)
    lse = torch.empty(inp["q"].shape[:2], dtype=torch.float64, device=dev)
    for r in range(lay.num_requests):
        q0, q1 = int(lay.q_indptr[r]), int(lay.q_indptr[r + 1])
        n, L, V = q1 - q0, int(lay.ctx_len[r]), int(lay.n_verify[r])
        if n == 0:
            continue
        T = L + n
        j = torch.arange(T, device=dev)
        see = torch.zeros(n, T, dtype=torch.bool, device=dev)
        see[:V] = j[None, :] <= L + torch.arange(V, device=dev)[:, None]
        at = V
        for prefix, lead, rows in (br[r] if br else [(V, 0, n - V)]):
            start = L + at
            own = (j >= start) & (j < start + rows)
            see[at:at + rows] = (j < L + prefix) | own
            for t in range(lead):
                see[at + t] = (j < L + prefix) | (own & (j <= start + t))
            at += rows
        pages = torch.as_tensor(lay.page_indices[int(lay.page_indptr[r]):int(lay.page_indptr[r + 1])].astype(np.int64),
                                device=dev)
        hide = torch.zeros(n, T, dtype=torch.float64, device=dev).masked_fill_(~see, -math.inf)
        for h in range(hkv):
            K = inp["k_cache"][pages, h].reshape(-1, d)[:T].double()
            Vt = inp["v_cache"][pages, h].transpose(1, 2).reshape(-1, d)[:T].double()
            q = inp["q"][q0:q1, h * g:(h + 1) * g].double().reshape(n * g, d)
            s = (q @ K.T).mul_(scale).view(n, g, T).add_(hide[:, None, :])
            top = s.amax(-1, keepdim=True)
            p = s.sub_(top).exp_()
            z = p.sum(-1, keepdim=True)
            out[q0:q1, h * g:(h + 1) * g] = ((p.view(n * g, T) @ Vt).view(n, g, d) / z)
            lse[q0:q1, h * g:(h + 1) * g] = (top + z.log())[..., 0]
    return dict(out=out, lse=lse)


def _exact_rows(x):
    """Per row: first place of the maximum, P_1st, P_2nd, entropy."""
    v = x.shape[1]
    place = torch.arange(v, device=x.device)
    am, p1, p2, ent = [], [], [], []
    for k in range(0, x.shape[0], 64):
        y = x[k:k + 64].double()
        m = y.amax(1, keepdim=True)
        first = torch.where(y == m, place, v).amin(1)
        dif = y - m
        e = dif.exp()
        rest = e.scatter(1, first[:, None], 0.0)
        z = rest.sum(1)
        am.append(first)
        p1.append(1.0 / (1.0 + z))
        p2.append(rest.amax(1) / (1.0 + z))
        ent.append(torch.log1p(z) - (e * dif).sum(1) / (1.0 + z))
    cat = lambda a: torch.cat(a) if a else torch.zeros(0, dtype=torch.float64, device=x.device)
    return cat(am), cat(p1), cat(p2), cat(ent)


def _exact_verified(lay, inp):
    am, _, _, ent = _exact_rows(inp["verify_logits"])
    bad = (inp["draft_tokens"] < 0) | (inp["draft_tokens"] != am)
    mean = torch.zeros(lay.num_requests, dtype=torch.float64, device=ent.device)
    for r in range(lay.num_requests):
        k0, k1 = int(lay.row_indptr[r]), int(lay.row_indptr[r + 1])
        if k1 > k0:
            miss = bad[k0:k1].nonzero()
            last = int(miss[0]) if len(miss) else k1 - k0 - 1
            mean[r] = ent[k0:k0 + last + 1].mean()
    return dict(row_argmax=None, accept_len=None, next_token=None, row_entropy=ent, accept_entropy=mean)


def _exact_drafted(inp):
    _, p1, p2, ent = _exact_rows(inp["draft_logits"])
    return dict(top1=None, top2=None, p1=p1, p2=p2, margin=p1 - p2, entropy=ent)


def exact(case, seed):
    kind = case["kind"]
    if kind == "decide":  # whole numbers, and a copy
        hist = torch.as_tensor(_decide_inputs(case, seed)["accept_entropy"]).double()
        return dict(plan=None, reused=None, sizes=None, entropy_hist=hist)
    lay, br = _structure(case, seed)
    res = {}
    if "ctx_min" in case:
        res.update(_exact_attention(case, lay, br, W.make_attention_inputs(lay, _dev())))
    if kind in ("step", "round", "verify", "draft"):
        inp = _logit_inputs(case, lay)
        if kind != "draft":
            res["verified"] = _exact_verified(lay, inp)
        if kind != "verify":
            res["drafted"] = _exact_drafted(inp)
    return res


def tolerance(case):
    if case["kind"] == "decide":
        return "exact"
    if "ctx_min" in case:
        # Output and probabilities are bf16: 2.2e-3 to 2.9e-3 measured against 64 bits.
        return dict(rel=1e-2, max=0.1, differ=0.0)
    # fp32 sums over the vocabulary: at most 2e-7 measured against 64 bits, where larger
    # logits can lose a few more ulps; indices come from the bf16 inputs and are exact.
    return dict(rel=2e-6, max=2e-5, differ=0.0)


# ---------------------------------------------------------------------------
# More cases of the same ranges
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = ((32, 8, 128), (32, 8, 128), (16, 4, 64), (8, 2, 128), (16, 2, 64), (8, 8, 128))
_BLOCKS = ("4,8,16,32", "2,2,2,2,4,4,4,8,8,16", "8,16", "16", "1,3,7,13", "3,5,11,16")
_VOCABS = (128256, 128250, 151936, 65537, 40000, 20000)


def _draw_attention(rng, kind):
    ctx_max = _log_int(rng, 128, 32768)
    ctx_min = max(16, int(ctx_max * rng.uniform(0.1, 1.0)))
    blocks = _BLOCKS if kind != "quadratic" else ("4,8", "8", "1,3,7", "4,8,16")
    case = _attn("", kind, _log_int(rng, 1, 160), (ctx_min, ctx_max), rng.choice(blocks), rng.choice(blocks),
                 rng.randrange(1 << 20), heads=rng.choice(_HEADS))
    del case["name"]
    while case["requests"] > 1:
        bytes_, flops = _attn_work(case)
        if bytes_ <= 5.0e9 and flops <= 3.0e11:
            break
        case["requests"] = case["requests"] * 2 // 3
    return case


def _draw_rows(rng, kind):
    blocks = rng.choice(_BLOCKS), rng.choice(_BLOCKS)
    case = _rows("", kind, _log_int(rng, 1, 64), "0" if kind == "draft" else blocks[0],
                 "0" if kind == "verify" else blocks[1], rng.choice(_VOCABS), rng.choice((0, 0, 0, 8, 11)),
                 kind != "draft" and rng.random() < 0.4, rng.randrange(1 << 20),
                 noalloc=kind == "round" and rng.random() < 0.3)
    del case["name"]
    return case


def draw(rng):
    kind = rng.choice(("attention", "attention", "attention", "attention", "overlap", "overlap", "quadratic", "round",
                       "round", "verify", "draft", "step", "decide"))
    if kind == "decide":
        return dict(kind="decide", requests=_log_int(rng, 32, 8192), bins=rng.choice((1, 8, 64)),
                    layout=rng.randrange(1 << 20))
    if kind == "step":
        case = _draw_attention(rng, kind)
        case["requests"] = min(case["requests"], 64)
        return case
    if kind in ("attention", "overlap", "quadratic"):
        return _draw_attention(rng, kind)
    return _draw_rows(rng, kind)
