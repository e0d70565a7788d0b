"""Timed cases of the verification step: what a target server does with this library, round after round.

A *step* is one pass of the four calls over a ragged batch of verification candidates (attention over the paged KV cache,
LM head, acceptance, commit) through `VerifyStep`.  Beside it stand the calls a server makes more often than whole steps
(attention runs once per transformer layer, the LM head once per model), candidates that form trees, an LM head on weights
that were not re-laid, and the draft side's integer work.  Sizes come from `paper_2605_08151_amd.workloads.CONFIGS`
where a case bears such a name, else they are generic.

Inputs are drawn on the GPU from the seed.  Activations have unit variance, the vocabulary matrix is scaled so that the
background logits have a standard deviation of 1.28, and every candidate row is aligned with one "planted" vocabulary entry
strongly enough to be its argmax, with a probability between about 0.1 and 1 at temperature 1, so that acceptance meets
rows as sharp and as flat as a language model's.  Drafts copy the planted entries for a geometric prefix (greedy requests)
or are drawn from the drafter's own distribution (sampled requests).
"""
import math

import numpy as np
import torch

from paper_2605_08151_amd import binding as sv
from paper_2605_08151_amd.step import VerifyStep

D, P = 128, 16                      # head dimension and tokens per page the library is built for
ROUND = 7                           # the round counter a server passes to acceptance
LARGEST_LM = 1204 * 151936 * 4096   # multiply-adds of the largest listed LM head
LARGEST_KV = 1_550_000              # key positions x kv heads of the largest listed attention


# ------------------------------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------------------------------
def _step(name, B, gamma, ctx, Hq, Hkv, H, V, temp, **more):
    """gamma: text "4" or "0,2,4,8" (dealt round-robin); ctx: "const c" | "uniform lo hi" | "lognormal median sigma lo hi";
    temp: temperature of the sampled requests, 0 = all greedy; temp_mix: every second request stays greedy."""
    return dict(kind="step", name=name, B=B, gamma=gamma, ctx=ctx, Hq=Hq, Hkv=Hkv, H=H, V=V, temp=temp, **more)


def listed():
    return [
        # The smallest batch of the repository's configurations: four chat requests on a small model.  Launches and latency.
        _step("step_tiny", 4, "4", "uniform 128 512", 8, 1, 1024, 32000, 0.0),
        # One user of a large model (batch size 1), sampling: the weight stream of the LM head is nearly everything.
        _step("step_single", 1, "4", "const 4000", 8, 1, 4096, 151936, 0.6),
        # An ordinary greedy batch with all kv heads on one GPU.
        _step("step_mid", 32, "4", "const 2048", 32, 8, 4096, 151936, 0.0),
        # Long drafts and rejection sampling on every request, one tensor-parallel rank's heads.
        _step("step_stochastic", 64, "8", "uniform 1024 4096", 8, 1, 4096, 151936, 0.7),
        # A few document-length requests: long contexts, few rows.
        _step("step_long", 8, "4", "uniform 32768 65536", 8, 1, 4096, 151936, 0.0),
        # The hybrid ordinary-parallel batch: plain decode rows beside candidates, half of the requests sampled, contexts
        # from 256 to 32768.  The largest case.
        _step("step_hybrid", 256, "0,2,4,8", "lognormal 4096 1.0 256 32768", 8, 1, 4096, 151936, 1.0, temp_mix=True),
        # Nothing a multiple of anything: an odd vocabulary, three query heads per kv head, ragged drafts, mixed requests.
        _step("step_odd", 13, "0,1,3,5,6,7", "uniform 37 3001", 12, 4, 1280, 50021, 0.8, temp_mix=True),
        # One layer's attention of an ordinary decode batch (no drafts): the call a server repeats for every layer.
        dict(kind="attn", name="attn_decode", B=128, gamma="0", ctx="lognormal 2048 0.7 128 8192", Hq=32, Hkv=8),
        # One layer's attention of a speculative batch on 4k-token conversations.
        dict(kind="attn", name="attn_verify", B=64, gamma="4", ctx="uniform 1024 4096", Hq=32, Hkv=8),
        # Candidates that form trees of up to 16 rows, greedy: attention, LM head, acceptance and commit for trees.
        dict(kind="tree", name="tree_step", B=16, gamma="7,15,11", ctx="uniform 512 4096", Hq=32, Hkv=8, H=4096, V=151936),
        # The LM head on weights as a checkpoint holds them (row-major), for a caller that cannot keep a re-laid copy.
        dict(kind="rowmajor", name="lm_head_rowmajor", M=128, H=4096, V=151936),
        # Integer work around a round: divergence of the drafts, rollback of their cache, compressed prompts of new requests,
        # the next round's candidates.
        dict(kind="round", name="draft_round", B=128, prefix=4000, gamma=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["attn"] * 3 + ["tree", "rowmajor", "round"])
    if kind == "round":
        return dict(kind="round", B=_log_int(rng, 1, 256), prefix=_log_int(rng, 50, 16000), gamma=rng.randint(1, 8))
    H = rng.choice([1024, 1280, 2048, 2560, 4096])
    V = _log_int(rng, 32000, 151936)
    V = rng.choice([V // 16 * 16, V // 4 * 4, V | 1])
    if kind == "rowmajor":
        return dict(kind=kind, M=_log_int(rng, 1, 320), H=H, V=V)
    B = _log_int(rng, 1, 256)
    Hq, Hkv = rng.choice([(8, 1), (32, 8), (16, 2), (12, 4), (64, 8)])
    most = 15 if kind == "tree" else 8
    most = min(most, 128 // (Hq // Hkv) - 1)
    gamma = rng.choice([[0], [most]] + [sorted(rng.randint(0, most) for _ in range(rng.randint(1, 4))) for _ in range(4)])
    if kind == "tree":
        gamma = [g + 1 for g in gamma if g < most] or [most]
    hi = _log_int(rng, 64, 65536)
    ctx = rng.choice(["const %d" % hi, "uniform %d %d" % (max(1, hi // rng.randint(2, 16)), hi),
                      "lognormal %d 1.0 %d %d" % (max(4, hi // 8), max(1, hi // 128), hi)])
    case = dict(kind=kind, B=B, gamma=",".join(map(str, gamma)), ctx=ctx, Hq=Hq, Hkv=Hkv)
    if kind != "attn":
        case.update(H=H, V=V)
    if kind == "step":
        case.update(temp=rng.choice([0.0, 0.0, 0.6, 1.0]), temp_mix=rng.random() < 0.5)
    while case["B"] > 1:                      # no more work than the largest listed case
        g, c = _lengths(case)
        keys = int((g + 1 + c).sum()) * Hkv
        if keys <= LARGEST_KV and int((g + 1).sum()) * case.get("H", 0) * case.get("V", 0) <= LARGEST_LM:
            break
        case["B"] = max(1, case["B"] * 3 // 4)
    return case


# ------------------------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------------------------
def _lengths(case):
    """gamma_i and committed lengths c_i of the case: evenly spaced quantiles of its distributions, paired the
    same way whatever the seed (prepare() shuffles the requests)."""
    B = case["B"]
    gammas = np.resize(np.array([int(x) for x in case["gamma"].split(",")], np.int64), B)
    kind, *a = case["ctx"].split()
    a = [float(x) for x in a]
    u = (np.arange(B) + 0.5) / B
    if kind == "const":
        c = np.full(B, a[0])
    elif kind == "uniform":
        c = a[0] + u * (a[1] - a[0])
    else:
        z = torch.special.ndtri(torch.from_numpy(u)).numpy()
        c = np.clip(a[0] * np.exp(a[1] * z), a[2], a[3])
    return gammas, np.floor(c).astype(np.int64)


def _paged_batch(case, rng, gen, with_cache=True):
    """Lengths, page table and free list (one int32 buffer, so that a server's per-round update of it is one copy), q, K/V."""
    B, Hq, Hkv = case["B"], case["Hq"], case["Hkv"]
    gammas, ctx = _lengths(case)
    order = rng.permutation(B)
    gammas, ctx = gammas[order], ctx[order]
    n = gammas + 1
    qo = np.zeros(B + 1, np.int32)
    qo[1:] = np.cumsum(n)
    M = int(qo[-1])
    pages = (ctx + n + P - 1) // P
    used = int(pages.sum())
    num_pages = used + max(1, used // 4)
    perm = rng.permutation(num_pages).astype(np.int32)
    max_pages = int(pages.max()) + 1
    table = np.full((B, max_pages), -1, np.int32)
    first = np.concatenate([[0], np.cumsum(pages)])
    for i in range(B):
        table[i, :pages[i]] = perm[first[i]:first[i + 1]]
    free = np.full(num_pages, -1, np.int32)
    free[:num_pages - used] = perm[used:]
    flat = np.concatenate([table.ravel(), ctx.astype(np.int32), free, np.array([num_pages - used], np.int32)])
    tables0 = torch.from_numpy(flat).cuda()
    tables = tables0.clone()
    cut = np.cumsum([B * max_pages, B, num_pages, 1])
    s = dict(B=B, M=M, gammas=gammas, ctx=ctx, gamma_max=int(gammas.max()), max_kv_len=int((ctx + n).max()), num_pages=num_pages,
             tables=tables, tables0=tables0, page_table=tables[:cut[0]].view(B, max_pages), seq_lens=tables[cut[0]:cut[1]],
             free_list=tables[cut[1]:cut[2]], free_count=tables[cut[2]:cut[3]], qo_np=qo, qo=torch.from_numpy(qo).cuda(),
             scale=1.0 / math.sqrt(D))
    if with_cache:
        for name, shape in (("q", (M, Hq, D)), ("k", (num_pages, Hkv, P, D)), ("v", (num_pages, Hkv, P, D))):
            s[name] = torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    return s


def _vocabulary(H, V, gen):
    return torch.empty((V, H), dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.28 / math.sqrt(H), generator=gen)


def _hidden(M, H, V, W, gen):
    """Rows aligned with one vocabulary entry each (its logit is 1.64 x strength above the background), and those entries."""
    planted = torch.randint(0, V, (M,), device="cuda", generator=gen)
    strength = torch.empty((M, 1), device="cuda").uniform_(6.5, 12.0, generator=gen)
    x = torch.empty((M, H), device="cuda").normal_(generator=gen) + strength * W[planted].float()
    return x.to(torch.bfloat16), planted


def _draft_distribution(planted, V, gen):
    """Probability rows of a drafter that mostly agrees with the target, and a token drawn from each."""
    n = planted.numel()
    probs = torch.empty((n, V), dtype=torch.float32, device="cuda")
    drawn = torch.empty(n, dtype=torch.int64, device="cuda")
    for lo in range(0, n, 64):
        part = planted[lo:lo + 64]
        rows = torch.empty((part.numel(), V), device="cuda").normal_(0.0, 1.28, generator=gen)
        boost = torch.empty((part.numel(), 1), device="cuda").uniform_(11.0, 18.0, generator=gen)
        rows.scatter_add_(1, part[:, None], boost)
        rows = torch.softmax(rows, dim=-1)
        probs[lo:lo + 64] = rows
        drawn[lo:lo + 64] = (rows / torch.empty_like(rows).exponential_(generator=gen)).argmax(1)
    return probs, drawn


def _draft_tokens(s, planted, V, rng):
    """Greedy drafts: draft j copies the target's choice on row j - 1 with probability 0.7, else it is any token."""
    tokens = rng.integers(0, V, s["M"])
    copied = rng.random(s["M"]) < 0.7
    copied[s["qo_np"][:-1]] = False                         # row 0 of a request: its last committed token
    at = np.nonzero(copied)[0]
    tokens[at] = planted[at - 1]
    return tokens


def _parents(s, rng):
    """Row-local parents of random candidate trees in topological order."""
    parent = np.full(s["M"], -1, np.int32)
    for i in range(s["B"]):
        for j in range(1, s["gammas"][i] + 1):
            parent[s["qo_np"][i] + j] = rng.integers(max(0, j - 4), j)
    return parent


def _prepare_step(case, rng, gen):
    s = _paged_batch(case, rng, gen)
    B, M, H, V = s["B"], s["M"], case["H"], case["V"]
    W = _vocabulary(H, V, gen)
    s["hidden"], planted = _hidden(M, H, V, W, gen)
    host = planted.cpu().numpy()
    step = VerifyStep(B, M, case["Hq"], case["Hkv"], D, H, V, s["gamma_max"], s["max_kv_len"])
    s["step"], s["Wp"] = step, step.pack_weights(W)
    if case["kind"] == "tree":
        parent = _parents(s, rng)
        tokens = rng.integers(0, V, M)
        row0 = np.repeat(s["qo_np"][:-1], s["gammas"] + 1)
        carry = (rng.random(M) < 0.5) & (parent >= 0)
        tokens[carry] = host[(row0 + parent)[carry]]
        s["parent"] = torch.from_numpy(parent).cuda()
        s["path"] = torch.zeros((B, s["gamma_max"] + 1), dtype=torch.int32, device="cuda")
        # the candidates' own K/V, which the model writes into the cache before it attends
        at = np.repeat(s["ctx"], s["gammas"] + 1) + np.arange(M) - row0
        owner = torch.from_numpy(np.repeat(np.arange(B), s["gammas"] + 1)).cuda()
        at = torch.from_numpy(at).cuda()
        s["new_page"], s["new_slot"] = s["page_table"][owner, at // P].long(), at % P
        s["new_k"] = s["k"][s["new_page"], :, s["new_slot"]].clone()
        s["new_v"] = s["v"][s["new_page"], :, s["new_slot"]].clone()
    else:
        tokens = _draft_tokens(s, host, V, rng)
        temp = np.full(B, case["temp"], np.float32)
        if case.get("temp_mix"):
            temp[::2] = 0.0
        s["temperature"] = torch.from_numpy(temp).cuda()
        s["seeds"], s["draft_probs"] = None, None
        if temp.any():
            s["seeds"] = torch.from_numpy(rng.integers(0, 2 ** 62, B)).cuda()
            later = np.ones(M, bool)
            later[s["qo_np"][:-1]] = False
            later = np.nonzero(later)[0]                    # rows 1 .. gamma_i of every request, in order
            if len(later):
                s["draft_probs"], drawn = _draft_distribution(planted[torch.from_numpy(later - 1).cuda()], V, gen)
                sampled = np.repeat(temp, s["gammas"] + 1)[later] > 0
                tokens[later[sampled]] = drawn.cpu().numpy()[sampled]
    s["tokens"] = torch.from_numpy(tokens.astype(np.int32)).cuda()
    return s


def _prepare_attn(case, rng, gen):
    s = _paged_batch(case, rng, gen)
    size = sv.spec_verify_attn_workspace_bytes(s["B"], s["M"], case["Hq"], case["Hkv"], D, s["max_kv_len"], s["gamma_max"] + 1)
    s["workspace"] = torch.empty(max(256, size), dtype=torch.uint8, device="cuda")
    s["out"] = torch.empty_like(s["q"])
    s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    return s


def _prepare_rowmajor(case, rng, gen):
    W = _vocabulary(case["H"], case["V"], gen)
    hidden, _ = _hidden(case["M"], case["H"], case["V"], W, gen)
    return dict(hidden=hidden, W=W, logits=torch.empty((case["M"], case["V"]), dtype=torch.float32, device="cuda"))


def _prepare_round(case, rng, gen):
    B, S, g = case["B"], case["prefix"], case["gamma"]
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    zeros = lambda *shape: torch.zeros(shape, dtype=torch.int32, device="cuda")
    lens = rng.permutation(np.maximum(1, (S * (0.5 + (np.arange(B) + 0.5) / (2 * B))).astype(np.int64)))
    indptr = np.concatenate([[0], np.cumsum(lens)])
    # the draft's own tokens: the verified prefix, with the last few tokens different in half of the requests
    verified = rng.integers(0, 151936, int(indptr[-1]))
    own = verified.copy()
    for i in range(0, B, 2):
        own[indptr[i + 1] - int(rng.integers(1, min(g + 1, lens[i]) + 1)):indptr[i + 1]] += 1
    s = _paged_batch(dict(B=B, gamma=str(g), ctx="const %d" % S, Hq=1, Hkv=1), rng, gen, with_cache=False)
    keep = s["ctx"] + rng.integers(-g, 1, B)
    accept = rng.integers(0, g + 1, B)
    out = rng.integers(0, 151936, (B, g + 1))
    out[np.arange(g + 1)[None, :] > accept[:, None]] = -1
    cont = rng.integers(0, 151936, (B, g + 1))
    cont[::2, 0] = out[np.arange(B), accept][::2]
    s.update(prefix=i32(verified), own=i32(own), indptr=i32(indptr), delta=zeros(B), keep=i32(np.maximum(keep, 0)),
             accept=i32(accept), out_tokens=i32(out), cont=i32(cont), cont_len=i32(np.full(B, g + 1)),
             repair=i32(rng.integers(0, 151936, (B, g))), repair_len=i32(np.full(B, g)),
             kept=zeros(len(verified)), kept_indptr=zeros(B + 1), next_tokens=zeros(B * (g + 1)), next_qo=zeros(B + 1),
             rollback=torch.zeros(B, dtype=torch.uint8, device="cuda"), stats=zeros(4), status=zeros(1), gamma_next=g)
    return s


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s = {"step": _prepare_step, "tree": _prepare_step, "attn": _prepare_attn, "rowmajor": _prepare_rowmajor,
         "round": _prepare_round}[case["kind"]](case, rng, gen)
    s["kind"] = case["kind"]
    return s


# ------------------------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------------------------
def _run_step(s):
    step = s["step"]
    s["tables"].copy_(s["tables0"])                         # the scheduler's page table and lengths of this round
    step.attn(s["q"], s["k"], s["v"], s["page_table"], s["seq_lens"], s["qo"], s["scale"])
    step.lm_head_packed(s["hidden"], s["Wp"])
    step.accept(s["tokens"], s["draft_probs"], s["temperature"], s["seeds"], ROUND, s["qo"])
    step.commit(s["page_table"], s["seq_lens"], s["qo"], s["free_list"], s["free_count"], P)
    return dict(attn=step.attn_out, lse=step.lse, logits=step.logits, accept_len=step.accept_len, tokens=step.out_tokens,
                rollback=step.rollback, stats=step.stats, status=step.status, tables=s["tables"])


def _run_tree(s):
    step = s["step"]
    s["tables"].copy_(s["tables0"])
    s["k"][s["new_page"], :, s["new_slot"]] = s["new_k"]    # the model appends the candidates' K/V
    s["v"][s["new_page"], :, s["new_slot"]] = s["new_v"]
    sv.spec_verify_attn_tree(s["q"], s["k"], s["v"], s["page_table"], s["seq_lens"], s["qo"], s["parent"], step.attn_out, step.lse,
                             s["max_kv_len"], s["gamma_max"] + 1, s["scale"], step.status, step.attn_ws)
    step.lm_head_packed(s["hidden"], s["Wp"])
    sv.spec_accept_tree(step.logits, s["tokens"], s["parent"], s["qo"], step.accept_len, step.out_tokens, s["path"], step.rollback,
                        step.stats, s["gamma_max"], step.status, step.accept_ws)
    sv.spec_kv_commit_tree(s["k"], s["v"], s["page_table"], s["seq_lens"], s["qo"], step.accept_len, s["path"], s["free_list"],
                           s["free_count"], step.status)
    return dict(attn=step.attn_out, lse=step.lse, logits=step.logits, accept_len=step.accept_len, tokens=step.out_tokens,
                path=s["path"], rollback=step.rollback, stats=step.stats, status=step.status, tables=s["tables"], k=s["k"], v=s["v"])


def _run_attn(s):
    sv.spec_verify_attn(s["q"], s["k"], s["v"], s["page_table"], s["seq_lens"], s["qo"], s["out"], None, s["max_kv_len"],
                        s["gamma_max"] + 1, s["scale"], s["status"], s["workspace"])
    return dict(attn=s["out"], status=s["status"])


def _run_rowmajor(s):
    sv.spec_lm_head(s["hidden"], s["W"], s["logits"])
    return s["logits"]


def _run_round(s):
    s["tables"].copy_(s["tables0"])
    sv.spec_divergence(s["prefix"], s["indptr"], s["own"], s["indptr"], s["delta"])
    sv.spec_kv_truncate(s["page_table"], s["seq_lens"], s["keep"], s["free_list"], s["free_count"], P, s["status"])
    sv.spec_compress_prompts(s["prefix"], s["indptr"], 1, 10, s["kept"], s["kept_indptr"], None)
    sv.spec_assemble_next(s["accept"], s["out_tokens"], s["qo"], s["cont"], s["cont_len"], s["repair"], s["repair_len"],
                          sv.MODE_ORDINARY, s["gamma_next"], s["next_tokens"], s["next_qo"], s["rollback"], s["stats"])
    return dict(delta=s["delta"], tables=s["tables"], kept=s["kept"], kept_indptr=s["kept_indptr"], next_tokens=s["next_tokens"],
                next_qo=s["next_qo"], rollback=s["rollback"], stats=s["stats"], status=s["status"])


def run(state):
    return {"step": _run_step, "tree": _run_tree, "attn": _run_attn, "rowmajor": _run_rowmajor, "round": _run_round}[state["kind"]](state)


# ------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------------------------
def work(case):
    if case["kind"] == "round":
        # both token streams of the divergence, the kept tokens read and written, a few integers per request
        tokens = 0.75 * case["B"] * case["prefix"]
        return dict(bytes=4.0 * (2.0 * tokens + 0.2 * tokens + case["B"] * (5 * case["gamma"] + 24)), flops=0.0)
    if case["kind"] == "rowmajor":
        M, H, V = case["M"], case["H"], case["V"]
        return dict(bytes=2.0 * V * H + 2.0 * M * H + 4.0 * M * V, flops=2.0 * M * V * H)
    g, c = _lengths(case)
    M, keys = int((g + 1).sum()), int((g + 1 + c).sum())
    bytes_ = 4.0 * D * keys * case["Hkv"] + 4.0 * D * M * case["Hq"]        # K and V once, q and out
    flops = 4.0 * D * case["Hq"] * float(((g + 1) * (c + (g + 2) / 2.0)).sum())
    if case["kind"] in ("step", "tree"):
        H, V = case["H"], case["V"]
        bytes_ += 2.0 * V * H + 2.0 * M * H + 4.0 * M * V                   # weights, hidden rows, logits written
        flops += 2.0 * M * V * H
        if case.get("temp", 0.0) > 0:
            sampled = case["B"] // 2 if case.get("temp_mix") else case["B"]
            bytes_ += 4.0 * V * sampled                                     # the drafter's row a rejected draft is compared with
    return dict(bytes=bytes_, flops=flops)


def tolerance(case):
    """bf16 attention outputs with bf16 probabilities inside (2^-9 each, averaged over the keys); fp32 logits summed over
    H products; whole values may differ only where two candidates are tied to within the rounding of a logit."""
    if case["kind"] == "round":
        return "exact"
    if case["kind"] == "rowmajor":
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 1e-2, "max": 5e-2, "differ": 0.005}
