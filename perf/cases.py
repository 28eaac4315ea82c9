"""The calls whose speed matters, as cases: what a decoding engine built on this
library calls at every step, over the sizes and options it is used with.

  listed()           the cases by name
  draw(rng)          one more case from the same ranges
  prepare(case, s)   what the engine holds before the call: inputs drawn on the
                     GPU from the seed, outputs, workspaces, step arguments
  run(state)         one pass through the public entry points
  work(case)         bytes and operations a pass cannot do without
  tolerance(case)    how far another correct implementation may be off
  exact(case, s)     the floating outputs (the probe logits) in 64 bits

Kinds of case:
  step     one whole step (switchsd_step), greedy (T = 0) or drawn (T > 0),
           with chain or tree drafts, one or several copy candidates, and for
           T > 0 with or without the draft's own distribution
  loop     decode steps with the commit, captured once in a HIP graph
  stages   the stage entry points in the order an engine calls them around the
           target's forward pass: match, probe, select and mask before it,
           verification and commit after it
  labels   copy-mode labels of whole sequences (probe training)

Inputs: Zipf contexts with copied spans and ragged lengths; every second
sequence ends inside a copied span and has a hidden state the probe reads as
copy-mode, the others draft neurally.  Logits are N(0, sigma) rounded to bf16,
with the accepted part of the drafts raised by 8.
"""
import math

import torch

from paper_2609_20186_amd import binding as B

DEV = "cuda"


# ------------------------------------------------------------------ cases

def listed():
    step = dict(kind="step", tree=False, W=1, T=0.0, q=False, sigma=1.0)
    return [
        # one user, short context, small vocabulary: launch latency is everything;
        # such a loop is captured in a HIP graph
        dict(name="loop_one_user", kind="loop", B=1, L=512, V=32000, d=1024, R=6, k=5, W=1,
             steps=32, sets=8, T=0.0, sigma=1.0),
        # the ordinary serving batch, greedy
        dict(step, name="greedy_chat", B=32, L=4096, V=128256, d=4096, R=8, k=7),
        # a large batch with the largest vocabulary, greedy
        dict(step, name="greedy_wide", B=64, L=8192, V=151936, d=5120, R=8, k=7),
        # few users with long documents, greedy: the context scan counts
        dict(step, name="greedy_long", B=8, L=32768, V=128256, d=8192, R=11, k=10),
        # tree drafts for a full batch, the largest call
        dict(step, name="greedy_tree", B=256, L=2048, V=128256, d=4096, R=60, k=7, tree=True),
        # ten copy candidates of twenty tokens
        dict(step, name="greedy_candidates", B=32, L=4096, V=128256, d=4096, R=201, k=20, W=10),
        # the ordinary serving batch at a sampling temperature
        dict(step, name="sampled_chat", B=32, L=4096, V=128256, d=4096, R=8, k=7, T=0.7),
        # long documents at a sampling temperature, wider logits
        dict(step, name="sampled_long", B=8, L=32768, V=128256, d=8192, R=11, k=10, T=1.0,
             sigma=2.0),
        # speculative sampling with the draft model's distribution
        dict(step, name="sampled_draft_q", B=32, L=4096, V=128256, d=4096, R=8, k=7, T=0.7,
             q=True),
        # ten copy candidates at a sampling temperature
        dict(step, name="sampled_candidates", B=32, L=4096, V=128256, d=4096, R=201, k=20, W=10,
             T=0.7),
        # an engine that runs the stages around its own forward pass; odd sizes
        dict(name="stages_odd", kind="stages", B=13, L=3001, V=50257, d=3072, R=41, k=10, W=4,
             T=0.0, sigma=1.0),
        # probe training labels of long documents
        dict(name="labels_long", kind="labels", B=8, L=32768, n=5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_LOGITS = 32 * 201 * 128256  # elements of one logits tensor of a drawn case


def draw(rng):
    kind = rng.choice(["step", "step", "sampled", "sampled", "sampled", "tree", "candidates",
                       "draft_q", "loop", "stages", "labels"])
    if kind == "labels":
        b = _log(rng, 1, 64)
        return dict(kind="labels", B=b, L=max(64, min(_log(rng, 256, 40000), 524288 // b)),
                    n=rng.choice([3, 5, 5, 8, 13]))
    T = rng.choice([0.3, 0.7, 1.0, 1.3])
    c = dict(kind="step", tree=False, W=1, T=0.0, q=False, sigma=rng.choice([1.0, 2.0, 3.0]))
    c["B"] = _log(rng, 1, 96)
    c["L"] = max(64, min(_log(rng, 200, 32768), 1048576 // c["B"]))
    c["V"] = rng.choice([32000, 128256, 151936, _log(rng, 8000, 160000) // 8 * 8])
    c["d"] = rng.choice([1024, 2048, 3072, 4096, 5120, 8192])
    c["k"] = rng.randint(2, 12)
    c["R"] = c["k"] + 1
    if kind in ("step", "tree", "stages") and rng.random() < 0.5:
        c["V"] = _log(rng, 8000, 160000)  # greedy verification takes any vocabulary
    if kind == "sampled":
        c["T"] = T
    if kind == "tree":
        c.update(tree=True, R=rng.randint(max(12, c["R"]), 64), T=rng.choice([0.0, 0.0, T]))
        if c["T"] > 0:
            c["V"] = c["V"] // 8 * 8
    if kind == "candidates":
        c["W"] = rng.randint(2, 10)
        c["R"] = 1 + c["W"] * c["k"]
        c["T"] = rng.choice([0.0, T])
    if kind == "draft_q":
        c.update(T=T, q=True, B=min(c["B"], 48))
    if kind == "loop":
        c = dict(kind="loop", B=_log(rng, 1, 6), L=_log(rng, 200, 8192), V=c["V"] // 8 * 8,
                 d=c["d"], R=c["R"], k=c["k"], W=1, steps=16, sets=2, T=rng.choice([0.0, T]),
                 sigma=c["sigma"])
    if kind == "stages":
        W = rng.randint(1, 6)
        c = dict(kind="stages", B=c["B"], L=c["L"], V=c["V"], d=c["d"], R=1 + W * c["k"], k=c["k"],
                 W=W, T=0.0, sigma=c["sigma"])
    while c["B"] * c["R"] * c["V"] * c.get("sets", 1) > MOST_LOGITS and c["B"] > 1:
        c["B"] //= 2
    return c


# ------------------------------------------------------------------ inputs

def _zipf(g, shape, V, s=1.1):
    """Truncated Zipf token ids (the continuous inverse CDF, rounded down)."""
    u = torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)
    a = 1.0 - s
    x = ((float(V + 1) ** a - 1.0) * u + 1.0) ** (1.0 / a)
    return (x.long() - 1).clamp_(0, V - 1).to(torch.int32)


def _contexts(g, Bn, L, V, k, W):
    """Contexts [B, L] with copied spans, their lengths, and which of them end
    inside a copied span: the last tokens of those repeat W earlier places."""
    x = _zipf(g, (Bn, L), V)
    span = 64
    nb = (L + span - 1) // span
    start = torch.arange(nb, device=DEV) * span
    shift = (torch.rand((Bn, nb), generator=g, device=DEV) * start).long() + 1
    copied = (torch.rand((Bn, nb), generator=g, device=DEV) < 0.3) & (start > 0)
    shift = torch.where(copied, shift, torch.zeros_like(shift)).repeat_interleave(span, 1)[:, :L]
    x = x.gather(1, (torch.arange(L, device=DEV) - shift).clamp_(min=0))
    lengths = L - (torch.rand(Bn, generator=g, device=DEV) * (L // 16)).long()
    copy = torch.arange(Bn, device=DEV) % 2 == 0
    # the last m tokens of a copying sequence, planted at W places, one every
    # (m + k + 2) tokens before the end
    m = max(2, min(24, L // (2 * (W + 1)) - k - 2))
    at = torch.arange(m, device=DEV)
    tail = (lengths - m)[:, None] + at
    tok = _zipf(g, (Bn, m), V, 1.01)  # rarer tokens than the context's
    for c in range(W + 1):
        pos = (tail - c * (m + k + 2)).clamp_(0, L - 1)
        x.scatter_(1, pos, torch.where(copy[:, None], tok, x.gather(1, pos)))
    return x.contiguous(), lengths.to(torch.int32), copy


def _draft(g, Bn, R, V, tree):
    ntok = _zipf(g, (Bn, R), V)
    ntok[:, 0] = -1
    if not tree:
        return ntok, None
    i = torch.arange(R, device=DEV)
    j = (torch.rand((Bn, R), generator=g, device=DEV) * 3).long()
    npar = ((i - 1) // 2 - j).clamp_(min=0)
    npar[:, 0] = -1
    return ntok, npar.to(torch.int32)


def _logits(g, Bn, R, V, sigma):
    t = torch.empty((Bn, R, V), dtype=torch.bfloat16, device=DEV)
    t.normal_(0.0, sigma, generator=g)
    return t.clamp_(-7.5 * sigma, 7.5 * sigma)


def _raise(logits, b, r, tok, on):
    """+8 at [b, r, tok] where on (index tensors of one shape)."""
    b, r, tok = b[on], r[on], tok[on].long()
    logits[b, r, tok] = logits[b, r, tok] + 8.0


def _plant(g, case, logits, x, lengths, copy, ntok, npar, nn):
    """Raises the accepted part of the drafts: a geometric share of a neural
    draft's nodes, the whole first candidate of a copying sequence."""
    Bn, R, k, W = case["B"], case["R"], case["k"], case["W"]
    i = torch.arange(1, R, device=DEV)
    bi = torch.arange(Bn, device=DEV)[:, None].expand(Bn, R - 1)
    par = (i - 1).expand(Bn, R - 1) if npar is None else npar[:, 1:].long()
    u = torch.rand((Bn, R - 1), generator=g, device=DEV)
    acc = u < 0.6 if npar is not None else (u < 0.6).cumprod(1).bool()
    acc = acc & ~copy[:, None] & (i < nn[:, None])
    _raise(logits, bi, par, ntok[:, 1:], acc)
    # candidate 0's continuation: the most recent planted place ends m + k + 2
    # tokens before the context does
    m = max(2, min(24, x.shape[1] // (2 * (W + 1)) - k - 2))
    n = min(k, R - 1)
    j = torch.arange(n, device=DEV)
    pos = (lengths.long()[:, None] - (m + k + 2) + j).clamp_(0, x.shape[1] - 1)
    bj = torch.arange(Bn, device=DEV)[:, None].expand(Bn, n)
    _raise(logits, bj, j.expand(Bn, n), x.gather(1, pos), copy[:, None].expand(Bn, n))


def _probe(g, case, copy):
    d = case["d"]
    w = torch.randn(d, generator=g, device=DEV) / math.sqrt(d)
    h = torch.randn((case["B"], d), generator=g, device=DEV).to(torch.bfloat16)
    z = h.double() @ w.double()
    return w, torch.where(((z >= 0) == copy)[:, None], h, -h).contiguous()


def _uniforms(g, Bn, R):
    lo = torch.randint(0, 1 << 32, (Bn, R), generator=g, device=DEV)
    return lo * (1 << 31) * 2 + torch.randint(0, 1 << 32, (Bn, R), generator=g, device=DEV)


def _draft_with_q(g, case, logits, ntok):
    """The draft model's logits (the target's with noise) and a chain drawn
    from them at the case's temperature."""
    q = torch.empty_like(logits)
    for b in range(case["B"]):
        n = torch.randn(logits[b].shape, generator=g, device=DEV)
        q[b] = logits[b].float() + 0.5 * n
        e = torch.empty_like(n).exponential_(generator=g)
        ntok[b, 1:] = (q[b].float() / case["T"] - e.log())[:-1].argmax(1).to(torch.int32)
    return q


def _inputs(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    Bn, R, V, L, W, k = (case[n] for n in ("B", "R", "V", "L", "W", "k"))
    x, lengths, copy = _contexts(g, Bn, L, V, k, W)
    w, hidden = _probe(g, case, copy)
    tree, T = case.get("tree", False), case["T"]
    sets = []
    for _ in range(case.get("sets", 1)):
        ntok, npar = _draft(g, Bn, R, V, tree)
        # a tree uses every node; with several candidates the chain is shorter
        # than their space
        n = R if tree or W == 1 else min(R, 8)
        nn = torch.full((Bn,), n, dtype=torch.int32, device=DEV)
        logits = _logits(g, Bn, R, V, case["sigma"])
        _plant(g, case, logits, x, lengths, copy, ntok, npar, nn)
        inp = dict(tokens=x, lengths=lengths, hidden=hidden, w=w, ntok=ntok, npar=npar, nn=nn,
                   logits=logits, bias=0.0)
        if T > 0:
            inp["uniforms"] = _uniforms(g, Bn, R)
            if case.get("q"):
                inp["draft_logits"] = _draft_with_q(g, case, logits, ntok)
                inp["accept_uniforms"] = _uniforms(g, Bn, R)
        sets.append(inp)
    return sets


# ------------------------------------------------------------------ passes

def prepare(case, seed):
    if case["kind"] == "labels":
        g = torch.Generator(device=DEV)
        g.manual_seed(seed)
        x, lengths, _ = _contexts(g, case["B"], case["L"], 128256, 8, 1)
        ws = torch.zeros(B.label_workspace_bytes(case["B"], case["L"]), dtype=torch.uint8,
                         device=DEV)
        return dict(kind="labels", n=case["n"], tokens=x, lengths=lengths, workspace=ws,
                    labels=torch.empty((case["B"], case["L"]), dtype=torch.uint8, device=DEV))
    sets = _inputs(case, seed)
    Bn, R, V, L, W, k, T = (case[n] for n in ("B", "R", "V", "L", "W", "k", "T"))
    cfg = B.make_cfg((3, 2, 1), 1, k, 0.0, W)
    out = B.alloc_outputs(Bn, R, k, W, device=DEV)
    ws = B.alloc_workspace(Bn, R, L, W, device=DEV)
    sws = B.alloc_sample_workspace(Bn, R, V, device=DEV) if T > 0 else None
    state = dict(kind=case["kind"], sets=sets, cfg=cfg, out=out, workspace=ws,
                 sample_workspace=sws)
    if case["kind"] == "stages":
        state["mask"] = torch.empty((Bn, R, (R + 31) // 32), dtype=torch.int32, device=DEV)
        state["draft_pos"] = torch.zeros(Bn, dtype=torch.int32, device=DEV)
        state["lag"] = torch.empty(Bn, dtype=torch.int32, device=DEV)
        return state
    more = {}
    if case["kind"] == "loop":
        more = dict(draft_pos=torch.zeros(Bn, dtype=torch.int32, device=DEV),
                    lag=torch.empty(Bn, dtype=torch.int32, device=DEV))
        state.update(more)
    state["args"] = [
        B.build_step_args(inp, out, cfg, temperature=T, uniforms=inp.get("uniforms"),
                          sample_workspace=sws, draft_logits=inp.get("draft_logits"),
                          accept_uniforms=inp.get("accept_uniforms"), **more) for inp in sets]
    if case["kind"] == "loop":
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for i in range(case["steps"]):
                B.switchsd_step(state["args"][i % len(sets)], ws)
        state["graph"] = graph
    return state


def run(state):
    kind = state["kind"]
    if kind == "step":
        B.switchsd_step(state["args"][0], state["workspace"])
        return state["out"]
    if kind == "loop":
        state["graph"].replay()
        inp = state["sets"][0]
        return dict(state["out"], tokens=inp["tokens"], lengths=inp["lengths"],
                    draft_pos=state["draft_pos"], lag=state["lag"])
    if kind == "labels":
        B.switchsd_copy_labels(state["tokens"], state["lengths"], state["n"], state["labels"],
                               state["workspace"])
        return state["labels"]
    inp, o, ws, cfg = state["sets"][0], state["out"], state["workspace"], state["cfg"]
    B.switchsd_ngram_match(inp["tokens"], inp["lengths"], cfg, o["match_n"], o["match_end"],
                           o["copy_len"], o["copy_tokens"], ws)
    B.switchsd_probe_score(inp["hidden"], inp["w"], inp["bias"], o["z"])
    B.switchsd_select_draft(o["match_n"], o["copy_len"], o["copy_tokens"], o["z"], inp["ntok"],
                            inp["npar"], inp["nn"], cfg, o["use_copy"], o["dtok"], o["dpar"],
                            o["dn"])
    B.switchsd_tree_mask(o["dpar"], o["dn"], state["mask"])
    # (the target's forward pass over the draft runs here and gives the logits)
    B.switchsd_verify_accept(inp["logits"], o["dtok"], o["dpar"], o["dn"], o["accept_len"],
                             o["accept_node"], o["bonus"], o["out_tokens"], o["amax"], ws)
    B.switchsd_commit(inp["tokens"], inp["lengths"], o["out_tokens"], o["accept_len"],
                      o["use_copy"], state["draft_pos"], state["lag"])
    return dict(o, mask=state["mask"], tokens=inp["tokens"], lengths=inp["lengths"],
                draft_pos=state["draft_pos"], lag=state["lag"])


# ------------------------------------------------------------------ work, tolerance, reference

def work(case):
    Bn, L = case["B"], case["L"]
    if case["kind"] == "labels":
        return dict(bytes=Bn * L * 5, flops=Bn * L * case["n"])
    R, V, W, k = case["R"], case["V"], case["W"], case["k"]
    ncopy = (Bn + 1) // 2
    if case.get("tree") or W > 1:  # the chosen draft's rows alone
        rows = ncopy * min(R, 1 + W * k) + (Bn - ncopy) * (R if case.get("tree") else min(R, 8))
    else:
        rows = Bn * R
    logits = rows * V * (2 if case.get("q") else 1)
    small = Bn * L * 4 + Bn * case["d"] * 2 + case["d"] * 4 + Bn * R * 4 * 5
    # a comparison per logit, or the twelve operations of an exponential's weight
    # and its sum
    once = dict(bytes=logits * 2 + small, flops=logits * (12 if case["T"] > 0 else 1))
    return {n: v * case.get("steps", 1) for n, v in once.items()}


def tolerance(case):
    # every output is a whole number but the probe logit, a 32-bit rounding of
    # a sum carried in more than 64 bits
    return "exact" if case["kind"] == "labels" else {"rel": 2.5e-7, "max": 1e-6, "differ": 0.0}


def exact(case, seed):
    if case["kind"] == "labels":
        return None
    if case["B"] * case["R"] * case["V"] > 4 * MOST_LOGITS:
        return None
    inp = _inputs(case, seed)[0]
    names = list(B.OUTPUTS)
    if case["kind"] == "stages":
        names += ["mask"]
    if case["kind"] in ("loop", "stages"):
        names += ["tokens", "lengths", "draft_pos", "lag"]
    out = dict.fromkeys(names)
    out["z"] = inp["hidden"].double() @ inp["w"].double() + inp["bias"]
    return out
