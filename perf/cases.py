"""What users of this library have it do, as timed cases: the trigger scan, verification steps of one sequence and of
several, prompts, and whole generations, each through the package's public calls.

Models have the shapes of the repository's configurations (tiny, small, 7B, 13B); the two large ones keep a few of
their layers, which are all alike.  The weights of a shape are fixed -- a deployment serves one model -- and the seed
draws what a request brings: prompts, drafts, references, caches.

Greedy decoding of a trained model has a clear favourite at nearly every position; iid random matrices do not, and a
rounding difference would then change all later tokens.  So the LM head is tied to the embedding along one cycle through
the vocabulary: embeddings N(0, 1), LM-head row next(v) = embedding of v / sqrt(d), all other matrices N(0, 0.02^2).  The
favourite after token t is next(t), at 11 .. 20 standard deviations of the other logits, whatever the rest of the context
is; every logit still depends on all of it.  So the outputs of a generation are known, references share spans with them
as in the paper's retrieval-augmented and cache-assisted settings, and acceptance lengths are what `prepare` chose.
"""
import math
import random

import numpy as np
import torch

import paper_2304_04487_amd as llma


class Model:
    def __init__(self, n_layers, d_model, n_heads, head_dim, d_ffn, vocab, dtype):
        self.n_layers, self.d_model, self.n_heads, self.head_dim = n_layers, d_model, n_heads, head_dim
        self.d_ffn, self.vocab, self.dtype = d_ffn, vocab, dtype
        self.rms_eps, self.rope_theta = 1e-6, 10000.0

    @property
    def item(self):
        return 2 if self.dtype == "bf16" else 4

    @property
    def layer_params(self):
        return 4 * self.d_model * self.d_model + 3 * self.d_model * self.d_ffn


MODELS = {
    "tiny": Model(2, 128, 4, 32, 512, 512, "fp32"),
    "small": Model(6, 512, 8, 64, 2048, 32000, "bf16"),
    "7b": Model(4, 4096, 32, 128, 11008, 32000, "bf16"),
    "13b": Model(2, 5120, 40, 128, 13824, 32000, "bf16"),
}


# ------------------------------------------------------------------------------------------------ what is measured
def listed():
    return [
        # one trigger lookup from host lists, as a serving loop of its own does before each step: a 3-document
        # reference of the retrieval-augmented workload's size
        {"name": "trigger_host_1472", "kind": "trigger_host", "y": 256, "ref": 1472, "docs": 3, "n": 1},
        # the same lookup on device memory against a large shared reference (a session's or a user's earlier answers)
        {"name": "trigger_device_600k", "kind": "trigger_device", "y": 700, "ref": 600011, "docs": 40, "n": 2},
        # the smallest model: nothing but launches and synchronisation
        {"name": "tiny_generate", "kind": "generate", "model": "tiny", "prompt": 64, "ref": 48, "docs": 1, "overlap": 0.8, "n": 1, "k": 4, "max_new": 32},
        # a draft-sized model, whole call: kernels of a few microseconds each
        {"name": "small_generate", "kind": "generate", "model": "small", "prompt": 512, "ref": 384, "docs": 1, "overlap": 0.6, "n": 2, "k": 8, "max_new": 96},
        # plain greedy decoding (k = 0), what every sequence without a match does
        {"name": "7b_plain_steps", "kind": "steps", "model": "7b", "past": 1001, "k": 0, "steps": 8},
        # the headline workload: prompt with three documents, n = 1, k = 8
        {"name": "7b_generate", "kind": "generate", "model": "7b", "prompt": 1536, "ref": 1472, "docs": 3, "overlap": 0.5, "n": 1, "k": 8, "max_new": 64},
        # verification steps with more than one row tile: 17 rows, and 33 rows over a long cache
        {"name": "13b_steps_k16", "kind": "steps", "model": "13b", "past": 2047, "k": 16, "steps": 6},
        {"name": "7b_steps_k32", "kind": "steps", "model": "7b", "past": 3500, "k": 32, "steps": 4},
        # time to first token: a short prompt (cache-assisted setting, chat turn) and a long one (two passes)
        {"name": "7b_prompt_190", "kind": "prompt", "model": "7b", "prompt": 190},
        {"name": "7b_prompt_2900", "kind": "prompt", "model": "7b", "prompt": 2900},
        # verification steps of 16 sequences over long given caches
        {"name": "7b_batch_16x4096", "kind": "batch", "model": "7b", "seqs": 16, "past": 4096, "k": 8, "steps": 6, "cache": "given"},
        # several short requests decoded together: ragged prompts, caches the library computed itself
        {"name": "7b_generate_batch_6", "kind": "generate_batch", "model": "7b", "seqs": 6, "prompt": 230, "ref": 704, "docs": 4, "overlap": 0.5, "n": 1, "k": 8, "max_new": 40},
    ]


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["trigger_host", "trigger_device", "generate", "steps", "steps", "prompt", "prompt", "batch", "generate_batch"])
    c = {"kind": kind}
    if kind == "trigger_host":
        return dict(c, y=log(4, 2048), ref=log(48, 100000), docs=rng.randint(1, 16), n=rng.randint(1, 3))
    if kind == "trigger_device":
        return dict(c, y=log(4, 4096), ref=log(2000, 600000), docs=rng.randint(1, 64), n=rng.randint(1, 3))
    if kind == "generate":
        m = rng.choice(["tiny", "small", "7b"])
        c.update(model=m, prompt=log(8, {"tiny": 100, "small": 1500, "7b": 1536}[m]), ref=log(60, 1500), docs=rng.randint(1, 4), overlap=rng.choice([0.4, 0.5, 0.6, 0.8]))
        return dict(c, n=rng.randint(1, 3), k=rng.randint(1, 16), max_new=rng.randint(12, 60))
    if kind == "steps":
        m = rng.choice(["small", "7b", "13b"])
        return dict(c, model=m, past=log(16, {"small": 3500, "7b": 3500, "13b": 2400}[m]), k=rng.randint(0, 32), steps=rng.randint(2, 4))
    if kind == "prompt":
        m = rng.choice(["small", "7b", "13b"])
        return dict(c, model=m, prompt=log(3, {"small": 2900, "7b": 2800, "13b": 2400}[m]))
    if kind == "batch":
        return dict(c, model=rng.choice(["small", "7b"]), seqs=rng.randint(2, 16), past=log(64, 4000), k=rng.randint(1, 8), steps=rng.randint(2, 5), cache=rng.choice(["given", "computed"]))
    return dict(c, model=rng.choice(["small", "7b"]), seqs=rng.randint(2, 6), prompt=log(12, 400), ref=log(60, 700), docs=rng.randint(1, 4), overlap=rng.choice([0.4, 0.6]),
                n=rng.randint(1, 2), k=rng.randint(2, 8), max_new=rng.randint(12, 40))


# ------------------------------------------------------------------------------------------------ models
_models = {}        # shape -> (host arrays as Context takes them, next-token table, gains and matrices for exact())


def _weights(name):
    if name in _models:
        return _models[name]
    m = MODELS[name]
    g = torch.Generator(device="cuda").manual_seed(2304)
    bf = m.dtype == "bf16"

    def host(t):
        """to pinned host memory (numpy): a new context then uploads it quickly"""
        t = t.to(torch.bfloat16).view(torch.uint16) if bf else t
        h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
        h.copy_(t)
        return h.numpy()

    def normal(*shape, std=0.02):
        return torch.randn(*shape, generator=g, device="cuda") * std

    def gain():
        return (1.0 + 0.4 * (torch.rand(m.d_model, generator=g, device="cuda") - 0.5)).cpu().numpy()

    order = torch.randperm(m.vocab, generator=g, device="cuda")
    nxt = torch.empty_like(order)
    nxt[order] = order.roll(-1)
    embed = normal(m.vocab, m.d_model, std=1.0)
    head = torch.empty_like(embed)
    head[nxt] = embed / math.sqrt(m.d_model)
    d, f = m.d_model, m.d_ffn
    w = {"embed": host(embed), "lm_head": host(head), "final_norm": gain(), "layers": []}
    for _ in range(m.n_layers):
        w["layers"].append({"wqkv": host(normal(3 * d, d)), "wo": host(normal(d, d)), "wgu": host(normal(2 * f, d)), "wd": host(normal(d, f)),
                            "norm1": gain(), "norm2": gain()})
    torch.cuda.synchronize()
    _models[name] = (w, nxt.cpu().numpy())
    return _models[name]


def _walk(nxt, token, n):
    out = np.empty(n, np.int32)
    for i in range(n):
        token = out[i] = nxt[token]
    return out


def _context(name, max_seq, max_batch=1, max_k=16, rows=1):
    ctx = llma.Context(MODELS[name], _weights(name)[0], max_seq=max_seq, max_batch=max_batch, max_k=max_k)
    ctx.enable_logits_dump(rows)
    return ctx


# ------------------------------------------------------------------------------------------------ requests
def _reference(rng, y, overlap, length, docs, vocab):
    """`length` token ids in `docs` documents: spans of y (12 tokens on average) cover the share `overlap` of it, all else is noise"""
    parts, pos, inside = [], 0, rng.random() < overlap
    while pos < len(y):
        mean = 12.0 if inside else 12.0 * (1 - overlap) / overlap
        n = min(len(y) - pos, 1 + int(rng.expovariate(1.0 / mean)))
        parts.append(list(y[pos:pos + n]) if inside else [rng.randrange(vocab) for _ in range(n)])
        pos, inside = pos + n, not inside
    pads = [0] * (len(parts) + 1)
    for _ in range(max(0, length - len(y))):                    # noise before, between and after them
        pads[rng.randrange(len(pads))] += 1
    ref = [t for n, p in zip(pads, parts + [[]]) for t in [rng.randrange(vocab) for _ in range(n)] + p]
    ref = np.array(ref[:length], np.int32)
    cuts = sorted(rng.randrange(len(ref) + 1) for _ in range(docs - 1))
    return ref, np.array([0] + cuts + [len(ref)], np.int32)


def _prompt(rng, n, vocab):
    return np.array([rng.randrange(vocab) for _ in range(n)], np.int32)


def _ragged(rng, n, most):
    return [most] + [max(2, int(most * rng.uniform(0.6, 1.0))) for _ in range(n - 1)]


def _step_plan(rng, nxt, vocab, token, k, steps):
    """drafts of consecutive steps (each right up to a drawn point), the tokens they will emit, and the rows the last step feeds"""
    drafts, emitted, rows = [], [], []
    for _ in range(steps):
        d = _walk(nxt, token, k)
        right = rng.randint(0, k)
        if right < k:
            d[right] = (d[right] + 1 + rng.randrange(vocab - 1)) % vocab
        rows = [token] + d.tolist()
        drafts.append(d)
        e = _walk(nxt, token, right + 1)
        emitted += e.tolist()
        token = int(e[-1])
    return drafts, emitted, rows


def _requests(case, seed):
    """everything the seed draws, on the host"""
    rng = random.Random("%s %s" % (seed, sorted((k, str(v)) for k, v in case.items() if k != "name")))
    kind, r = case["kind"], {}
    if kind.startswith("trigger"):
        y = _prompt(rng, case["y"], 32000)
        noise = np.random.RandomState(rng.randrange(1 << 30)).randint(0, 32000, case["ref"]).astype(np.int32)
        for _ in range(max(1, case["ref"] // 300)):             # spans of the output so far, the current tail among them
            n = min(len(y), len(noise), 1 + int(rng.expovariate(1 / 12.0)))
            a, b = rng.randrange(len(y) - n + 1), rng.randrange(len(noise) - n + 1)
            noise[b:b + n] = y[a:a + n]
        n = min(case["n"] + 3, len(y), len(noise) - 1)
        b = rng.randrange(len(noise) - n)
        noise[b:b + n] = y[len(y) - n:]
        cuts = [rng.randrange(case["ref"] + 1) for _ in range(case["docs"] - 1)]
        cuts = sorted(b if b < c <= b + n else c for c in cuts)  # the tail and the token after it lie in one document
        offs = np.array([0] + cuts + [case["ref"]], np.int32)
        return {"y": y, "ref": noise, "offs": offs}
    m, nxt = MODELS[case["model"]], _weights(case["model"])[1]
    if kind in ("prompt", "generate"):
        r["prompt"] = _prompt(rng, case["prompt"], m.vocab)
        if kind == "generate":
            r["y"] = _walk(nxt, r["prompt"][-1], case["max_new"])
            r["ref"], r["offs"] = _reference(rng, r["y"], case["overlap"], case["ref"], case["docs"], m.vocab)
    elif kind == "steps":
        r["prompt"] = _prompt(rng, case["past"] + 1, m.vocab)
        r["drafts"], r["emitted"], r["rows"] = _step_plan(rng, nxt, m.vocab, int(r["prompt"][-1]), case["k"], case["steps"])
    elif kind == "batch":
        r["pasts"] = _ragged(rng, case["seqs"], case["past"])
        r["prompts"] = [_prompt(rng, n + 1, m.vocab) for n in r["pasts"]]
        r["plans"] = [_step_plan(rng, nxt, m.vocab, int(p[-1]), case["k"], case["steps"]) for p in r["prompts"]]
        r["kv_seed"] = rng.randrange(1 << 40)
    else:
        r["prompts"] = [_prompt(rng, n, m.vocab) for n in _ragged(rng, case["seqs"], case["prompt"])]
        r["ys"] = [_walk(nxt, p[-1], case["max_new"]) for p in r["prompts"]]
        r["refs"] = [_reference(rng, y, case["overlap"], case["ref"], case["docs"], m.vocab) for y in r["ys"]]
    return r


def _given_kv(m, kv_seed, seq, layer, length):
    """K and V of one given cache: N(0, 1), [heads, length, head_dim]"""
    g = torch.Generator(device="cuda").manual_seed(kv_seed + 1009 * seq + layer)
    kv = torch.randn(2, m.n_heads, length, m.head_dim, generator=g, device="cuda", dtype=torch.float32)
    return kv.to(torch.bfloat16 if m.dtype == "bf16" else torch.float32)


# ------------------------------------------------------------------------------------------------ prepare / run
def _whole(rows, count, width=()):
    """rows as an int32 array of `count` entries, the unused ones -1: how many there are depends on what was accepted"""
    out = np.full((count,) + width, -1, np.int32)
    out[:len(rows)] = rows
    return out


def prepare(case, seed):
    kind, r = case["kind"], _requests(case, seed)
    s = dict(r, kind=kind, case=case)
    if kind == "trigger_device":
        s.update({k: torch.from_numpy(r[k]).cuda() for k in ("y", "ref", "offs")}, result=torch.zeros(3, dtype=torch.int32, device="cuda"))
    elif kind == "prompt":
        s["ctx"] = _context(case["model"], case["prompt"] + 64)
    elif kind == "generate":
        s["ctx"] = _context(case["model"], case["prompt"] + case["max_new"] + case["k"] + 1, max_k=max(case["k"], 1), rows=case["k"] + 1)
    elif kind == "steps":
        s["ctx"] = _context(case["model"], case["past"] + (case["steps"] + 1) * (case["k"] + 1), max_k=max(16, case["k"]), rows=case["k"] + 1)
        s["ctx"].prefill(r["prompt"])
    elif kind == "batch":
        m, rows = MODELS[case["model"]], case["seqs"] * (case["k"] + 1)
        s["ctx"] = _context(case["model"], case["past"] + (case["steps"] + 1) * (case["k"] + 1), max_batch=case["seqs"], max_k=case["k"], rows=rows)
        for b, p in enumerate(r["prompts"]):
            if case["cache"] == "computed":
                s["ctx"].prefill(p, seq=b)
            else:
                for layer in range(m.n_layers):
                    k, v = _given_kv(m, r["kv_seed"], b, layer, r["pasts"][b])
                    s["ctx"].kv_import(b, layer, k, v, r["pasts"][b])
        s["drafts"] = [np.stack([p[0][i] for p in r["plans"]]) for i in range(case["steps"])]
        torch.cuda.synchronize()
    elif kind == "generate_batch":
        s["ctx"] = _context(case["model"], case["prompt"] + case["max_new"] + case["k"] + 1, max_batch=case["seqs"], max_k=case["k"], rows=case["seqs"] * (case["k"] + 1))
    return s


def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "trigger_host":
        return np.array(llma.llma_find_trigger(s["y"], s["ref"], s["offs"], case["n"]), dtype=np.int32)
    if kind == "trigger_device":
        llma.llma_find_trigger_static(s["y"], s["ref"], s["offs"], case["n"], s["result"])
        return s["result"]
    ctx = s["ctx"]
    if kind == "prompt":                    # up to the first token and its logits
        ctx.reset()
        ctx.prefill(s["prompt"])
        out = ctx.verify_step([])[2]
        return {"tokens": np.array(out, np.int32), "logits": ctx._dump[:1]}
    if kind == "generate":                  # and the logits of the token that would come next
        tokens, trace = ctx.generate(s["prompt"], s["ref"], s["offs"], case["n"], case["k"], case["max_new"])
        more = ctx.verify_step([])[2]
        return {"tokens": tokens, "trace": _whole(trace, case["max_new"], (4,)), "next": np.array(more, np.int32), "logits": ctx._dump[:1]}
    if kind == "steps":                     # from the same point of the sequence each time; logits of the last step
        ctx.truncate(case["past"])
        ctx.set_pending(s["prompt"][-1])
        out = []
        for d in s["drafts"]:
            out += ctx.verify_step(d)[2]
        return {"tokens": _whole(out, case["steps"] * (case["k"] + 1)), "logits": ctx._dump[:case["k"] + 1]}
    if kind == "batch":
        seqs = list(range(case["seqs"]))
        for b in seqs:
            ctx.truncate(s["pasts"][b], seq=b)
            ctx.set_pending(s["prompts"][b][-1], seq=b)
        out = [[] for _ in seqs]
        for d in s["drafts"]:
            emitted = ctx.verify_step_batch(seqs, d)[2]
            for b in seqs:
                out[b] += emitted[b]
        return {"tokens": np.stack([_whole(o, case["steps"] * (case["k"] + 1)) for o in out]), "logits": ctx._dump[:len(seqs) * (case["k"] + 1)]}
    res = ctx.generate_batch(s["prompts"], s["refs"], case["n"], case["k"], case["max_new"])
    seqs = list(range(case["seqs"]))
    ctx.verify_step_batch(seqs, np.zeros((len(seqs), 0), np.int32))
    return {"tokens": np.stack([t for t, _ in res]), "trace": np.stack([_whole(t, case["max_new"], (4,)) for _, t in res]), "logits": ctx._dump[:len(seqs)]}


# ------------------------------------------------------------------------------------------------ what it takes
def _trace(nxt, prompt, ref, offs, y, n, k, max_new):
    """rows fed by each step of the method on these inputs"""
    ref, y, rows, i = ref.tolist(), y.tolist(), [], 0
    doc = np.searchsorted(offs, np.arange(len(ref)), side="right") - 1
    while i < max_new:
        best = None
        for p in range(len(ref)) if i >= n else ():
            pos = p - int(offs[doc[p]])
            if pos < n or ref[p - n:p] != y[i - n:i]:
                continue
            score = n
            while score < min(pos, i) and ref[p - 1 - score] == y[i - 1 - score]:
                score += 1
            if best is None or score > best[0]:
                best = (score, p)
        drafts = []
        if best:
            drafts = ref[best[1]:min(best[1] + k, int(offs[doc[best[1]] + 1]))][:max(0, max_new - i - 1)]
        a = 0
        while a < len(drafts) and drafts[a] == y[i + a]:
            a += 1
        rows.append((i, 1 + len(drafts)))
        i += a + 1
    return rows


def _forward(m, rows, past, head_rows):
    """bytes and operations of one forward: each matrix once, the cache once, the new cache rows, the logits of head_rows rows"""
    w = m.n_layers * m.layer_params
    kv = 2 * m.n_layers * m.d_model
    by = (w + m.vocab * m.d_model * (head_rows > 0)) * m.item + kv * sum(past) * m.item + kv * sum(rows) * m.item + 4 * m.vocab * head_rows
    fl = 2 * (w * sum(rows) + m.vocab * m.d_model * head_rows) + 4 * m.n_layers * m.d_model * sum(r * p + r * (r + 1) / 2 for r, p in zip(rows, past))
    return np.array([by, fl], float)


def work(case):
    kind = case["kind"]
    if kind.startswith("trigger"):
        return {"bytes": 4 * (case["y"] + case["ref"] + case["docs"] + 4), "flops": 0}
    m = MODELS[case["model"]]
    t = np.zeros(2)
    if kind == "prompt":
        if case["prompt"] > 1:
            t += _forward(m, [case["prompt"] - 1], [0], 0)
        t += _forward(m, [1], [case["prompt"] - 1], 1)
    elif kind == "steps":
        for i in range(case["steps"]):
            t += _forward(m, [case["k"] + 1], [case["past"] + i * (1 + case["k"] // 2)], case["k"] + 1)
    elif kind == "batch":
        for i in range(case["steps"]):
            t += _forward(m, [case["k"] + 1] * case["seqs"], [0.8 * case["past"] + 0.2 * case["past"] / case["seqs"] + i * (1 + case["k"] / 2)] * case["seqs"], case["seqs"] * (case["k"] + 1))
    else:                                   # steps as the method takes them on one set of requests
        r = _requests(case, 0)
        one = kind == "generate"
        prompts, refs, ys = ([r["prompt"]], [(r["ref"], r["offs"])], [r["y"]]) if one else (r["prompts"], r["refs"], r["ys"])
        nxt = _weights(case["model"])[1]
        traces = [_trace(nxt, p, *f, y, case["n"], case["k"], case["max_new"]) for p, f, y in zip(prompts, refs, ys)]
        for p in prompts:
            t += _forward(m, [len(p) - 1], [0], 0) if len(p) > 1 else 0
        for i in range(max(len(x) for x in traces)):
            live = [(x[i], p) for x, p in zip(traces, prompts) if i < len(x)]
            t += _forward(m, [x[1] for x, _ in live], [len(p) - 1 + x[0] for x, p in live], sum(x[1] for x, _ in live))
        t += _forward(m, [1] * len(prompts), [len(p) - 1 + case["max_new"] for p in prompts], len(prompts))
    return {"bytes": float(t[0]), "flops": float(t[1])}


def tolerance(case):
    # Trigger positions, tokens, accepted lengths and traces: exact (the favourite leads by far).  Logits, against exact()
    # over 30 cases of these ranges: fp32 model rel 0.9e-7 .. 1.2e-7, max 2.8e-7; bf16 models (activations and caches as
    # bf16 pairs or bf16 + 8 bits, sums in fp32) rel 0.3e-5 .. 8.6e-5, max 3.9e-4.  About four times that.
    if case["kind"].startswith("trigger"):
        return "exact"
    if MODELS[case["model"]].dtype == "fp32":
        return {"rel": 1e-6, "max": 4e-6, "differ": 0.0}
    return {"rel": 3.5e-4, "max": 1.6e-3, "differ": 0.0}


# ------------------------------------------------------------------------------------------------ the same in 64 bits
def _logits64(name, tokens, rows, given=None):
    """float64 logits of the last `rows` positions; tokens: the ids after the given cache (list of (K, V) per layer) if any"""
    m, (w, _) = MODELS[name], _weights(name)
    H, dh, d, f = m.n_heads, m.head_dim, m.d_model, m.d_ffn

    def mat(a):
        t = torch.from_numpy(a).cuda()
        return (t.view(torch.bfloat16) if m.dtype == "bf16" else t).double()

    def norm(x, g):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + m.rms_eps) * torch.from_numpy(g).cuda().double()

    ids = torch.as_tensor(np.asarray(tokens, np.int64), device="cuda")
    R, P = len(ids), given[0][0].shape[1] if given else 0
    pos = torch.arange(P, P + R, device="cuda", dtype=torch.float64)
    ang = pos[:, None] * (m.rope_theta ** (-2.0 * torch.arange(dh // 2, device="cuda", dtype=torch.float64) / dh))[None]
    cos, sin = torch.cos(ang), torch.sin(ang)

    def rot(x):                             # [H, R, dh]
        a, b = x[..., :dh // 2], x[..., dh // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    h = mat(w["embed"])[ids]
    for i, lw in enumerate(w["layers"]):
        qkv = norm(h, lw["norm1"]) @ mat(lw["wqkv"]).T
        q, k, v = (t.reshape(R, H, dh).transpose(0, 1) for t in qkv.split(d, 1))
        q, k = rot(q), rot(k)
        if given:
            k, v = torch.cat([given[i][0].double(), k], 1), torch.cat([given[i][1].double(), v], 1)
        o = torch.empty(R, d, dtype=torch.float64, device="cuda")
        mask = torch.arange(P + R, device="cuda")[None] > (P + torch.arange(R, device="cuda"))[:, None]
        for hh in range(H):
            sc = (q[hh] @ k[hh].T) / math.sqrt(dh)
            o[:, hh * dh:(hh + 1) * dh] = torch.softmax(sc.masked_fill(mask, -math.inf), -1) @ v[hh]
        h = h + o @ mat(lw["wo"]).T
        if i == m.n_layers - 1:
            h = h[-rows:]
        gu = norm(h, lw["norm2"]) @ mat(lw["wgu"]).T
        h = h + (torch.nn.functional.silu(gu[:, :f]) * gu[:, f:]) @ mat(lw["wd"]).T
    return norm(h[-rows:], w["final_norm"]) @ mat(w["lm_head"]).T


def exact(case, seed):
    kind = case["kind"]
    if kind.startswith("trigger"):
        return None
    r, name = _requests(case, seed), case["model"]
    if kind == "prompt":
        return {"tokens": None, "logits": _logits64(name, r["prompt"], 1)}
    if kind == "generate":
        return {"tokens": None, "trace": None, "next": None, "logits": _logits64(name, np.concatenate([r["prompt"], r["y"]]), 1)}

    def history(prompt, plan):              # all tokens before the last step's rows, then those rows
        _, emitted, rows = plan
        upto = [int(t) for t in prompt] + emitted
        last = len(upto) - 1 - upto[::-1].index(rows[0])        # (a cycle of `vocab` tokens: the pending one occurs last here)
        return upto[:last] + rows

    if kind == "steps":
        return {"tokens": None, "logits": _logits64(name, history(r["prompt"], (r["drafts"], r["emitted"], r["rows"])), case["k"] + 1)}
    if kind == "batch":
        m, out = MODELS[name], []
        for b, p in enumerate(r["prompts"]):
            toks, given = history(p, r["plans"][b]), None
            if case["cache"] == "given":
                given = [tuple(_given_kv(m, r["kv_seed"], b, layer, r["pasts"][b])) for layer in range(m.n_layers)]
                toks = toks[len(p) - 1:]
            out.append(_logits64(name, toks, case["k"] + 1, given))
        return {"tokens": None, "logits": torch.cat(out)}
    return {"tokens": None, "trace": None, "logits": torch.cat([_logits64(name, np.concatenate([p, y]), 1) for p, y in zip(r["prompts"], r["ys"])])}
