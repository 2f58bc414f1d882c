"""Performance cases of the SPD library: what a program that uses it has it do, through the public calls.

Three kinds of call, over the sizes the configurations, tests and benchmark of this repository use:

  attn     one ragged paged decode attention (spd_decode_attention, or its form without a workspace);
  steps    decoding: a rollback to the prompt (a regeneration), then `steps` pipeline steps in one logged call,
           with drafts forced to the greedy tokens at an acceptance pattern, greedy or sampled;
  prefill  a new request: a handle over resident weights, the prompt's prefill, its first token, logits and caches.

Weights are N(0, 0.02) in the model's storage type and prompts are uniform, made on the GPU from the seed alone."""
import math
import random

import numpy as np
import torch

import synth
from paper_2605_30852_amd import binding as B
from paper_2605_30852_amd.engine import DeviceWeights, Engine

MODELS = {"tiny": synth.TINY, "mid": synth.MID, "wide": synth.WIDE, "gqa8": synth.GQA8, "mha": synth.MHA,
          "4b": synth.B4, "9b": synth.B9}


# ------------------------------------------------------------------------------------------------ the cases
def _attn(name, rows, keys, hq, hkv, dh, dtype, chunk, noalloc):
    return {"name": name, "kind": "attn", "rows": rows, "keys": keys, "hq": hq, "hkv": hkv, "dh": dh,
            "dtype": dtype, "chunk": chunk, "noalloc": noalloc}


def _steps(name, model, n, ls, prompt, steps, accept, chunk=0, top_k=0, own_head=0, post=False, logits=False):
    return {"name": name, "kind": "steps", "model": model, "n": n, "ls": ls, "prompt": prompt, "steps": steps,
            "accept": accept, "chunk": chunk, "top_k": top_k, "own_head": own_head, "post": post, "logits": logits}


def _prefill(name, model, n, ls, prompt, chunk=0):
    return {"name": name, "kind": "prefill", "model": model, "n": n, "ls": ls, "prompt": prompt, "chunk": chunk}


def listed():
    return [
        # one short row, the smallest call: a serving loop that must not allocate
        _attn("attn_1x300", 1, 300, 8, 2, 64, "bf16", 64, True),
        # the in-flight rows of one layer at the benchmark's 2048-token context and split size
        _attn("attn_4x2051", 4, 2051, 32, 8, 128, "bf16", 128, False),
        # a full pipeline of rows at the long-context configuration
        _attn("attn_8x32776", 8, 32776, 32, 8, 128, "bf16", 2048, False),
        # the CPU-sized fp32 model: launch latency
        _steps("steps_tiny_f32", "tiny", 2, 1, 64, 32, 0.7),
        # the benchmark's headline workload, every draft accepted
        _steps("steps_4b_n4", "4b", 4, 1, 2048, 24, 1.0, chunk=128),
        # plain greedy decoding through the same library (the benchmark's reference decoder)
        _steps("steps_4b_n1", "4b", 1, 1, 300, 12, 1.0, logits=True),
        # a wide pipeline over a two-layer draft module, sampled at the paper's top-k 50, with rejections
        _steps("steps_9b_n8_sampled", "9b", 8, 2, 200, 20, 0.9, top_k=50, logits=True),
        # a long context, eight stages, rejections, the draft module's own head
        _steps("steps_wide_n8_5000", "wide", 8, 2, 5000, 32, 0.6, own_head=2048),
        # a short request to a small model
        _prefill("prefill_mid_45", "mid", 3, 1, 45),
        # an ordinary request to the headline model
        _prefill("prefill_4b_384", "4b", 4, 1, 384),
        # a long one, ragged
        _prefill("prefill_4b_1501", "4b", 4, 1, 1501, chunk=128),
        # a long context: attention counts
        _prefill("prefill_wide_6000", "wide", 5, 2, 6000),
    ]


def draw(rng):
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))

    kind = rng.choice(["attn", "steps", "prefill"])
    if kind == "attn":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        keys = log_int(16, 32776 if dtype == "bf16" else 12000)
        hkv, g = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4, 8])
        smallest = (keys + 63) // 64
        chunk = 16 * rng.randint((smallest + 15) // 16, max((smallest + 15) // 16, min(128, (keys + 15) // 16)))
        c = _attn("", rng.randint(1, 8), keys, hkv * g, hkv, rng.choice([64, 128]), dtype, chunk, False)
        c["noalloc"] = c["rows"] * hkv * ((keys + chunk - 1) // chunk) <= 2048 and rng.random() < 0.5
    else:
        name = rng.choice(["tiny", "mid", "wide", "gqa8", "mha", "4b", "4b", "9b"])
        sh = MODELS[name]
        n, ls = rng.randint(1, min(8, sh.n_layers)), rng.choice([1, 1, 2])
        if kind == "prefill":
            longest = {"4b": 1501, "9b": 800, "wide": 6000, "tiny": 1500}.get(name, 4000)
            c = _prefill("", name, n, ls, log_int(1, longest))
        else:
            longest = {"4b": 600, "9b": 300, "wide": 3000, "tiny": 800}.get(name, 2000)
            own = rng.choice([0, 0, 0, sh.vocab // 4])
            c = _steps("", name, n, ls, log_int(1, longest), rng.randint(n + 4, 12 if name == "9b" else 24), rng.choice([1.0, 0.9, 0.7, 0.5]),
                       top_k=rng.choice([0, 0, 0, 8, 50]), own_head=own, post=rng.random() < 0.15,
                       logits=rng.random() < 0.5)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ inputs
def _shape(case):
    return MODELS[case["model"]].with_(n_stages=case["n"], pdm_layers=case["ls"], pdm_vocab=case.get("own_head", 0))


def _tensors(sh, seed):
    """Every weight of the model by name, on the GPU (norm gains near one, so that they count)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = torch.bfloat16 if sh.dtype == "bf16" else torch.float32
    t = {}
    for name, s in sh.tensor_shapes().items():
        if synth.is_norm(name):
            t[name] = 1.0 + 0.1 * torch.randn(s, generator=g, device="cuda", dtype=torch.float32)
        elif name != "pdm.lm_head":
            t[name] = torch.empty(s, dtype=dt, device="cuda").normal_(0.0, 0.02, generator=g)
    if sh.pdm_vocab:
        ids = np.sort(np.random.RandomState(seed % (1 << 31)).permutation(sh.vocab)[: sh.pdm_vocab])
        t["pdm.vocab_map"] = torch.from_numpy(ids.astype(np.int32)).cuda()
        t["pdm.lm_head"] = t["lm_head"][t["pdm.vocab_map"].long()].contiguous()
    return t


def _weights(sh, seed):
    w = DeviceWeights.__new__(DeviceWeights)
    w.shape, w.seed, w.t = sh, seed, _tensors(sh, seed)
    return w


def _prompt(sh, seed, length):
    return np.random.RandomState((seed + 1) % (1 << 31)).randint(0, sh.vocab, length).astype(np.int32)


def _mask(case):
    """Whether the draft of the i-th position after the first token is forced to the greedy token: one
    pattern for every seed, so that a case always walks through the same pipeline states."""
    return np.random.RandomState(4).random_sample(case["steps"] + 2 * case["n"] + 8) < case["accept"]


def _forced(ref, mask, vocab):
    """Drafts of the positions after the first token: the greedy token, or another one."""
    return [int(t) if m else (int(t) + 1) % vocab for t, m in zip(ref[1:], mask)]


def _attn_inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    pages = (case["keys"] + 15) // 16 + 1
    pool = torch.empty(pages, 2, case["hkv"], 16, case["dh"], dtype=dt, device="cuda").normal_(0.0, 1.0, generator=g)
    q = torch.empty(case["rows"], case["hq"], case["dh"], device="cuda").normal_(0.0, 1.5, generator=g)
    table = torch.from_numpy(np.random.RandomState(seed % (1 << 31)).permutation(pages).astype(np.int32)).cuda()
    # the in-flight rows of neighbouring stages: one key apart, the deepest the shortest
    lens = np.array([max(1, case["keys"] - i) for i in range(case["rows"])], dtype=np.int32)
    return pool, q, table, lens


def _greedy(eng, prompt, need):
    """The prompt's greedy continuation, `need` tokens, from the handle's own decoding."""
    ref = [eng.spd_prefill(prompt)]
    while len(ref) < need:
        at = len(prompt) + len(ref)
        new = [r["verified_token"] for r in eng.spd_run_steps(eng.n, want_log=True) if r["verified_pos"] == at]
        ref += new
        eng.spd_rollback(at, new[0])
    return ref


def prepare(case, seed):
    if case["kind"] == "attn":
        pool, q, table, lens = _attn_inputs(case, seed)
        s = {"case": case, "pool": pool, "q": q, "table": table, "lens": lens, "out": torch.empty_like(q)}
        if not case["noalloc"]:
            s["ws_bytes"] = B.decode_attention_workspace_bytes(case["rows"], case["hkv"], case["dh"], lens, case["chunk"])
            s["ws"] = torch.empty(s["ws_bytes"] + 256, dtype=torch.uint8, device="cuda")
            s["ws_at"] = (s["ws"].data_ptr() + 255) // 256 * 256
        return s
    sh = _shape(case)
    w, prompt = _weights(sh, seed), _prompt(sh, seed, case["prompt"])
    if case["kind"] == "prefill":
        return {"case": case, "w": w, "prompt": prompt, "max_tokens": case["prompt"] + 64}
    n, steps, P = case["n"], case["steps"], case["prompt"]
    need = steps + n + 4  # greedy tokens from position P on
    rows = P + need + 2 * n + 16
    eng = Engine(w, max_tokens=rows, n=n, pdm_layers=case["ls"], attn_chunk=case["chunk"])
    ref = _greedy(eng if not case["top_k"] else
                  Engine(w, max_tokens=rows, n=n, pdm_layers=case["ls"], attn_chunk=case["chunk"]), prompt, need)
    if case["top_k"]:
        u = np.zeros((rows, 3), dtype=np.float32)  # keep what the target gives mass to, else its likeliest token
        u[:, 0] = np.random.RandomState((seed + 3) % (1 << 31)).random_sample(rows) * 0.999
        eng.spd_set_sampling(case["top_k"], 1.0, u)
        assert eng.spd_prefill(prompt) == ref[0]
    eng.spd_set_graph(True)
    eng.spd_set_pdm_schedule(case["post"])
    eng.spd_rollback(P, ref[0])
    eng.spd_set_forced_drafts(_forced(ref, _mask(case), sh.vocab), P + 1)
    eng.spd_set_debug(case["logits"])
    return {"case": case, "w": w, "eng": eng, "first": ref[0]}


# ------------------------------------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    if case["kind"] == "attn":
        bf16 = B.SPD_BF16 if case["dtype"] == "bf16" else B.SPD_F32
        stream = torch.cuda.current_stream().cuda_stream
        args = (state["q"].data_ptr(), state["pool"].data_ptr(), state["table"].data_ptr(), state["pool"].shape[0],
                state["lens"], case["hq"], case["hkv"], case["dh"], bf16, case["chunk"], state["out"].data_ptr())
        if case["noalloc"]:
            B.spd_decode_attention_noalloc(*args, stream)
        else:
            B.spd_decode_attention(*args, state["ws_at"], state["ws_bytes"], stream)
        return state["out"]
    if case["kind"] == "steps":
        eng = state["eng"]
        eng.spd_rollback(case["prompt"], state["first"])
        log = eng.spd_run_steps(case["steps"], want_log=True)
        out = {"decisions": np.array([r["decision"] for r in log], dtype=np.int32),
               "tokens": np.array([r["verified_token"] for r in log], dtype=np.int32),
               "resid": _inflight(eng.resid(), log[-1]["committed_len"], log[-1]["inflight"]),
               "draft_rows": eng.pdm_hidden()[: log[-2]["inflight"]]}
        if case["logits"]:
            out["draft_logits"] = eng.pdm_logits()
            if log[-1]["exited_pos"] >= 0:
                out["logits"] = eng.exit_logits()
        return out
    sh = state["w"].shape
    eng = Engine(state["w"], max_tokens=state["max_tokens"], n=case["n"], pdm_layers=case["ls"],
                 attn_chunk=case["chunk"])
    eng.spd_set_debug(True)
    first = eng.spd_prefill(state["prompt"])
    out = {"first": first, "logits": eng.exit_logits()}
    for name, pdm, layer in (("kv", 0, sh.n_layers - 1), ("draft_kv", 1, case["ls"] - 1)):
        k, v = B.spd_read_kv(eng.h, pdm, layer, 0, case["prompt"], sh.n_kv_heads, sh.head_dim, sh.dtype == "bf16")
        for part, x in (("k", k), ("v", v)):
            x = torch.from_numpy(x.view(np.int16) if sh.dtype == "bf16" else x)
            out[name + "." + part] = x.view(torch.bfloat16) if sh.dtype == "bf16" else x
    eng.close()
    return out


def _inflight(resid, c, a):
    """The residual rows of the in-flight positions c .. c + a - 1 (position q lives in row q mod n)."""
    return resid[[(c + i) % len(resid) for i in range(a)]]


# ------------------------------------------------------------------------------------------------ costs
def _walk(case, ref, mask, vocab):
    """The pipeline's states before each step and after the last, as (c, a, token at each position): the
    staircase fills, the oldest token exits, a wrong successor is replaced and the pipeline refills.
    ref: the greedy tokens from the prompt's end on."""
    P, n = case["prompt"], case["n"]
    drafts = _forced(ref, mask, vocab)
    toks, c, a = {P: ref[0]}, P, 1
    states, log = [(c, a, dict(toks))], []
    for _ in range(case["steps"]):
        q = c + a
        draft = drafts[q - P - 1]
        if a < n:
            toks[q] = draft
            a += 1
            log.append((0, -1))
        else:
            y = ref[c + 1 - P]
            c += 1
            if (toks[c] if n > 1 else draft) == y:
                toks[q] = draft
                log.append((1, y))
            else:
                toks, a = {p: t for p, t in toks.items() if p < c}, 1
                toks[c] = y
                log.append((2, y))
        states.append((c, a, dict(toks)))
    return states, log


def work(case):
    if case["kind"] == "attn":
        e = 2 if case["dtype"] == "bf16" else 4
        lens = [max(1, case["keys"] - i) for i in range(case["rows"])]
        qd = case["hq"] * case["dh"]
        return {"bytes": max(lens) * 2 * case["hkv"] * case["dh"] * e + 8 * case["rows"] * qd,
                "flops": 4 * sum(lens) * qd}
    sh = _shape(case)
    e = 2 if sh.dtype == "bf16" else 4
    d, n, ls, L, P = sh.d_model, case["n"], case["ls"], sh.n_layers, case["prompt"]
    layer = d * (sh.q_dim + 2 * sh.kv_dim) + sh.q_dim * d + 3 * d * sh.ffn_dim  # weights of one layer
    kv = 2 * sh.kv_dim * e                                                      # cache bytes of one key
    head, fc = sh.vocab * d, n * d * d
    if case["kind"] == "prefill":
        pairs = P * (P + 1) // 2
        return {"bytes": ((L + ls) * layer + head + fc) * e + P * ((L + ls) * kv + d * e),
                "flops": 2 * P * ((L + ls) * layer + fc) + 4 * pairs * sh.q_dim * (L + ls) + 2 * head}
    # the pattern of states does not depend on the tokens: any distinct successors give it
    states, _ = _walk(case, list(range(case["steps"] + 2 * n + 4)), _mask(case), 1 << 30)
    bts = fl = 0
    own = sh.pdm_vocab * d
    for c, a, _t in states[:-1]:
        stages = [(s * L // n, (s + 1) * L // n) for s in range(min(a, n))]
        layers = sum(b - t for t, b in stages)
        exits = a == n
        bts += (layers + ls) * layer * e + fc * e + ((head if exits or not own else 0) + own) * e
        bts += (layers + ls) * (c + a) * kv
        fl += 2 * layers * layer + 2 * a * (ls * layer + fc) + 2 * head * (1 if own else 2)
        fl += 4 * (c + a) * sh.q_dim * (layers + a * ls)
    return {"bytes": bts, "flops": fl}


def tolerance(case):
    if case["kind"] == "attn":
        return {"rel": 1e-5, "max": 2e-4}
    if MODELS[case["model"]].dtype == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    # fp32 sums in another order now and then round a stored bf16 key or value the other way, which every
    # layer after it carries on until most stored values sit one rounding apart: up to 4e-3 from the 64-bit
    # result measured over these sizes (2^-8 is one such rounding)
    return {"rel": 1.6e-2, "max": 1e-1, "differ": 1e-3}


# ------------------------------------------------------------------------------------------------ in 64 bits
class _Cache:
    def __init__(self, rows, sh):
        self.k = torch.zeros(rows, sh.n_kv_heads, sh.head_dim, dtype=torch.float64, device="cuda")
        self.v = torch.zeros_like(self.k)


def _norm(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, pos, sh):
    half = sh.head_dim // 2
    inv = sh.rope_base ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / sh.head_dim)
    ang = pos.double()[:, None] * inv
    cos, sin = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)


def _layer(sh, t, pre, x, p0, cache):
    """One decoder layer over rows at positions p0 ..; keys and values are stored in the model's type."""
    r = x.shape[0]
    pos = torch.arange(p0, p0 + r, device="cuda")
    h = _norm(x, t[pre + "attn_norm"], sh.rms_eps)
    mm = lambda a, name: a @ t[pre + name].double().t()  # noqa: E731
    q = _rope(mm(h, "wq").view(r, sh.n_q_heads, sh.head_dim), pos, sh)
    k = _rope(mm(h, "wk").view(r, sh.n_kv_heads, sh.head_dim), pos, sh)
    v = mm(h, "wv").view(r, sh.n_kv_heads, sh.head_dim)
    if sh.dtype == "bf16":
        k, v = k.float().bfloat16().double(), v.float().bfloat16().double()
    cache.k[p0: p0 + r], cache.v[p0: p0 + r] = k, v
    o = torch.empty_like(q)
    G, end = sh.n_q_heads // sh.n_kv_heads, p0 + r
    for g in range(sh.n_kv_heads):
        kk, vv = cache.k[:end, g], cache.v[:end, g]
        for r0 in range(0, r, 1024):
            qq = q[r0: r0 + 1024, g * G: (g + 1) * G]
            m = qq.shape[0]
            s = (qq.reshape(m * G, -1) @ kk.t()).view(m, G, end) / math.sqrt(sh.head_dim)
            s.masked_fill_((torch.arange(end, device="cuda")[None] > pos[r0: r0 + m, None])[:, None, :], -math.inf)
            o[r0: r0 + m, g * G: (g + 1) * G] = (torch.softmax(s, -1).view(m * G, end) @ vv).view(m, G, -1)
    x = x + mm(o.reshape(r, -1), "wo")
    h = _norm(x, t[pre + "mlp_norm"], sh.rms_eps)
    gate = mm(h, "wg")
    return x + mm(gate * torch.sigmoid(gate) * mm(h, "wu"), "wd")


class _Model:
    """The target and the draft module in 64 bits over their own caches."""

    def __init__(self, case, seed, rows):
        self.sh, self.case = _shape(case), case
        self.t = _tensors(self.sh, seed)
        self.caches = [_Cache(rows, self.sh) for _ in range(self.sh.n_layers)]
        self.pdm_caches = [_Cache(rows, self.sh) for _ in range(self.sh.pdm_layers)]
        self.beta = [s * self.sh.n_layers // case["n"] for s in range(case["n"] + 1)]

    def forward(self, toks, p0):
        """The rows' anchors (stage inputs) and the residual after the last layer: [n + 1] of [rows][d]."""
        x = self.t["embed"][torch.as_tensor(np.asarray(toks, dtype=np.int64), device="cuda")].double()
        at = [x]
        for l in range(self.sh.n_layers):
            x = _layer(self.sh, self.t, "layer.%d." % l, x, p0, self.caches[l])
            if l + 1 in self.beta[1:]:
                at.append(x)
        return at

    def head(self, x, norm="final_norm", w="lm_head"):
        return _norm(x, self.t[norm], self.sh.rms_eps) @ self.t[w].double().t()

    def draft(self, at, elig, p0):
        """The draft module over rows at p0 ..; row i sees its first elig[i] anchors."""
        d, n = self.sh.d_model, self.case["n"]
        f = torch.cat([torch.where((torch.as_tensor(elig, device="cuda") > j)[:, None], at[j], 0.0) for j in range(n)], -1)
        x = f @ self.t["pdm.in"].double().t()
        for l in range(self.sh.pdm_layers):
            x = _layer(self.sh, self.t, "pdm.layer.%d." % l, x, p0, self.pdm_caches[l])
        return x


def _exact_attn(case, seed):
    pool, q, table, lens = _attn_inputs(case, seed)
    kv = pool[table.long()].double().permute(1, 2, 0, 3, 4).reshape(2, case["hkv"], -1, case["dh"])
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    G = case["hq"] // case["hkv"]
    for i, n in enumerate(lens.tolist()):
        for g in range(case["hkv"]):
            s = q[i, g * G: (g + 1) * G].double() @ kv[0, g, :n].t() / math.sqrt(case["dh"])
            out[i, g * G: (g + 1) * G] = torch.softmax(s, -1) @ kv[1, g, :n]
    return out


def exact(case, seed):
    with torch.no_grad():
        if case["kind"] == "attn":
            return _exact_attn(case, seed)
        sh = _shape(case)
        if case.get("top_k") and sh.vocab < 50000:
            return None  # a wrong draft is too often among the target's top-k, and is then kept
        P, n = case["prompt"], case["n"]
        m = _Model(case, seed, P + case.get("steps", 0) + 2 * n + 8)
        prompt = _prompt(sh, seed, P)
        at = m.forward(prompt, 0)
        logits = m.head(at[n][-1:])[0]
        if case["kind"] == "prefill":
            out = {"first": None, "logits": logits}
            m.draft(at, [n] * P, 0)
            for name, c in (("kv", m.caches[-1]), ("draft_kv", m.pdm_caches[-1])):
                out[name + ".k"], out[name + ".v"] = c.k[:P], c.v[:P]
            return out
        ref = [int(logits.argmax())]
        rows = [at]
        while len(ref) < case["steps"] + n + 4:
            a1 = m.forward(ref[-1:], P + len(ref) - 1)
            rows.append(a1)
            ref.append(int(m.head(a1[n])[0].argmax()))
        full = [torch.cat([r[j] for r in rows]) for j in range(n + 1)]  # the greedy rows' anchors
        states, log = _walk(case, ref, _mask(case), sh.vocab)
        out = {"decisions": None, "tokens": None}
        # the in-flight rows after the last step: the token at position c + i is a - 1 - i stages deep
        c, a, toks = states[-1]
        at = m.forward([toks[c + i] for i in range(a)], c)
        out["resid"] = torch.stack([at[a - 1 - i][i] for i in range(a)])
        # the draft module's rows of the last step, over the features before it (or after, one stage deeper)
        c, a, toks = states[-2]
        m.draft([f[:c] for f in full], [n] * c, 0)
        at = m.forward([toks[c + i] for i in range(a)], c)
        deep = 1 if case["post"] else 0
        x = m.draft(at, [min(a - 1 - i + deep, n - 1) + 1 for i in range(a)], c)
        out["draft_rows"] = x
        if case["logits"]:
            out["draft_logits"] = m.head(x[-1:], "pdm.norm", "pdm.lm_head" if sh.pdm_vocab else "lm_head")[0]
            if log[-1][0]:
                out["logits"] = m.head(at[n][:1])[0]
        return out
