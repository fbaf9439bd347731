"""Performance cases of the length-prediction path: what a serving system asks
of it, through ``OutletsPredictor``, from one small model call to full batches.

A case is one of three kinds:

``life``
    Requests arrive, get their static prediction (``prefill``), then ``steps``
    dynamic re-predictions (``step``, one generated token each), optionally
    the draft model head's distribution, and leave (``release``).  With
    ``steps`` = 0 it is a prefill batch.
``step``
    One re-prediction of a standing batch whose caches are already filled;
    every pass appends one token per request.
``probe``
    The MLP-probe baseline: its static prediction, ``steps`` updates, release.

Shapes are the repository's own: the tiny fp32 layer and the draft layers of
the 8B (bf16) and 70B (e4m3 weights, bf16 activations) target models.  Lengths
come from the case alone; states, and token ids, from the seed.  The weights
are one fixed random model per shape.
"""
import functools
import math
import random
import types
import zlib

import numpy as np
import torch

from paper_2609_01068_amd.predictor import OutletsPredictor

MODELS = {
    "tiny": dict(d=256, n_q=4, n_kv=2, head_dim=64, ffn=688, head_hidden=128, rope_theta=1e4, vocab=512,
                 rms_eps=1e-5, weight="f32", act="f32", scales=(1.0, 1.0, 1.0)),
    "8b": dict(d=4096, n_q=32, n_kv=8, head_dim=128, ffn=14336, head_hidden=1024, rope_theta=5e5, vocab=128256,
               rms_eps=1e-5, weight="bf16", act="bf16", scales=(1.0, 4.0, 16.0)),
    "70b": dict(d=8192, n_q=64, n_kv=8, head_dim=128, ffn=28672, head_hidden=2048, rope_theta=5e5, vocab=128256,
                rms_eps=1e-5, weight="e4m3", act="bf16", scales=(1.0, 4.0, 16.0)),
}
BIG = ("w_proj", "w_q", "w_k", "w_v", "w_o", "w_gate", "w_up", "w_down", "w_attn_gate", "w_lm")
CHUNK = 32768      # prompt tokens of one cache-filling prefill call of a ``step`` case
GROW = 3072        # tokens a standing batch may grow by before its requests are replaced


def _case(kind, model, requests, lo, hi, lens_seed, median=0, sigma=0.0, **more):
    c = dict(kind=kind, model=model, requests=requests, lo=lo, hi=hi, median=median, sigma=sigma,
             lens_seed=lens_seed, steps=0, hdraft=False, gate=False, embed=False, draft=False, noalloc=False)
    c.update(more)
    return c


def listed():
    return [
        # the fp32 layer, the smallest call there is: latency and launches
        _case("life", "tiny", 4, 16, 64, 0, name="tiny-life-4", steps=8, hdraft=True),
        # one user: a prompt, then its length predicted again after each token
        _case("life", "8b", 1, 777, 777, 0, name="8b-life-1", steps=8, hdraft=True),
        # a small serving batch of short chat prompts
        _case("life", "8b", 24, 9, 50, 1, name="8b-life-24", steps=8),
        # a middle-sized serving batch of short chat prompts
        _case("life", "8b", 130, 9, 50, 2, name="8b-life-130", steps=8, hdraft=True),
        # a prompt batch of a prefill instance, ragged lengths
        _case("life", "8b", 32, 32, 4096, 0, 512, 1.0, name="8b-prefill-32"),
        # a saturated prefill instance: everything that fits one call
        _case("life", "8b", 256, 16, 8192, 0, 1024, 1.2, name="8b-prefill-256"),
        # a full decode instance: 512 requests in flight, 2.2M cached tokens
        _case("step", "8b", 512, 256, 8192, 0, name="8b-step-512", hdraft=True),
        # a few requests with long caches, in a loop that must not allocate
        _case("step", "8b", 6, 3000, 16000, 3, name="8b-step-6-long", hdraft=True, noalloc=True),
        # every optional part: output gate, input embeddings, draft model head
        _case("life", "8b", 11, 60, 2000, 4, 400, 0.9, name="8b-options-11", steps=2, hdraft=True, gate=True,
              embed=True, draft=True),
        # the 70B layer with e4m3 weights, a large prompt batch
        _case("life", "70b", 64, 64, 16384, 0, 2048, 1.0, name="70b-prefill-64"),
        # the 70B layer re-predicting a middle-sized serving batch
        _case("life", "70b", 40, 9, 50, 5, name="70b-life-40", steps=6, hdraft=True),
        # the baseline predictor on a prompt batch
        _case("probe", "8b", 32, 32, 4096, 0, 512, 1.0, name="8b-probe-32", steps=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["life", "life", "prefill", "prefill", "step", "probe", "tiny", "70b"])
    seed = rng.randrange(1 << 30)
    if kind == "tiny":
        return _case("life", "tiny", _log(rng, 1, 24), 1, _log(rng, 8, 100), seed, steps=rng.randint(0, 8),
                     hdraft=rng.random() < 0.5, gate=rng.random() < 0.25)
    if kind == "step":
        n = _log(rng, 1, 512)
        hi = _log(rng, 200, 8192)
        return _case("step", "8b", n, rng.randint(1, hi), hi, seed, hdraft=rng.random() < 0.5,
                     noalloc=rng.random() < 0.3)
    if kind == "life":      # decoding: short prompts, several steps
        n = _log(rng, 1, 512)
        return _case("life", "8b", n, 1, rng.randint(4, 60), seed, steps=rng.randint(2, 8),
                     hdraft=rng.random() < 0.5, gate=rng.random() < 0.2)
    if kind == "70b":
        n = _log(rng, 1, 64)
        return _case("life", "70b", n, 1, _log(rng, 20, 3000), seed, steps=rng.randint(0, 3),
                     hdraft=rng.random() < 0.5)
    n = _log(rng, 1, 128)
    lo, hi = _log(rng, 1, 64), _log(rng, 100, 8192)
    med = max(lo, hi // 6)
    if kind == "probe":
        return _case("probe", "8b", n, lo, hi, seed, med, 1.0, steps=rng.randint(0, 3))
    return _case("life", "8b", n, lo, hi, seed, med, 1.0, steps=rng.randint(0, 1), hdraft=rng.random() < 0.5,
                 gate=rng.random() < 0.2, embed=rng.random() < 0.2)


# ---------------------------------------------------------------- inputs

def _shape(case):
    m = MODELS[case["model"]]
    return m, types.SimpleNamespace(**m)


@functools.lru_cache(maxsize=None)
def _lens(n, lo, hi, median, sigma, seed):
    r = random.Random(seed)
    if not sigma:
        return tuple(r.randint(lo, hi) for _ in range(n))
    return tuple(int(min(hi, max(lo, round(math.exp(r.gauss(math.log(median), sigma)))))) for _ in range(n))


def _lengths(case):
    return _lens(*(case[k] for k in ("requests", "lo", "hi", "median", "sigma", "lens_seed")))


def _weight_shapes(case):
    m, _ = _shape(case)
    d, q, kv, h1 = m["d"], m["n_q"] * m["head_dim"], m["n_kv"] * m["head_dim"], m["head_hidden"]
    ka = 2 * d if case["embed"] else d
    s = dict(w_proj=(d, 3 * d), w_q=(q, ka), w_k=(kv, ka), w_v=(kv, ka), w_o=(d, q), w_gate=(m["ffn"], d),
             w_up=(m["ffn"], d), w_down=(d, m["ffn"]), gamma_attn=(d,), gamma_mlp=(d,), gamma_final=(d,),
             head_w1=(h1, 2 * d), head_b1=(h1,), head_w2=(h1,), head_b2=(1,))
    if case["gate"]:
        s["w_attn_gate"] = (q, ka)
    if case["draft"]:
        s["w_lm"] = (m["vocab"], d)
    if case["embed"]:
        s["embed"], s["gamma_emb"] = (m["vocab"], d), (d,)
    if case["kind"] == "probe":
        s.update(probe_w1=(h1, 2 * d), probe_b1=(h1,), probe_w2=(h1,), probe_b2=(1,))
    return s


@functools.lru_cache(maxsize=None)
def _weight(model, name, shape):
    """One weight of the model as the predictor takes it: a host array, or
    (codes, row scales) for e4m3."""
    fmt = MODELS[model]["weight"]
    g = torch.Generator(device="cuda")
    g.manual_seed(zlib.crc32(("%s %s %s" % (model, name, shape)).encode()))
    x = torch.randn(shape, generator=g, device="cuda") * 0.02
    if name.startswith("gamma"):
        x = 1.0 + x
    if fmt == "f32":
        return x.cpu().numpy()
    if fmt == "e4m3" and name in BIG:
        s = (x.abs().amax(dim=1) / 448.0).to(torch.bfloat16)
        codes = (x / s.float()[:, None]).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
        return codes.view(torch.uint8).cpu().numpy(), s.view(torch.int16).cpu().numpy().view(np.uint16)
    return x.to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)


def _weights(case):
    return {k: _weight(case["model"], k, s) for k, s in _weight_shapes(case).items()}


def _states(case, seed, stream, rows):
    """Target-model states of `rows` tokens at the three depths."""
    m, _ = _shape(case)
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + stream) & 0x7FFFFFFFFFFF)
    dt = torch.float32 if m["act"] == "f32" else torch.bfloat16
    out = [torch.empty((rows, m["d"]), dtype=dt, device="cuda") for _ in m["scales"]]
    for r in range(0, rows, CHUNK):
        for x, scale in zip(out, m["scales"]):
            n = min(CHUNK, rows - r)
            x[r:r + n] = torch.randn((n, m["d"]), generator=g, device="cuda") * scale
    return out


def _tokens(case, seed, stream, rows):
    if not case["embed"]:
        return None
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + 500_000 + stream) & 0x7FFFFFFFFFFF)
    return torch.randint(0, MODELS[case["model"]]["vocab"], (rows,), generator=g, device="cuda", dtype=torch.int32)


def _calls(case):
    """The prefill calls that admit the case's requests: [(first, end)]."""
    lens, calls = _lengths(case), []
    if case["kind"] != "step":
        return [(0, len(lens))]
    i = 0
    while i < len(lens):
        j, t = i, 0
        while j < len(lens) and (j == i or t + lens[j] <= CHUNK):
            t += lens[j]
            j += 1
        calls.append((i, j))
        i = j
    return calls


def _admit(s):
    case, lens = s["case"], _lengths(s["case"])
    for i, j in _calls(case):
        x = _states(case, s["seed"], i, sum(lens[i:j]))
        s["pred"].prefill(list(range(i, j)), lens[i:j], *x)
    s["left"] = GROW


def prepare(case, seed):
    m, shape = _shape(case)
    lens, n = _lengths(case), case["requests"]
    grow = GROW if case["kind"] == "step" else case["steps"]
    batch = max(max(sum(lens[i:j]) for i, j in _calls(case)), n)
    pred = OutletsPredictor(
        shape, m["weight"], m["act"], _weights(case), max_slots=n, max_seq_len=max(lens) + grow,
        num_pages=sum((x + grow + 15) // 16 for x in lens), max_batch_tokens=batch, max_batch_requests=n)
    s = dict(case=case, seed=seed, pred=pred, slots=list(range(n)), lens=list(lens))
    if case["kind"] == "step":
        _admit(s)
    else:
        s["prompt"] = _states(case, seed, 0, sum(lens))
        s["prompt_tokens"] = _tokens(case, seed, 0, sum(lens))
    steps = 1 if case["kind"] == "step" else case["steps"]
    s["steps"] = [(_states(case, seed, 1000 + k, n), _tokens(case, seed, 1000 + k, n)) for k in range(steps)]
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    case, pred, slots = s["case"], s["pred"], s["slots"]
    if case["kind"] == "probe":
        z = [pred.probe_prefill(slots, s["lens"], s["prompt"][1])]
        z += [pred.probe_step(slots, x[1]) for x, _ in s["steps"]]
        pred.probe_release(slots)
        return {"z": z}
    hd = case["hdraft"]
    if case["kind"] == "step":
        if s["left"] == 0:          # every request has reached its end: new ones take their place
            pred.release(slots)
            _admit(s)
        s["left"] -= 1
        z, h = pred.step(slots, *s["steps"][0][0], want_hdraft=hd, noalloc=case["noalloc"])
        return {"z": [z], "h": [h]}
    z, h = pred.prefill(slots, s["lens"], *s["prompt"], want_hdraft=hd, tokens=s["prompt_tokens"])
    out = {"z": [z], "h": [h], "p": []}
    for x, tok in s["steps"]:
        z, h = pred.step(slots, *x, want_hdraft=hd, tokens=tok, noalloc=case["noalloc"])
        out["z"].append(z)
        out["h"].append(h)
    if case["draft"]:
        out["p"].append(pred.draft_distribution(len(slots)))
    pred.release(slots)
    return out


# ---------------------------------------------------------------- work and tolerance

def work(case):
    m, _ = _shape(case)
    lens, n = _lengths(case), case["requests"]
    T, d, q, kv = sum(lens), m["d"], m["n_q"] * m["head_dim"], m["n_kv"] * m["head_dim"]
    wb, ab = {"f32": 4, "bf16": 2, "e4m3": 1}[m["weight"]], 4 if m["act"] == "f32" else 2
    h1 = m["head_hidden"]
    head_b, head_f = 2 * d * h1 * (4 if wb == 4 else 2), 2 * 2 * d * h1 * n
    if case["kind"] == "probe":
        return {"bytes": T * d * ab + head_b + case["steps"] * (n * d * (ab + 8) + head_b),
                "flops": T * d + (1 + case["steps"]) * head_f}
    ka = 2 * d if case["embed"] else d
    params = 3 * d * d + (q + 2 * kv + (q if case["gate"] else 0)) * ka + d * q + 3 * d * m["ffn"]

    def call(tokens, cached, pairs):
        byt = params * wb + head_b + tokens * (3 * d + 2 * kv + (d if case["hdraft"] else 0)) * ab
        byt += tokens * (d * ab + 4) * (1 if case["embed"] else 0) + cached * 2 * kv * ab + n * 4
        return byt, 2 * params * tokens + 4 * q * pairs + head_f

    total = [0, 0]

    def add(c):
        total[0] += c[0]
        total[1] += c[1]

    if case["kind"] == "life":
        add(call(T, 0, sum(x * (x + 1) // 2 for x in lens)))
    for k in range(1 if case["kind"] == "step" else case["steps"]):
        add(call(n, T + k * n, T + (k + 1) * n))
    if case["draft"]:
        add((m["vocab"] * d * wb + 4 * n * m["vocab"], 2 * n * m["vocab"] * d))
    return {"bytes": total[0], "flops": total[1]}


def tolerance(case):
    """About four times the error seen against 64 bits where an output has
    many elements, with room for a single z near zero: fp32 layer 5e-7 to
    8e-7, probe (its input kept to 16 mantissa bits) 2e-7 to 7e-7, bf16
    activations 1.7e-3 to 1.9e-3 (h_draft) and up to 1.0e-3 (z)."""
    if MODELS[case["model"]]["act"] == "f32":
        return {"rel": 1e-5}
    if case["kind"] == "probe":
        return {"rel": 2e-5}
    return {"rel": 8e-3}


# ---------------------------------------------------------------- the same in 64 bits

def _wide(model, name, shape):
    w = _weight(model, name, shape)
    if isinstance(w, tuple):
        codes = torch.from_numpy(w[0]).cuda().view(torch.float8_e4m3fn).float().double()
        return codes * torch.from_numpy(w[1].view(np.int16)).view(torch.bfloat16).cuda().double()[:, None]
    t = torch.from_numpy(w if w.dtype == np.float32 else w.view(np.int16)).cuda()
    return t.double() if w.dtype == np.float32 else t.view(torch.bfloat16).double()


class _Exact:
    def __init__(self, case):
        self.case, (self.m, _) = case, _shape(case)
        self.w = {k: _wide(case["model"], k, s) for k, s in _weight_shapes(case).items()}
        self.cache, self.sum, self.count = {}, {}, {}

    def norm(self, x, gamma):
        return x / torch.sqrt((x * x).mean(dim=1, keepdim=True) + self.m["rms_eps"]) * self.w[gamma]

    def rope(self, x, pos):
        half = self.m["head_dim"] // 2
        ang = pos.double()[:, None] * self.m["rope_theta"] ** (-torch.arange(half, device="cuda").double() / half)
        c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * c - b * s, b * c + a * s], dim=-1)

    def attend(self, q, k, v, first):
        """q [t, n_q, hd] at positions first.. over k, v [n, n_kv, hd]."""
        n_kv, hd = self.m["n_kv"], self.m["head_dim"]
        G = self.m["n_q"] // n_kv
        kt, vt = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()
        out = torch.empty_like(q)
        step = max(1, min(512, (1 << 28) // (self.m["n_q"] * max(1, len(k)))))
        for t in range(0, len(q), step):
            u = q[t:t + step]
            n = first + t + len(u)
            s = torch.matmul(u.reshape(len(u), n_kv, G, hd).permute(1, 2, 0, 3).reshape(n_kv, -1, hd),
                             kt[:, :, :n]) / math.sqrt(hd)
            s = s.reshape(n_kv, G, len(u), n)
            late = torch.arange(n, device="cuda")[None, :] > torch.arange(first + t, n, device="cuda")[:, None]
            p = torch.softmax(s.masked_fill(late, -math.inf), dim=-1).reshape(n_kv, -1, n)
            o = torch.matmul(p, vt[:, :n]).reshape(n_kv, G, len(u), hd)
            out[t:t + step] = o.permute(2, 0, 1, 3).reshape(len(u), n_kv * G, hd)
        return out

    def rows(self, x, tokens, reqs, lens, every):
        """The layer over packed rows; h_draft of each, or None when only
        their keys and values are wanted."""
        w, m = self.w, self.m
        starts = [self.count.get(r, 0) for r in reqs]
        pos = torch.cat([torch.arange(s, s + n, device="cuda") for s, n in zip(starts, lens)])
        f = torch.cat([t.double() for t in x], dim=1) @ w["w_proj"].T
        a = self.norm(f, "gamma_attn")
        if self.case["embed"]:
            e = w["embed"][tokens.long()]
            a = torch.cat([self.norm(e, "gamma_emb"), a], dim=1)
        k = self.rope((a @ w["w_k"].T).reshape(-1, m["n_kv"], m["head_dim"]), pos)
        v = (a @ w["w_v"].T).reshape(-1, m["n_kv"], m["head_dim"])
        at = 0
        spans = []
        for r, n in zip(reqs, lens):
            old = self.cache.get(r)
            new = (k[at:at + n], v[at:at + n])
            self.cache[r] = tuple(torch.cat([o, y]) for o, y in zip(old, new)) if old else new
            spans.append((at, at + n))
            at += n
        for r, n in zip(reqs, lens):
            self.count[r] = self.count.get(r, 0) + n
        if not every:
            return None
        q = self.rope((a @ w["w_q"].T).reshape(-1, m["n_q"], m["head_dim"]), pos)
        o = torch.empty_like(q)
        for r, s, (b, e) in zip(reqs, starts, spans):
            o[b:e] = self.attend(q[b:e], *self.cache[r], s)
        o = o.reshape(len(o), -1)
        if self.case["gate"]:
            o = o * torch.sigmoid(a @ w["w_attn_gate"].T)
        x1 = f + o @ w["w_o"].T
        b = self.norm(x1, "gamma_mlp")
        x2 = x1 + (torch.nn.functional.silu(b @ w["w_gate"].T) * (b @ w["w_up"].T)) @ w["w_down"].T
        return self.norm(x2, "gamma_final")

    def head(self, h, reqs, lens, counts, prefix="head"):
        w, rows, at = self.w, [], 0
        for r, n, c in zip(reqs, lens, counts):
            self.sum[r] = self.sum.get(r, 0) + h[at:at + n].sum(dim=0)
            at += n
            rows.append(torch.cat([self.sum[r] / c, h[at - 1]]))
        y = torch.relu(torch.stack(rows) @ w[prefix + "_w1"].T + w[prefix + "_b1"])
        return y @ w[prefix + "_w2"] + w[prefix + "_b2"]


def exact(case, seed):
    lens, n = _lengths(case), case["requests"]
    everyone, ones = list(range(n)), [1] * n
    full = work(case)["flops"] < 6e14 if case["kind"] != "step" else sum(lens) < 200_000
    E = _Exact(case)
    if case["kind"] == "probe":
        h, out, count = _states(case, seed, 0, sum(lens))[1], [], list(lens)
        for k in range(case["steps"] + 1):
            out.append(E.head(h.double(), everyone, lens if k == 0 else ones, count, "probe"))
            if k < case["steps"]:
                h, count = _states(case, seed, 1000 + k, n)[1], [c + 1 for c in count]
        return {"z": out}
    if not full and case["kind"] == "life":
        return None
    out = {"z": [], "h": [], "p": []}
    keep = case["hdraft"]
    if case["kind"] == "step":
        for i, j in _calls(case):
            h = E.rows(_states(case, seed, i, sum(lens[i:j])), None, everyone[i:j], lens[i:j], full)
            if full:
                E.head(h, everyone[i:j], lens[i:j], lens[i:j])
        h = E.rows(_states(case, seed, 1000, n), None, everyone, ones, True)
        z = E.head(h, everyone, ones, [x + 1 for x in lens]) if full else None
        return {"z": [z], "h": [h if keep else None]}
    x, tok = _states(case, seed, 0, sum(lens)), _tokens(case, seed, 0, sum(lens))
    parts, at, i = [], 0, 0
    while i < n:            # the prompts, some thousand rows at a time
        j, t = i, 0
        while j < n and (j == i or t + lens[j] <= CHUNK // 2):
            t += lens[j]
            j += 1
        h = E.rows([y[at:at + t] for y in x], None if tok is None else tok[at:at + t], everyone[i:j], lens[i:j], True)
        parts.append((E.head(h, everyone[i:j], lens[i:j], lens[i:j]), h if keep else None))
        if not case["steps"]:
            for r in everyone[i:j]:
                del E.cache[r]
        at, i = at + t, j
    out["z"].append(torch.cat([p[0] for p in parts]))
    out["h"].append(torch.cat([p[1] for p in parts]) if keep else None)
    for k in range(case["steps"]):
        h = E.rows(_states(case, seed, 1000 + k, n), _tokens(case, seed, 1000 + k, n), everyone, ones, True)
        out["z"].append(E.head(h, everyone, ones, [x + k + 1 for x in lens]))
        out["h"].append(h if keep else None)
    if case["draft"]:
        out["p"].append(torch.softmax(h @ E.w["w_lm"].T, dim=1))      # of the newest step
    return out
