"""Workloads of the multi-byte-prediction decoder, for timing and comparing builds.

Every case is one request served whole, through the public entry points: prefill a batch
of prompts and decode (threshold acceptance, sampled, or with verification), or the
full-sequence forward with its losses.  Shapes are those of the repository's workloads
(a tiny float32 model, d = 1024 models with the LCA head, the MLP head, learned
boundaries or no MB head, and a d = 2048 model) at batch sizes 1 to 64.

A program that serves requests loads its weights and creates its handle once, so both
are kept here per model and capacity; prompts, continuations, drafts and uniforms come
from the seed.  Decoding is fed with a given continuation (accept's override), 1..n bytes
per step, each further byte with probability one half: two correct builds then stay on
the same bytes even where two candidates are nearly equal.  Only the verification cases
commit what the model accepts, which is sure there: the unembedding makes the model
prefer one successor of every byte by a wide margin.
"""
from __future__ import annotations

import ctypes
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2608_15454_amd import SELF_VERIFY, THRESHOLD, Decoder, make_config, weight_manifest

SPACE, EPS, ROPE_BASE, MAX_PATCH = 0x20, 1e-6, 1e5, 16
TAU = 0.75
TEMPERATURE, TOP_P = 0.7, 0.9
EXACT_MAX_FLOPS = 3.5e14  # about 10 s of float64 products


def _arch(d, heads, enc, lm, nb, mb, head="lca", dtype="bf16", boundary="space"):
    return dict(d_model=d, n_heads=heads, d_ff=4 * d, n_enc=enc, n_lm=lm, n_nb=nb, n_mb=mb, head=head, dtype=dtype,
                rope_base=ROPE_BASE, rms_eps=EPS, attn_scale=1.0, max_patch=MAX_PATCH, window_mode=0, boundary=boundary)


MODELS = {
    "tiny_f32": _arch(128, 4, 1, 2, 1, 1, dtype="f32"),
    "small_f32": _arch(256, 4, 2, 2, 2, 2, dtype="f32"),
    "lca_d1024": _arch(1024, 16, 2, 16, 2, 2),
    "mlp_d1024": _arch(1024, 16, 2, 16, 2, 3, head="mlp"),
    "fxt_d1024": _arch(1024, 16, 2, 16, 4, 0),
    "learned_d1024": _arch(1024, 16, 2, 16, 2, 2, boundary="learned"),
    "lca_d2048": _arch(2048, 32, 2, 16, 2, 2),
}


def listed():
    return [
        # the smallest call: float32 weights, per-kernel path, launches and host work
        dict(name="tiny_f32_b1", kind="generate", model="tiny_f32", batch=1, prompt=256, n=3, steps=16),
        # one user, long prompt: latency of the first bytes, then of every step
        dict(name="prompt_b1", kind="generate", model="lca_d1024", batch=1, prompt=3001, n=3, steps=0),
        dict(name="generate_b1", kind="generate", model="lca_d1024", batch=1, prompt=4096, n=3, steps=64),
        # the parameter-matched baseline head, and segments from the boundary predictor
        dict(name="mlp_b1", kind="generate", model="mlp_d1024", batch=1, prompt=1024, n=3, steps=32),
        dict(name="learned_b1", kind="generate", model="learned_d1024", batch=1, prompt=1024, n=3, steps=24),
        # a few users, sampled decoding at the settings of an instruction-following task
        dict(name="sampled_b8", kind="sampled", model="lca_d1024", batch=8, prompt=777, n=5, steps=24),
        # a full server: decoding short requests, and taking in long prompts
        dict(name="generate_b64", kind="generate", model="lca_d1024", batch=64, prompt=512, n=5, steps=32),
        dict(name="prompt_b64", kind="generate", model="lca_d1024", batch=64, prompt=2048, n=5, steps=0),
        # drafts checked by a next-byte model, and by the model itself at d = 2048
        dict(name="extverify_b1", kind="external", model="fxt_d1024", batch=1, prompt=2048, n=7, steps=24),
        dict(name="selfverify_d2048_b16", kind="selfverify", model="lca_d2048", batch=16, prompt=2048, n=7, steps=16),
        # scoring a whole sequence: both heads at every position and the losses
        dict(name="forward_t4096", kind="forward", model="lca_d1024", batch=1, prompt=4096, n=0, steps=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["generate"] * 5 + ["sampled", "external", "selfverify", "forward", "forward"])
    if kind == "forward":
        model = rng.choice(["lca_d1024", "lca_d1024", "learned_d1024", "fxt_d1024", "small_f32"])
        return dict(kind=kind, model=model, batch=1, prompt=_log_int(rng, 64, 6000), n=0, steps=0)
    if kind == "external":
        return dict(kind=kind, model="fxt_d1024", batch=_log_int(rng, 1, 8), prompt=_log_int(rng, 64, 3000),
                    n=rng.randint(1, 7), steps=rng.randint(4, 24))
    if kind == "selfverify":
        return dict(kind=kind, model=rng.choice(["lca_d2048", "lca_d1024"]), batch=_log_int(rng, 1, 16),
                    prompt=_log_int(rng, 64, 2048), n=rng.randint(2, 8), steps=rng.randint(4, 12))
    model = rng.choice(["lca_d1024"] * 4 + ["mlp_d1024", "learned_d1024", "lca_d2048", "small_f32", "tiny_f32"])
    small = model in ("tiny_f32", "small_f32")
    batch = _log_int(rng, 1, 16 if small or model == "lca_d2048" else 64)
    most = 512 if model == "tiny_f32" else 1024 if model in ("small_f32", "lca_d2048") else 4096 if batch <= 16 else 2048
    n = rng.randint(2, 4) if model == "mlp_d1024" else rng.randint(2, 8)
    steps = 0 if kind == "generate" and rng.random() < 0.3 else rng.randint(8, 32)
    return dict(kind=kind, model=model, batch=batch, prompt=_log_int(rng, 40, most), n=n, steps=steps)


# ------------------------------------------------------------------ what a program keeps
_weights, _decoders = {}, {}
_PERM = None


def _successor():
    """The byte the model prefers after every byte: a permutation whose cycle through the
    space has six bytes, so that text that follows it has words of five letters."""
    global _PERM
    if _PERM is None:
        order = np.random.default_rng(7).permutation([b for b in range(256) if b != SPACE])
        _PERM = np.zeros(256, dtype=np.uint8)
        for cycle in ([SPACE] + [int(b) for b in order[:5]], [int(b) for b in order[5:]]):
            for a, b in zip(cycle, cycle[1:] + cycle[:1]):
                _PERM[a] = b
    return _PERM


def _word():
    """The bytes of the space's cycle."""
    s, out = _successor(), [SPACE]
    while s[out[-1]] != SPACE:
        out.append(int(s[out[-1]]))
    return out


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _weights_of(name):
    """Random weights of the architecture, N(0, 0.02^2) and norm gains around 1, with an
    embedding the states keep hold of and an unembedding that reads it back as the
    successor byte; the boundary predictor looks for the space."""
    if name in _weights:
        return _weights[name]
    m = MODELS[name]
    d = m["d_model"]
    emb_std = 1.5 if d <= 1024 else 6.0  # the blocks add more to the states of wider models
    g = torch.Generator(device=_device()).manual_seed(20)
    rand = lambda *shape: torch.randn(*shape, generator=g, device=_device())  # noqa: E731
    out = {}
    for key, (rows, cols) in weight_manifest(make_config(SimpleNamespace(**m), max_batch=1, max_ctx=64)):
        if key == "emb":
            w = rand(rows, cols) * emb_std
            emb = w.bfloat16().float()
        elif key == "unembed":
            w = rand(rows, cols) * 0.02
            w[torch.from_numpy(_successor().astype(np.int64)).to(w.device)] += emb * (18.0 / (d * emb_std))
        elif key == "bp.w":
            w = (emb[SPACE] * (8.0 / (0.65 * math.sqrt(d) * float(emb[SPACE].norm())))).reshape(rows, cols)
        elif key == "bp.b":
            w = torch.full((rows, cols), -4.0, device=_device())
        elif key.endswith("norm"):
            w = 1.0 + 0.2 * (2.0 * torch.rand(rows, cols, generator=g, device=_device()) - 1.0)
        else:
            w = rand(rows, cols) * 0.02
        if m["dtype"] == "bf16":
            w = w.bfloat16().float()
        out[key] = w.cpu().numpy()
    _weights[name] = out
    return out


def _decoder(case):
    m = MODELS[case["model"]]
    max_ctx = case["prompt"] + (case["steps"] + 1) * (case["n"] + 1) + 8
    key = (case["model"], case["batch"], max_ctx)
    if key not in _decoders:
        cfg = make_config(SimpleNamespace(**m), max_batch=case["batch"], max_ctx=max_ctx, max_n=8)
        _decoders[key] = Decoder(cfg, _weights_of(case["model"]))
    return _decoders[key]


# ------------------------------------------------------------------------------- inputs
def _text(rng, length):
    """Bytes that are a space with probability 1/6, else Zipf(1.1) over the others."""
    p = np.arange(1, 256, dtype=np.float64) ** -1.1
    others = np.random.default_rng(77).permutation([b for b in range(256) if b != SPACE])
    out = others[rng.choice(255, size=length, p=p / p.sum())]
    out[rng.random(length) < 1.0 / 6.0] = SPACE
    return out.astype(np.uint8)


def _inputs(case, seed):
    """Prompts (rows of a batch of several differ in length, down to half), and per step
    the continuation's bytes and counts, or the drafts of an external verification."""
    rng = np.random.default_rng(int(seed))
    B, T, n, steps, word, succ = case["batch"], case["prompt"], case["n"], case["steps"], _word(), _successor()
    prompts = []
    for _ in range(B):
        length = T if B == 1 else int(rng.integers((T + 1) // 2, T + 1))
        x = _text(rng, length)
        if case["kind"] in ("external", "selfverify"):
            x[-1] = word[int(rng.integers(len(word)))]
        prompts.append(x)
    got = SimpleNamespace(prompts=prompts)
    if case["kind"] in ("generate", "sampled"):
        got.counts = np.minimum(n, rng.geometric(0.5, size=(steps, B))).astype(np.int32)
        got.bytes = np.zeros((steps, B, 8), dtype=np.uint8)
        for i in range(steps):
            for b in range(B):
                got.bytes[i, b, : got.counts[i, b]] = _text(rng, int(got.counts[i, b]))
        if case["kind"] == "sampled":
            got.uniforms = rng.random((steps + 1, B, 3 * n), dtype=np.float32)
    elif case["kind"] == "external":
        # drafts that agree with the verifier for 0..n bytes, then do not
        got.drafts = np.zeros((steps, B, n), dtype=np.uint8)
        got.seqs = [[] for _ in range(B)]  # what is committed before each round
        for b in range(B):
            x = [int(v) for v in prompts[b]]
            for i in range(steps):
                got.seqs[b].append(list(x))
                good = min(n, int(rng.geometric(0.3)) - 1)
                got.drafts[i, b] = rng.integers(0, 256, size=n)
                for k in range(good):
                    x.append(int(succ[x[-1]]))
                    got.drafts[i, b, k] = x[-1]
                if good < n:
                    got.drafts[i, b, good] = (int(succ[x[-1]]) + int(rng.integers(1, 256))) % 256
                x.append(int(succ[x[-1]]))  # the verifier's own byte after the kept drafts
    return got


def prepare(case, seed):
    dec = _decoder(case)
    s = _inputs(case, seed)
    s.case, s.dec = case, dec
    B, n, steps, dev = case["batch"], case["n"], case["steps"], dec.device
    if case["kind"] == "forward":
        s.work = torch.empty(dec.L.mbp_forward_workspace_bytes(ctypes.byref(dec.cfg), case["prompt"]), dtype=torch.uint8,
                             device=dev)
        return s
    rounds = steps if case["kind"] == "external" else steps + 1
    rows = n + 1 if case["kind"] == "external" else n
    s.logits = torch.zeros((rounds, B, rows, 256), dtype=torch.float32, device=dev)
    s.cand = torch.zeros((rounds, B, rows), dtype=torch.uint8, device=dev)
    s.prob = torch.zeros((rounds, B, rows), dtype=torch.float32, device=dev)
    s.lens = torch.zeros((rounds, B), dtype=torch.int32, device=dev)
    if case["kind"] == "external":
        s.drafts = torch.from_numpy(s.drafts).to(dev)
    if case["kind"] == "sampled":
        s.uniforms = torch.from_numpy(s.uniforms).to(dev)
    return s


# ---------------------------------------------------------------------------- one request
def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def run(state):
    s, dec, case = state, state.dec, state.case
    kind, n, steps = case["kind"], case["n"], case["steps"]
    if kind == "forward":
        nll, loss = dec.forward(s.prompts[0], work=s.work)
        return {"nll": nll, "loss": loss}
    L, h = dec.L, dec.h
    dec.prefill(s.prompts)
    if kind == "external":
        for i in range(steps):
            dec._check(L.mbp_verify_draft(h, _ptr(s.drafts[i]), n, _ptr(s.cand[i]), _ptr(s.lens[i])))
            dec._check(L.mbp_get_logits(h, _ptr(s.logits[i])))
            dec.accept()
        return {"logits": s.logits, "bytes": s.cand, "lens": s.lens}
    for i in range(steps + 1):
        out = _ptr(s.cand[i]), _ptr(s.prob[i]), _ptr(s.lens[i])
        if kind == "sampled":
            dec._check(L.mbp_decode_step_sampled(h, n, TAU, THRESHOLD, TEMPERATURE, TOP_P, _ptr(s.uniforms[i]), *out))
        else:
            dec._check(L.mbp_decode_step(h, n, TAU, SELF_VERIFY if kind == "selfverify" else THRESHOLD, *out))
        dec._check(L.mbp_get_logits(h, _ptr(s.logits[i])))
        if kind == "selfverify":
            dec.accept()
        elif i < steps:
            dec._check(L.mbp_accept(h, s.bytes[i].ctypes.data, s.counts[i].ctypes.data))
    if kind == "sampled":
        return {"logits": s.logits, "cand": s.cand}
    if kind == "selfverify":
        return {"logits": s.logits, "lens": s.lens}
    return {"logits": s.logits, "prob": s.prob}


# ------------------------------------------------------------------------- work and limits
def _segments(x):
    q, prev = [], -1
    for i, b in enumerate(x):
        if int(b) == SPACE or i - prev >= MAX_PATCH:
            q.append(i)
            prev = i
    return q


def work(case):
    """Flops: two per weight and row that meets it, four per head dimension and visible
    (query, key) pair.  Bytes: for the prompt and for every step, the weights of the
    modules that have rows then, once; the keys and values its rows see, once per
    sequence and layer, and those it adds; logits."""
    m = MODELS[case["model"]]
    d, dff, wb = m["d_model"], m["d_ff"], 4 if m["dtype"] == "f32" else 2
    per_layer = 4 * d * d + 3 * d * dff
    s = _inputs(case, 1)
    B, n, steps, kind = case["batch"], case["n"], case["steps"], case["kind"]
    trunk = m["n_enc"] + m["n_nb"]
    head_layer = 3 * d * dff if m["head"] == "mlp" else per_layer
    mb_layers = 0 if n < 2 else n - 1 if m["head"] == "mlp" else m["n_mb"]
    kv = 2 * d * wb  # a key and a value of one layer
    flops = nbytes = 0.0
    seqs = [list(p) for p in s.prompts]

    def commit(adds):
        """Adds adds[b] to every row; returns flops and bytes of the pass."""
        f = y = 0.0
        rows = lat_rows = 0
        for b, add in enumerate(adds):
            if len(add) == 0:
                continue
            x = seqs[b]
            k0, t0 = len(_segments(x)) + 1 if x else 0, len(x)
            x.extend(int(v) for v in add)
            k1, t1 = len(_segments(x)) + 1, len(x)
            rows += t1 - t0
            lat_rows += k1 - k0
            f += 4.0 * d * (trunk * (t1 * (t1 + 1) - t0 * (t0 + 1)) / 2 + m["n_lm"] * (k1 * (k1 + 1) - k0 * (k0 + 1)) / 2)
            y += kv * (trunk * t1 + (m["n_lm"] * k1 if k1 > k0 else 0))
        f += 2.0 * per_layer * (trunk * rows + m["n_lm"] * lat_rows)
        y += per_layer * wb * (trunk + (m["n_lm"] if lat_rows else 0))
        return f, y

    prompts, seqs = seqs, [[] for _ in seqs]
    f, y = commit(prompts)
    flops, nbytes = flops + f, nbytes + y
    if kind == "forward":
        T = case["prompt"]
        heads = 2 if m["n_mb"] else 1
        flops += 2.0 * per_layer * m["n_mb"] * T + heads * 2.0 * 256 * d * T
        nbytes += per_layer * wb * m["n_mb"] + 256 * d * wb + 8.0 * T
        return {"bytes": nbytes, "flops": flops}
    for i in range(steps + (kind != "external")):
        rows = n + 1 if kind == "external" else n
        flops += 2.0 * 256 * d * B * rows
        nbytes += 256 * d * wb + B * rows * 1024
        if kind != "external" and mb_layers:
            new = B * (n - 1 if m["head"] == "mlp" else max(1, n - 2))
            flops += 2.0 * head_layer * (new if m["head"] != "mlp" else B) * mb_layers
            nbytes += head_layer * wb * mb_layers
        if kind in ("external", "selfverify"):
            keep = [len(x) for x in seqs]
            drafts = s.drafts[i] if kind == "external" else np.full((B, n), 0x61, dtype=np.uint8)
            f, y = commit(list(drafts))
            flops, nbytes = flops + f, nbytes + y
            for b in range(B):
                seqs[b] = seqs[b][: keep[b] + (n + 1) // 2 if kind == "external" else keep[b] + 1]
        elif i < steps:
            f, y = commit([s.bytes[i, b, : s.counts[i, b]] for b in range(B)])
            flops, nbytes = flops + f, nbytes + y
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the error measured against 64 bits: float32 models are 2e-7 to 6e-7
    off; bfloat16 ones, whose keys and values are kept in float16, 2e-5 to 1e-4 (up to 3e-5
    in the losses)."""
    m = MODELS[case["model"]]
    if m["dtype"] == "f32":
        return {"rel": 3e-6, "differ": 0.01}
    if case["kind"] == "forward":
        return {"rel": 1.2e-4, "differ": 0.01}
    return {"rel": 4e-4, "differ": 0.01}


# ------------------------------------------------------- the same in plain torch, 64 bits
class _Exact:
    def __init__(self, name):
        self.m = SimpleNamespace(**MODELS[name])
        self.dev = _device()
        self.W = {k: torch.from_numpy(v).to(self.dev).double().squeeze() for k, v in _weights_of(name).items()}
        self.dh = self.m.d_model // self.m.n_heads

    def norm(self, x, gain):
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * gain

    def rope(self, x, pos):
        ang = pos.double()[:, None] * ROPE_BASE ** (-torch.arange(0, self.dh, 2, device=self.dev).double() / self.dh)
        c, s = ang.cos()[:, None], ang.sin()[:, None]
        a, b = x[..., 0::2], x[..., 1::2]
        return torch.stack((a * c - b * s, a * s + b * c), -1).flatten(-2)

    def attend(self, q, k, v, mask):
        """mask: None for causal, else rows by keys."""
        T, H, dh = q.shape
        out = torch.empty_like(q)
        for h in range(H):
            for i0 in range(0, T, 2048):
                i1 = min(T, i0 + 2048)
                j1 = i1 if mask is None else T
                s = (q[i0:i1, h] @ k[:j1, h].T) / math.sqrt(dh)
                see = (torch.arange(j1, device=self.dev)[None, :] <= torch.arange(i0, i1, device=self.dev)[:, None]
                       if mask is None else mask[i0:i1])
                out[i0:i1, h] = s.masked_fill_(~see, -math.inf).softmax(-1) @ v[:j1, h]
        return out.reshape(T, H * dh)

    def stack(self, x, name, layers, pos, mask=None):
        T, H = x.shape[0], self.m.n_heads
        for i in range(layers):
            w = lambda k: self.W["%s.%d.%s" % (name, i, k)]  # noqa: B023, E731
            u = self.norm(x, w("attn_norm"))
            q, k, v = ((u @ w(t).T).view(T, H, self.dh) for t in ("wq", "wk", "wv"))
            x = x + self.attend(self.rope(q, pos), self.rope(k, pos), v, mask) @ w("wo").T
            x = x + self.ffn(self.norm(x, w("ffn_norm")), w)
        return x

    @staticmethod
    def ffn(u, w):
        return (torch.nn.functional.silu(u @ w("w_gate").T) * (u @ w("w_up").T)) @ w("w_down").T

    def head(self, x, gain):
        return self.norm(x, gain) @ self.W["unembed"].T

    def trunk(self, x):
        m, W = self.m, self.W
        xt = torch.tensor([int(v) for v in x], device=self.dev)
        pos = torch.arange(len(xt), device=self.dev)
        he = self.stack(W["emb"][xt], "enc", m.n_enc, pos)
        if m.boundary == "learned":
            z = (he @ W["bp.w"]) * torch.rsqrt(he.square().mean(-1) + EPS) + W["bp.b"]
            ends = (z >= 0).tolist()
            q, prev = [], -1
            for i, e in enumerate(ends):
                if e or i - prev >= MAX_PATCH:
                    q.append(i)
                    prev = i
        else:
            q = _segments(x)
        lo = [0] + [v + 1 for v in q[:-1]]
        lat = torch.stack([W["bos"]] + [he[a: b + 1].mean(0) for a, b in zip(lo, q)])
        out = self.stack(lat, "lm", m.n_lm, torch.arange(len(lat), device=self.dev))
        group = torch.searchsorted(torch.tensor(q, device=self.dev), pos, right=True) if q else torch.zeros_like(pos)
        h1 = self.stack(out[group] + he, "nt", m.n_nb, pos)
        return SimpleNamespace(q=q, z=lat + out, group=group, h1=h1)

    def lca(self, g):
        i = torch.arange(len(g), device=self.dev)
        return ((g[None, :] == g[:, None]) & (i[None, :] <= i[:, None])) | (g[None, :] == g[:, None] - 1)

    def candidates(self, t, last, n):
        """The n x 256 logits of the step whose last committed byte is `last`."""
        m, W = self.m, self.W
        rows = [self.head(t.h1[last: last + 1], W["nt_norm"])]
        if n >= 2 and m.head == "mlp":
            for k in range(n - 1):
                w = lambda key: W["mlp.%d.%s" % (k, key)]  # noqa: B023, E731
                h = t.h1[last: last + 1]
                rows.append(self.head(h + self.ffn(self.norm(h, w("norm")), w), W["nt_norm"]))
        elif n >= 2:
            g = int(t.group[last])
            start = t.q[g - 2] if g >= 2 else 0
            pos = torch.arange(start, last + n - 1, device=self.dev)
            grp = torch.cat([t.group[start: last + 1], torch.full((n - 2,), g, device=self.dev)])
            h = self.stack(t.z[grp], "mb", m.n_mb, pos, self.lca(grp))
            rows.append(self.head(h[last - start: last - start + n - 1], W["mb_norm"]))
        return torch.cat(rows)


def _exact_flops(case):
    m = MODELS[case["model"]]
    d, T = m["d_model"], case["prompt"] + case["steps"] * case["n"]
    one = 2.0 * 16 * d * d * T * (m["n_enc"] + m["n_nb"] + m["n_mb"] + m["n_lm"] / 5) + 4.0 * d * T * T * (m["n_enc"] + m["n_nb"])
    return one * case["batch"] * (case["steps"] if case["kind"] == "external" else 1)


@torch.no_grad()
def exact(case, seed):
    if _exact_flops(case) > EXACT_MAX_FLOPS:
        return None
    s, E = _inputs(case, seed), _Exact(case["model"])
    B, n, steps, kind = case["batch"], case["n"], case["steps"], case["kind"]
    if kind == "forward":
        x, T = s.prompts[0], case["prompt"]
        t = E.trunk(x)
        nll = torch.zeros((2, T), dtype=torch.float64, device=E.dev)
        xt = torch.from_numpy(x.astype(np.int64)).to(E.dev)
        rows = [E.head(t.h1, E.W["nt_norm"])]
        if E.m.n_mb:
            pos = torch.arange(T, device=E.dev)
            rows.append(E.head(E.stack(t.z[t.group], "mb", E.m.n_mb, pos, E.lca(t.group)), E.W["mb_norm"]))
        for k, lg in enumerate(rows):
            left = T - 1 - k
            if left > 0:
                nll[k, :left] = -lg[:left].log_softmax(-1).gather(1, xt[k + 1:, None])[:, 0]
        a, b, rate = float(nll[0].sum()), float(nll[1].sum()), len(t.q) / T
        bp = max(rate - 1.0, 0.0)
        return {"nll": nll, "loss": torch.tensor([a, b, a + b, bp, a + b + bp, len(t.q)], dtype=torch.float64)}
    rounds, rows = (steps, n + 1) if kind == "external" else (steps + 1, n)
    logits = torch.zeros((rounds, B, rows, 256), dtype=torch.float64, device=E.dev)
    for b in range(B):
        if kind == "external":
            for i in range(steps):
                x = s.seqs[b][i]
                t = E.trunk(x + [int(v) for v in s.drafts[i, b]])
                logits[i, b] = E.head(t.h1[len(x) - 1:], E.W["nt_norm"])
            continue
        x = [int(v) for v in s.prompts[b]]
        if kind == "selfverify":
            # what follows is taken to be each byte's successor, and taken again from
            # where the model keeps another byte
            def follow(x, length):
                while len(x) < length:
                    x.append(int(_successor()[x[-1]]))
                return x, E.trunk(x)

            last, length = len(x) - 1, len(x) + (steps + 1) * n
            x, t = follow(x, length)
            for i in range(steps + 1):
                logits[i, b] = E.candidates(t, last, n)
                c, k = logits[i, b].argmax(-1).tolist(), 0
                while k < n:
                    greedy = int(E.head(t.h1[last + k], E.W["nt_norm"]).argmax())
                    if c[k] != greedy:
                        break
                    k += 1
                    if x[last + k] != greedy:
                        x, t = follow(x[: last + k] + [greedy], length)
                last += k
            continue
        last = [len(x) - 1]
        for i in range(steps):
            x += [int(v) for v in s.bytes[i, b, : s.counts[i, b]]]
            last.append(len(x) - 1)
        t = E.trunk(x)
        for i, at in enumerate(last):
            logits[i, b] = E.candidates(t, at, n)
    if kind == "external":
        return {"logits": logits, "bytes": None, "lens": None}
    if kind == "selfverify":
        return {"logits": logits, "lens": None}
    if kind == "sampled":
        return {"logits": logits, "cand": None}
    return {"logits": logits, "prob": logits.softmax(-1).amax(-1)}
