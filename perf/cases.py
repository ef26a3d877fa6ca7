"""The work this library does for its users, as cases that can be timed and compared.

A case is a dict of plain values. `prepare` makes what a program holds before the call (inputs on
the GPU, workspaces, the transposed frozen head, n-gram sets with their history), `run` is one
pass through the public entry points, `exact` the same result from plain torch in 64 bits.

Kinds:
  update      one whole in-episode update: n-gram weights, weighted CE forward and backward, the
              attention block's backward (bf16), the LoRA gradients of q, k, v and o
  ngram       exposure and weights of the update tokens against the flat history (Eq. 8-9)
  ngram_set   the same from persistent per-episode sets: append the previous update, weigh the new
  repetition  the sequence-level filter: update text against every previous one (Eq. 6-7)
  ce          token-weighted CE through the frozen LM head, with or without its backward (Eq. 10)
  attn        backward of the adapted attention block
  lora_grad   LoRA gradients of q, k, v and o of every episode of a batch
  adapter     the adapter step on every layer's parameters and the swap into serving
  serve       grouped multi-adapter forward of concurrent episodes (decoding and prefill)
"""
import math

import numpy as np
import torch

import paper_2607_03441_amd as attt

DH = 128        # head dimension of the attention block
W_MIN = 0.05    # weight floor
LR = 5e-4       # adapter step
DEV = "cuda"


# ---- the cases ---------------------------------------------------------------------------------
def listed():
    return [
        # the smallest whole update (fp32, one adapted projection): launches and latency count
        dict(name="update_tiny_fp32", kind="update", dtype="f32", E=1, N=512, H=2048, n=4, d=256, kv=0, V=4096,
             rank=8, copy=0.4),
        # a small model's whole update in bf16: 2048 tokens, 16 heads over 4
        dict(name="update_small_bf16", kind="update", dtype="bf16", E=1, N=2048, H=16384, n=3, d=2048, kv=4, V=32000,
             rank=16, copy=0.3),
        # 16 concurrent stuck episodes against half a million history tokens each
        dict(name="ngram_stuck16", kind="ngram", E=16, N=65536, H=524288, n=3, V=128256, copy=0.9),
        # the per-update n-gram work of 16 concurrent episodes on persistent sets
        dict(name="ngram_set_update16", kind="ngram_set", E=16, N=16000, H=131072, n=4, V=128256, copy=0.35),
        # the sequence-level filter over 16 episodes of 33 texts
        dict(name="repetition16", kind="repetition", E=16, texts=33, words=4096, V=128256, copy=0.35),
        # the Llama-8B head, forward and backward: the largest single call
        dict(name="ce_llama8b", kind="ce", dtype="bf16", E=1, N=8192, d=4096, V=128256, grad=True),
        # the loss alone over three ragged episodes (evaluating an update without a step)
        dict(name="ce_eval_ragged", kind="ce", dtype="bf16", E=3, N=3001, d=4096, V=128256, grad=False),
        # the Llama-8B attention block's backward over one long update
        dict(name="attn_llama8b", kind="attn", E=1, N=8192, heads=32, kv=8),
        # the adapter gradients of the same update
        dict(name="lora_grad_llama8b", kind="lora_grad", dtype="bf16", E=1, N=8192, d=4096, kv=8, rank=16),
        # after the update: the step on all 32 layers' adapters and their swap into serving
        dict(name="adapter_step_swap", kind="adapter", layers=32, d=4096, kv=8, rank=16),
        # one decoding step of 16 concurrent episodes through one layer's q, k, v and o
        dict(name="serve_decode16", kind="serve", E=16, rows=1, d=4096, kv=8, rank=16),
        # prefill of 16 episodes of 512 tokens through the same adapters
        dict(name="serve_prefill16", kind="serve", E=16, rows=512, d=4096, kv=8, rank=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng, most):
    """(d, kv): a hidden size of whole heads and a number of key/value heads that divides them."""
    kv = rng.choice([1, 2, 4, 8])
    g = rng.randint(1, max(1, most // kv))
    return kv * g * DH, kv


def draw(rng):
    kind = rng.choice(["update", "update", "ngram", "ngram", "ngram_set", "repetition", "ce", "ce", "ce", "attn",
                       "attn", "lora_grad", "lora_grad", "adapter", "serve", "serve", "serve"])
    if kind == "update":
        if rng.random() < 0.4:
            return dict(kind=kind, dtype="f32", E=rng.randint(1, 3), N=_log(rng, 64, 1024), H=_log(rng, 256, 16384),
                        n=rng.randint(2, 5), d=8 * _log(rng, 8, 64), kv=0, V=_log(rng, 500, 8192),
                        rank=rng.randint(4, 16), copy=round(rng.uniform(0.2, 0.9), 2))
        d, kv = _heads(rng, 20)
        return dict(kind=kind, dtype="bf16", E=rng.randint(1, 4), N=_log(rng, 128, 4096), H=_log(rng, 1024, 65536),
                    n=rng.randint(2, 5), d=d, kv=kv, V=_log(rng, 8000, 64000), rank=rng.choice([8, 16, 24, 32]),
                    copy=round(rng.uniform(0.2, 0.9), 2))
    if kind == "ngram":
        E = rng.randint(1, 16)
        return dict(kind=kind, E=E, N=E * _log(rng, 200, 4096), H=_log(rng, 1000, 524288), n=rng.randint(2, 6),
                    V=_log(rng, 4000, 152000), copy=round(rng.uniform(0.2, 0.95), 2))
    if kind == "ngram_set":
        E = rng.randint(1, 16)
        return dict(kind=kind, E=E, N=E * _log(rng, 100, 4096), H=_log(rng, 1000, 131072), n=rng.randint(2, 6),
                    V=_log(rng, 4000, 152000), copy=round(rng.uniform(0.2, 0.95), 2))
    if kind == "repetition":
        return dict(kind=kind, E=rng.randint(1, 16), texts=rng.randint(2, 65), words=_log(rng, 60, 8192),
                    V=_log(rng, 4000, 152000), copy=round(rng.uniform(0.2, 0.95), 2))
    if kind == "ce":
        grad = rng.random() < 0.7
        if rng.random() < 0.25:
            return dict(kind=kind, dtype="f32", E=rng.randint(1, 4), N=_log(rng, 64, 1024), d=8 * _log(rng, 8, 64),
                        V=_log(rng, 500, 8192), grad=grad)
        while True:
            c = dict(kind=kind, dtype="bf16", E=rng.randint(1, 8), N=_log(rng, 100, 8192), d=8 * _log(rng, 128, 640),
                     V=_log(rng, 16000, 152000), grad=grad)
            if c["N"] * c["d"] * c["V"] < 4.0e12:
                return c
    if kind == "attn":
        while True:
            d, kv = _heads(rng, 40)
            c = dict(kind=kind, E=rng.randint(1, 8), N=_log(rng, 200, 8192), heads=d // DH, kv=kv)
            if _pairs(c) * c["heads"] < 2.0e9:
                return c
    if kind == "lora_grad":
        d, kv = _heads(rng, 40)
        return dict(kind=kind, dtype="bf16", E=rng.randint(1, 8), N=_log(rng, 200, 16384), d=d, kv=kv,
                    rank=rng.choice([4, 8, 16, 32, 64]))
    if kind == "adapter":
        d, kv = _heads(rng, 40)
        return dict(kind=kind, layers=rng.randint(1, 32), d=d, kv=kv, rank=rng.choice([4, 8, 16, 32]))
    d, kv = _heads(rng, 40)
    return dict(kind=kind, E=rng.randint(1, 16), rows=1 if rng.random() < 0.4 else _log(rng, 2, 1024), d=d, kv=kv,
                rank=rng.choice([4, 8, 16, 32]))


# ---- inputs ------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(g, shape, std, dtype):
    return (torch.randn(shape, generator=g, device=DEV) * std).to(dtype)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _offsets(E, N):
    """Ragged episodes: offsets [E+1] of N rows, weights 3, 2, 4, 1, 3, ... in turn."""
    w = np.array([(3, 2, 4, 1)[e % 4] for e in range(E)], np.float64)
    return np.concatenate([[0], np.floor(np.cumsum(w) / w.sum() * N + 0.5)]).astype(np.int64)


def _pairs(case):
    L = np.diff(_offsets(case["E"], case["N"])).astype(np.float64)
    return float((L * (L + 1) / 2).sum())


def _text(g, total, vocab, copy):
    """Token ids with the repetition of agent text: Zipf-distributed fresh tokens, cut into spans of
    4 to 32, each span a copy of an earlier one with probability `copy`."""
    ranks = torch.arange(1, vocab + 1, device=DEV, dtype=torch.float64)
    cdf = torch.cumsum(ranks ** -1.1, 0)
    u = torch.rand(total, generator=g, device=DEV, dtype=torch.float64) * cdf[-1]
    fresh = torch.searchsorted(cdf, u).clamp_(max=vocab - 1)
    lens = torch.randint(4, 33, (total // 4 + 2,), generator=g, device=DEV)
    ends = torch.cumsum(lens, 0)
    pos = torch.arange(total, device=DEV)
    seg = torch.searchsorted(ends, pos, right=True)
    begin = (ends - lens)[seg]
    src = (torch.rand(lens.shape, generator=g, device=DEV, dtype=torch.float64)[seg] * (begin - 32).clamp(min=0)).long()
    copied = (torch.rand(lens.shape, generator=g, device=DEV)[seg] < copy) & (begin > 64)
    idx = torch.where(copied, src + (pos - begin), pos)
    for _ in range(14):
        idx = idx[idx]
    perm = torch.randperm(vocab, generator=g, device=DEV)
    return perm[fresh[idx]].to(torch.int32)


def _token_inputs(case, g, extra=0):
    """Per episode a history of H tokens and a new text; `extra`: texts of the same length before it."""
    off = _offsets(case["E"], case["N"])
    hist, texts = [], [[] for _ in range(extra + 1)]
    for L in np.diff(off):
        t = _text(g, case["H"] + int(L) * (extra + 1), case["V"], case["copy"])
        hist.append(t[:case["H"]])
        for k in range(extra + 1):
            texts[k].append(t[case["H"] + k * int(L):case["H"] + (k + 1) * int(L)])
    hoff = np.arange(case["E"] + 1, dtype=np.int64) * case["H"]
    return torch.cat(hist), hoff, [torch.cat(x) for x in texts], off


def _u8(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def _ce_inputs(case, g):
    dt = _dtype(case)
    N, d, V = case["N"], case["d"], case["V"]
    return _randn(g, (N, d), 1.0, dt), _randn(g, (V, d), 0.02, dt)


def _projections(case):
    """(name, d_out, input) of the adapted projections; q, k and v read one input."""
    d = case["d"]
    if not case["kv"]:
        return [("o", d, "xo")]
    return [("q", d, "x"), ("k", case["kv"] * DH, "x"), ("v", case["kv"] * DH, "x"), ("o", d, "xo")]


def _lora_inputs(case, g, dy):
    """Adapter problems of every episode. `dy`: per projection the upstream gradient [N, d_out]."""
    dt, N, d, r = _dtype(case), case["N"], case["d"], case["rank"]
    off = _offsets(case["E"], N)
    xs = {k: _randn(g, (N, d), 1.0, dt) for k in ("x", "xo")}
    flat, problems = {}, []
    for name, d_out, x in _projections(case):
        A, B = _randn(g, (case["E"], r, d), 0.02, dt), _randn(g, (case["E"], d_out, r), 0.02, dt)
        dA, dB = torch.zeros(A.shape, device=DEV), torch.zeros(B.shape, device=DEV)
        flat[name] = (xs[x], A, B, dA, dB)
        for e in range(case["E"]):
            rows = slice(int(off[e]), int(off[e + 1]))
            problems.append((e, dict(x=xs[x][rows], dy=dy[name][rows], A=A[e], B=B[e], dA=dA[e], dB=dB[e],
                                     scale=16.0 / r)))
    # episodes in order, each one's projections together; q, k and v share one view of x
    problems.sort(key=lambda p: p[0])
    out, views = [], {}
    for _, p in problems:
        key = (p["x"].data_ptr(), p["x"].shape[0])
        p["x"] = views.setdefault(key, p["x"])
        out.append(p)
    return out, flat


def _adapter_shapes(case):
    r = case["rank"]
    return [s for _, d_out, _ in _projections(case) for s in ((r, case["d"]), (d_out, r))]


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("update", "ngram"):
        hist, hoff, (tok,), off = _token_inputs(case, g)
        s.update(hist=hist, hoff=hoff, tok=tok, off=off, ws_ng=_u8(attt.ngram_workspace_size(hoff, off, case["n"])),
                 fw=(torch.empty_like(tok), torch.empty(tok.shape, dtype=torch.float32, device=DEV)))
    if kind == "ngram_set":
        hist, hoff, (prev, new), off = _token_inputs(case, g, extra=1)
        cap = case["H"] + 2 * int(np.diff(off).max()) + 64
        nbytes = attt.ngram_set_size(cap, case["n"])
        sets = [_u8(nbytes) for _ in range(case["E"])]
        attt.ngram_set_init(sets, cap, case["n"])
        attt.ngram_set_append(sets, hist, hoff, cap, case["n"])
        s.update(sets=sets, cap=cap, prev=prev, new=new, off=off, hist=hist, hoff=hoff)
        s["fw"] = (torch.empty_like(new), torch.empty(new.shape, dtype=torch.float32, device=DEV))
    if kind == "repetition":
        words = torch.cat([_text(g, case["texts"] * case["words"], case["V"], case["copy"]) for _ in range(case["E"])])
        toff = np.arange(case["E"] * case["texts"] + 1, dtype=np.int64) * case["words"]
        eoff = np.arange(case["E"] + 1, dtype=np.int64) * case["texts"]
        s.update(words=words, toff=toff, eoff=eoff, toff_dev=torch.from_numpy(toff).to(DEV),
                 ws=_u8(attt.repetition_workspace_size(toff, eoff)))
    if kind in ("update", "ce"):
        h, W = _ce_inputs(case, g)
        dt = attt.BF16 if case["dtype"] == "bf16" else attt.F32
        grad = case.get("grad", True)
        Wt = attt.ce_head_transpose(W) if grad and case["dtype"] == "bf16" else None
        N, E = case["N"], case["E"]
        off = _offsets(E, N)
        if kind == "ce":
            labels = torch.randint(0, case["V"], (N,), generator=g, device=DEV, dtype=torch.int32)
            s["w"] = 1.0 / (1.0 + torch.randint(0, 20, (N,), generator=g, device=DEV).float())
        else:
            labels = s["tok"]
        s.update(h=h, W=W, Wt=Wt, labels=labels, off=off, grad=grad,
                 ws_ce=_u8(attt.ce_workspace_size(N, case["d"], case["V"], dt, want_grad=grad, head_t=Wt is not None)),
                 ce_out=(torch.empty(E, device=DEV), torch.empty(N, device=DEV), torch.empty_like(h) if grad else None))
    if kind == "attn" or (kind == "update" and case["kv"]):
        N, H, kv = case["N"], case.get("heads") or case["d"] // DH, case["kv"]
        bf = torch.bfloat16
        s.update(q=_randn(g, (N, H, DH), 1.0, bf), k=_randn(g, (N, kv, DH), 1.0, bf), v=_randn(g, (N, kv, DH), 1.0, bf),
                 do=_randn(g, (N, H, DH), 0.05, bf), off=_offsets(case["E"], N))
        s["at_out"] = (torch.empty_like(s["q"]), torch.empty_like(s["k"]), torch.empty_like(s["v"]),
                       torch.empty(H, N, device=DEV), torch.empty(H, N, device=DEV))
    if kind in ("update", "lora_grad"):
        N = case["N"]
        if kind == "lora_grad":
            dy = {name: _randn(g, (N, d_out), 1.0 / N, _dtype(case)) for name, d_out, _ in _projections(case)}
        else:
            dy = {"o": s["ce_out"][2]}
            if case["kv"]:
                dy.update({name: t.view(N, -1) for name, t in zip("qkv", s["at_out"])})
        s["problems"], s["lora"] = _lora_inputs(case, g, dy)
        s["dy"] = dy
        s["ws_lora"] = _u8(attt.lora_workspace_size(s["problems"], attt.BF16 if case["dtype"] == "bf16" else attt.F32))
    if kind == "adapter":
        shapes = _adapter_shapes(case) * case["layers"]
        n = sum(a * b for a, b in shapes)
        master, grad = _randn(g, (n,), 0.02, torch.float32), _randn(g, (n,), 0.01, torch.float32)
        train, slot = torch.empty(n, dtype=torch.bfloat16, device=DEV), torch.empty(n, dtype=torch.bfloat16, device=DEV)
        params, pairs, o = [], [], 0
        for a, b in shapes:
            e = o + a * b
            params.append(dict(param=master[o:e], grad=grad[o:e], param_bf16=train[o:e]))
            pairs.append((master[o:e], slot[o:e]))
            o = e
        s.update(master=master, grad=grad, train=train, slot=slot, params=params, pairs=pairs)
    if kind == "serve":
        # one batch buffer per projection, an episode's rows contiguous in it, as the base GEMM writes it
        bf, E, L, d, r = torch.bfloat16, case["E"], case["rows"], case["d"], case["rank"]
        xs = {k: _randn(g, (E, L, d), 1.0, bf) for k in ("x", "xo")}
        s.update(xs=xs, y={}, AB={}, problems=[])
        for name, d_out, _ in _projections(case):
            s["y"][name] = _randn(g, (E, L, d_out), 1.0, bf)
            s["AB"][name] = (_randn(g, (E, r, d), 0.02, bf), _randn(g, (E, d_out, r), 0.02, bf))
        for e in range(E):
            x1 = {k: v[e] for k, v in xs.items()}
            for name, _, x in _projections(case):
                A, B = s["AB"][name]
                s["problems"].append(dict(x=x1[x], y=s["y"][name][e], A=A[e], B=B[e], scale=16.0 / r))
    return s


# ---- one pass ----------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    out = {}
    if kind in ("update", "ngram"):
        out["f"], out["w"] = attt.ngram_weights(s["hist"], s["hoff"], s["tok"], s["off"], n=case["n"], w_min=W_MIN,
                                                workspace=s["ws_ng"], out=s["fw"])
    if kind == "ngram_set":
        attt.ngram_set_append(s["sets"], s["prev"], s["off"], s["cap"], case["n"])
        out["f"], out["w"] = attt.ngram_set_weights(s["sets"], s["new"], s["off"], s["cap"], case["n"], W_MIN, out=s["fw"])
    if kind == "repetition":
        r = attt.update_repetition(s["words"], s["toff"], s["eoff"], text_offsets_dev=s["toff_dev"], want_pairs=True,
                                   workspace=s["ws"])
        out = dict(zip(("rho", "nu", "skip", "best", "pairs"), r))
    if kind in ("update", "ce"):
        w = out["w"] if kind == "update" else s["w"]
        loss, lse, dh = attt.weighted_ce_fwd_bwd(s["h"], s["W"], s["labels"], w, row_offsets=s["off"],
                                                 want_grad=s["grad"], workspace=s["ws_ce"], out=s["ce_out"],
                                                 lm_head_t=s["Wt"])
        out.update(loss=loss, lse=lse)
        if dh is not None:
            out["dh"] = dh
    if "at_out" in s:
        r = attt.attention_bwd(s["q"], s["k"], s["v"], s["do"], row_offsets=s["off"], out=s["at_out"])
        out.update(zip(("dq", "dk", "dv", "at_lse", "at_d"), r))
    if kind in ("update", "lora_grad"):
        attt.lora_grad(s["problems"], workspace=s["ws_lora"])
        for name, (_, _, _, dA, dB) in s["lora"].items():
            out["dA_" + name], out["dB_" + name] = dA, dB
    if kind == "adapter":
        attt.lora_sgd_step(s["params"], LR, zero_grad=True)
        attt.lora_hot_swap(s["pairs"])
        out = dict(master=s["master"], grad=s["grad"], train=s["train"], slot=s["slot"])
    if kind == "serve":
        attt.lora_forward(s["problems"])
        out = dict(s["y"])
    return out


# ---- what a pass cannot do without --------------------------------------------------------------
def work(case):
    kind = case["kind"]
    nbytes = flops = 0.0
    if kind in ("update", "ngram"):
        nbytes += 4.0 * case["E"] * case["H"] + 12.0 * case["N"]
    if kind == "ngram_set":
        # tokens in, f and w out, one record read and one updated per token
        nbytes += 16.0 * case["N"] + 3.0 * (12 + 4 * case["n"]) * case["N"]
    if kind == "repetition":
        nbytes += 4.0 * case["E"] * case["texts"] * case["words"] + 8.0 * case["E"] * case["texts"]
    if kind in ("update", "ce"):
        N, d, V, esz = case["N"], case["d"], case["V"], 2 if case["dtype"] == "bf16" else 4
        grad = case.get("grad", True)
        flops += (4.0 if grad else 2.0) * N * d * V
        nbytes += esz * (float(N) * d * (2 if grad else 1) + float(V) * d) + 12.0 * N
    if kind == "attn" or (kind == "update" and case["kv"]):
        H = case.get("heads") or case["d"] // DH
        flops += 14.0 * DH * _pairs(case) * H
        nbytes += 2.0 * case["N"] * DH * (3 * H + 4 * case["kv"]) + 8.0 * case["N"] * H
    if kind in ("update", "lora_grad"):
        N, d, r, esz = case["N"], case["d"], case["rank"], 2 if case["dtype"] == "bf16" else 4
        ps = _projections(case)
        nbytes += esz * N * d * len({x for _, _, x in ps})
        for _, d_out, _ in ps:
            flops += 4.0 * N * r * (d + d_out)
            nbytes += esz * N * d_out + (esz + 8.0) * case["E"] * r * (d + d_out)
    if kind == "adapter":
        n = case["layers"] * sum(a * b for a, b in _adapter_shapes(case))
        nbytes += 18.0 * n + 6.0 * n
        flops += 2.0 * n
    if kind == "serve":
        E, L, d, r = case["E"], case["rows"], case["d"], case["rank"]
        ps = _projections(case)
        nbytes += 2.0 * E * L * d * len({x for _, _, x in ps})
        for _, d_out, _ in ps:
            nbytes += 4.0 * E * L * d_out + 2.0 * E * r * (d + d_out)
            flops += 2.0 * E * L * r * (d + d_out)
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    kind = case["kind"]
    if kind in ("ngram", "ngram_set", "repetition", "adapter"):
        return "exact"  # integers and correctly rounded functions of them; two roundings per element
    if case.get("dtype") == "f32":
        return dict(rel=1e-5)
    if kind == "ce" and not case["grad"]:
        return dict(rel=1e-5)  # float32 sums of exact bf16 products
    if kind == "lora_grad":
        return dict(rel=1e-5)  # float32 results; the low-rank factors between the passes carry 16 bits
    return dict(rel=1e-2, max=4e-2)


# ---- the same in 64 bits --------------------------------------------------------------------------
def _exact_counts(hist, x, n):
    """Occurrences in hist of the n-gram of x starting at each position (int64 [len(x) - n + 1])."""
    both = torch.cat([hist, x]).long()
    base = int(both.max()) + 1
    ids = both
    for k in range(1, n):
        ids = torch.unique(ids[:-1] * base + both[k:], return_inverse=True)[1]
    nh = max(0, hist.numel() - n + 1)
    if x.numel() < n:
        return torch.zeros(0, dtype=torch.int64, device=DEV)
    cnt = torch.bincount(ids[:nh], minlength=int(ids.max()) + 1) if nh else torch.zeros(int(ids.max()) + 1, dtype=torch.int64, device=DEV)
    return cnt[ids[hist.numel():]]


def _exact_weights(hists, texts, n):
    ws = []
    for hist, x in zip(hists, texts):
        c = torch.zeros(x.numel() + n - 1, dtype=torch.int64, device=DEV)
        got = _exact_counts(hist, x, n)
        c[n - 1:n - 1 + got.numel()] = got
        f = c.unfold(0, n, 1).max(1)[0] if x.numel() else c[:0]
        ws.append(torch.clamp(1.0 / (1.0 + f.double()), min=float(np.float32(W_MIN))))
    return torch.cat(ws)


def _cut(t, off):
    return [t[int(a):int(b)] for a, b in zip(off[:-1], off[1:])]


def _exact_ce(s, w):
    case, off = s["case"], s["off"]
    h, W, N = s["h"].double(), s["W"].double(), case["N"]
    L = np.diff(off)
    per = torch.from_numpy(np.repeat(L, L)).to(DEV).double()
    lse = torch.empty(N, dtype=torch.float64, device=DEV)
    loss = torch.zeros(case["E"], dtype=torch.float64, device=DEV)
    dh = torch.empty(h.shape, dtype=torch.float64, device=DEV) if s["grad"] else None
    ce = torch.empty(N, dtype=torch.float64, device=DEV)
    step = max(1, min(N, (1 << 28) // case["V"]))
    for a in range(0, N, step):
        b = min(N, a + step)
        z = h[a:b] @ W.t()
        y = s["labels"][a:b].long()[:, None]
        lse[a:b] = torch.logsumexp(z, 1)
        ce[a:b] = lse[a:b] - z.gather(1, y)[:, 0]
        if dh is not None:
            z.sub_(lse[a:b, None]).exp_()
            z.scatter_add_(1, y, torch.full(y.shape, -1.0, dtype=torch.float64, device=DEV))
            dh[a:b] = (z * (w[a:b] / per[a:b])[:, None]) @ W
    for e, part in enumerate(_cut(w * ce / per, off)):
        loss[e] = part.sum()
    out = dict(loss=loss, lse=lse)
    if dh is not None:
        out["dh"] = dh
    return out


def _exact_attn(s):
    q, k, v, do = (s[n].double() for n in ("q", "k", "v", "do"))
    N, H = q.shape[:2]
    g = H // k.shape[1]
    scale = 1.0 / math.sqrt(DH)
    dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
    lse, D = (torch.zeros(H, N, dtype=torch.float64, device=DEV) for _ in range(2))
    for a, b in zip(s["off"][:-1], s["off"][1:]):
        r = slice(int(a), int(b))
        mask = torch.ones(int(b - a), int(b - a), dtype=torch.bool, device=DEV).triu(1)
        for h in range(H):
            Q, K, V, dO = q[r, h], k[r, h // g], v[r, h // g], do[r, h]
            S = (Q @ K.t()).mul_(scale).masked_fill_(mask, -math.inf)
            lse[h, r] = torch.logsumexp(S, 1)
            P = S.sub_(lse[h, r][:, None]).exp_()
            dP = dO @ V.t()
            D[h, r] = (P * dP).sum(1)
            dv[r, h // g] += P.t() @ dO
            dS = P.mul_(dP.sub_(D[h, r][:, None]))
            dq[r, h] = scale * (dS @ K)
            dk[r, h // g] += scale * (dS.t() @ Q)
    return dict(dq=dq, dk=dk, dv=dv, at_lse=lse, at_d=D)


def _exact_lora(s, dy):
    case, out = s["case"], {}
    off = _offsets(case["E"], case["N"])
    scale = 16.0 / case["rank"]
    for name, (x, A, B, _, _) in s["lora"].items():
        xs, ys = _cut(x.double(), off), _cut(dy[name].double(), off)
        out["dA_" + name] = torch.stack([(scale * (ys[e] @ B[e].double())).t() @ xs[e] for e in range(case["E"])])
        out["dB_" + name] = torch.stack([scale * (ys[e].t() @ (xs[e] @ A[e].double().t())) for e in range(case["E"])])
    return out


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    out = {}
    if kind in ("update", "ngram"):
        out["f"] = None
        out["w"] = _exact_weights(_cut(s["hist"], s["hoff"]), _cut(s["tok"], s["off"]), case["n"])
    if kind == "ngram_set":
        hists = [torch.cat(p) for p in zip(_cut(s["hist"], s["hoff"]), _cut(s["prev"], s["off"]))]
        out = dict(f=None, w=_exact_weights(hists, _cut(s["new"], s["off"]), case["n"]))
    if kind == "repetition":
        words, rho = s["words"].cpu().numpy().reshape(case["E"], case["texts"], case["words"]), []
        for ep in words:
            sets = [set(t.tolist()) for t in ep]
            rho.append(max(len(sets[-1] & p) / len(sets[-1] | p) for p in sets[:-1]))
        rho = torch.tensor(rho, dtype=torch.float64)
        out = dict(rho=rho, nu=1.0 - rho, skip=None, best=None, pairs=None)
    if kind in ("update", "ce"):
        out.update(_exact_ce(s, out["w"] if kind == "update" else s["w"].double()))
    if "at_out" in s:
        out.update(_exact_attn(s))
    if kind in ("update", "lora_grad"):
        dy = s["dy"] if kind == "lora_grad" else {"o": out["dh"]}
        if kind == "update" and case["kv"]:
            dy.update({n: out["d" + n].reshape(case["N"], -1) for n in "qkv"})
        out.update(_exact_lora(s, dy))
    if kind == "adapter":
        p = s["master"].double() - float(np.float32(LR)) * s["grad"].double()
        out = dict(master=p, grad=torch.zeros_like(p), train=p, slot=p)
    if kind == "serve":
        for name, _, x in _projections(case):
            A, B = s["AB"][name]
            y = [s["y"][name][e].double() + (16.0 / case["rank"]) * ((s["xs"][x][e].double() @ A[e].double().t())
                                                                      @ B[e].double().t()) for e in range(case["E"])]
            out[name] = torch.stack(y)
    return out
