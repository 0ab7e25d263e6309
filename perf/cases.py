"""Workloads of the AirCache hot path that are timed and compared between versions of the library.

One pass is one request as a serving program issues it through the binding: the prompt's layers are scored, the
budgets set, every layer compacted, and then tokens are decoded over the compacted cache.  The outputs are the
attention outputs of every decoded token, which depend on everything before them (scores, elite sets, budgets,
selection, gather, append).  `exact` is the same method in plain fp64 torch.

Fields of a case: dtype and head_dim d of the tensors; L layers, hq query heads over hkv KV heads, B sequences of
n_sys + n_vis + n_text tokens (lengths of a batch differ by +-jitter); the observation window (kind text: the last
`window` text tokens, 0 = all of them, and the threshold alpha; kind visual: the last `window` visual tokens); the
budget mode; `steps` decoded tokens; by_layer: scoring and decode are called one layer at a time, as a model does
that calls attention layer by layer; graph: the decode step is recorded into a HIP graph and replayed;
token_major: tensors are stored [B][token][head][d].
"""
from __future__ import annotations

import math
import random
from typing import NamedTuple

import torch

import paper_2503_23956_amd as A

_DEFAULTS = dict(dtype="bf16", d=128, L=28, hq=28, hkv=4, B=1, n_sys=14, n_vis=7290, n_text=128, jitter=0.0,
                 kind="text", window=0, alpha=0.9, retention=0.10, mode=0, causal=False, steps=1, by_layer=False,
                 graph=False, token_major=False)


def _case(name, **kw):
    return dict(_DEFAULTS, name=name, **kw)


def listed():
    return [
        # The smallest call: two fp32 layers with few heads of 64 elements, a continuous candidate span of 16 text
        # tokens; what a unit test, a notebook or a debugging session in full precision does.  Launch latency.
        _case("tiny-f32", dtype="f32", d=64, L=2, hq=4, hkv=2, n_sys=16, n_vis=576, n_text=64, window=16),
        # Full-precision evaluation of the 7B geometry (fp32 tensors, heads of 128), one ordinary image.
        _case("f32-d128", dtype="f32", n_vis=2304, steps=8),
        # A small model with heads of 64 elements in bf16 (seven query heads per KV head), one large image, a short answer.
        _case("bf16-d64", d=64, L=24, hq=14, hkv=2, steps=32),
        # One large image, 7B geometry: compression and the first token.  What a yes/no question costs.
        _case("prompt-7b", steps=1),
        # The same with an answer of ordinary length, all layers of a step in one call.
        _case("answer-7b", steps=128),
        # The same in a model that calls the library layer by layer, eagerly: four units per launch.
        _case("layerwise-7b", steps=8, by_layer=True),
        # Layer by layer with the decode step recorded once and replayed from a HIP graph.
        _case("graph-7b", steps=8, by_layer=True, graph=True),
        # A batch of 16 prompts of differing lengths, one ordinary image each.
        _case("batch-16", B=16, n_vis=2304, n_text=256, jitter=0.10, steps=32),
        # Four video prompts of 32 frames with long questions.
        _case("video-4", B=4, n_vis=6272, n_text=512, steps=32),
        # 72B geometry, two long prompts: the largest.
        _case("72b", L=80, hq=64, hkv=8, B=2, n_vis=16384, n_text=512, steps=8),
        # Observation window of the last 32 text tokens, no threshold (the continuous window of the ablations).
        _case("window-text-32", window=32, alpha=0.0),
        # Observation window of the last 32 visual tokens.
        _case("window-visual-32", kind="visual", window=32, alpha=0.0),
    ]


def _cost(case):
    w = work(case)
    return w["bytes"] * (1 if case["dtype"] == "bf16" and case["d"] == 128 else 4) + w["flops"] / 50


def draw(rng):
    """Another case of the same ranges: sizes spread over their logarithm, odd ones among them."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    largest = max(_cost(c) for c in listed() if c["name"] == "72b")
    while True:
        dtype, d = rng.choice([("bf16", 128)] * 5 + [("bf16", 64)] * 2 + [("f32", 64), ("f32", 128)])
        hkv, g = rng.choice([(4, 7), (2, 7), (8, 8), (2, 2), (8, 4), (4, 8), (1, 12), (3, 5)])
        kind, window, alpha = rng.choice([("text", 0, 0.9)] * 5 + [("text", 0, 0.6), ("text", log_int(2, 64), 0.9),
                                                                  ("text", log_int(2, 48), 0.0), ("visual", log_int(2, 48), 0.0)])
        batch = rng.choice([1, 1, 1, 2, 3, 4, 8, 16])
        c = dict(_DEFAULTS, dtype=dtype, d=d, L=log_int(2, 80), hq=hkv * g, hkv=hkv, B=batch, n_sys=rng.randrange(0, 40),
                 n_vis=log_int(60, 16384), n_text=log_int(8, 512), jitter=rng.choice([0.0, 0.1]) if batch > 1 else 0.0,
                 kind=kind, window=window, alpha=alpha, retention=rng.choice([0.01, 0.05, 0.10, 0.10, 0.25, 0.50, 1.0]),
                 mode=rng.choice([0, 0, 0, 1, 2, 3]), causal=kind == "text" and rng.random() < 0.2, steps=log_int(1, 64),
                 token_major=rng.random() < 0.3)
        c["by_layer"] = rng.random() < 0.2
        c["graph"] = dtype == "bf16" and d == 128 and c["by_layer"] and rng.random() < 0.3
        if kind == "visual":
            c["window"] = min(c["window"], c["n_vis"] // 2)
        bytes_held = c["L"] * c["B"] * c["hkv"] * (c["n_vis"] + c["n_text"]) * d * (2 if dtype == "bf16" else 4) * 2
        if bytes_held < 6e9 and _cost(c) <= largest:
            return c


class _Seq(NamedTuple):
    """[system | visual | text] of one prompt and its candidate window."""
    seq_len: int
    vis_start: int
    vis_len: int
    win_start: int
    win_len: int

    @property
    def text_start(self):
        return self.vis_start + self.vis_len

    @property
    def n_text(self):
        return self.seq_len - self.text_start


def _seqs(case):
    rng = random.Random(20250323)
    out = []
    for _ in range(case["B"]):
        u, u2 = (rng.uniform(-case["jitter"], case["jitter"]) for _ in range(2))
        n_vis, n_text = max(1, round(case["n_vis"] * (1 + u))), max(1, round(case["n_text"] * (1 + u2)))
        seq_len = case["n_sys"] + n_vis + n_text
        if case["kind"] == "visual":
            win = min(case["window"], n_vis)
            out.append(_Seq(seq_len, case["n_sys"], n_vis, case["n_sys"] + n_vis - win, win))
        else:
            win = min(case["window"], n_text) if case["window"] else n_text
            out.append(_Seq(seq_len, case["n_sys"], n_vis, seq_len - win, win))
    return out


def _tensors(case, seed, device):
    """Seeded prompt tensors with a head effect: a share of the visual keys (1-20 % over the layers) is shifted along
    a direction per (layer, sequence, KV head), the text queries lean towards it and the text keys lean by an amount
    per layer, so that strengths, skewnesses and budgets differ between the layers.  Returns q, k, v lists over the
    layers (indexed [B][head][token][d]) and q_new, k_new, v_new [steps][L][B][head][d]."""
    seqs = _seqs(case)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    L, B, hq, hkv, d = case["L"], case["B"], case["hq"], case["hkv"], case["d"]
    S = max(s.seq_len for s in seqs)
    n_q = max(s.win_len if case["kind"] == "visual" else s.n_text for s in seqs)
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    host = random.Random(seed)
    share = [0.01 + 0.19 * i / max(1, L - 1) for i in range(L)]
    host.shuffle(share)

    def randn(*shape):
        return torch.randn(shape, generator=gen, device=device, dtype=torch.float32)

    def store(x):  # [B][head][token][d] -> storage type and memory order
        if case["token_major"]:
            return x.to(dt).transpose(1, 2).contiguous().transpose(1, 2)
        return x.to(dt)

    tok = torch.arange(S, device=device)[None, :]
    vis_end = torch.tensor([s.text_start for s in seqs], device=device)[:, None]
    is_vis, is_text = (tok >= case["n_sys"]) & (tok < vis_end), tok >= vis_end
    q, k, v = [], [], []
    for l in range(L):
        u = randn(B, hkv, 1, d)
        u /= u.norm(dim=-1, keepdim=True)
        salient = is_vis & (torch.rand((B, S), generator=gen, device=device) < share[l])
        lean = 2.0 * salient + host.uniform(0.0, 6.0) * is_text
        k.append(store(randn(B, hkv, S, d).addcmul_(lean[:, None, :, None].to(torch.float32), u)))
        v.append(store(randn(B, hkv, S, d)))
        q.append(store(randn(B, hq, n_q, d) + 1.5 * math.sqrt(d) * u.repeat_interleave(hq // hkv, dim=1)))
    n = case["steps"]
    return (seqs, q, k, v, randn(n, L, B, hq, d).to(dt), randn(n, L, B, hkv, d).to(dt), randn(n, L, B, hkv, d).to(dt))


def prepare(case, seed):
    device = torch.device("cuda:0")
    seqs, q, k, v, qn, kn, vn = _tensors(case, seed, device)
    L = case["L"]
    cfg = A.make_config(
        n_layers=L, n_q_heads=case["hq"], n_kv_heads=case["hkv"], head_dim=case["d"], batch=case["B"],
        max_vis_len=max(s.vis_len for s in seqs), max_nonvis_len=max(s.seq_len - s.vis_len for s in seqs),
        max_window=max(s.win_len for s in seqs), max_decode_steps=case["steps"],
        dtype=A.AIR_BF16 if case["dtype"] == "bf16" else A.AIR_F32, alpha=case["alpha"], retention=case["retention"],
        budget_mode=case["mode"], window_kind=A.AIR_WINDOW_VISUAL if case["kind"] == "visual" else A.AIR_WINDOW_TEXT,
        device_steps=int(case["graph"]), causal_text=int(case["causal"]))
    cache = A.AirCache(cfg, device)
    st = dict(case=case, cache=cache, out=torch.empty_like(qn), all_layers=cache.prepare(q, k, v, seqs))
    if case["by_layer"]:
        st["layer"] = [cache.prepare(q[l:l + 1], k[l:l + 1], v[l:l + 1], seqs) for l in range(L)]
    if case["graph"]:  # static buffers of the recorded step
        st["now"] = [qn[0].clone(), kn[0].clone(), vn[0].clone(), torch.empty_like(qn[0])]
        st["new"] = (qn, kn, vn)
        _compress(st)
        torch.cuda.synchronize()
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            for l in range(L):
                cache.air_decode_attn(l, l + 1, *(x[l] for x in st["now"]))
        torch.cuda.synchronize()
    elif case["by_layer"]:
        st["new"] = [[(qn[t, l], kn[t, l], vn[t, l], st["out"][t, l]) for l in range(L)] for t in range(case["steps"])]
    else:
        st["new"] = [(qn[t], kn[t], vn[t], st["out"][t]) for t in range(case["steps"])]
    st["hold"] = (qn, kn, vn)
    return st


def _compress(st):
    cache, L = st["cache"], st["case"]["L"]
    cache.air_reset()
    if st["case"]["by_layer"]:
        for l in range(L):
            cache.air_score(l, l + 1, prepared=st["layer"][l])
    else:
        cache.air_score(0, L, prepared=st["all_layers"])
    cache.air_budget()
    cache.air_select_compact(0, L, prepared=st["all_layers"])


def run(st):
    case, cache, L = st["case"], st["cache"], st["case"]["L"]
    _compress(st)
    if case["graph"]:
        for t in range(case["steps"]):
            for x, new in zip(st["now"], st["new"]):
                x.copy_(new[t])
            st["graph"].replay()
            st["out"][t].copy_(st["now"][3])
    elif case["by_layer"]:
        for step in st["new"]:
            for l in range(L):
                cache.air_decode_attn(l, l + 1, *step[l])
    else:
        for step in st["new"]:
            cache.air_decode_attn(0, L, *step)
    return st["out"]


def work(case):
    """Bytes: the keys that are scored and the queries and keys of the window once, the kept rows of K and V read and
    written once, the cache once per decoded token, the new tokens and the outputs.  Flops: the window's logits (one
    row per head with a threshold) and the two products of every decoded token."""
    e = 2 if case["dtype"] == "bf16" else 4
    row, g = case["d"] * e, case["hq"] // case["hkv"]
    nbytes = flops = 0.0
    for s in _seqs(case):
        rows = s.win_len if case["alpha"] == 0.0 else 1
        text = 0 if case["kind"] == "visual" else s.win_len
        keep = s.seq_len - s.vis_len + max(1.0, case["retention"] * s.vis_len)
        t = case["steps"]
        cached = t * keep + t * (t + 1) / 2  # rows read over all steps, the appended ones included
        unit = (s.vis_len + text) * row + g * rows * row + 4 * keep * row
        unit += 2 * cached * row + t * (2 * g + 2) * row
        nbytes += case["L"] * case["hkv"] * unit
        flops += case["L"] * case["hq"] * 2.0 * case["d"] * (rows * (s.vis_len + (rows if text else 0)) + text + 2 * cached)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """bf16: probabilities of the second product and the outputs are rounded to bf16 (2^-9 each): 0.0023 measured against
    fp64 with heads of 128 elements; four times that, which also covers a pair of tokens of equal score (to fp32 rounding)
    that change places at a layer's budget.  fp32: sums of up to some thousand products in another order, 5e-7 measured."""
    return {"rel": 1e-2, "max": 0.3} if case["dtype"] == "bf16" else {"rel": 1e-5}


def _budgets(case, n_vis, s_t, s_k):
    """Per-layer budgets of one sequence: shares of strength and skewness, clamped to [1, n_vis], largest remainder."""
    L, r = case["L"], case["retention"]
    sk = [max(x, 0.0) for x in s_k]
    a = [x / sum(s_t) if sum(s_t) > 0 else 1 / L for x in s_t]
    b = [x / sum(sk) if sum(sk) > 0 else 1 / L for x in sk]
    share = {0: [0.5 * (x + y) for x, y in zip(a, b)], 1: [1 / L] * L, 2: a, 3: b}[case["mode"]]
    lo, hi = 1.0, float(n_vis)
    total = min(max(math.floor(r * n_vis * L + 0.5), L), L * n_vis)
    x, free, left = [0.0] * L, set(range(L)), float(total)
    while free:
        whole = sum(share[l] for l in sorted(free))
        for l in free:
            x[l] = share[l] / whole * left if whole > 0 else left / len(free)
        over = sum(x[l] - hi for l in free if x[l] > hi)
        under = sum(lo - x[l] for l in free if x[l] < lo)
        if over == 0.0 and under == 0.0:
            break
        pin = [l for l in free if (x[l] > hi if over >= under else x[l] < lo)]
        for l in pin:
            x[l] = hi if over >= under else lo
            left -= x[l]
            free.discard(l)
    k = [max(1, min(math.floor(v), n_vis)) for v in x]
    frac = [v - n for v, n in zip(x, k)]
    rest = total - sum(k)
    while rest > 0:
        best = max((l for l in range(L) if k[l] < n_vis), key=lambda l: (frac[l], -l), default=None)
        if best is None:
            break
        k[best] += 1
        frac[best] = -1.0
        rest -= 1
    return k


def exact(case, seed):
    device = torch.device("cuda:0")
    seqs, q, k, v, qn, kn, vn = _tensors(case, seed, device)
    L, B, hq, hkv, d = case["L"], case["B"], case["hq"], case["hkv"], case["d"]
    g = hq // hkv
    out = torch.empty((case["steps"], L, B, hq, d), dtype=torch.float64, device=device)
    for b, s in enumerate(seqs):
        scores, s_t, s_k = [], [], []
        for l in range(L):
            kb = k[l][b, :, :s.seq_len].double()
            qb = q[l][b].double()
            imp = torch.zeros((hkv, s.vis_len), dtype=torch.float64, device=device)
            kv = kb[:, s.vis_start:s.text_start]
            if case["kind"] == "visual":
                pos = torch.arange(s.win_len, device=device) + (s.win_start - s.vis_start)
                hidden = torch.arange(s.vis_len, device=device)[None, :] > pos[:, None]
                for h in range(hq):
                    logits = (qb[h, :s.win_len] @ kv[h // g].T / math.sqrt(d)).masked_fill(hidden, -math.inf)
                    imp[h // g] += torch.softmax(logits, dim=1).mean(dim=0) / g
            else:
                w0 = s.win_start - s.text_start
                for h in range(hq):
                    kw = kb[h // g, s.win_start:s.win_start + s.win_len]
                    if case["alpha"] == 0.0:
                        rows = torch.arange(s.win_len, device=device)
                    else:
                        ref = kw @ qb[h, w0 + s.win_len - 1] / math.sqrt(d)
                        rows = torch.nonzero(torch.exp(ref - ref.max()) >= case["alpha"])[:, 0]
                    qe = qb[h, w0 + rows]
                    text = qe @ kw[rows].T
                    if case["causal"]:
                        text = text.masked_fill(rows[None, :] > rows[:, None], -math.inf)
                    logits = torch.cat([qe @ kv[h // g].T, text], dim=1) / math.sqrt(d)
                    imp[h // g] += torch.softmax(logits, dim=1)[:, :s.vis_len].mean(dim=0) / g
            scores.append(imp)
            n = s.vis_len
            c = imp - imp.mean(dim=1, keepdim=True)
            sigma = (c.square().sum(dim=1) / max(1, n - 1)).sqrt()
            flat = sigma <= 1e-6 * imp.mean(dim=1).abs()
            skew = n / max(1.0, (n - 1.0) * (n - 2.0)) * c.pow(3).sum(dim=1) / sigma.pow(3)
            skew = torch.where(flat, torch.zeros_like(skew), skew) if n >= 3 else torch.zeros_like(skew)
            s_t.append(imp.sum(dim=1).mean())
            s_k.append(skew.mean())
        budgets = _budgets(case, s.vis_len, torch.stack(s_t).tolist(), torch.stack(s_k).tolist())
        for l in range(L):
            # ties at the budget go to the lower token index: a stable sort in falling order
            kept = torch.sort(torch.sort(scores[l], dim=1, descending=True, stable=True)[1][:, :budgets[l]], dim=1)[0]
            rows = torch.cat([torch.arange(s.vis_start, device=device).expand(hkv, -1), s.vis_start + kept,
                              torch.arange(s.text_start, s.seq_len, device=device).expand(hkv, -1)], dim=1)
            rows = rows[:, :, None].expand(-1, -1, d)
            kc = torch.cat([k[l][b].double().gather(1, rows), kn[:, l, b].double().transpose(0, 1)], dim=1)
            vc = torch.cat([v[l][b].double().gather(1, rows), vn[:, l, b].double().transpose(0, 1)], dim=1)
            t0 = rows.shape[1]
            qs = qn[:, l, b].double().view(case["steps"], hkv, g, d).transpose(0, 1).reshape(hkv, case["steps"] * g, d)
            step = torch.arange(case["steps"], device=device).repeat_interleave(g)
            later = torch.arange(kc.shape[1], device=device)[None, :] > t0 + step[:, None]
            p = torch.softmax((qs @ kc.transpose(1, 2).contiguous() / math.sqrt(d)).masked_fill(later, -math.inf), dim=2)
            out[:, l, b] = (p @ vc).view(hkv, case["steps"], g, d).transpose(0, 1).reshape(case["steps"], hq, d)
    return out
