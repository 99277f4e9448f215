"""What a user of this framework has it do, as measurable cases.

Three kinds of pass, each through the Python binding:

- ``serve``: a batch of requests through attention layers.  The cache is emptied, the prompts
  compacted (``prefill``), then ``steps`` tokens decoded; with ``park`` the compressed caches are
  exported at the end, as a session that is set aside.  With ``graph`` the same calls are captured
  once, when the program starts, and a pass is one replay (a serving loop for small batches).
- ``attend``: prompts through one layer with attention for every prompt token
  (``prefill_attend``), then the first decoded token.
- ``train``: the training-time forward and backward of one layer.

Layer shapes are those of ``workloads/synthetic.py`` and of the tests; inputs have that module's
distributions (N(0, 1) activations, decision logits that append with probability 1 / CR).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2403_09636_amd as dmc

DEVICE = "cuda"
SERVE = dict(kind="serve", layers=1, batch=1, hq=32, hkv=32, d=128, dtype="bf16", page=32, n=1024,
             steps=16, cr="mix", ragged=False, fused=False, window=0, omega="lead",
             decision="per_head", bias=0.0, graph=False, park=False)
ATTEND = dict(SERVE, kind="attend", steps=1)
TRAIN = dict(kind="train", batch=1, hq=32, hkv=32, d=128, dtype="bf16", n=1024, window=12,
             omega="lead", cr="mix")


def listed():
    return [
        # The parity workload "tiny": one sequence from an empty cache, four small heads, fp32,
        # called step by step: nothing but latency.
        dict(SERVE, name="tiny_fp32", hq=4, hkv=4, d=64, dtype="fp32", n=0, steps=64, park=True),
        # One chat turn on four layers of the 7B shape, then parked; captured in a graph.
        dict(SERVE, name="chat_b1_graph", layers=4, n=1024, steps=8, graph=True, park=True),
        # The Llama-2-7B layer workload: batch 16, 4096-token prompts, then decoding.
        dict(SERVE, name="serve_7b", batch=16, n=4096, steps=32),
        # The Llama-2-70B grouped-query layer; prompt compaction weighs as much as decoding.
        dict(SERVE, name="serve_70b", batch=32, hq=64, hkv=8, n=4096, steps=8, cr="two"),
        # The 13B shape at long context with very uneven heads (10 % of them keep everything).
        dict(SERVE, name="serve_skew", batch=6, hq=40, hkv=40, n=8192, steps=16, cr="skew"),
        # Ragged prompts from a fused projection, grouped-query heads, window grouping as the
        # model was trained with (w = 12), importance averaged over the group, caches parked.
        dict(SERVE, name="serve_window_ragged", batch=13, hq=32, hkv=8, n=1999, steps=24,
             ragged=True, fused=True, window=12, omega="group_mean", park=True),
        # Prompt attention of the 7B layer, and of the 70B layer with ragged prompts.
        dict(ATTEND, name="attend_7b", batch=4, n=4096),
        dict(ATTEND, name="attend_70b_ragged", batch=4, hq=64, hkv=8, n=4096, cr="two",
             ragged=True, fused=True),
        # A short odd prompt in fp32 (debugging and parity work runs in fp32).
        dict(ATTEND, name="attend_fp32_odd", batch=3, hq=16, hkv=8, d=64, dtype="fp32", n=777,
             page=16, ragged=True),
        # One 7B layer of continued pre-training: 4096-token sequences, c = 5, tau = 0.1, w = 12.
        dict(TRAIN, name="train_7b", batch=2, n=4096),
        # A grouped-query layer at an odd sequence length.
        dict(TRAIN, name="train_gqa_odd", batch=3, hq=32, hkv=8, n=1501),
        # fp32 training at the size of a gradient check or a small model.
        dict(TRAIN, name="train_fp32", batch=2, hq=8, hkv=4, d=64, dtype="fp32", n=640),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["serve", "serve", "attend", "attend", "train", "train"])
    fp32 = rng.random() < 0.25
    g = rng.choice([1, 1, 2, 4, 8])
    hkv = rng.choice([4, 8, 16, 32]) if g <= 2 else rng.choice([2, 4, 8])
    shape = dict(hq=hkv * g, hkv=hkv, d=rng.choice([64, 128, 128]),
                 dtype="fp32" if fp32 else "bf16")
    if kind == "train":
        n = _log_int(rng, 48, 900 if fp32 else 4096)
        top = (8 << 20 if fp32 else 512 << 20) * 2 // (n * n * hkv * g)   # (query, key) pairs
        return dict(TRAIN, **shape, batch=rng.randint(1, max(1, min(6, top))), n=n,
                    window=rng.choice([1, 5, 12, 12, 12, 31]),
                    omega=rng.choice(["lead", "lead", "uniform"]), cr=rng.choice(["mix", "two"]))
    common = dict(shape, cr=rng.choice(["mix", "two", "skew"]), ragged=rng.random() < 0.5,
                  fused=rng.random() < 0.5, window=rng.choice([0, 0, 0, 4, 12]),
                  omega=rng.choice(["lead", "lead", "group_mean", "uniform"]),
                  decision=rng.choice(["per_head", "per_head", "per_head", "shared_layer"]),
                  bias=rng.choice([0.0, 0.0, 1.5]), page=rng.choice([16, 32, 32, 32, 64]))
    if kind == "attend":
        n = _log_int(rng, 24, 900 if fp32 else 4096)
        top = (12 << 20 if fp32 else 512 << 20) * 2 // (n * n * hkv * g)
        return dict(ATTEND, **common, n=n, batch=rng.randint(1, max(1, min(6, top))))
    n = _log_int(rng, 24, 8192)
    layers = rng.randint(1, 3) if n < 2000 else 1
    row = n * hkv * shape["d"] * (8 if fp32 else 4) * layers   # bytes of one request's prompt K, V
    top = max(1, min(40, (384 << 20) // row))
    return dict(SERVE, **dict(common, n=n, batch=_log_int(rng, 1, top), layers=layers,
                              steps=rng.randint(4, 24), graph=rng.random() < 0.4,
                              park=rng.random() < 0.3))


# ---------------------------------------------------------------------------
# Inputs and passes
# ---------------------------------------------------------------------------

def _crs(case):
    """Compression ratio of every kv head: 1, 2, 4, 8 in turn; 2; or every tenth head 1 and the
    others spread over 16 .. 32."""
    h = case["hkv"]
    if case["cr"] == "two":
        return np.full(h, 2.0)
    if case["cr"] == "skew":
        return np.array([1.0 if i % 10 == 3 else 16.0 * 2.0 ** ((i * 7 % 10) / 9) for i in range(h)])
    return np.array([(1.0, 2.0, 4.0, 8.0)[i % 4] for i in range(h)])


def _dtype(case):
    return torch.float32 if case["dtype"] == "fp32" else torch.bfloat16


def _generator(seed, stream):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed((seed * 1009 + stream) & 0x7FFFFFFFFFFF)
    return gen


def _qkv(case, gen, lead, fused=False):
    """q [*lead, Hq, d], k, v [*lead, Hkv, d] ~ N(0, 1), k[..., 0] decision logits that append
    with probability 1 / CR; three tensors, or views of one projection."""
    hq, hkv, d, dt = case["hq"], case["hkv"], case["d"], _dtype(case)

    def rows(h):
        return torch.randn((*lead, h, d), generator=gen, device=DEVICE, dtype=dt)

    if fused:
        x = rows(hq + 2 * hkv)
        q, k, v = x[..., :hq, :], x[..., hq:hq + hkv, :], x[..., hq + hkv:, :]
    else:
        q, k, v = rows(hq), rows(hkv), rows(hkv)
    u = torch.rand((*lead, hkv), generator=gen, device=DEVICE).clamp(1e-6, 1 - 1e-6)
    lam = torch.log(u) - torch.log1p(-u)
    cr = torch.as_tensor(_crs(case), dtype=torch.float32, device=DEVICE).expand_as(lam)
    logits = torch.where(cr > 1, lam + torch.log((cr - 1).clamp_min(1e-30)), -(1 + lam.abs()))
    k[..., 0] = (logits + case["bias"]).to(dt)
    return q, k, v


def _request_inputs(case, seed):
    """Prompts per layer, prompt lengths, and the decode steps' inputs per layer."""
    B, n, S = case["batch"], case["n"], case["steps"]
    prompts, tokens = [], []
    for layer in range(case["layers"]):
        prompts.append(_qkv(case, _generator(seed, 2 * layer), (B, n), case["fused"]) if n else None)
        tokens.append(_qkv(case, _generator(seed, 2 * layer + 1), (S, B)))
    lens = None
    if case["ragged"] and n:
        lens = torch.randint(max(1, n // 4), n + 1, (B,), generator=_generator(seed, 999),
                             device=DEVICE, dtype=torch.int32)
        lens[B // 2] = n
    return prompts, lens, tokens


def _train_inputs(case, seed):
    """q, k, v ~ N(0, 1) with k[..., 0] = c + log(CR - 1) + N(0, 0.3) (c - 3 for CR 1), logistic
    noise, the incoming gradient, and the compression loss's gradient (one value)."""
    gen = _generator(seed, 0)
    B, n, hq, hkv, d, dt = (case["batch"], case["n"], case["hq"], case["hkv"], case["d"],
                            _dtype(case))

    def rows(h):
        return torch.randn((B, n, h, d), generator=gen, device=DEVICE, dtype=dt)

    q, k, v, dout = rows(hq), rows(hkv), rows(hkv), rows(hq)
    cr = torch.as_tensor(_crs(case), dtype=torch.float32, device=DEVICE)
    k0 = torch.where(cr > 1, 5.0 + torch.log((cr - 1).clamp_min(1e-30)), torch.full_like(cr, 2.0))
    k[..., 0] = (k0 + 0.3 * torch.randn((B, n, hkv), generator=gen, device=DEVICE)).to(dt)
    u = torch.rand((B, n, hkv), generator=gen, device=DEVICE).clamp(1e-6, 1 - 1e-6)
    noise = torch.log(u) - torch.log1p(-u)
    return q, k, v, noise, dout, torch.full((B, n, hkv), -0.05, device=DEVICE)


def prepare(case, seed):
    if case["kind"] == "train":
        cfg = dmc.make_train_config(case["batch"], case["n"], case["hq"], case["hkv"], case["d"],
                                    case["dtype"], window=case["window"], omega_src=case["omega"])
        return {"case": case, "trainer": dmc.DMCTrainer(cfg, DEVICE),
                "inputs": _train_inputs(case, seed)}
    B, n, S, L = case["batch"], case["n"], case["steps"], case["layers"]
    cfg = dmc.make_config(L, B, case["hq"], case["hkv"], case["d"], case["dtype"],
                          page_size=case["page"], max_slots_per_seq=n + S,
                          max_prompt_len=max(n, 1), decision_bias=case["bias"],
                          omega_src=case["omega"], decision_src=case["decision"],
                          window=case["window"])
    state = {"case": case, "cache": dmc.DMCCache(cfg, DEVICE),
             "inputs": _request_inputs(case, seed),
             "out": torch.empty((L, S, B, case["hq"], case["d"]), dtype=_dtype(case), device=DEVICE),
             "slots": torch.empty((L, S, B, case["hkv"]), dtype=torch.int32, device=DEVICE)}
    if case["kind"] == "attend":
        state["prompt_out"] = torch.empty((B, n, case["hq"], case["d"]), dtype=_dtype(case),
                                          device=DEVICE)
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _serve(state)
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            state["captured"] = _serve(state)
        state["graph"] = graph
    return state


def _serve(state):
    case, cache = state["case"], state["cache"]
    prompts, lens, tokens = state["inputs"]
    cache.reset()
    if case["n"]:
        for layer, (q, k, v) in enumerate(prompts):
            if case["kind"] == "attend":
                cache.prefill_attend(layer, k, v, q, out=state["prompt_out"], prompt_lens=lens)
            else:
                cache.prefill(layer, k, v, q, prompt_lens=lens)
    for s in range(case["steps"]):
        for layer, (q, k, v) in enumerate(tokens):
            cache.decode_step(layer, q[s], k[s], v[s], out=state["out"][layer, s],
                              slot_index=state["slots"][layer, s])
    result = {"out": state["out"], "slots": state["slots"]}
    if case["kind"] == "attend":
        result["prompt_out"] = state["prompt_out"]
    if case["park"]:
        result["parked"] = [cache.export(layer) for layer in range(case["layers"])]
    return result


def run(state):
    if state["case"]["kind"] == "train":
        trainer, (q, k, v, noise, dout, dalpha) = state["trainer"], state["inputs"]
        alpha = torch.empty_like(noise)
        out = trainer.forward(q, k, v, noise, alpha=alpha)
        dq, dk, dv = trainer.backward(q, k, v, noise, out, dout, dalpha=dalpha)
        return {"out": out, "alpha": alpha, "dq": dq, "dk": dk, "dv": dv}
    if "graph" in state:
        state["graph"].replay()
        return state["captured"]
    return _serve(state)


# ---------------------------------------------------------------------------
# Work and tolerance
# ---------------------------------------------------------------------------

def work(case):
    B, n, hq, hkv, d = (case[x] for x in ("batch", "n", "hq", "hkv", "d"))
    es, G = (4 if case["dtype"] == "fp32" else 2), hq // hkv
    if case["kind"] == "train":
        pairs = B * hq * n * (n + 1) / 2
        rows = B * n * d * es
        return {"bytes": rows * (4 * hq + 4 * hkv) + 3 * 4 * B * n * hkv, "flops": 12 * d * pairs}
    # prompt lengths uniform over [n / 4, n] when ragged
    tokens, squares = (0.625 * n, 0.4375 * n * n) if case["ragged"] else (n, n * n)
    crs = _crs(case)
    if case["decision"] == "shared_layer":
        crs = np.full(hkv, crs[0])
    L, S = case["layers"], case["steps"]
    slots = [min(tokens, 1 + tokens / c) if n else 0 for c in crs]   # after the prompt, per head
    row = 2 * d * es                                                 # one K and V row
    moved = B * sum(tokens * (row + 2 * es) + s * row for s in slots)
    flops = B * hkv * tokens * 4 * d
    if case["kind"] == "attend":
        moved += 2 * B * tokens * hq * d * es
        flops += 4 * d * G * B * sum(squares / (2 * c) + tokens for c in crs)
    for s in range(S):
        held = B * sum(x + s / c for x, c in zip(slots, crs))
        moved += held * row + B * hkv * (row + (2 * G + 2) * d * es + 16) + 4 * held / case["page"]
        flops += 4 * d * G * held
    if case["park"]:
        moved += B * hkv * row * (n + S) + B * sum(slots) * row
    return {"bytes": L * moved, "flops": L * flops}


def tolerance(case):
    """About four times the distance from the 64-bit values that every output was measured to
    have (bf16 0.002 - 0.004, mostly the rounding of the output itself and of the probabilities;
    fp32 1e-7 - 9e-7).  Slot indices are whole numbers and exact."""
    return {"rel": 5e-6} if case["dtype"] == "fp32" else {"rel": 0.012}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------

def _omega(case, q):
    """Importance [..., Hkv] of queries [..., Hq, d], and alpha's source heads."""
    hkv, G = case["hkv"], case["hq"] // case["hkv"]
    w = torch.sigmoid(q[..., 0].double()).clamp_min(2.0 ** -100).unflatten(-1, (hkv, G))
    w = w.mean(-1) if case["omega"] == "group_mean" else w[..., 0]
    return torch.ones_like(w) if case["omega"] == "uniform" else w


def _neurons(case, q, k):
    """(accumulate, omega) [..., Hkv] of each token."""
    acc = k[..., 0].float() > case["bias"]
    w = _omega(case, q)
    if case["decision"] == "shared_layer":
        acc, w = acc[..., :1].expand_as(acc), w[..., :1].expand_as(w)
    return acc, w


def _zero_first(x):
    x = x.double()
    x[..., 0] = 0
    return x


class _Exact64:
    """One layer's caches [B, Hkv] in float64: slots, counts, z, and the last w raw tokens."""

    def __init__(self, case):
        B, h, d = case["batch"], case["hkv"], case["d"]
        cap = case["n"] + case["steps"]
        self.case = case
        self.K = torch.zeros((B, h, cap, d), dtype=torch.float64, device=DEVICE)
        self.V = torch.zeros_like(self.K)
        self.len = torch.zeros((B, h), dtype=torch.int64, device=DEVICE)
        self.z = torch.zeros((B, h), dtype=torch.float64, device=DEVICE)
        w = case["window"]
        self.recent = [torch.zeros((B, h, w, x), dtype=torch.float64, device=DEVICE)
                       for x in (d, d, 1)]

    def prompt(self, b, q, k, v, nb, attend):
        """Row b's prompt q [n, Hq, d], k, v [n, Hkv, d]; attention outputs if asked."""
        case, W = self.case, self.case["window"]
        n, hq, d = q.shape
        G = hq // case["hkv"]
        acc, om = _neurons(case, q[:nb], k[:nb])
        kz, vd = _zero_first(k[:nb]), v[:nb].double()
        out = torch.zeros((n, hq, d), dtype=torch.float64, device=DEVICE) if attend else None
        t = torch.arange(nb, device=DEVICE)
        for h in range(case["hkv"]):
            start = ~acc[:, h]
            start[0] = True
            seg = torch.cumsum(start, 0) - 1
            L = int(seg[-1]) + 1
            first = torch.nonzero(start)[:, 0]                     # [L]
            end = torch.cat([first[1:], torch.tensor([nb], device=DEVICE)])
            lo = first[seg] if W == 0 else torch.maximum(first[seg], t - W + 1)
            w = om[:, h, None]
            if W:
                w_slot = torch.where((t >= end[seg] - W)[:, None], w, torch.zeros_like(w))
            else:
                w_slot = w
            zs = torch.zeros((L, 1), dtype=torch.float64, device=DEVICE).index_add_(0, seg, w_slot)
            Ks = torch.zeros((L, d), dtype=torch.float64, device=DEVICE)
            Vs = torch.zeros_like(Ks)
            Ks.index_add_(0, seg, w_slot * kz[:, h])
            Vs.index_add_(0, seg, w_slot * vd[:, h])
            Ks /= zs
            Vs /= zs
            self.K[b, h, :L], self.V[b, h, :L] = Ks, Vs
            self.len[b, h], self.z[b, h] = L, zs[-1, 0]
            for i in range(W):
                src = nb - W + i
                if src >= int(first[-1]):
                    for buf, val in zip(self.recent, (kz[src, h], vd[src, h], w[src])):
                        buf[b, h, i] = val
            if not attend:
                continue

            def open_mean(x):   # running mean of each token's own segment
                c = torch.cat([torch.zeros((1, x.shape[1]), dtype=torch.float64, device=DEVICE),
                               torch.cumsum(w * x, 0)])
                return c[1:] - c[lo]

            zo = open_mean(torch.ones_like(w))
            Ko, Vo = open_mean(kz[:, h]) / zo, open_mean(vd[:, h]) / zo
            hidden = torch.arange(L, device=DEVICE)[None, :] >= seg[:, None]
            for j in range(h * G, (h + 1) * G):
                qj = _zero_first(q[:nb, j])
                s = torch.cat([(qj @ Ks.t().contiguous()).masked_fill_(hidden, -math.inf),
                               (qj * Ko).sum(1, keepdim=True)], 1) / math.sqrt(d)
                p = torch.softmax(s, 1)
                out[:nb, j] = p[:, :L] @ Vs + p[:, L:] * Vo
        return out

    def step(self, q, k, v):
        case, W = self.case, self.case["window"]
        B, h, cap, d = self.K.shape
        G = q.shape[1] // h
        acc, om = _neurons(case, q, k)
        kz, vd = _zero_first(k), v.double()
        acc = acc & (self.len > 0)
        if W:
            keep = acc[..., None, None].double()
            for buf, val in zip(self.recent, (kz, vd, om[..., None])):
                buf[:, :, :-1] = buf[:, :, 1:].clone()
                buf[:, :, -1] = val
            self.recent[2][:, :, :-1] *= keep
            wk, wv, ww = self.recent
            znew = ww.sum((2, 3))
            ck, cv = (ww * wk).sum(2) / znew[..., None], (ww * wv).sum(2) / znew[..., None]
        slot = torch.where(acc, self.len - 1, self.len)
        at = slot[..., None, None].expand(B, h, 1, d)
        if not W:
            zold = torch.where(acc, self.z, torch.zeros_like(self.z))
            znew = zold + om
            ck, cv = ((x.gather(2, at)[:, :, 0] * zold[..., None] + y * om[..., None])
                      / znew[..., None] for x, y in ((self.K, kz), (self.V, vd)))
        self.K.scatter_(2, at, ck[:, :, None])
        self.V.scatter_(2, at, cv[:, :, None])
        self.z = znew
        self.len = slot + 1
        qz = _zero_first(q).reshape(B * h, G, d)
        s = torch.bmm(self.K.reshape(B * h, cap, d), qz.transpose(1, 2).contiguous()) / math.sqrt(d)
        past = torch.arange(cap, device=DEVICE)[None, :] >= self.len.reshape(-1, 1)
        p = torch.softmax(s.masked_fill_(past[..., None], -math.inf), 1)
        out = torch.bmm(p.transpose(1, 2).contiguous(), self.V.reshape(B * h, cap, d))
        return out.reshape(B, h * G, d), slot.to(torch.int32)


def _exact_serve(case, seed):
    prompts, lens, tokens = _request_inputs(case, seed)
    outs, slots, prompt_out, parked = [], [], None, []
    for layer in range(case["layers"]):
        ref = _Exact64(case)
        if case["n"]:
            q, k, v = prompts[layer]
            rows = []
            for b in range(case["batch"]):
                nb = case["n"] if lens is None else int(lens[b])
                rows.append(ref.prompt(b, q[b], k[b], v[b], nb, case["kind"] == "attend"))
            if case["kind"] == "attend":
                prompt_out = torch.stack(rows)
        got = [ref.step(*(x[s] for x in tokens[layer])) for s in range(case["steps"])]
        outs.append(torch.stack([o for o, _ in got]))
        slots.append(torch.stack([s for _, s in got]))
        parked.append((ref.K, ref.V, ref.z))
    result = {"out": torch.stack(outs), "slots": torch.stack(slots)}
    if case["kind"] == "attend":
        result["prompt_out"] = prompt_out
    if case["park"]:
        result["parked"] = parked
    return result


def _exact_train(case, seed):
    q, k, v, noise, dout, dalpha = _train_inputs(case, seed)
    n, hkv, d, W = case["n"], case["hkv"], case["d"], case["window"]
    G = case["hq"] // hkv
    res = {"out": torch.empty_like(q, dtype=torch.float64),
           "alpha": torch.empty_like(noise, dtype=torch.float64)}
    grads = [torch.empty_like(x, dtype=torch.float64) for x in (q, k, v)]
    future = torch.ones((n, n), dtype=torch.bool, device=DEVICE).triu(1)
    eye = torch.eye(n, dtype=torch.bool, device=DEVICE)
    for b in range(case["batch"]):
        for h in range(hkv):
            heads = slice(h * G, (h + 1) * G)
            qu, ku, vu = (x.double().requires_grad_(True)
                          for x in (q[b, :, heads], k[b, :, h], v[b, :, h]))
            x = (ku[:, 0] - 5.0 + noise[b, :, h].double()) / float(np.float32(0.1))
            al = torch.sigmoid(x)
            om = torch.sigmoid(qu[:, 0, 0]).clamp_min(2.0 ** -100)
            if case["omega"] == "uniform":
                om = torch.ones_like(om)
            kz = torch.cat([torch.zeros_like(ku[:, :1]), ku[:, 1:]], 1)
            # state j: tokens j, j - 1, .. j - w + 1, weights omega_t prod_{r = t + 1 .. j} alpha_r
            P, sk, sv, z = torch.ones_like(al), 0.0, 0.0, 0.0
            for i in range(min(W, n)):
                pad = (0, 0, i, 0)
                c = P * torch.nn.functional.pad(om[:n - i], (i, 0))
                sk = sk + c[:, None] * torch.nn.functional.pad(kz[:n - i], pad)
                sv = sv + c[:, None] * torch.nn.functional.pad(vu[:n - i], pad)
                z = z + c
                P = P * torch.nn.functional.pad(al[:n - i], (i, 0))
            K, V = sk / z[:, None], sv / z[:, None]
            col = torch.cat([torch.nn.functional.logsigmoid(-x[1:]), torch.zeros_like(x[:1])])
            bias = col[None, :].expand(n, n).masked_fill(eye, 0.0).masked_fill(future, -math.inf)
            Kt = K.t().contiguous()
            loss = (al * dalpha[b, :, h].double()).sum()
            for j in range(G):
                qz = torch.cat([torch.zeros_like(qu[:, j, :1]), qu[:, j, 1:]], 1)
                o = torch.softmax(qz @ Kt / math.sqrt(d) + bias, 1) @ V
                res["out"][b, :, h * G + j] = o.detach()
                loss = loss + (o * dout[b, :, h * G + j].double()).sum()
            res["alpha"][b, :, h] = al.detach()
            gq, gk, gv = torch.autograd.grad(loss, (qu, ku, vu))
            grads[0][b, :, heads], grads[1][b, :, h], grads[2][b, :, h] = gq, gk, gv
    res.update(zip(("dq", "dk", "dv"), grads))
    return res


def exact(case, seed):
    """What ``run`` returns, in float64 from the definitions (on the GPU, plain torch)."""
    return _exact_train(case, seed) if case["kind"] == "train" else _exact_serve(case, seed)
