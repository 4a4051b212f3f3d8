"""The calls whose speed matters: what a serving or fine-tuning program makes this library do.

One case is one pass through the public binding (``paper_2607_28848_amd.dsv``) with the buffers, weights, workspace
and (except where the batch changes with every pass) the plan that such a program keeps.  Shapes are the projections
of Llama-3-8B and Llama-3-70B as the workloads of this repository have them, and generic sizes; batches mix one-token
decode segments, prefill segments and fine-tuning segments.  Inputs have the distributions of ``workloads.py``.

Fields of a case:
    what      "fwd", "bwd", "step" (plan, forward and backward) or "adamw"
    set       a key of SETS, or "generic" with K, N and count (projections on one input)
    api       "grouped", "single" or "noalloc" (forward only)
    decode, prefill, prefill_len, ragged, train, train_len, table
              one-token segments; prefill segments and their mean length (ragged: log-normal lengths); fine-tuning
              segments and their length; the number the table's order, lengths and adapters are drawn from
    adapters, rank        adapters of the stack and their rank (0: ranks 8, 16, 32, 64 by turns)
    dropout   LoRA dropout of the fine-tuning rows
    wt        the backward has the transposed weight as well
    keep_h    the forward keeps h for the backward (else the backward computes it again)
    dtype     "bf16" or "f32"
"""
import math
import random

import torch

from paper_2607_28848_amd import dsv

# Projections that share one input run as one call: [[(K, N), ...] for each call].
SETS = {
    "8b_qkv": [[(4096, 4096), (4096, 1024), (4096, 1024)]],
    "8b_o": [[(4096, 4096)]],
    "8b_gate": [[(4096, 14336)]],
    "8b_gate_up": [[(4096, 14336), (4096, 14336)]],
    "8b_down": [[(14336, 4096)]],
    "8b_layer": [[(4096, 4096), (4096, 1024), (4096, 1024)], [(4096, 4096)], [(4096, 14336), (4096, 14336)],
                 [(14336, 4096)]],
    "70b_up_down": [[(8192, 28672)], [(28672, 8192)]],
}
BASE = dict(what="fwd", set="generic", K=0, N=0, count=1, api="grouped", decode=0, prefill=0, prefill_len=0,
            ragged=False, train=0, train_len=0, table=0, adapters=32, rank=16, dropout=0.0, wt=False, keep_h=True,
            dtype="bf16")


def listed():
    return [dict(BASE, name=name, **fields) for name, fields in (
        # One decode step of a small serving batch through the attention projections: launches and latency.
        ("decode8_qkv", dict(set="8b_qkv", decode=8, adapters=32, rank=16)),
        # One decode step of a busy server through the wide MLP projections, adapters of several ranks.
        ("decode64_gate_up", dict(set="8b_gate_up", decode=64, adapters=64, rank=0)),
        # A chunked-prefill step: decode tokens beside a ragged chunk, from a loop that must not allocate.
        ("chunk365_o_noalloc", dict(set="8b_o", api="noalloc", decode=48, prefill=1, prefill_len=317, rank=16)),
        # Plain prefill of several prompts of uneven length, inference only.
        ("prefill_ragged_gate_up", dict(set="8b_gate_up", prefill=6, prefill_len=250, ragged=True, table=3, rank=0)),
        # The paper's fine-tuning setting: 256 training tokens with dropout 0.05 co-batched with serving traffic,
        # forward and backward of the attention projections.
        ("ft256_dropout_qkv_step", dict(what="step", set="8b_qkv", decode=32, prefill=2, prefill_len=256, train=2,
                                        train_len=128, dropout=0.05, wt=True)),
        # The backward of 256 accumulated fine-tuning tokens alone, as the paper's backward process runs it.
        ("ft256_gate_up_bwd", dict(what="bwd", set="8b_gate_up", train=2, train_len=128, wt=True)),
        # Residual-only retention without a second copy of the weight: h computed again, one long ragged sample.
        ("ft1000_down_recompute_bwd", dict(what="bwd", set="8b_down", api="single", train=1, train_len=1000,
                                           keep_h=False)),
        # The framework's flagship batch, one transformer layer as a model can call it (q/k/v, o, gate/up, down).
        ("mixed_8b_layer_step", dict(what="step", set="8b_layer", prefill=8, prefill_len=512, train=2,
                                     train_len=1024, wt=True)),
        # Decode-heavy co-serving: 256 one-token entries over 64 adapters of four ranks and one long training sample.
        ("decode_heavy_gate_step", dict(what="step", set="8b_gate", api="single", decode=256, train=1,
                                        train_len=2048, adapters=64, rank=0)),
        # The largest: the MLP projections of the 70B layer, ragged prefill and 8192 fine-tuning tokens, rank 64.
        ("mixed_70b_up_down_step", dict(what="step", set="70b_up_down", prefill=16, prefill_len=510, ragged=True,
                                        train=4, train_len=2048, adapters=16, rank=64, wt=True)),
        # fp32 layer, forward and backward (the smallest workload of the benchmark).
        ("f32_512_step", dict(what="step", K=512, N=512, api="single", prefill=2, prefill_len=96, train=1,
                              train_len=64, adapters=2, rank=8, dtype="f32")),
        # The optimizer step of one layer's adapter.
        ("adamw_8b_layer", dict(what="adamw", set="8b_layer", train=1, train_len=256)),
    )]


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    c = dict(BASE, table=rng.randrange(1, 1 << 20))
    kind = rng.choice(("decode", "decode", "prefill", "prefill", "step", "step", "bwd", "f32", "adamw"))
    c["set"] = rng.choice(("8b_qkv", "8b_o", "8b_gate_up", "8b_down", "8b_gate", "generic"))
    if c["set"] == "generic":
        c.update(K=8 * log_int(64, 1024), N=8 * log_int(64, 1024), count=rng.randint(1, 3))
    c["adapters"], c["rank"] = log_int(2, 64), rng.choice((8, 16, 16, 32, 64, 0))
    n_proj = c["count"] if c["set"] == "generic" else len(SETS[c["set"]][0])
    if kind == "decode":
        c.update(decode=log_int(1, 256))
    elif kind == "prefill":
        c.update(decode=rng.choice((0, log_int(1, 64))), prefill=rng.randint(1, 6), prefill_len=log_int(16, 400),
                 ragged=rng.random() < 0.6)
    elif kind in ("step", "bwd"):
        c.update(what=kind, train=rng.randint(1, 3), train_len=log_int(32, 1024), keep_h=rng.random() < 0.75,
                 wt=rng.random() < 0.5, dropout=rng.choice((0.0, 0.0, 0.05)))
        if kind == "step":
            c.update(decode=rng.choice((0, log_int(1, 128))), prefill=rng.randint(0, 4),
                     prefill_len=log_int(32, 512), ragged=rng.random() < 0.6)
    elif kind == "f32":
        c.update(what=rng.choice(("fwd", "step")), set="generic", K=8 * log_int(16, 128), N=8 * log_int(16, 128),
                 count=1, dtype="f32", prefill=rng.randint(1, 3), prefill_len=log_int(8, 128), train=1,
                 train_len=log_int(16, 128), adapters=rng.randint(2, 8), rank=rng.choice((8, 16)))
        n_proj = 1
    else:
        c.update(what="adamw", train=1, train_len=log_int(16, 256))
    if n_proj == 1 and not c["wt"] and c["what"] != "adamw":
        c["api"] = rng.choice(("grouped", "single", "noalloc") if c["what"] == "fwd" and c["dtype"] == "bf16"
                              else ("grouped", "single"))
    return c


# ---- the batch ------------------------------------------------------------------------------------------------------
def calls(case):
    """[[(K, N), ...]]: the projections of each call."""
    if case["set"] == "generic":
        return [[(case["K"], case["N"])] * case["count"]]
    return SETS[case["set"]]


def table(case):
    """(segments, ranks): the segment table and the adapters' ranks; training segments are on adapter 1 % adapters."""
    rng = random.Random(case["table"])
    n_ad = case["adapters"]
    pieces = [(1, rng.randrange(n_ad), 0) for _ in range(case["decode"])]
    for _ in range(case["prefill"]):
        n = case["prefill_len"]
        if case["ragged"]:
            n = max(1, min(4 * n, int(round(rng.lognormvariate(math.log(0.8 * n), 0.7)))))
        pieces.append((n, rng.randrange(n_ad), 0))
    pieces += [(case["train_len"], 1 % n_ad, 1)] * case["train"]
    rng.shuffle(pieces)
    segs, start = [], 0
    for n, a, t in pieces:
        segs.append((start, n, a, t))
        start += n
    ranks = [case["rank"] or (8, 16, 32, 64)[a % 4] for a in range(n_ad)]
    return segs, ranks


def _tokens(segs):
    return sum(s[1] for s in segs), sum(s[1] for s in segs if s[3])


def _rows(segs, dev):
    """(adapter of each row, training rows)."""
    ad = torch.tensor([a for _, n, a, _ in segs for _ in range(n)], device=dev)
    tr = torch.tensor([i for s, n, _, t in segs if t for i in range(s, s + n)], dtype=torch.long, device=dev)
    return ad, tr


def _strided(case, values):
    """values [rows][n] in a buffer with the recommended row stride where the call takes one."""
    if case["api"] != "grouped":
        return values.contiguous()
    n = values.shape[1]
    buf = torch.zeros((values.shape[0], dsv.row_stride(n, dsv.BF16 if case["dtype"] == "bf16" else dsv.F32)),
                      dtype=values.dtype, device=values.device)[:, :n]
    buf.copy_(values)
    return buf


def inputs(case, seed):
    """The tensors of every call: [[dict per projection]], from the seed alone."""
    dev, dt = "cuda", torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    segs, ranks = table(case)
    T, Tt = _tokens(segs)
    r_max = max(ranks)
    gen = torch.Generator(device=dev).manual_seed(1000003 * (seed % (1 << 30)) + case["table"])
    pad = torch.arange(r_max, device=dev)[None, :] >= torch.tensor(ranks, device=dev)[:, None]  # [n_ad][r_max]

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.float32)

    out = []
    for group in calls(case):
        X = _strided(case, normal(T, group[0][0]).to(dt))
        projs = []
        for K, N in group:
            A = (torch.rand((len(ranks), r_max, K), generator=gen, device=dev) * 2 - 1) / math.sqrt(K)
            B = normal(len(ranks), N, r_max) * 0.02
            A.masked_fill_(pad[:, :, None], 0)
            B.masked_fill_(pad[:, None, :], 0)
            p = dict(K=K, N=N, X=X, A=A.to(dt), B=B.to(dt))
            if case["what"] != "adamw":
                p["W"] = _strided(case, (normal(N, K) / math.sqrt(K)).to(dt))
            if case["what"] in ("bwd", "step"):
                p["dY"] = _strided(case, normal(Tt, N).to(dt))
            projs.append(p)
        out.append(projs)
    return out


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    code = dsv.BF16 if case["dtype"] == "bf16" else dsv.F32
    segs, ranks = table(case)
    T, Tt = _tokens(segs)
    r_max, n_ad = max(ranks), len(ranks)
    scales = [2.0] * n_ad
    st = dict(case=case, dev=dev, segs=segs, T=T, ranks=ranks, scales=scales, r_max=r_max, t=0)
    st["calls"] = groups = inputs(case, seed)
    plan = st["plan"] = dsv.segments_build(segs, T, ranks, scales, r_max, device=dev)
    drop = case["dropout"]
    ws = 256
    for ci, group in enumerate(groups):
        shapes = [(p["K"], p["N"]) for p in group]
        for pi, p in enumerate(group):
            K, N = p["K"], p["N"]
            p["H"] = torch.zeros((Tt, r_max), dtype=dt, device=dev) if Tt and case["keep_h"] else None
            if case["what"] in ("fwd", "step"):
                p["Y"] = _strided(case, torch.zeros((T, N), dtype=dt, device=dev))
            if case["what"] in ("bwd", "step"):
                p["dA"] = torch.zeros((n_ad, r_max, K), dtype=torch.float32, device=dev)
                p["dB"] = torch.zeros((n_ad, N, r_max), dtype=torch.float32, device=dev)
                p["dX"] = _strided(case, torch.zeros((Tt, K), dtype=dt, device=dev))
                p["Wt"] = _strided(case, p["W"].t().contiguous()) if case["wt"] else None
            p["drop"] = None
            if drop:
                mask = torch.zeros(dsv.dropout_mask_words(plan, K), dtype=torch.int32, device=dev)
                # a step's backward reads the mask its forward drew; a backward alone draws it from the seed again
                p["drop"] = (drop, 77 + seed % 1000, 16 * ci + pi) + ((mask,) if case["what"] == "step" else ())
            if case["what"] == "bwd" and case["keep_h"]:  # h as the forward left it
                ad, tr = _rows(segs, dev)
                x = p["X"][tr].float()
                if drop:
                    x = x * keep_mask(p["drop"], Tt, K, dev) / (1 - drop)
                p["H"].copy_(x @ p["A"][segs_train_adapter(segs)].float().t())
            if case["what"] == "adamw":
                gen = torch.Generator(device=dev).manual_seed(seed % (1 << 30) + 31 * ci + pi)

                def noise(t, std):
                    return torch.randn(t.shape, generator=gen, device=dev) * std
                p["dA"], p["dB"] = noise(p["A"], 1e-2), noise(p["B"], 1e-2)
                p["A_master"], p["B_master"] = p["A"].float() + noise(p["A"], 1e-6), p["B"].float() + noise(p["B"], 1e-6)
                p["A_m"], p["B_m"] = noise(p["A"], 1e-3), noise(p["B"], 1e-3)
                p["A_v"], p["B_v"] = noise(p["A"], 1e-2).square(), noise(p["B"], 1e-2).square()
        if case["what"] != "adamw":
            if case["api"] == "grouped":
                ws = max(ws, dsv.fwd_grouped_workspace_bytes(plan, code, shapes),
                         dsv.bwd_grouped_workspace_bytes(plan, code, shapes) if Tt else 0)
            else:
                K, N = shapes[0]
                ws = max(ws, dsv.fwd_workspace_bytes(plan, code, K, N),
                         dsv.bwd_workspace_bytes(plan, code, K, N, dropout=drop > 0) if Tt else 0)
    st["workspace"] = torch.empty(ws, dtype=torch.uint8, device=dev)
    return st


def segs_train_adapter(segs):
    return next(a for _, _, a, t in segs if t)


# ---- one pass -------------------------------------------------------------------------------------------------------
def run(st):
    case, plan, ws = st["case"], st["plan"], st["workspace"]
    what, api = case["what"], case["api"]
    if what == "adamw":
        st["t"] += 1
        projs = [p for group in st["calls"] for p in group]
        dsv.adamw_step_grouped(plan, 10 + st["t"], [
            (p["dA"], p["dB"], p["A_master"], p["B_master"], p["A_m"], p["A_v"], p["B_m"], p["B_v"], p["A"], p["B"])
            for p in projs])
        return [[p[k] for k in ("A", "B", "A_master", "B_master", "A_m", "A_v", "B_m", "B_v")] for p in projs]
    if what == "step":  # the batch, and with it the plan, is another one in every step
        plan = dsv.segments_build(st["segs"], st["T"], st["ranks"], st["scales"], st["r_max"], device=st["dev"])
    if what in ("fwd", "step"):
        for group in st["calls"]:
            if api == "grouped":
                drops = [p["drop"] for p in group] if case["dropout"] else None
                dsv.cobatch_fwd_grouped(plan, [(p["X"], p["W"], p["A"], p["B"], p["Y"], p["H"]) for p in group],
                                        workspace=ws, keep_h=case["keep_h"], dropouts=drops)
            elif api == "noalloc":
                p = group[0]
                dsv.cobatch_fwd_noalloc(plan, p["X"], p["W"], p["A"], p["B"], p["Y"], p["H"])
            else:
                p = group[0]
                dsv.cobatch_fwd(plan, p["X"], p["W"], p["A"], p["B"], p["Y"], p["H"], workspace=ws,
                                keep_h=case["keep_h"], dropout=p["drop"])
    if what in ("bwd", "step"):
        for group in reversed(st["calls"]):
            if api == "grouped":
                drops = [p["drop"] for p in group] if case["dropout"] else None
                dsv.lora_bwd_grouped(plan, [(p["X"], p["W"], p["A"], p["B"], p["H"], p["dY"], p["dA"], p["dB"], p["dX"])
                                            for p in group], workspace=ws, dropouts=drops,
                                     wts=[p["Wt"] for p in group] if case["wt"] else None)
            else:
                p = group[0]
                dsv.lora_bwd(plan, p["X"], p["W"], p["A"], p["B"], p["H"], p["dY"], dA=p["dA"], dB=p["dB"], dX=p["dX"],
                             workspace=ws, dropout=p["drop"])
    return [[p[k] for k in _outputs(case)] for group in st["calls"] for p in group]


def _outputs(case):
    keys = ("Y", "H") if case["what"] in ("fwd", "step") and case["train"] and case["keep_h"] else \
        ("Y",) if case["what"] in ("fwd", "step") else ()
    return keys + (("dA", "dB", "dX") if case["what"] in ("bwd", "step") else ())


# ---- the same in 64 bits --------------------------------------------------------------------------------------------
def keep_mask(drop, Tt, K, dev):
    """The elements LoRA dropout keeps (1.0 / 0.0, [Tt][K]): Philox4x32-10 at counter (k / 4, row, offset), key seed."""
    p, seed, offset = drop[:3]
    lo = 0xFFFFFFFF

    def mul(m, c):  # the two 32-bit halves of m * c, 32-bit numbers held in int64
        a, b = (m >> 16) * c, (m & 0xFFFF) * c
        t = a + (b >> 16)
        return t >> 16, ((t & 0xFFFF) << 16) | (b & 0xFFFF)

    c0 = torch.arange((K + 3) // 4, device=dev)[None, :].expand(Tt, -1)
    c1 = torch.arange(Tt, device=dev)[:, None].expand_as(c0)
    c2, c3 = torch.full_like(c0, offset & lo), torch.full_like(c0, offset >> 32)
    k0, k1 = seed & lo, seed >> 32
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c0)
        h1, l1 = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & lo, (k1 + 0xBB67AE85) & lo
    words = torch.stack((c0, c1, c2, c3), dim=-1).reshape(Tt, -1)[:, :K]
    return (words >= math.floor(p * 2.0 ** 32)).double()


def exact(case, seed):
    st = prepare(case, seed)
    dev, segs = st["dev"], st["segs"]
    ad, tr = _rows(segs, dev)
    out = []
    for group in st["calls"]:
        for p in group:
            if case["what"] == "adamw":
                out.append(_exact_adamw(p, segs_train_adapter(segs), st["ranks"], 11))
                continue
            X, W = p["X"].double(), p["W"].double()
            Xa = X.clone()  # the low-rank branch's input
            mask = None
            if case["dropout"] and len(tr):
                mask = keep_mask(p["drop"], len(tr), p["K"], dev) / (1 - case["dropout"])
                Xa[tr] *= mask
            res = {}
            if case["what"] in ("fwd", "step"):
                Y = X @ W.t()
                for a in set(ad.tolist()):
                    rows = (ad == a).nonzero()[:, 0]
                    Y[rows] += 2.0 * (Xa[rows] @ p["A"][a].double().t()) @ p["B"][a].double().t()
                res["Y"] = Y
            if len(tr):
                a = segs_train_adapter(segs)
                A, B, x = p["A"][a].double(), p["B"][a].double(), Xa[tr]
                res["H"] = x @ A.t()
                if case["what"] in ("bwd", "step"):
                    dY = p["dY"].double()
                    h = p["H"].double() if case["what"] == "bwd" and p["H"] is not None else res["H"]
                    g = 2.0 * dY @ B
                    res["dA"], res["dB"] = torch.zeros_like(p["dA"]).double(), torch.zeros_like(p["dB"]).double()
                    res["dA"][a], res["dB"][a] = g.t() @ x, 2.0 * dY.t() @ h
                    low = g @ A
                    res["dX"] = dY @ W + (low * mask if mask is not None else low)
            out.append([res[k] for k in _outputs(case)])
    return out


def _exact_adamw(p, a, ranks, step, lr=1e-3, b1=0.9, b2=0.999, eps=1e-8, wd=0.01):
    r = ranks[a]
    out = {}
    for x in ("A", "B"):
        at = (a, slice(0, r)) if x == "A" else (a, slice(None), slice(0, r))
        w, m, v, low = (p[k].double().clone() for k in (x + "_master", x + "_m", x + "_v", x))
        g = p["d" + x].double()[at]
        m[at] = b1 * m[at] + (1 - b1) * g
        v[at] = b2 * v[at] + (1 - b2) * g * g
        w[at] = w[at] * (1 - lr * wd) - lr * (m[at] / (1 - b1 ** step)) / ((v[at] / (1 - b2 ** step)).sqrt() + eps)
        low[at] = w[at]
        out.update({x: low, x + "_master": w, x + "_m": m, x + "_v": v})
    return [out[k] for k in ("A", "B", "A_master", "B_master", "A_m", "A_v", "B_m", "B_v")]


# ---- what it takes and how exact it is -----------------------------------------------------------------------------
def work(case):
    segs, ranks = table(case)
    T, Tt = _tokens(segs)
    e = 2 if case["dtype"] == "bf16" else 4
    touched = {a for _, _, a, _ in segs}
    flops = nbytes = 0
    for group in calls(case):
        K0 = group[0][0]
        what = case["what"]
        if what in ("fwd", "step"):
            nbytes += e * T * K0
        elif what == "bwd":
            nbytes += e * Tt * K0
        for K, N in group:
            r = ranks[segs_train_adapter(segs)] if Tt else 0
            if what == "adamw":  # gradient, master and moments read; master, moments and bf16 copy written
                nbytes += 30 * r * (K + N)
                flops += 15 * r * (K + N)
                continue
            nbytes += e * N * K + e * sum(ranks[a] for a in touched) * (K + N)
            if what in ("fwd", "step"):
                nbytes += e * T * N + (e * Tt * r if case["keep_h"] else 0)
                flops += 2 * T * K * N + sum(2 * n * ranks[a] * (K + N) for _, n, a, _ in segs)
            if what in ("bwd", "step"):
                nbytes += e * Tt * (N + K) + 4 * r * (K + N)
                flops += 2 * Tt * K * N + 4 * Tt * r * (K + N)
                if not case["keep_h"]:
                    flops += 2 * Tt * K * r
                if what == "bwd" and case["keep_h"]:
                    nbytes += e * Tt * r
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["what"] == "adamw":
        # fp32 elementwise; the bf16 copy of a master next to a rounding boundary differs by one step of 2^-8
        return {"rel": 1e-4, "max": 1e-2}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    # bf16 results and intermediates (h, g) rounded once each: 1.7e-3 .. 2e-3 from the 64-bit result
    return {"rel": 7e-3, "max": 6e-2}
