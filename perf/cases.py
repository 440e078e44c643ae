"""The work that users of this library have it do, as measurable cases: packing a batch, training steps of each model
family and regime, the preference step, and single kernels (attention, a projection, the optimizer) through their own
entry points.  Architectures and length recipes are those of the benchmark configurations, at reduced depth: every layer
of a model does the same work, so one or two stand for all of them.

listed() names the cases, draw() gives others of the same ranges, prepare() builds what a program holds before the call,
run() is one pass, work() what a pass cannot do without, exact() the result in 64-bit torch, tolerance() what another
correct implementation at the same precision may differ by.
"""
import math

import numpy as np
import torch

from paper_2503_22673_amd import binding as B

DEV = "cuda"
SEVEN = ("q", "k", "v", "o", "gate", "up", "down")
# widths, adapter rank and targets, rotary base, length recipe (median, lowest, highest; median 0: uniform), turns, assistant share
ARCH = {
    "tiny": dict(d=128, hq=4, hkv=4, dh=32, ffn=344, vocab=1024, rank=8, alpha=16.0, targets=("q", "k", "v", "o"), base=1e4,
                 lens=(0, 48, 320), share=0.30),
    "1b": dict(d=2048, hq=32, hkv=8, dh=64, ffn=8192, vocab=32000, rank=16, alpha=32.0, targets=SEVEN, base=1e4,
               lens=(1200, 128, 4096), share=0.25),
    "8b": dict(d=4096, hq=32, hkv=8, dh=128, ffn=14336, vocab=128256, rank=64, alpha=128.0, targets=SEVEN, base=5e5,
               lens=(2000, 256, 16384), share=0.20),
    "8x7b": dict(d=4096, hq=32, hkv=8, dh=128, ffn=14336, vocab=32000, rank=16, alpha=32.0, targets=("q", "k", "v", "o", "router"),
                 base=1e6, lens=(0, 64, 1024), share=0.25, experts=8),
}
EPS = 1e-5
BETA = 0.1                                               # of the preference loss
NF4 = (-1.0, -0.6961928009986877, -0.5250730514526367, -0.39491748809814453, -0.28444138169288635, -0.18477343022823334,
       -0.09105003625154495, 0.0, 0.07958029955625534, 0.16093020141124725, 0.24611230194568634, 0.33791524171829224,
       0.44070982933044434, 0.5626170039176941, 0.7229568362236023, 1.0)


def listed():
    return [
        # one batch of host trajectories to packed rows on the device, at the size of an 8B run: once per step, the only upload
        dict(name="pack_8b_batch", kind="pack", arch="8b", rows=4, row_len=16384),
        # the float32 tier on a toy model: what a unit test or a first experiment runs; all latency and launches
        dict(name="step_tiny_fp32", kind="step", arch="tiny", layers=2, rows=1, row_len=512, train="lora", recompute=0, fp32=True),
        # adapters on a quantised base, one short ragged row: the smallest call a program with little data makes
        dict(name="step_1b_nf4_short", kind="step", arch="1b", layers=2, rows=1, row_len=1003, train="nf4", recompute=0, fp32=False),
        # the 1B adapter run at its benchmark batch
        dict(name="step_1b_lora", kind="step", arch="1b", layers=2, rows=8, row_len=4096, train="lora", recompute=0, fp32=False),
        # full fine-tuning of the 1B model: weight gradients of everything, the embedding and the head among them
        dict(name="step_1b_full", kind="step", arch="1b", layers=1, rows=4, row_len=4096, train="full", recompute=0, fp32=False),
        # the headline workload (8B, rank 64 on seven projections, selective recompute), one 16k row of its four
        dict(name="step_8b_lora", kind="step", arch="8b", layers=2, rows=1, row_len=16384, train="lora", recompute=2, fp32=False),
        # a sparse layer at 8x7B widths: routing, grouped experts, combine; many short trajectories
        dict(name="step_8x7b_lora", kind="step", arch="8x7b", layers=1, rows=1, row_len=8192, train="lora", recompute=0, fp32=False),
        # preference tuning: reference log-probabilities of the base model, then the policy's step on the pairs
        dict(name="dpo_1b", kind="step", arch="1b", layers=1, rows=2, row_len=4096, train="dpo", recompute=0, fp32=False),
        # attention alone: forward at 8B heads over one long trajectory with short ones around it, backward at 1B heads
        dict(name="attn_fwd_8b_long", kind="attn", arch="8b", tokens=24576, longest=16384, direction="fwd"),
        dict(name="attn_bwd_1b", kind="attn", arch="1b", tokens=8191, longest=4096, direction="bwd"),
        # one projection with its adapter and the residual over the tokens of a single mid-sized trajectory
        dict(name="gemm_8b_down", kind="gemm", arch="8b", tokens=1531, proj="down"),
        # the optimizer over all adapters of an 8B model
        dict(name="adamw_8b_lora", kind="adamw", arch="8b", layers=32, rank=64, train="lora"),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("step", "step", "step", "step", "attn", "attn", "gemm", "pack", "adamw"))
    if kind == "pack":
        return dict(kind=kind, arch=rng.choice(("1b", "8b", "8x7b")), rows=rng.randint(1, 8), row_len=size(512, 16384))
    if kind == "attn":
        n = size(512, 24576)
        return dict(kind=kind, arch=rng.choice(("1b", "8b")), tokens=n, longest=max(64, min(n, size(256, 16384))), direction=rng.choice(("fwd", "bwd")))
    if kind == "gemm":
        return dict(kind=kind, arch=rng.choice(("1b", "8b")), tokens=size(256, 16384), proj=rng.choice(SEVEN))
    if kind == "adamw":
        if rng.random() < 0.5:
            return dict(kind=kind, arch=rng.choice(("1b", "8b")), layers=rng.randint(1, 32), rank=rng.randint(4, 64), train="lora")
        return dict(kind=kind, arch="1b", layers=rng.randint(1, 4), vocab=size(1000, 32000), train="full")
    arch = rng.choice(("tiny", "1b", "1b", "8b", "8x7b"))
    if arch == "tiny":
        return dict(kind=kind, arch=arch, layers=rng.randint(1, 3), rows=rng.randint(1, 2), row_len=size(384, 1024), train=rng.choice(("lora", "full")),
                    recompute=rng.choice((0, 1)), fp32=True)
    train = "lora" if arch == "8x7b" else rng.choice(("lora", "lora", "nf4", "dpo", "full") if arch == "1b" else ("lora", "nf4"))
    rows = rng.randint(1, 4)
    return dict(kind=kind, arch=arch, layers=1 if train in ("full", "dpo") or arch == "8x7b" else rng.randint(1, 2), rows=rows,
                row_len=size(512, 8192 if arch == "8x7b" else 16384) // rows + 256, train=train, recompute=rng.choice((0, 1, 2)), fp32=False)


# ------------------------------------------------------------------------------------------------ inputs from the seed

def _lengths(case):
    """Trajectory lengths that fill the rows, from the recipe: those of the case, so that every seed packs alike."""
    med, lo, hi = ARCH[case["arch"]]["lens"]
    g, left, out = np.random.Generator(np.random.Philox(key=[7, case["rows"] * 65537 + case["row_len"]])), case["rows"] * case["row_len"], []
    while left > 0:
        x = g.integers(lo, hi + 1) if med == 0 else np.clip(round(math.exp(math.log(med) + 0.6 * g.standard_normal())), lo, hi)
        out.append(min(int(x), case["row_len"]))
        left -= out[-1]
    return out


def _trajectories(case, seed):
    """Host arrays of as_pack: turn tokens, offsets and roles, trajectory offsets.  system, then user / assistant / tool /
    assistant ...; assistant turns hold about the recipe's share of the tokens; token frequencies fall off as 1 / rank^1.1."""
    a = ARCH[case["arch"]]
    g = np.random.Generator(np.random.Philox(key=[seed, 1]))
    offs, roles, traj = [0], [], [0]
    for n in _lengths(case):
        turns = min(int(g.integers(2, 13)), max(1, n // 8))
        r = [1, 2][-turns:] if turns <= 2 else [0] + [(1, 2, 3, 2)[i % 4] for i in range(turns - 1)]
        k = sum(x == 2 for x in r)
        w = np.array([a["share"] * (turns - k) / (k * (1 - a["share"])) if x == 2 and k < turns else 1.0 for x in r]) * g.uniform(0.5, 1.5, turns)
        ends = np.maximum(np.arange(1, turns + 1), np.round(np.cumsum(w / w.sum()) * n)).astype(np.int64)
        ends[-1] = n
        offs += (offs[-1] + ends).tolist()
        roles += r
        traj.append(len(roles))
    p = np.cumsum(np.arange(1, a["vocab"] + 1, dtype=np.float64) ** -1.1)
    toks = np.minimum(np.searchsorted(p / p[-1], g.random(offs[-1])), a["vocab"] - 1).astype(np.int32)
    return toks, np.asarray(offs, np.int32), np.asarray(roles, np.uint8), np.asarray(traj, np.int32)


def _packed(case, seed):
    """What packing these trajectories gives (next fit, tail pads as segments of their own), from the definition."""
    toks, offs, roles, traj = _trajectories(case, seed)
    rows, width, row, fill, cu = case["rows"], case["row_len"], 0, 0, [0]
    tok, mask = np.zeros(rows * width, np.int64), np.zeros(rows * width, bool)
    for i in range(len(traj) - 1):
        b, e = int(offs[traj[i]]), int(offs[traj[i + 1]])
        if fill and fill + e - b > width:
            row, fill = row + 1, 0
            cu.append(row * width)
        if row >= rows:
            break
        pos = row * width + fill
        tok[pos:pos + e - b] = toks[b:e]
        for t in range(traj[i], traj[i + 1]):
            mask[pos + offs[t] - b:pos + offs[t + 1] - b] = roles[t] == 2
        cu.append(pos + e - b)
        row, fill = divmod(pos + e - b, width)
    if fill:
        row += 1
        cu.append(row * width)
    return tok[:row * width], mask[:row * width], cu


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 16 + stream)
    return g


def _weights(case, seed):
    """Random weights of the architecture, N(0, 0.02), gains about 1; embeddings of unit scale, the scale a trained model's
    residual stream has.  Sparse models: router rows and embeddings that make every token's choice clear, as training does."""
    a, g, L = ARCH[case["arch"]], _gen(seed, 1), case["layers"]
    dt = torch.float32 if case["fp32"] else torch.bfloat16
    D, Dkv, d, F, V, E = a["hq"] * a["dh"], a["hkv"] * a["dh"], a["d"], a["ffn"], a["vocab"], a.get("experts", 0)

    def mat(*shape, std=0.02):
        return torch.empty(shape, dtype=dt, device=DEV).normal_(0.0, std, generator=g)

    def gain():
        return (1.0 + 0.1 * torch.empty(d, device=DEV).normal_(generator=g)).to(dt)

    P = dict(embed=mat(V, d, std=0.02 if case["fp32"] else 1.0), head=mat(V, d), g_final=gain(), layers=[])
    ex = (E,) if E else ()
    for _ in range(L):
        W = dict(g1=gain(), wq=mat(D, d), wk=mat(Dkv, d), wv=mat(Dkv, d), wo=mat(d, D), g2=gain(),
                 wgate=mat(*ex, F, d), wup=mat(*ex, F, d), wdown=mat(*ex, d, F))
        if E:
            basis = torch.linalg.qr(torch.empty(d, E, device=DEV).normal_(generator=g))[0]
            first = torch.randint(0, E, (V,), generator=g, device=DEV)
            second = (first + torch.randint(1, E, (V,), generator=g, device=DEV)) % E
            P["embed"] = (8.0 * math.sqrt(d) * (basis.T[first] + 0.8 * basis.T[second]) + 0.5 * P["embed"].float()).to(dt)
            W["wrouter"] = (0.16 * basis.T).to(dt).contiguous()
        P["layers"].append(W)
    return P


def _dims(a, t):
    D, Dkv = a["hq"] * a["dh"], a["hkv"] * a["dh"]
    return {"q": (a["d"], D), "k": (a["d"], Dkv), "v": (a["d"], Dkv), "o": (D, a["d"]), "gate": (a["d"], a["ffn"]), "up": (a["d"], a["ffn"]),
            "down": (a["ffn"], a["d"]), "router": (a["d"], a.get("experts", 0))}[t]


def _adapters(case, seed):
    if case["train"] == "full":
        return None
    a, g = ARCH[case["arch"]], _gen(seed, 2)
    new = lambda *s: torch.empty(s, dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=g)  # noqa: E731
    return [{t: (new(a["rank"], _dims(a, t)[0]), new(_dims(a, t)[1], a["rank"])) for t in a["targets"]} for _ in range(case["layers"])]


def _config(case):
    a, full = ARCH[case["arch"]], case.get("train") == "full"
    mask = 0
    for t in () if full else a["targets"]:
        mask |= 1 << B.TARGETS.index(t)
    return B.ModelConfig(B.C.sizeof(B.ModelConfig), case.get("layers", 1), a["d"], a["hq"], a["hkv"], a["dh"], a["ffn"], a["vocab"], a.get("experts", 0),
                         2 if a.get("experts") else 0, EPS, a["base"], 0 if full else a["rank"], 0.0 if full else a["alpha"], mask,
                         B.AS_FP32 if case.get("fp32") else B.AS_BF16, B.AS_FULL if full else B.AS_LORA, case.get("recompute", 0),
                         B.AS_W_NF4 if case.get("train") == "nf4" else B.AS_W_DENSE)


def _segments(case, seed):
    """Segment boundaries of an attention call: one trajectory of `longest` tokens among shorter ones."""
    n, g = case["tokens"], np.random.Generator(np.random.Philox(key=[seed, 5]))
    shape = np.random.Generator(np.random.Philox(key=[9, n]))
    lens, left = [min(n, case["longest"])], n - min(n, case["longest"])
    while left > 0:
        x = int(np.clip(round(math.exp(math.log(900) + 0.6 * shape.standard_normal())), 32, case["longest"]))
        lens.append(min(x, left))
        left -= lens[-1]
    return [0] + np.cumsum([lens[i] for i in g.permutation(len(lens))]).tolist()


def _attn_inputs(case, seed):
    a, g, n = ARCH[case["arch"]], _gen(seed, 3), case["tokens"]
    D, W = a["hq"] * a["dh"], (a["hq"] + 2 * a["hkv"]) * a["dh"]
    new = lambda *s: torch.empty(s, dtype=torch.bfloat16, device=DEV).normal_(generator=g)  # noqa: E731
    return _segments(case, seed), new(n, W), new(n, D)


def _gemm_inputs(case, seed):
    a, g = ARCH[case["arch"]], _gen(seed, 4)
    K, N = _dims(a, case["proj"])
    new = lambda s, *shape: torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, s, generator=g)  # noqa: E731
    rp = -(-a["rank"] // 64) * 64                        # the adapter's columns are padded to whole 64-wide steps
    u, b2 = new(1.0, case["tokens"], rp), new(0.04, N, rp)
    u[:, a["rank"]:] = 0
    b2[:, a["rank"]:] = 0
    res = new(1.0, case["tokens"], N) if case["proj"] in ("o", "down") else None
    return new(1.0, case["tokens"], K), new(0.02, N, K), u, b2, res


def _adam_sizes(case):
    a = ARCH[case["arch"]]
    if case["train"] == "lora":
        return [n for _ in range(case["layers"]) for t in a["targets"] for n in (case["rank"] * _dims(a, t)[0], case["rank"] * _dims(a, t)[1])]
    layer = [a["d"], a["d"]] + [_dims(a, t)[0] * _dims(a, t)[1] for t in SEVEN]
    return [case["vocab"] * a["d"], case["vocab"] * a["d"], a["d"]] + layer * case["layers"]


ADAM = dict(lr=2e-5, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)


def _adam_inputs(case, seed):
    g, n = _gen(seed, 5), sum(_adam_sizes(case))
    new = lambda s: torch.empty(n, dtype=torch.float32, device=DEV).normal_(0.0, s, generator=g)  # noqa: E731
    return new(0.02), new(1e-3), new(1e-4), new(1e-3).square_()


# ------------------------------------------------------------------------------------------------------- one pass of a case

def prepare(case, seed):
    s = dict(case=case, ctx=B.Context(_config(case)))
    ctx = s["ctx"]
    if case["kind"] == "pack":
        s["host"] = _trajectories(case, seed)
        s["out"] = (torch.empty(case["rows"] * case["row_len"], dtype=torch.int32, device=DEV),
                    torch.empty(len(s["host"][3]) + case["rows"], dtype=torch.int32, device=DEV),
                    torch.empty(case["rows"] * case["row_len"], dtype=torch.uint8, device=DEV))
    elif case["kind"] == "attn":
        cu, s["qkv"], s["d_o"] = _attn_inputs(case, seed)
        lens = torch.tensor([e - b for b, e in zip(cu, cu[1:])], device=DEV)
        s["start"] = torch.repeat_interleave(torch.tensor(cu[:-1], dtype=torch.int32, device=DEV), lens)
        s["end"] = torch.repeat_interleave(torch.tensor(cu[1:], dtype=torch.int32, device=DEV), lens)
        if case["direction"] == "bwd":
            s["o"], s["lse"] = ctx.op_attention_fwd(s["qkv"], s["start"])
    elif case["kind"] == "gemm":
        s["x"], s["w"], s["u"], s["b2"], s["res"] = _gemm_inputs(case, seed)
        s["tail"] = torch.empty(B.GEMM_TAIL_SCRATCH_BYTES, dtype=torch.uint8, device=DEV)
    elif case["kind"] == "adamw":
        flat = _adam_inputs(case, seed)
        sizes = _adam_sizes(case)
        s["flat"] = dict(zip(("w", "g", "m", "v"), flat))
        s["lists"] = [list(torch.split(t, sizes)) for t in flat]
        s["low"] = torch.empty(sum(sizes), dtype=torch.bfloat16, device=DEV) if case["train"] == "full" else None
        s["low_list"] = list(torch.split(s["low"], sizes)) if s["low"] is not None else None
    else:
        P = _weights(case, seed)
        if case["train"] == "nf4":
            for W in P["layers"]:
                for k in ("q", "k", "v", "o", "gate", "up", "down"):
                    W["w" + k], W["a" + k] = ctx.nf4_quantize(W["w" + k])
        s["model"] = B.DeviceModel(ctx, P, _adapters(case, seed))
        pk = ctx.pack(*_trajectories(case, seed), case["row_len"], case["rows"])
        s["batch"] = dict(tokens=pk["tokens"], cu_seqlens=pk["cu_seqlens"], h_cu_seqlens=pk["cu_seqlens"].cpu().numpy(), loss_mask=pk["loss_mask"],
                          n_rows=pk["n_rows"], row_len=case["row_len"], seg_skip=pk["seg_skip"])
        s["ws"] = torch.empty(ctx.workspace_bytes(pk["n_rows"], case["row_len"]), dtype=torch.uint8, device=DEV)
        s["pairs"] = np.asarray(_pairs(pk["seg_skip"]), np.int32)
        s["out"] = dict(loss=torch.zeros(1, device=DEV), loss_sum=torch.zeros(1, device=DEV), count=torch.zeros(1, dtype=torch.int32, device=DEV))
    return s


def _pairs(skip):
    """Neighbouring segments that bear loss are the chosen and the rejected trajectory of a pair."""
    live = [i for i, x in enumerate(skip) if not x]
    return [(live[i], live[i + 1]) for i in range(0, len(live) - 1, 2)]


def run(s):
    case, ctx = s["case"], s["ctx"]
    if case["kind"] == "pack":
        pk = ctx.pack(*s["host"], case["row_len"], case["rows"], outputs=s["out"])
        return dict(tokens=pk["tokens"], cu=pk["cu_seqlens"], mask=pk["loss_mask"], skip=pk["seg_skip"])
    if case["kind"] == "attn":
        if case["direction"] == "fwd":
            o, lse = ctx.op_attention_fwd(s["qkv"], s["start"])
            return dict(o=o, lse=lse)
        return dict(dqkv=ctx.op_attention_bwd(s["qkv"], s["start"], s["end"], s["o"], s["lse"], s["d_o"]))
    if case["kind"] == "gemm":
        return dict(y=ctx.op_gemm(s["x"], s["w"], s["u"], s["b2"], R=s["res"], tail_scratch=s["tail"]))
    if case["kind"] == "adamw":
        w, g, m, v = s["lists"]
        ctx.adamw_update(w, s["low_list"], g, m, v, [1] * len(w), 10, **ADAM)
        out = dict(w=s["flat"]["w"], m=s["flat"]["m"], v=s["flat"]["v"])
        return out if s["low"] is None else dict(out, low=s["low"])
    model = s["model"]
    if case["train"] == "dpo":
        ref = ctx.sequence_logps(model, workspace=s["ws"], adapters=False, **s["batch"])
        r = ctx.dpo_step(model, workspace=s["ws"], pairs=s["pairs"], ref_logp=ref, beta=BETA, **s["batch"])
        out = dict(ref=ref, logp=r["logp"], loss=r["stats"][:1])
    else:
        ctx.train_step(model, workspace=s["ws"], out=s["out"], **s["batch"])
        out = dict(s["out"])
    out["grads"] = model.w_grads if case["train"] == "full" else [{t: dict(a=g[0], b=g[1]) for t, g in L.items()} for L in model.lora_grads]
    return out


# ------------------------------------------------------------------------------------------------- what a pass cannot do without

def work(case):
    a = ARCH[case["arch"]]
    D, Dkv, d, F, V, E, r = a["hq"] * a["dh"], a["hkv"] * a["dh"], a["d"], a["ffn"], a["vocab"], a.get("experts", 0), a["rank"]
    if case["kind"] == "pack":
        n = case["rows"] * case["row_len"]
        return dict(bytes=9.0 * n, flops=0.0)
    if case["kind"] == "attn":
        cu, n = _segments(case, 0), case["tokens"]
        sq, qkv = float(sum((e - b) ** 2 for b, e in zip(cu, cu[1:]))), n * (D + 2 * Dkv) * 2.0
        return dict(bytes=qkv + n * D * 2.0, flops=2.0 * D * sq) if case["direction"] == "fwd" else dict(bytes=2 * qkv + 2 * n * D * 2.0, flops=5.0 * D * sq)
    if case["kind"] == "gemm":
        K, N = _dims(a, case["proj"])
        n = case["tokens"]
        return dict(bytes=2.0 * (n * (K + r) + N * (K + r) + n * N * (2 if case["proj"] in ("o", "down") else 1)), flops=2.0 * n * N * (K + r))
    if case["kind"] == "adamw":
        return dict(bytes=(28.0 + (2.0 if case["train"] == "full" else 0.0)) * sum(_adam_sizes(case)), flops=0.0)
    _, mask, cu = _packed(case, 0)
    keep = [(b, e) for b, e in zip(cu, cu[1:]) if mask[b + 1:e].any()]
    n, sq, tgt = float(sum(e - b for b, e in keep)), float(sum((e - b) ** 2 for b, e in keep)), float(sum(mask[b + 1:e].sum() for b, e in keep))
    L, full, dpo = case["layers"], case["train"] == "full", case["train"] == "dpo"
    p_qkv, p_ffn = d * (D + 2 * Dkv), 3 * d * F
    p_layer = p_qkv + D * d + (2 * p_ffn + d * E if E else p_ffn)
    flops = (6.0 if full else 4.0) * L * p_layer * n + 7.0 * D * L * sq + (6.0 if full else 4.0) * d * V * tgt
    if not full:                                         # nothing below the first layer's projections takes a gradient
        flops += 6.0 * r * sum(sum(_dims(a, t)) for t in a["targets"]) * L * n - 2.0 * p_qkv * n
    if dpo:
        flops += 2.0 * L * p_layer * n + 2.0 * D * L * sq + 2.0 * 2.0 * d * V * tgt
    params = L * (p_qkv + D * d + max(E, 1) * p_ffn + d * E)
    size = 4.0 if case["fp32"] else 2.0
    byts = size * (params + 2 * V * d) if case["train"] != "nf4" else 4.5 / 8 * params + size * 2 * V * d
    byts -= size * max(0.0, V - n) * d                   # only the rows of the batch's tokens are read from the embedding
    byts += 4.0 * (params + 2 * V * d) if full else 8.0 * L * r * sum(sum(_dims(a, t)) for t in a["targets"])
    return dict(bytes=byts, flops=flops)


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    if case["kind"] == "adamw":
        return dict(rel=1e-6, max=1e-2)                  # 2e-7 seen; a 16-bit copy may round the other way
    if case.get("fp32"):
        return dict(rel=5e-6, max=1e-3)                  # 1e-6 seen
    if case["kind"] == "step":
        return dict(rel=0.03, max=0.8)                   # 4e-3 .. 1e-2 seen: activations are stored in 16 bits
    return dict(rel=0.01, max=0.3)                       # 1.7e-3 .. 2.4e-3 seen: one rounding of the result, one of the probabilities


# --------------------------------------------------------------------------------------------------------- results in 64 bits

def _attention64(q, k, v):
    """Causal attention of one segment: q [n, hq, dh], k, v [n, hkv, dh] -> [n, hq * dh] and the log-sum-exps [n, hq]."""
    n, hq, dh = q.shape
    grp = hq // k.shape[1]
    hidden = torch.ones(n, n, dtype=torch.bool, device=q.device).triu_(1)

    def group(qg, kg, vg):                               # the query heads of one KV head: [n, grp, dh], [n, dh], [n, dh]
        s = torch.matmul(qg.transpose(0, 1).reshape(-1, dh), kg.T).view(grp, n, n) / math.sqrt(dh)
        s = s.masked_fill(hidden, -math.inf)
        lse = torch.logsumexp(s, 2)
        return torch.matmul((s - lse[:, :, None]).exp().view(-1, n), vg).view(grp, n, dh), lse

    outs = [torch.utils.checkpoint.checkpoint(group, q[:, g * grp:(g + 1) * grp], k[:, g], v[:, g], use_reentrant=False) for g in range(k.shape[1])]
    return torch.cat([o for o, _ in outs]).transpose(0, 1).reshape(n, hq * dh), torch.cat([x for _, x in outs]).T


def _step64(case, seed):
    a = ARCH[case["arch"]]
    tok, mask, cu = _packed(case, seed)
    W, ad, full = _weights(case, seed), _adapters(case, seed), case["train"] == "full"
    f64 = lambda t: t.double().requires_grad_(full)  # noqa: E731
    layers = []
    for Wl in W["layers"]:
        if case["train"] == "nf4":
            lv = torch.tensor(NF4, dtype=torch.float32, device=DEV)
            for k in ("q", "k", "v", "o", "gate", "up", "down"):
                x = Wl["w" + k].float().view(-1, 64)
                top = x.abs().amax(1, keepdim=True)
                code = torch.bucketize(x / torch.where(top > 0, top, torch.ones_like(top)), (lv[:-1] + lv[1:]) * 0.5, right=True)
                Wl["w" + k] = (lv[code].double() * top.double()).view_as(Wl["w" + k])
        layers.append({k: f64(v) for k, v in Wl.items()})
    embed, head, g_final = f64(W["embed"]), f64(W["head"]), f64(W["g_final"])
    lora = None if full else [{t: (A.double().requires_grad_(), Bm.double().requires_grad_()) for t, (A, Bm) in Ld.items()} for Ld in ad]
    del W
    keep = [(b, e) for b, e in zip(cu, cu[1:]) if mask[b + 1:e].any()]
    ids = torch.from_numpy(np.concatenate([tok[b:e] for b, e in keep])).to(DEV)
    ends = np.cumsum([e - b for b, e in keep]).tolist()
    segs = list(zip([0] + ends[:-1], ends))
    where = torch.from_numpy(np.concatenate([np.append(mask[b + 1:e], False) for b, e in keep])).to(DEV).nonzero()[:, 0]
    label = ids[where + 1]
    pos = torch.cat([torch.arange(e - b, device=DEV) for b, e in segs]).double()
    half = a["dh"] // 2
    ang = pos[:, None] * float(a["base"]) ** (-torch.arange(half, device=DEV).double() / half)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def norm(x, g):
        return x * torch.rsqrt(x.square().mean(1, keepdim=True) + EPS) * g

    def rope(x):
        x1, x2 = x[..., :half], x[..., half:]
        return torch.cat((x1 * cos - x2 * sin, x1 * sin + x2 * cos), -1)

    def losses(adapters):
        def lin(l, x, w, t):
            y = x @ w.T
            if adapters and not full and t in lora[l]:
                A, Bm = lora[l][t]
                y = y + a["alpha"] / a["rank"] * ((x @ A.T) @ Bm.T)
            return y

        def ffn(x, Wg, Wu, Wd, l=0, plain=True):
            if plain:
                return (torch.nn.functional.silu(x @ Wg.T) * (x @ Wu.T)) @ Wd.T
            return lin(l, torch.nn.functional.silu(lin(l, x, Wg, "gate")) * lin(l, x, Wu, "up"), Wd, "down")

        h = embed[ids]
        for l, Wl in enumerate(layers):
            x = norm(h, Wl["g1"])
            q, k, v = (lin(l, x, Wl["w" + t], t).view(len(ids), -1, a["dh"]) for t in "qkv")
            q, k = rope(q), rope(k)
            h = h + lin(l, torch.cat([_attention64(q[b:e], k[b:e], v[b:e])[0] for b, e in segs]), Wl["wo"], "o")
            x = norm(h, Wl["g2"])
            if "wrouter" not in Wl:
                h = h + ffn(x, Wl["wgate"], Wl["wup"], Wl["wdown"], l, False)
                continue
            val, sel = lin(l, x, Wl["wrouter"], "router").topk(2, 1)
            p, y = val.softmax(1), torch.zeros_like(h)
            for e in range(a["experts"]):
                t, slot = (sel == e).nonzero(as_tuple=True)
                y = y.index_add(0, t, p[t, slot][:, None] * ffn(x[t], Wl["wgate"][e], Wl["wup"][e], Wl["wdown"][e]))
            h = h + y
        z = norm(h[where], g_final) @ head.T
        return torch.logsumexp(z, 1) - z.gather(1, label[:, None])[:, 0]

    def logps(rows):
        at = torch.searchsorted(torch.tensor(ends, device=DEV), where, right=True)
        return torch.zeros(len(segs), dtype=torch.float64, device=DEV).index_add(0, at, -rows)

    if case["train"] == "dpo":
        with torch.no_grad():
            ref = logps(losses(False))
        pi = logps(losses(True))
        index = {i: j for j, i in enumerate(i for i, (b, e) in enumerate(zip(cu, cu[1:])) if mask[b + 1:e].any())}
        skip = [i not in index for i in range(len(cu) - 1)]
        pc, pr = ([index[p[j]] for p in _pairs(skip)] for j in (0, 1))
        loss = torch.nn.functional.softplus(-BETA * ((pi - ref)[pc] - (pi - ref)[pr])).mean()
        spread = lambda x: torch.zeros(len(cu) - 1, dtype=torch.float64, device=DEV).index_add(0, torch.tensor(list(index), device=DEV), x.detach())  # noqa: E731
        out = dict(ref=spread(ref), logp=spread(pi), loss=loss.detach()[None])
    else:
        rows = losses(True)
        loss = rows.mean()
        out = dict(loss=loss.detach()[None], loss_sum=rows.detach().sum()[None], count=None)
    loss.backward()
    if full:
        out["grads"] = dict(embed=embed.grad, head=head.grad, g_final=g_final.grad, layers=[{k: t.grad for k, t in Wl.items()} for Wl in layers])
    else:
        out["grads"] = [{t: dict(a=A.grad, b=Bm.grad) for t, (A, Bm) in Ld.items()} for Ld in lora]
    return out


def exact(case, seed):
    a = ARCH[case["arch"]]
    if case["kind"] == "pack":
        return None                                      # whole numbers only
    if case["kind"] == "attn":
        cu, qkv, d_o = _attn_inputs(case, seed)
        x = qkv.double().view(len(qkv), -1, a["dh"]).requires_grad_(case["direction"] == "bwd")
        q, k, v = x.split((a["hq"], a["hkv"], a["hkv"]), 1)
        parts = [_attention64(q[b:e], k[b:e], v[b:e]) for b, e in zip(cu, cu[1:])]
        o = torch.cat([p[0] for p in parts])
        if case["direction"] == "fwd":
            return dict(o=o, lse=torch.cat([p[1] for p in parts]))
        o.backward(d_o.double())
        return dict(dqkv=x.grad.view(len(qkv), -1))
    if case["kind"] == "gemm":
        x, w, u, b2, res = (t if t is None else t.double() for t in _gemm_inputs(case, seed))
        y = x @ w.T + u @ b2.T
        return dict(y=y if res is None else y + res)
    if case["kind"] == "adamw":
        w, g, m, v = (t.double() for t in _adam_inputs(case, seed))
        b1, b2 = ADAM["beta1"], ADAM["beta2"]
        m, v = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
        w = w - ADAM["lr"] * (m / (1 - b1 ** 10) / ((v / (1 - b2 ** 10)).sqrt() + ADAM["eps"]) + ADAM["weight_decay"] * w)
        out = dict(w=w, m=m, v=v)
        return dict(out, low=w) if case["train"] == "full" else out
    return _step64(case, seed)
