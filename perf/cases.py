"""Timing cases of the norm-test + AdamW library: the calls a training program makes, over the sizes it makes them at.

One case is a plain dict:

    op       "step"     fused step, statistics only or AdamW only (by `flags`), rows in one (J, ld) matrix
             "rows"     the same step with every row an allocation of its own
             "clipped"  the two-phase gradient-clipped step
             "shard"    one parameter shard's clipped step: partial sums + stored mean, host combination, AdamW
             "layers"   a step followed by the per-layer table
    J, d     gradient vectors and coordinates;  dtype "bf16" or "f32" of the gradients
    padded   row stride rounded up to 64 elements (False: a contiguous (J, d) tensor, as torch.stack gives)
    flags    "full", "stats", "adamw" or "partial" (the fused step of a shard);  coord: coordinate-wise test too
    dist     input distribution: "flat", "blocks" (per-parameter-block scales) or "heavy" (Student-t noise, per sample)
    layers   number of parameter tensors in the per-layer table

What the paths read and write is device memory, so inputs, state, workspace and result stay on the GPU between calls,
as a training loop keeps them.  w, m, v are updated in place by every pass.
"""
from __future__ import annotations

import math

import torch

from paper_2412_21124_amd import binding as B
from paper_2412_21124_amd import synth

DEVICE = "cuda:0"
_ALL_SHARDS = 8
_CHUNK_VALUES = 1 << 27   # gradient values widened to 64 bits at a time in exact()


def _case(name, op, J, d, dtype, *, padded=True, flags="full", coord=False, dist="flat", layers=0):
    c = {"op": op, "J": J, "d": d, "dtype": dtype, "padded": padded, "flags": flags, "coord": coord, "dist": dist,
         "layers": layers}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest calls: a probe or an adapter of odd size, five workers, rows stacked without padding
        _case("small_odd", "step", 5, 100_003, "f32", padded=False),
        # the benchmark's tiny workload: launches and latency
        _case("tiny", "step", 4, 1 << 20, "f32"),
        # per-example gradients of a small model of odd size, stacked without padding
        _case("per_sample_odd", "step", 128, 1_000_003, "bf16", padded=False, dist="heavy"),
        # worker gradients of a mid-sized model whose length is no multiple of anything, stacked without padding
        _case("odd_medium", "step", 8, 30_000_001, "bf16", padded=False),
        # the 148-tensor GPT-2-small-sized workload: test, coordinate-wise test, update and the per-layer table
        _case("gpt2_layers", "layers", 8, 124_439_808, "bf16", coord=True, dist="blocks", layers=148),
        # the same vector on the steps between tests (test interval above one): mean and update alone
        _case("gpt2_skip", "step", 8, 124_439_808, "bf16", flags="adamw", dist="blocks"),
        # the paper's 304.6M-parameter model with its four workers' gradients in buffers of their own
        _case("paper_300m_rows", "rows", 4, 304_600_000, "bf16"),
        # the same model's step with the global gradient norm clipped, as the paper's runs have it
        _case("paper_300m_clipped", "clipped", 4, 304_600_000, "bf16"),
        # one of eight shards of the 1.1B-parameter model, clipped: sums and mean, combination on the host, update
        _case("shard_clipped", "shard", 4, 137_500_000, "bf16"),
        # one of eight shards of a 7B-parameter model, 16 micro-batch gradients, fused partial step
        _case("fsdp_shard", "step", 16, 875_000_000, "bf16", flags="partial"),
        # 512 per-example gradients of a 16.8M-parameter model
        _case("per_sample", "step", 512, 1 << 24, "bf16", dist="heavy"),
        # the headline: 1.5e9 coordinates, eight workers
        _case("flat_1p5b", "step", 8, 1_500_000_000, "bf16"),
    ]


def draw(rng):
    """One more case: sizes log-uniform from a thousand coordinates to 12 GB of traffic, odd lengths and unpadded rows among them."""
    op = rng.choice(["step", "step", "step", "step", "rows", "rows", "clipped", "shard", "layers"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    J = rng.choice([2, 3, 4, 4, 5, 6, 8, 8, 12, 16, 16, 20, 24, 32, 48, 64, 100, 128, 256, 512])
    per_coord = J * (2 if dtype == "bf16" else 4) + 24
    d = int(math.exp(rng.uniform(math.log(1000), math.log(12e9 / per_coord))))
    if rng.random() < 0.5:
        d = max(64, d // 64 * 64)   # tensor dimensions are mostly multiples of 64; the sum of all of them need not be
    flags = rng.choice(["full", "full", "full", "stats", "adamw", "partial"]) if op in ("step", "rows") else "full"
    coord = op != "shard" and flags in ("full", "stats") and rng.random() < 0.25
    return _case(None, op, J, d, dtype, padded=rng.random() < 0.5, flags=flags, coord=coord,
                 dist="heavy" if J > 32 else rng.choice(["flat", "blocks"]),
                 layers=rng.choice([1, 12, 75, 148, 300]) if op == "layers" else 0)


def _hyper(case):
    J = case["J"]
    if J > 32:   # per-sample statistics: the batch is the rows
        return synth.Hyper(lr=4e-4, step=10, b_k=J, b_max=8192, round_to=1, ddof=1)
    return synth.Hyper(lr=4e-4, step=10, b_k=256, b_max=8192, round_to=16 * J, ddof=1)


def _flags(case):
    if case["op"] == "shard":
        return B.NT_DO_STATS | B.NT_PARTIAL | B.NT_WRITE_GBAR
    f = {"full": B.NT_DO_STATS | B.NT_DO_ADAMW, "stats": B.NT_DO_STATS, "adamw": B.NT_DO_ADAMW,
         "partial": B.NT_DO_STATS | B.NT_DO_ADAMW | B.NT_PARTIAL}[case["flags"]]
    return f | (B.NT_COORD_TEST if case["coord"] else 0)


def _sizes(case):
    """Parameter tensors of the vector: the GPT-2-small list at its own length, else that list's proportions."""
    base = synth.gpt2_small_blocks()
    d, n = case["d"], case["layers"] or 64
    if d == sum(base) and n == len(base):
        return base
    n = min(n, d)
    weights = [base[i % len(base)] for i in range(n)]
    edges = [round(d * s / sum(weights)) for s in _running(weights)]
    return [b - a for a, b in zip([0] + edges[:-1], edges[:-1] + [d])]


def _running(xs):
    total, out = 0, []
    for x in xs:
        total += x
        out.append(total)
    return out


def _workload(case, seed):
    d, J = case["d"], case["J"]
    ld = (d + 63) // 64 * 64 if case["padded"] else d
    kw = {"mu": "normal", "mu_scale": 1e-2, "noise": "normal"}
    if case["dist"] in ("blocks", "heavy"):
        kw.update(mu="sign", block_sizes=_sizes(case))
    if case["dist"] == "heavy":
        kw.update(noise="student_t3")
    return synth.make("case", J, d, gdtype=torch.bfloat16 if case["dtype"] == "bf16" else torch.float32, sigma=1e-2,
                      hyper=_hyper(case), seed=seed, device=DEVICE, ld=ld, **kw)


def prepare(case, seed):
    wl = _workload(case, seed)
    J, d, h = case["J"], case["d"], wl.hyper
    hyper = B.make_hyper(lr=h.lr, beta1=h.beta1, beta2=h.beta2, eps=h.eps, weight_decay=h.weight_decay, eta=h.eta,
                         step=h.step, b_k=h.b_k, b_max=h.b_max, round_to=h.round_to, ddof=h.ddof, flags=_flags(case))
    s = {"case": case, "hyper": hyper, "d": d, "grads": wl.grads, "w": wl.w, "m": wl.m, "v": wl.v, "shard": None}
    need = B.normtest_workspace_bytes_for(B.NT_BF16 if case["dtype"] == "bf16" else B.NT_F32, J, d,
                                          hyper.flags | B.NT_WRITE_GBAR)
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEVICE)
    s["result"] = torch.zeros(B.RESULT_BYTES, dtype=torch.uint8, device=DEVICE)
    if case["op"] == "rows":
        s["rows"] = [wl.grads[j, :d].clone() for j in range(J)]
        s["grads"] = None
        s["table"] = B.make_row_table(s["rows"])
    if case["op"] in ("clipped", "shard"):
        s["gbar"] = torch.empty(d, dtype=torch.float32, device=DEVICE)
    if case["op"] == "shard" or case["flags"] == "partial":
        s["shard"] = B.nt_shard_info(3, _ALL_SHARDS, 3 * d, _ALL_SHARDS * d)
    if case["op"] == "layers":
        s["offsets"] = torch.tensor([0] + _running(_sizes(case)), dtype=torch.int64, device=DEVICE)
        s["layers"] = torch.zeros((s["offsets"].numel() - 1) * B.LAYER_BYTES, dtype=torch.uint8, device=DEVICE)
    return s


def _record(result):
    """Views of the step's record.  The sums' low-order parts are left out: they are rounding residue, with no digits of their own."""
    f, i = result.view(torch.float64), result.view(torch.int64)
    return {"sums": f[0:3], "derived": f[6:10], "counts": i[10:12], "pass_status": result.view(torch.int32)[24:26],
            "max_ratio": f[13:14]}


def run(s):
    case, kw = s["case"], {"d": s["d"], "workspace": s["workspace"], "result": s["result"], "shard": s["shard"]}
    w, m, v = s["w"], s["m"], s["v"]
    op = case["op"]
    if op in ("step", "layers"):
        B.normtest_step(s["grads"], w, m, v, s["hyper"], **kw)
    elif op == "rows":
        B.normtest_step_rows(s["rows"], w, m, v, s["hyper"], table=s["table"], **kw)
    elif op == "clipped":
        B.normtest_step_clipped(s["grads"], w, m, v, s["gbar"], 1.0, s["hyper"], **kw)
    else:
        B.normtest_step(s["grads"], None, None, None, s["hyper"], gbar_out=s["gbar"], **kw)
        # every rank reads its partial sums and combines all of them; here they stand for all shards
        whole = B.normtest_combine([B.read_result(s["result"])], case["J"], s["hyper"])
        B.normtest_adamw_gbar(s["gbar"], w, m, v, s["hyper"], B.normtest_clip_coef(whole.gbar_sq, 1.0))
    out = _record(s["result"])
    if case["flags"] != "stats":
        out.update(w=w, m=m, v=v)
    if "gbar" in s:
        out["gbar"] = s["gbar"]
    if op == "layers":
        B.normtest_layer_stats(s["grads"], s["offsets"], s["workspace"], d=s["d"], layers=s["layers"])
        L = s["offsets"].numel() - 1
        out["layer_stats"] = s["layers"].view(torch.float64).view(L, -1)[:, :6]
        out["layer_counts"] = s["layers"].view(torch.int64).view(L, -1)[:, 6:8]
        out["layer_max_ratio"] = s["layers"].view(torch.float64).view(L, -1)[:, 9]
    return out


def work(case):
    J, d = case["J"], case["d"]
    rows = J * (2 if case["dtype"] == "bf16" else 4)
    state = 0 if case["flags"] == "stats" else 24
    mean = 4 if case["op"] in ("clipped", "shard") else 0   # the mean is handed back; its second reading is not counted
    flops = (1 if case["flags"] == "adamw" else 6) * J + (12 if state else 0)
    return {"bytes": d * (rows + state + mean), "flops": d * flops}


def tolerance(case):
    # 32-bit state and means: a few roundings per coordinate; sums of squares: 32-bit terms, 64-bit sums.  Against
    # 64 bits w, m, v are 3e-8 to 8e-8 off and the sums up to 1.2e-8; single values of w, where the update cancels it, more
    return {"rel": 4e-7, "max": 4e-5}


def exact(case, seed):
    """The first pass on prepare(case, seed) in 64 bits."""
    s, hy = prepare(case, seed), _hyper(case)
    J, d, op = case["J"], case["d"], case["op"]
    f64 = torch.float64
    grads = s["grads"] if s["grads"] is not None else None
    stats, update = case["flags"] != "adamw", case["flags"] != "stats"
    edges = s["offsets"].tolist() if op == "layers" else [0, d]
    L = len(edges) - 1
    sums = torch.zeros((L, 3), dtype=f64, device=DEVICE)
    ratio = torch.zeros(L, dtype=f64, device=DEVICE)
    gbar = torch.empty(d, dtype=f64, device=DEVICE) if (update or "gbar" in s) else None
    step = max(1, _CHUNK_VALUES // J)
    for l in range(L):
        for lo in range(edges[l], edges[l + 1], step):
            hi = min(edges[l + 1], lo + step)
            x = torch.stack([r[lo:hi] for r in s["rows"]]) if grads is None else grads[:, lo:hi]
            x = x.to(f64)
            gb = x.mean(0)
            if gbar is not None:
                gbar[lo:hi] = gb
            if not stats:
                continue
            centred = (x - gb).square_().sum(0)
            sums[l] += torch.stack([x.square().sum(), (gb * J).square().sum(), centred.sum()])
            if case["coord"]:
                rho = centred / (hy.eta ** 2 * hy.b_k * (J - hy.ddof) * gb * gb)
                ratio[l] = torch.maximum(ratio[l], torch.where(centred == 0, 0.0, rho).max())
    nan = float("nan")

    def derived(a):
        g2, var = a[..., 1] / J ** 2, a[..., 2] / (J - hy.ddof)
        return torch.stack([g2, var, var / (hy.eta ** 2 * g2)], -1)

    total = sums.sum(0)
    partial = op == "shard" or case["flags"] == "partial"
    clip = 1.0
    if op in ("clipped", "shard"):
        clip = min(1.0, 1.0 / (math.sqrt(float(total[1])) / J + 1e-6))
    three = [nan, nan, nan] if (partial or not stats) else derived(total).tolist()
    out = {"sums": total if stats else torch.full((3,), nan, dtype=f64),
           "derived": torch.tensor(three + [clip if op == "clipped" else 1.0], dtype=f64),
           "counts": None, "pass_status": None,
           "max_ratio": ratio.max().reshape(1) if case["coord"] else torch.tensor([-1.0], dtype=f64)}
    if update:
        # one array at a time: at the largest size every 64-bit vector is 12 GB
        w, m, v = s["w"], s["m"], s["v"]
        em, ev, ew = (torch.empty(d, dtype=f64, device=DEVICE) for _ in range(3))
        bc1, bc2 = 1 - hy.beta1 ** hy.step, 1 - hy.beta2 ** hy.step
        for lo in range(0, d, 1 << 26):
            at = slice(lo, min(d, lo + (1 << 26)))
            g = gbar[at] * clip
            em[at] = hy.beta1 * m[at].to(f64) + (1 - hy.beta1) * g
            ev[at] = hy.beta2 * v[at].to(f64) + (1 - hy.beta2) * g * g
            ew[at] = (1 - hy.lr * hy.weight_decay) * w[at].to(f64) \
                - hy.lr * (em[at] / bc1) / ((ev[at] / bc2).sqrt() + hy.eps)
        out.update(w=ew, m=em, v=ev)
    if "gbar" in s:
        out["gbar"] = gbar
    if op == "layers":
        out["layer_stats"] = torch.cat([sums, derived(sums)], -1)
        out["layer_counts"] = None
        out["layer_max_ratio"] = ratio if case["coord"] else torch.full((L,), -1.0, dtype=f64)
    return out
