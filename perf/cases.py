"""The work a user of this library has it do, as cases that can be timed and compared.

A case is one call a training program makes per iteration: the fused compression step in its
forms (deterministic top-k, HEAVYMIX, momentum and error kept in the sketch, inside the
training loop with the weight update), the separate calls of a program that runs one worker
per GPU, and the estimate without a context. Sizes are those of this repository's workloads
(`synth`), of the warm-up schedule of its training integration, and odd ones in between.

Gradients are drawn on the GPU with the workloads' distributions: Laplace with log-uniform
layer scales, Student-t(3) with a few coordinates 100 times larger (heavy hitters), and row-sparse
embedding gradients over a dense half.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2108_06004_amd as gs
from paper_2108_06004_amd.train import DensitySchedule, GlobalSketchSGD

DEV = "cuda:0"
RHO = 0.9
MERSENNE = (1 << 31) - 1
# the warm-up of the training integration: (density, learning rate) of the first epochs
WARMUP = [(0.25, 0.1), (0.0725, 0.03), (0.015, 0.01), (0.004, 0.01)]


def listed():
    def case(name, call, d, P, r, c, k, grads, **more):
        return dict(name=name, call=call, d=d, P=P, r=r, c=c, k=k, grads=grads, **more)

    return [
        # the smallest model: launches and latency decide
        case("step-65k-p4", "step", 65_536, 4, 5, 4_096, 655, "heavy", layout="interleaved"),
        # a ResNet-20-sized model in the training loop: fused step and weight update
        case("train-270k-p4", "train", 270_000, 4, 5, 27_000, 2_700, "layers", layout="worker_major", epoch=9),
        # an odd size and a worker count that is no multiple of four
        case("step-1.2M-p6", "step", 1_234_567, 6, 5, 61_729, 12_345, "layers", layout="interleaved"),
        # many small workers simulated on one GPU
        case("step-2M-p32", "step", 2_000_003, 32, 5, 100_003, 20_000, "layers", layout="interleaved"),
        # estimates of every coordinate by a program that holds no context (monitoring, capture)
        case("estimate-4M", "static", 4_000_000, 4, 5, 400_000, 40_000, "layers"),
        # a VGG-16-sized model
        case("step-14.7M-p4", "step", 14_700_000, 4, 5, 1_470_000, 14_700, "heavy", layout="interleaved"),
        # the same in the first warm-up epoch of the training loop: a quarter of the coordinates
        case("warmup-14.7M-p4", "train", 14_700_000, 4, 5, 1_470_000, 3_675_000, "heavy", layout="worker_major",
             epoch=0),
        # the same with momentum and error kept in the sketch
        case("sketch-state-14.7M-p4", "sketch_state", 14_700_000, 4, 5, 1_470_000, 14_700, "heavy",
             layout="worker_major"),
        # a ResNet-50-sized model, one worker per GPU: its calls around its own exchange
        case("worker-25.6M-p1", "calls", 25_600_000, 1, 5, 256_000, 25_600, "layers", layout="worker_major"),
        # a ResNet-50-sized model, eight workers: the benchmark's step
        case("step-25.6M-p8", "step", 25_600_000, 8, 5, 256_000, 25_600, "layers", layout="interleaved"),
        # the same with HEAVYMIX as printed
        case("heavymix-25.6M-p8", "heavymix", 25_600_000, 8, 5, 256_000, 25_600, "layers", layout="interleaved"),
        # an LSTM language model's size, sixteen workers, row-sparse embedding gradients
        case("step-66M-p16", "step", 66_000_000, 16, 7, 1_320_000, 66_000, "rows", layout="interleaved"),
    ]


def draw(rng):
    call = rng.choice(["step", "step", "step", "train", "heavymix", "sketch_state", "calls", "static"])
    P = 1 if call == "calls" else rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 8, 12, 16, 24, 32])
    # at most the largest listed case's work; the simulated many-worker runs are small models
    most = min(66e6, 1e9 / P, 8e7 / P if P > 16 else 1e9)
    if call == "static":
        most = gs.GS_STATIC_MAX_D
    if call == "train":
        most = min(most, 15e6)
    d = int(round(math.exp(rng.uniform(math.log(50_000), math.log(most)))))
    if rng.random() < 0.3:
        d -= d % 1000
    r = rng.choice([3, 4, 5, 5, 5, 7])
    c = max(64, int(d / math.exp(rng.uniform(math.log(8), math.log(100)))))
    if call == "train" and rng.random() < 0.5:
        epoch = rng.randrange(len(WARMUP))
        k = math.ceil(WARMUP[epoch][0] * d)
    else:
        epoch = 9
        k = max(1, int(d * math.exp(rng.uniform(math.log(5e-4), math.log(1e-2)))))
    grads = rng.choice(["layers", "heavy"])
    layout = rng.choice(["interleaved", "worker_major"])
    if call == "sketch_state":  # needs heavy hitters that the sketch can recover: k well below c
        grads, layout = "heavy", "worker_major"
        c = max(c, d // 16)
        k = max(1, d // 1000)
    if call in ("train", "calls"):
        layout = "worker_major"
    case = dict(call=call, d=d, P=P, r=r, c=c, k=k, grads=grads)
    if call != "static":
        case["layout"] = layout
    if call == "train":
        case["epoch"] = epoch
    return case


def _hash_params(r, seed):
    g = np.random.default_rng([seed, 77])
    return {n: g.integers(lo, MERSENNE, size=r, dtype=np.int64).astype(np.uint32)
            for n, lo in (("a", 1), ("b", 0), ("a2", 1), ("b2", 0))}


def _scales(case, seed):
    """Scale of each coordinate of the layered gradients: 53 (20 below 1M coordinates) layers."""
    d = case["d"]
    n = 53 if d >= 1_000_000 else 20
    g = np.random.default_rng([seed, 78])
    s = 10.0 ** g.uniform(-5.0 if n == 53 else -4.0, -2.0, size=n)
    return torch.repeat_interleave(torch.tensor(s, dtype=torch.float32, device=DEV), -(-d // n))[:d]


def _values(case, seed, gen):
    """One [P][d] array of the case's gradient distribution."""
    d, P = case["d"], case["P"]
    out = torch.empty((P, d), dtype=torch.float32, device=DEV)
    if case["grads"] == "layers":
        scale = _scales(case, seed)
        for q in range(P):
            u = torch.rand(d, generator=gen, device=DEV) - 0.5
            out[q] = -scale * torch.sign(u) * torch.log1p(-2.0 * torch.abs(u).clamp(max=0.4999999))
    elif case["grads"] == "heavy":
        big = torch.randperm(d, generator=torch.Generator(device=DEV).manual_seed(seed * 31 + 7),
                             device=DEV)[:max(1, d // 1000)]
        for q in range(P):
            z = torch.randn((4, d), generator=gen, device=DEV)
            row = 1e-3 * z[0] / torch.sqrt((z[1] ** 2 + z[2] ** 2 + z[3] ** 2) / 3.0)
            row[big] = row[big] * 100.0
            out[q] = row
    else:  # rows: an embedding of 1,500 columns with 2% of its rows active, then a dense half
        cols = 1_500
        rows = d // 2 // cols
        for q in range(P):
            row = 1e-4 * torch.randn(d, generator=gen, device=DEV)
            active = torch.rand(rows, generator=gen, device=DEV) < 0.02
            row[:rows * cols] *= (100.0 * active.float()).repeat_interleave(cols)
            out[q] = row
    return out


def _inputs(case, seed):
    """Gradients, momentum, error ([P][d] each) and the hash family of a step in mid-training."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 1_000_003 + 17)
    hp = _hash_params(case["r"], seed)
    g = _values(case, seed, gen)
    u = _values(case, seed, gen).mul_(2.0)
    v = _values(case, seed, gen).mul_(4.0)
    return g, u, v, hp, gen


def _hashes(case, hp, j, dev=DEV):
    i = torch.arange(case["d"], dtype=torch.int64, device=dev)
    col = (i * int(hp["a"][j]) + int(hp["b"][j])) % MERSENNE % case["c"]
    odd = (i * int(hp["a2"][j]) + int(hp["b2"][j])) % MERSENNE % 2
    return col, (2 * odd - 1)


def _sketch64(case, hp, x):
    """Count Sketch of a [d] vector in 64 bits."""
    out = torch.zeros((case["r"], case["c"]), dtype=torch.float64, device=DEV)
    for j in range(case["r"]):
        col, sign = _hashes(case, hp, j)
        out[j].index_add_(0, col, x * sign)
    return out


def _estimate64(case, hp, table):
    vals = []
    for j in range(case["r"]):
        col, sign = _hashes(case, hp, j)
        vals.append(table[j][col] * sign)
    r = case["r"]
    # selection network by columns: r is small
    for a in range(r):
        for t in range(a & 1, r - 1, 2):
            lo, hi = torch.minimum(vals[t], vals[t + 1]), torch.maximum(vals[t], vals[t + 1])
            vals[t], vals[t + 1] = lo, hi
    return vals[r // 2] if r % 2 else (vals[r // 2 - 1] + vals[r // 2]) * 0.5


def _top(key, k):
    """The k largest keys, ties to the lower index, ascending."""
    order = torch.sort(key, descending=True, stable=True).indices[:k]
    return torch.sort(order).values


def prepare(case, seed):
    d, P, r, c, k, call = (case[n] for n in ("d", "P", "r", "c", "k", "call"))
    g, u, v, hp, gen = _inputs(case, seed)
    st = dict(case=case, g=g)
    if call == "static":
        st.update(merged=_sketch64(case, hp, g.double().sum(0)).float(), hp=hp)
        st["est"] = torch.empty(d, dtype=torch.float32, device=DEV)
        st["idx"] = torch.empty(k, dtype=torch.int32, device=DEV)
        del st["g"]
        return st
    if call == "train":
        epoch = case["epoch"]
        sched = DensitySchedule((k - 0.5) / d if epoch >= len(WARMUP) else 0.01, 0.1, WARMUP)
        opt = GlobalSketchSGD(d, P, r, c, hp, sched, rho=RHO, device=DEV)
        opt.u.copy_(u)
        opt.v.copy_(v)
        st.update(opt=opt, w=torch.randn(d, generator=gen, device=DEV), epoch=epoch)
        return st
    ctx = gs.GsContext(d, P, r, c, k, hp, rho=RHO, state_layout=case["layout"])
    st["ctx"] = ctx
    f32 = dict(dtype=torch.float32, device=DEV)
    st["merged"] = torch.empty((r, c), **f32)
    st["idx"] = torch.empty(k, dtype=torch.int32, device=DEV)
    st["values"] = torch.empty(k, **f32)
    if call == "sketch_state":
        st["U"] = _sketch64(case, hp, u.double().sum(0)).float()
        st["E"] = _sketch64(case, hp, v.double().sum(0)).float()
        return st
    st["u"], st["v"] = ctx.to_state(u), ctx.to_state(v)
    if call == "heavymix":
        st["rnd"] = torch.empty(d, dtype=torch.int32, device=DEV).random_(-(1 << 31), 1 << 31, generator=gen)
        st["n_heavy"] = torch.empty(1, dtype=torch.int64, device=DEV)
    if call == "calls":
        st["tables"] = torch.empty((P, r, c), **f32)
    return st


def run(st):
    case = st["case"]
    call, k = case["call"], case["k"]
    if call == "static":
        gs.gs_unsketch_topk_static(case["d"], case["r"], case["c"], st["hp"], st["merged"], k, st["est"], st["idx"])
        return {n: st[n] for n in ("est", "idx")}
    if call == "train":
        opt = st["opt"]
        got = opt.step(st["g"], st["w"], epoch=st["epoch"])["k"]
        return dict(w=st["w"], u=opt.u, v=opt.v, merged=opt.merged, idx=opt.idx[:got], values=opt.values[:got])
    ctx = st["ctx"]
    if call == "sketch_state":
        ctx.step_sketch_momentum(st["g"], st["U"], st["E"], k, st["merged"], st["idx"], st["values"])
        return {n: st[n] for n in ("U", "E", "merged", "idx", "values")}
    if call == "heavymix":
        ctx.step_heavymix(st["g"], st["u"], st["v"], k, st["rnd"], st["merged"], st["idx"], st["values"],
                          n_heavy=st["n_heavy"])
        return {n: st[n] for n in ("u", "v", "merged", "idx", "values", "n_heavy")}
    if call == "calls":  # one worker: its table would be all-reduced before the selection
        ctx.accumulate(st["g"], st["u"], st["v"])
        ctx.sketch(st["v"], st["tables"])
        ctx.merge(st["tables"], st["merged"])
        ctx.unsketch_topk(st["merged"], k, st["idx"])
        ctx.gather_reset(st["idx"], k, st["u"], st["v"], st["values"])
    else:
        ctx.step(st["g"], st["u"], st["v"], k, st["merged"], st["idx"], st["values"])
    return {n: st[n] for n in ("u", "v", "merged", "idx", "values")}


def work(case):
    """Each input read once, each output written once (interleaved rows without their padding)."""
    d, P, r, c, k, call = (case[n] for n in ("d", "P", "r", "c", "k", "call"))
    if call == "static":
        return {"bytes": 4 * r * c + 4 * d + 4 * k, "flops": r * d}
    if call == "sketch_state":
        return {"bytes": 4 * P * d + 20 * r * c + 8 * k, "flops": (P * r + r) * d}
    b = 20 * P * d + 8 * r * c + 12 * P * k + 8 * k
    if call == "heavymix":
        b += 4 * d
    if call == "train":
        b += 8 * k
    return {"bytes": b, "flops": (3 * P + P * r + r) * d}


def tolerance(case):
    # fp32 results of a few rounded operations each; the cells are 64-bit sums rounded once.
    # Measured against 64 bits over the listed and some drawn cases: at most 1.4e-7 (E), 7.3e-8
    # (merged), 5.6e-8 (values), 3.6e-8 (u, v) and 2.8e-8 (est).
    return {"rel": 6e-7, "max": 1e-5, "differ": 0.002}


def exact(case, seed):
    d, P, r, c, k, call = (case[n] for n in ("d", "P", "r", "c", "k", "call"))
    g, u, v, hp, gen = _inputs(case, seed)
    rho = float(np.float32(RHO))
    if call == "static":
        merged = _sketch64(case, hp, g.double().sum(0)).float().double()
        est = _estimate64(case, hp, merged)
        return dict(est=est, idx=_top(est.abs(), k))
    if call == "sketch_state":
        S = _sketch64(case, hp, g.double().sum(0))
        U = rho * _sketch64(case, hp, u.double().sum(0)).float().double() + S
        E = _sketch64(case, hp, v.double().sum(0)).float().double() + U
        est = _estimate64(case, hp, E)
        idx = _top(est.abs(), k)
        values = est[idx]
        for j in range(r):
            col, sign = _hashes(case, hp, j)
            col, sign = col[idx], sign[idx]
            E[j].index_add_(0, col, -values * sign)
            U[j][col] = 0.0
        return dict(U=U, E=E, merged=S, idx=idx, values=values)
    w = torch.randn(d, generator=gen, device=DEV).double() if call == "train" else None
    rnd = None
    if call == "heavymix":
        rnd = torch.empty(d, dtype=torch.int32, device=DEV).random_(-(1 << 31), 1 << 31, generator=gen)
    total = torch.zeros(d, dtype=torch.float64, device=DEV)
    for q in range(P):  # worker by worker: the sum that is sketched needs no [P][d] in 64 bits
        total += v[q].double() + (rho * u[q].double() + g[q].double())
    merged = _sketch64(case, hp, total)
    est = _estimate64(case, hp, merged)
    more = {}
    if call == "heavymix":
        theta = (merged ** 2).sum(1).median() / k if r % 2 else None
        if theta is None:
            rows = torch.sort((merged ** 2).sum(1)).values
            theta = 0.5 * (rows[r // 2 - 1] + rows[r // 2]) / k
        heavy = est ** 2 >= theta
        draws = (rnd.to(torch.int64) & 0xffffffff) >> 1
        key = torch.where(heavy, est.abs() + 2.0 ** 32, draws.double())
        more["n_heavy"] = heavy.sum().reshape(1)
        if int(heavy.sum()) >= k:
            key = torch.where(heavy, est.abs(), torch.full_like(est, -1.0))
    else:
        key = est.abs()
    idx = _top(key, k)
    del est, key
    out = dict(merged=merged, idx=idx, values=total[idx], **more)
    del total
    if case["P"] * d > 3e8:  # the state in 64 bits is left out where it would not fit beside the rest
        return dict(out, u=None, v=None)
    u64 = rho * u.double() + g.double()
    v64 = v.double() + u64
    u64[:, idx] = 0.0
    v64[:, idx] = 0.0
    if case["layout"] == "interleaved":
        PP = gs.state_stride(P)

        def rows(x):
            y = torch.zeros((d, PP), dtype=torch.float64, device=DEV)
            y[:, :P] = x.t()
            return y

        u64, v64 = rows(u64), rows(v64)
    out.update(u=u64, v=v64)
    if call == "train":
        epoch = case["epoch"]
        lr = WARMUP[epoch][1] if epoch < len(WARMUP) else 0.1
        w[idx] -= float(np.float32(lr / P)) * out["values"]
        out["w"] = w
    return out
