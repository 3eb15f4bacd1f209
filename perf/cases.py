"""The work that a user of this library has it do, as cases that can be timed and checked.

Three kinds of pass, all through the binding's public calls:

  gemv   a loop over the layers of a model, one dpllm_gemv per layer at a fixed bitwidth: what a program does that picks
         its bitwidths itself, or serves a small batch.  Every layer has its own weights, as in a model.
  calls  a loop over the linears of some Transformer blocks, each dpllm_estimate followed by dpllm_gemv at the bitwidth
         the estimate left on the device: how the library sits inside a program that runs its own attention between.
  step   dpllm_decode_step over all linears of a model; either every linear has its input ready ("chain": False), or the
         buffers are chained the way a Transformer block chains them.

Weights are random p-bit codes with Gaussian-quantile tables per row (what a non-uniform quantiser produces),
scaled so that activations keep their size from layer to layer; activations are N(0, 1) with one channel in a
hundred twenty times larger; the projections are Gaussian.  Thresholds lie a few to some tens of per cent from the
estimates of the inputs at hand, half of them on either side, so that about half of the linears take the wider code.
"""
import math

import numpy as np
import torch

import paper_2508_06041_amd as dp

# (rows, columns) of q, k, v, o, gate, up, down
SHAPES = {
    "7b": [(4096, 4096)] * 4 + [(11008, 4096)] * 2 + [(4096, 11008)],
    "8b": [(4096, 4096), (1024, 4096), (1024, 4096), (4096, 4096)] + [(14336, 4096)] * 2 + [(4096, 14336)],
    "70b": [(8192, 8192), (1024, 8192), (1024, 8192), (8192, 8192)] + [(28672, 8192)] * 2 + [(8192, 28672)],
}
RANK = 64


def _gemv(name, out, in_, p, kmin, k, batch, layers):
    c = {"kind": "gemv", "out": out, "in": in_, "p": p, "kmin": kmin, "k": k, "batch": batch, "layers": layers}
    return dict(c, name=name) if name else c


def _calls(name, model, p, l, h, hybrid, blocks):
    c = {"kind": "calls", "model": model, "p": p, "l": l, "h": h, "hybrid": hybrid, "blocks": blocks}
    return dict(c, name=name) if name else c


def _step(name, model, p, l, h, hybrid, blocks, chain, ahead):
    c = {"kind": "step", "model": model, "p": p, "l": l, "h": h, "hybrid": hybrid, "blocks": blocks, "chain": chain, "ahead": ahead}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one key or value projection of a grouped-query model, alone
        _gemv("gemv_1024x4096_k3", 1024, 4096, 8, 3, 3, 1, 1),
        # an attention projection of every layer in turn
        _gemv("gemv_4096x4096_k4", 4096, 4096, 8, 3, 4, 1, 16),
        # odd sizes: rows that are no multiple of 64, columns that are no multiple of 128
        _gemv("gemv_2500x6688_k7", 2500, 6688, 7, 3, 7, 1, 8),
        # a two-bit child model
        _gemv("gemv_4096x11008_k2", 4096, 11008, 4, 2, 2, 1, 8),
        # few rows of long columns, the largest batch
        _gemv("gemv_4096x14336_k3_b8", 4096, 14336, 8, 3, 3, 8, 8),
        # many rows, an ordinary small batch
        _gemv("gemv_14336x4096_k6_b4", 14336, 4096, 8, 3, 6, 4, 8),
        # the widest projection of the largest model
        _gemv("gemv_28672x8192_k6", 28672, 8192, 6, 3, 6, 1, 4),
        # linear by linear inside a program of its own
        _calls("calls_7b", "7b", 8, 4, 5, False, 2),
        # a whole token: buffers chained, every selector on its linear's own input
        _step("chain_7b", "7b", 8, 3, 4, False, 32, True, False),
        # the same with every second linear on the linear regression and selectors that read an earlier vector
        _step("chain_8b_ahead", "8b", 8, 5, 6, True, 16, True, True),
        # all linears of a token in one group: streaming throughput
        _step("step_7b", "7b", 8, 3, 4, False, 32, False, False),
        # part of the largest model, the hybrid of both estimators
        _step("step_70b", "70b", 6, 4, 5, True, 8, False, False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemv", "gemv", "gemv", "calls", "step"])
    if kind == "gemv":
        out, in_ = _log_int(rng, 192, 28672), 32 * _log_int(rng, 8, 896)
        while out * in_ > 28672 * 8192:
            out, in_ = _log_int(rng, 192, 28672), 32 * _log_int(rng, 8, 896)
        p = rng.randint(3, 8)
        kmin = rng.randint(2, 3)
        k = rng.randint(kmin, p)
        batch = rng.choice([1, 1, 1, 2, 3, 4, 5, 6, 7, 8])
        layers = max(1, min(16, int(3e8 / (out * in_ * p / 8))))
        return _gemv(None, out, in_, p, kmin, k, batch, rng.randint(1, layers))
    model = rng.choice(["7b", "8b", "70b"])
    l = rng.randint(3, 5)
    p = rng.randint(l + 1, 8) if model != "70b" else 6
    hybrid = rng.random() < 0.5
    if kind == "calls":
        return _calls(None, model, p, l, l + 1, hybrid, rng.randint(1, 3))
    blocks = _log_int(rng, 2, 24) if model != "70b" else rng.randint(1, 4)
    chain = rng.random() < 0.5
    return _step(None, model, p, l, l + 1, hybrid, blocks, chain, chain and rng.random() < 0.5)


# ---- inputs ---------------------------------------------------------------------------------------------------
def _gen(*key):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(np.random.SeedSequence([int(k) for k in key]).generate_state(1, np.uint64)[0] >> 1))
    return g


def _unit_tables(p, kmin):
    """{k: fp64 [2^k]}: Gaussian quantiles and the means of their children, each of unit mean square."""
    n = 1 << p
    q = torch.special.ndtri((torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) / n)
    tables = {k: q.reshape(1 << k, -1).mean(dim=1) for k in range(kmin, p + 1)}
    return {k: t / t.square().mean().sqrt() for k, t in tables.items()}


def _weights(seed, i, out, in_, p, kmin, units):
    """planes int32 [p][out][in / 32] and {k: fp16 [out][2^k]} of linear i."""
    g = _gen(seed, 1, i)
    planes = torch.randint(-2 ** 31, 2 ** 31, (p, out, in_ // 32), dtype=torch.int32, device="cuda", generator=g)
    s = torch.exp(0.5 * torch.randn(out, generator=g, device="cuda", dtype=torch.float64))
    s /= s.square().mean().sqrt() * math.sqrt(in_)
    return planes, {k: (s[:, None] * t[None, :]).half() for k, t in units.items()}


def _activations(seed, i, n, in_):
    g = _gen(seed, 2, i)
    x = torch.randn(n, in_, generator=g, device="cuda")
    x[:, torch.randperm(in_, generator=g, device="cuda")[:max(1, in_ // 100)]] *= 20.0
    return x.half()


def _projection(seed, i, in_):
    """G of linear i: with these weights ||(W_h - W_l) x|| is some tenth of ||W x||."""
    return (torch.randn(RANK, in_, generator=_gen(seed, 3, i), device="cuda") * (0.1 / math.sqrt(in_))).half()


def _choices(seed, n):
    """Per linear: whether its estimate lies above its threshold, and the threshold over the estimate."""
    rng = np.random.default_rng([seed, 4])
    wide = rng.random(n) < 0.5
    return wide, np.where(wide, rng.uniform(0.6, 0.95, n), rng.uniform(1.05, 1.6, n))


def _linreg(case, i):
    return case["hybrid"] and i % 2 == 1


LINREG = (0.011, 0.25)   # alpha, beta


def _linears(case):
    return SHAPES[case["model"]] * case["blocks"]


def _chain(case):
    """Per linear the buffer it reads, the one it writes, and the one its selector reads.  Buffer 0 is the input of the
    token; linear i writes buffer i + 1."""
    src, sel = [], []
    res = 0                                   # the residual the block starts from
    before = None                             # the attention output of the block before
    for b in range(case["blocks"]):
        q, o, gate, down = 7 * b + 1, 7 * b + 4, 7 * b + 5, 7 * b + 7
        src += [res, res, res, q, o, o, gate]
        qkv = res if before is None else before
        sel += [qkv, qkv, qkv, q, res, res, gate] if case["ahead"] else src[-7:]
        res, before = down, o
    return src, sel


def prepare(case, seed):
    if case["kind"] == "gemv":
        return _prepare_gemv(case, seed)
    shapes = _linears(case)
    n, l, h = len(shapes), case["l"], case["h"]
    units = _unit_tables(case["p"], 3)
    m = dp.Model(n)
    for i, (out, in_) in enumerate(shapes):
        planes, luts = _weights(seed, i, out, in_, case["p"], 3, units)
        m.dpllm_load_linear(i, planes, luts, 3)
        del planes, luts
    wide, ratio = _choices(seed, n)
    y = torch.zeros(sum(out for out, _ in shapes), dtype=torch.float16, device="cuda")
    ys = list(torch.split(y, [out for out, _ in shapes]))
    k = torch.zeros(n, dtype=torch.int32, device="cuda")
    e = torch.zeros(n, dtype=torch.float32, device="cuda")
    # thresholds from a calibration pass with every selector pinned to its side
    kinds = [(dp.DPLLM_SEL_LINREG, None) if _linreg(case, i) else (dp.DPLLM_SEL_PROJ, _projection(seed, i, in_))
             for i, (_, in_) in enumerate(shapes)]
    for i, (kind, G) in enumerate(kinds):
        m.dpllm_set_selector(i, l, h, kind, G=G, alpha=LINREG[0], beta=LINREG[1], T=-math.inf if wide[i] else math.inf)
    s = {"kind": case["kind"], "model": m, "y": y, "ys": ys, "k": k, "e": e}
    if case["kind"] == "calls":
        s["xs"] = [_activations(seed, i, 1, in_)[0] for i, (_, in_) in enumerate(shapes)]
        s["pair"] = (l, h)
        s["es"], s["ks"] = list(torch.split(e, 1)), list(torch.split(k, 1))
    else:
        if case["chain"]:
            src, sel = _chain(case)
            buffers = [_activations(seed, 0, 1, shapes[0][1])[0]] + ys
            xs = [buffers[j] for j in src]
            if case["ahead"]:
                for i in range(n):
                    if sel[i] != src[i]:
                        m.dpllm_set_selector_input(i, buffers[sel[i]])
        else:
            by_width = {in_: _activations(seed, in_, 1, in_)[0] for _, in_ in shapes}
            xs = [by_width[in_] for _, in_ in shapes]
        s["keep"] = xs
        s["xp"], s["yp"] = m.pointers(xs), m.pointers(ys)
    run(s)
    for i, est in enumerate(e.tolist()):
        m.dpllm_set_threshold(i, l, h, float(np.float32(est * ratio[i])))
    return s


def _prepare_gemv(case, seed):
    m = dp.Model(case["layers"])
    units = _unit_tables(case["p"], case["kmin"])
    xs = []
    for i in range(case["layers"]):
        planes, luts = _weights(seed, i, case["out"], case["in"], case["p"], case["kmin"], units)
        m.dpllm_load_linear(i, planes, luts, case["kmin"])
        del planes, luts
        x = _activations(seed, i, case["batch"], case["in"])
        xs.append(x if case["batch"] > 1 else x[0])
    shape = (case["out"],) if case["batch"] == 1 else (case["batch"], case["out"])
    y = torch.zeros((case["layers"],) + shape, dtype=torch.float16, device="cuda")
    return {"kind": "gemv", "model": m, "k": case["k"], "xs": xs, "y": y, "ys": list(y.unbind(0))}


# ---- one pass -------------------------------------------------------------------------------------------------
def run(state):
    m = state["model"]
    if state["kind"] == "gemv":
        k = state["k"]
        for i, (x, y) in enumerate(zip(state["xs"], state["ys"])):
            m.dpllm_gemv(i, k, x, y=y)
        return state["y"]
    if state["kind"] == "calls":
        l, h = state["pair"]
        for i, (x, y, e, k) in enumerate(zip(state["xs"], state["ys"], state["es"], state["ks"])):
            m.dpllm_estimate(i, l, h, x, e_out=e, k_out=k)
            m.dpllm_gemv(i, -1, x, y=y, k_dev=k)
    else:
        m.dpllm_decode_step(state["xp"], state["yp"], state["k"], state["e"])
    return {"y": state["y"], "k": state["k"], "e": state["e"]}


# ---- what a pass cannot do without ------------------------------------------------------------------------------
def work(case):
    if case["kind"] == "gemv":
        out, in_, k, b = case["out"], case["in"], case["k"], case["batch"]
        one = out * in_ * k / 8 + out * (2 << k) + 2 * b * (in_ + out)
        return {"bytes": case["layers"] * one, "flops": case["layers"] * 2.0 * b * out * in_}
    # about half of the linears run at either bitwidth
    mean_bits, mean_table = (case["l"] + case["h"]) / 2, ((2 << case["l"]) + (2 << case["h"])) / 2
    byts = flops = 0.0
    for i, (out, in_) in enumerate(_linears(case)):
        rows = 0 if _linreg(case, i) else RANK
        byts += out * in_ * mean_bits / 8 + out * mean_table + 2 * (in_ + out) + 2 * rows * in_ + 8
        flops += 2.0 * in_ * (out + max(1, rows))
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    # results are fp16 (half a unit in the last place is 2.4e-4 of a value, about 2e-4 in the 2-norm); chained, that
    # rounding is fed on through four linears per block.  Bitwidths are the same: thresholds keep their distance
    if case["kind"] == "step" and case["chain"]:
        return {"rel": 6e-3, "max": 0.06, "differ": 0.0}
    return {"rel": 1e-3, "max": 4e-3, "differ": 0.0}


def _dense_product(planes, lut, k, x):
    """x [B][in] (fp64) times the k-bit weights [out][in], in fp64: the code of a weight is its bits in planes 0 .. k - 1,
    most significant first; column c is bit c mod 32 of word c / 32."""
    _, out, nw = planes.shape
    y = torch.empty(x.shape[0], out, dtype=torch.float64, device="cuda")
    bit = torch.arange(32, device="cuda", dtype=torch.int32)
    step = max(1, (1 << 24) // (nw * 32))
    for r in range(0, out, step):
        code = torch.zeros((), dtype=torch.int32, device="cuda")
        for b in range(k):
            code = code * 2 + ((planes[b, r:r + step, :, None] >> bit) & 1)
        w = torch.gather(lut[r:r + step].double(), 1, code.reshape(code.shape[0], -1).long())
        y[:, r:r + step] = (w @ x.T).T
    return y


def exact(case, seed):
    if case["kind"] == "gemv":
        units = _unit_tables(case["p"], case["kmin"])
        ys = []
        for i in range(case["layers"]):
            planes, luts = _weights(seed, i, case["out"], case["in"], case["p"], case["kmin"], units)
            x = _activations(seed, i, case["batch"], case["in"]).double()
            y = _dense_product(planes, luts[case["k"]], case["k"], x)
            ys.append(y if case["batch"] > 1 else y[0])
        return torch.stack(ys)
    shapes = _linears(case)
    units = _unit_tables(case["p"], 3)
    wide, _ = _choices(seed, len(shapes))
    chain = case["kind"] == "step" and case["chain"]
    if chain:
        src, sel = _chain(case)
        buffers = [_activations(seed, 0, 1, shapes[0][1])[0].double()]
    ys, ks, es = [], [], []
    for i, (out, in_) in enumerate(shapes):
        if chain:
            x, xsel = buffers[src[i]], buffers[sel[i]]
        else:
            x = xsel = _activations(seed, i if case["kind"] == "calls" else in_, 1, in_)[0].double()
        if _linreg(case, i):
            alpha, beta = (float(np.float32(v)) for v in LINREG)
            est = alpha * float(xsel.norm()) + beta
        else:
            est = float((_projection(seed, i, in_).double() @ xsel).norm())
        k = case["h"] if wide[i] else case["l"]
        planes, luts = _weights(seed, i, out, in_, case["p"], 3, units)
        y = _dense_product(planes, luts[k], k, x[None])[0]
        if chain:
            buffers.append(y)
        ys.append(y)
        ks.append(k)
        es.append(est)
    return {"y": torch.cat(ys), "k": None, "e": torch.tensor(es, dtype=torch.float64, device="cuda")}
