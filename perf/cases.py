"""The workloads this library is used for, as cases that can be timed and compared.

A case is one call of the library on one model: which step (`op`), the model's matrices (`net` and its sizes), the rank,
the bits and block of the error quantiser or the kept share of the count sketch, and the type of the gradients.  Inputs
are synthetic and come from the seed alone: gradients with the distributions of the workloads in
`paper_2312_08538_amd/workloads.py`, and an error state such as a run has after some steps (codes and scales, or a
sketch table), so that no path sees the all-zero state of a run's first step only.

A state can be stepped again and again.  On gradients that never change the error grows without bound (real training
changes them), so every sixteenth pass starts by clearing the error, as `bench.py` does.
"""
from __future__ import annotations

import math

import torch

from paper_2312_08538_amd import binding as B
from paper_2312_08538_amd import workloads as wl

DTYPES = {"f32": wl.F32, "bf16": wl.BF16}
DISTS = {"normal": 1e-3, "normal_fanin": 1.0, "laplace": 1e-3, "student_t3": 1e-3}
RESET_EVERY = 16          # passes on one state between two clearings of its error
SKETCH_KEEP, SKETCH_BETA = 0.2, 0.9       # an fp16 table of a fifth of the rows or columns: 90 % of an fp32 error saved
RK_GROUP = 10             # random-k keeps one coordinate of ten


# ------------------------------------------------------------------------------------------------ models
def layout_of(case):
    """(rows, cols) of every compressed matrix, in model order."""
    net, d = case["net"], case["d"]
    if net == "matrix":
        return [(case["rows"], d)]
    if net == "resnet":                     # the 18-layer residual network with `d` channels in its first stage
        L = [(d, 3 * 49)] + [(d, 9 * d)] * 4
        for s in (1, 2, 3):
            i, o = d << (s - 1), d << s
            L += [(o, 9 * i), (o, 9 * o), (o, i), (o, 9 * o), (o, 9 * o)]
        return L + [(case["out"], 8 * d)]
    if net == "gpt":                        # decoder-only transformer, tied embedding
        return [(case["out"], d)] + [(d, 3 * d), (d, d), (d, 4 * d), (4 * d, d)] * case["layers"]
    if net == "transformer":                # encoder and decoder of `layers` layers each
        L = [(case["out"], d)]
        L += ([(d, d)] * 4 + [(d, 4 * d), (4 * d, d)]) * case["layers"]
        return L + ([(d, d)] * 8 + [(d, 4 * d), (4 * d, d)]) * case["layers"]
    if net == "recurrent":                  # LSTM language model, tied embedding
        return [(case["out"], d)] + [(4 * d, d)] * (2 * case["layers"])
    raise ValueError(net)


def elements_of(case):
    return sum(n * m for n, m in layout_of(case))


def listed():
    def c(name, op, net, d, rank, dtype, dist, bits=4, block=128, rows=0, out=0, layers=0):
        return {"name": name, "op": op, "net": net, "d": d, "rows": rows, "out": out, "layers": layers, "rank": rank,
                "bits": bits, "block": block, "dtype": dtype, "dist": dist}

    return [
        # one small matrix, the least a caller can ask for: launches and the host path
        c("tiny", "step", "matrix", 128, 2, "f32", "normal", bits=8, block=64, rows=256),
        # image classification: 21 convolution and dense matrices of very different sizes, 147 columns among them
        c("cnn", "step", "resnet", 64, 4, "f32", "normal_fanin", out=1000),
        # a recurrent language model: no dimension is a multiple of a block or of 16 bytes' worth of codes
        c("recurrent", "step", "recurrent", 650, 4, "f32", "laplace", out=33278, layers=2),
        # language-model fine-tuning in fp32
        c("lm", "step", "gpt", 768, 4, "f32", "laplace", out=50257, layers=12),
        # translation in bf16 with ternary codes
        c("translation", "step", "transformer", 1024, 8, "bf16", "normal", bits=2, block=256, out=32768, layers=6),
        # pre-training of a 1.3 G-parameter model in bf16 at a high rank: the largest
        c("large", "step", "gpt", 2048, 32, "bf16", "student_t3", out=50304, layers=24),
        # the same method with two error vectors (Algorithm 3)
        c("lm_iconef", "iconef_step", "gpt", 768, 4, "f32", "laplace", out=50257, layers=12),
        # the count sketch as the error compressor, in its row form ...
        c("translation_sketch", "sketch_step", "transformer", 1024, 8, "bf16", "normal", out=32768, layers=6),
        # ... and in its column form, on the network the paper's sketch experiments use
        c("cnn_sketch_columns", "sketch_columns_step", "resnet", 64, 4, "f32", "normal_fanin", out=1000),
        # element-wise gradient compressors, which stream the gradient and the error: the sign with one scale per matrix ...
        c("translation_sign", "sign_step", "transformer", 1024, 8, "bf16", "normal", bits=2, block=256, out=32768, layers=6),
        # ... and random-k with two error vectors, the paper's setting for Algorithm 3
        c("large_random_k", "iconef_random_k_step", "gpt", 2048, 32, "bf16", "student_t3", out=50304, layers=24),
        # decompression: the weights take the compressed gradient (what follows every step)
        c("large_update", "update", "gpt", 2048, 32, "bf16", "student_t3", out=50304, layers=24),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another model of the families above with another compressor setting."""
    while True:
        op = rng.choice(["step"] * 6 + ["iconef_step", "sketch_step", "sketch_columns_step", "sign_step", "iconef_random_k_step",
                                        "update"])
        net = rng.choice(["matrix", "resnet", "gpt", "transformer", "recurrent"])
        case = {"op": op, "net": net, "rows": 0, "out": 0, "layers": 0}
        if net == "matrix":
            case["rows"] = _log_int(rng, 64, 16384)
            case["d"] = _log_int(rng, 64, 8192) if rng.random() < 0.5 else 64 * _log_int(rng, 1, 128)
        elif net == "resnet":
            case.update(d=8 * rng.randint(3, 12), out=rng.choice([10, 100, 1000]))
        elif net == "recurrent":
            case.update(d=_log_int(rng, 96, 1500), out=_log_int(rng, 2000, 50000), layers=rng.randint(1, 3))
        else:
            case.update(d=64 * _log_int(rng, 2, 32), out=_log_int(rng, 2000, 50304), layers=_log_int(rng, 1, 12))
        case["rank"] = rng.choice([1, 2, 4, 4, 8, 8, 16, 32])
        case["bits"] = rng.choice([2, 4, 4, 8])
        case["block"] = rng.choice([64, 128, 128, 256, 512])
        case["dtype"] = rng.choice(["f32", "bf16"])
        case["dist"] = rng.choice(sorted(DISTS))
        layout = layout_of(case)
        # no costlier than the largest listed case: high ranks are the costly ones where they do not run on the bf16
        # matrix cores (blocks of 128 4-bit codes)
        if case["rank"] > min(min(n, m) for n, m in layout):
            continue
        if elements_of(case) * max(1, case["rank"] // 4) > 1.2e8 and not op.startswith(("sign", "iconef_random")):
            continue
        if elements_of(case) > 2.5e8:
            continue
        return case


# ------------------------------------------------------------------------------------------------ inputs
def _codes(flat, gen, n_elems, bits, word_off):
    """Codes of one matrix: a normal variable rounded to the levels, fields beyond the last element zero."""
    per, s = 32 // bits, (1 << (bits - 1)) - 1
    words = -(-n_elems // per)
    step = 1 << 24
    shift = torch.arange(per, device=flat.device, dtype=torch.int32) * bits
    for w0 in range(0, words, step):
        w1 = min(words, w0 + step)
        q = torch.randn((w1 - w0) * per, device=flat.device, generator=gen)
        q = q.mul_(max(1.0, s / 3.0) * 0.7).round_().clamp_(-s, s).to(torch.int32)
        q[max(0, n_elems - w0 * per):] = 0
        q = (q & ((1 << bits) - 1)).view(-1, per) << shift
        flat[word_off + w0:word_off + w1] = q.sum(1).to(torch.int32)


def _error(model, layout, gen, size, codes, scales):
    """An error vector whose entries are of the order of `size`[l] in matrix l."""
    for (n, m), o, sz in zip(layout, model.offsets, size):
        blocks = -(-n * m // model.block)
        _codes(codes, gen, n * m, model.bits, o["word_off"])
        scales[o["scale_off"]:o["scale_off"] + blocks] = torch.rand(blocks, device=scales.device, generator=gen).add_(2.0).mul_(sz)


def prepare(case, seed):
    dev = "cuda:0"
    layout, rank, dtype, op = layout_of(case), case["rank"], DTYPES[case["dtype"]], case["op"]
    w = wl.Workload("case", seed & 0x3FFFFFFF, tuple(layout), rank, case["bits"], case["block"], dtype, case["dist"],
                    DISTS[case["dist"]], 0x5EED0000 + (seed & 0xFFFF))
    gen = torch.Generator(device=dev)
    gen.manual_seed((seed << 8) ^ 0x5EED)
    size = [w.scale / math.sqrt(m) if w.dist == "normal_fanin" else w.scale for _, m in layout]
    if op in ("sketch_step", "sketch_columns_step"):
        columns = op == "sketch_columns_step"
        buckets = [max(1, int(m * SKETCH_KEEP)) for _, m in layout] if columns else wl.sketch_rows(layout, SKETCH_KEEP)
        model = B.SketchModel(layout, buckets, rank, SKETCH_BETA, B.TABLE_F16, dtype, w.lib_seed, columns=columns)
        buf = model.alloc(dev)
        for (n, m), o, k, sz in zip(layout, model.offsets, buckets, size):
            cells = n * k if columns else k * m
            buf["table"][o["table_off"]:o["table_off"] + cells] = torch.randn(cells, device=dev, generator=gen).mul_(2 * sz).half()
    else:
        model = B.Model(layout, rank, case["bits"], case["block"], dtype, w.lib_seed)
        buf = {"P": torch.zeros(model.sizes["p_elems"], device=dev), "Q": torch.zeros(model.sizes["q_elems"], device=dev)}
        if op != "update":
            buf = model.alloc(dev)
            _error(model, layout, gen, size, buf["codes"], buf["scales"])
    state = {"op": op, "model": model, "buf": buf, "passes": 0}
    if op == "update":
        for (n, m), o, sz in zip(layout, model.offsets, size):
            buf["P"][o["p_off"]:o["p_off"] + n * rank] = torch.randn(n * rank, device=dev, generator=gen).mul_(n ** -0.5)
            buf["Q"][o["q_off"]:o["q_off"] + m * rank] = torch.randn(m * rank, device=dev, generator=gen).mul_(sz * math.sqrt(n))
        state["params"] = torch.randn(model.sizes["grad_elems"], device=dev, generator=gen).mul_(0.02)
        return state
    wl.device_fill_gradients(w, seed & 0xFFFF, buf["grads"], [o["grad_off"] for o in model.offsets])
    wl.device_q0(w, buf["Q"], [o["q_off"] for o in model.offsets])
    if op in ("iconef_step", "iconef_random_k_step"):
        s = (1 << (case["bits"] - 1)) - 1
        buf["codes2"], buf["scales2"] = torch.zeros_like(buf["codes"]), torch.zeros_like(buf["scales"])
        _error(model, layout, gen, [sz / s for sz in size], buf["codes2"], buf["scales2"])
    if op == "iconef_random_k_step":
        B.conef_rk_configure(model.ctx, [min(RK_GROUP, n * m) for n, m in layout])
        state["delta"] = torch.zeros(B.conef_rk_sizes(model.ctx)["delta_elems"], device=dev)
    if op == "sign_step":
        state["signs"] = torch.zeros(B.conef_ss_sizes(model.ctx)["sign_words"], dtype=torch.int32, device=dev)
        state["norms"] = torch.zeros(len(layout), device=dev)
    return state


# ------------------------------------------------------------------------------------------------ one pass
def run(state):
    op, model, buf, t = state["op"], state["model"], state["buf"], state["passes"]
    state["passes"] = t + 1
    st = B.Model.stream_handle()
    if op == "update":
        B.conef_apply_update(model.ctx, buf["P"], buf["Q"], state["params"], st)
        return {"params": state["params"]}
    clear = t % RESET_EVERY == RESET_EVERY - 1
    if op in ("sketch_step", "sketch_columns_step"):
        if clear:
            buf["table"].zero_()
        model.step(buf)
        return {"P": buf["P"], "Q": buf["Q"], "table": buf["table"]}
    if clear:
        B.conef_reset_error(model.ctx, buf["codes"], buf["scales"], st)
        if "codes2" in buf:
            B.conef_reset_error(model.ctx, buf["codes2"], buf["scales2"], st)
    if op == "step":
        model.step(buf, t)
        return {"P": buf["P"], "Q": buf["Q"], "codes": buf["codes"], "scales": buf["scales"]}
    if op == "iconef_step":
        B.conef_i_step(model.ctx, buf["grads"], buf["codes"], buf["scales"], buf["codes2"], buf["scales2"], buf["Q"], buf["P"],
                       buf["Q"], buf["ws"], t, st)
        return {k: buf[k] for k in ("P", "Q", "codes", "scales", "codes2", "scales2")}
    if op == "sign_step":
        B.conef_ss_step(model.ctx, buf["grads"], buf["codes"], buf["scales"], state["signs"], state["norms"], buf["ws"], t, st)
        return {"signs": state["signs"], "norms": state["norms"], "codes": buf["codes"], "scales": buf["scales"]}
    if op == "iconef_random_k_step":
        B.conef_i_rk_step(model.ctx, buf["grads"], buf["codes"], buf["scales"], buf["codes2"], buf["scales2"], state["delta"], t, st)
        return dict({k: buf[k] for k in ("codes", "scales", "codes2", "scales2")}, delta=state["delta"])
    raise ValueError(op)


def work(case):
    """Bytes: the gradient once, the error state read and written once, what is sent written once.  Operations: two per
    element and column of a factor for each of the three products of a rank-r step."""
    layout, op, r = layout_of(case), case["op"], case["rank"]
    n_el = sum(n * m for n, m in layout)
    factors = 4 * r * sum(n + m for n, m in layout)
    grad = n_el * (4 if case["dtype"] == "f32" else 2)
    error = n_el * (case["bits"] / 8 + 4 / case["block"])
    if op == "update":
        return {"bytes": 8 * n_el + factors, "flops": 2 * r * n_el}
    if op in ("sketch_step", "sketch_columns_step"):
        return {"bytes": grad + 2 * 2 * SKETCH_KEEP * n_el + 1.5 * factors, "flops": 6 * r * n_el}
    if op == "step":
        return {"bytes": grad + 2 * error + 1.5 * factors, "flops": 6 * r * n_el}
    if op == "iconef_step":
        return {"bytes": grad + 4 * error + 1.5 * factors, "flops": 6 * r * n_el}
    if op == "sign_step":
        return {"bytes": grad + 2 * error + n_el / 8, "flops": 4 * n_el}
    return {"bytes": grad + 4 * error + 4 * n_el / RK_GROUP, "flops": 4 * n_el}


def tolerance(case):
    op = case["op"]
    if op == "iconef_random_k_step":
        return "exact"                  # element-wise fp32 arithmetic in a stated order
    if op == "update":
        return {"rel": 1e-6}            # one fp32 chain per entry
    if op in ("sketch_step", "sketch_columns_step"):
        # fp16 table: a last-bit difference of a factor moves a few entries by one unit in the last place
        return {"rel": 1e-4, "max": 5e-3}
    # fp32 factors; a code whose value lies at a rounding boundary may fall to the other side (a few in ten million), and
    # in the next pass such an element may set the scale of its block
    return {"rel": 1e-5, "max": 0.3, "differ": 1e-4}
