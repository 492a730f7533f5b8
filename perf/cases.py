"""Timed cases of the library: what its users call, over the sizes they call it with.

Convolution layers of ResNet-50-like networks (the layer set that bench.py times, plus ragged ones of
the kind the tests use), matrix products of the square sizes and of the sizes of the paper's
GEMM table.  Inputs follow synth.workloads: N(0,1) activations, N(0, 2/(C R S)) filters, bias
U[-0.1, 0.1), matrices U[-1, 1).
"""
import math

import torch

import paper_2006_02230_amd as P


def _conv(name, N, C, H, W, K, R, S, stride, pad, form="fp32", bias=True, act="relu"):
    c = {"kind": "conv", "form": form, "N": N, "C": C, "H": H, "W": W, "K": K, "R": R, "S": S, "stride": stride,
         "pad": pad, "bias": bias, "act": act}
    if name:
        c["name"] = name
    return c


def _gemm(name, M, N, K, accumulate=False):
    c = {"kind": "sgemm", "M": M, "N": N, "K": K, "accumulate": accumulate}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one image through one mid-size layer: the latency of a single small call
        _conv("conv_one_image", 1, 64, 56, 56, 64, 3, 3, 1, 1, bias=False, act="none"),
        # the first layer of the network: three channels, large strided filter
        _conv("conv_stem", 32, 3, 224, 224, 64, 7, 7, 2, 3),
        # the work horse, called as the benchmark calls it: with the filter's [K][R][S][C] copy
        _conv("conv_3x3_copy", 32, 128, 28, 28, 128, 3, 3, 1, 1, form="tap"),
        # the last stage: few pixels, long reduction, KCRS filter only
        _conv("conv_3x3_deep", 32, 512, 7, 7, 512, 3, 3, 1, 1),
        # bottleneck expansion: short reduction, large output, bound by memory
        _conv("conv_1x1_expand", 32, 64, 56, 56, 256, 1, 1, 1, 0),
        # strided projection shortcut
        _conv("conv_1x1_stride2", 32, 1024, 14, 14, 2048, 1, 1, 2, 0),
        # nothing a multiple of a tile: odd channels, pixels and batch
        _conv("conv_ragged", 7, 83, 35, 29, 201, 3, 3, 1, 1, act="relu6"),
        # bfloat16 layer between layers that keep the blocked layout
        _conv("conv_bf16_blocked", 64, 256, 14, 14, 256, 3, 3, 1, 1, form="bf16_blocked"),
        # bfloat16 layer on plain NCHW / KCRS tensors: layout passes and convolution
        _conv("conv_bf16_plain", 64, 64, 56, 56, 256, 1, 1, 1, 0, form="bf16"),
        # the large square product
        _gemm("sgemm_4096", 4096, 4096, 4096),
        # a size of the paper's GEMM table: few rows, long reduction
        _gemm("sgemm_128x2048x4096", 128, 2048, 4096),
        # odd everywhere, accumulated onto a matrix the caller has
        _gemm("sgemm_ragged", 1001, 777, 1531, accumulate=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A call of the same ranges: any layer of a CNN, or a product up to the largest listed one."""
    while True:
        if rng.random() < 0.7:
            R = rng.choice([1, 1, 3, 3, 3, 5, 7])
            stride = rng.choice([1, 1, 1, 2])
            C = rng.choice([3, 64, 128, 256, 512, _log_int(rng, 4, 1024), _log_int(rng, 4, 1024)])
            K = rng.choice([64, 128, 256, 512, _log_int(rng, 16, 2048), _log_int(rng, 16, 2048)])
            H = rng.choice([7, 14, 28, 56, _log_int(rng, 7, 128)])
            W = H if rng.random() < 0.6 else _log_int(rng, 7, 128)
            N = rng.choice([1, 32, 64, _log_int(rng, 1, 64)])
            form = rng.choice(["fp32", "fp32", "tap", "bf16_blocked", "bf16"])
            if form == "tap" and R == 1:
                form = "fp32"
            case = _conv(None, N, C, H, W, K, R, R, stride, R // 2, form=form, bias=rng.random() < 0.8,
                         act=rng.choice(["none", "relu", "relu", "relu6"]))
        else:
            case = _gemm(None, _log_int(rng, 64, 4096), _log_int(rng, 64, 4096), _log_int(rng, 32, 8192),
                         accumulate=rng.random() < 0.3)
        w = work(case)
        if w["flops"] <= 4e10 and w["bytes"] <= 6e8 and w["flops"] >= 2e7:
            return case


def _out_hw(c):
    return (c["H"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["S"]) // c["stride"] + 1


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape, sigma=1.0):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32) * sigma

    def uniform(*shape):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float32) * 2 - 1

    if case["kind"] == "sgemm":
        M, N, K = case["M"], case["N"], case["K"]
        return uniform(M, K), uniform(K, N), (uniform(M, N) if case["accumulate"] else None)
    x = normal(case["N"], case["C"], case["H"], case["W"])
    w = normal(case["K"], case["C"], case["R"], case["S"], sigma=math.sqrt(2.0 / (case["C"] * case["R"] * case["S"])))
    b = uniform(case["K"]) * 0.1 if case["bias"] else None
    if case["form"].startswith("bf16"):
        x, w = x.to(torch.bfloat16), w.to(torch.bfloat16)
    return x, w, b


def prepare(case, seed):
    if case["kind"] == "sgemm":
        A, B, C0 = _inputs(case, seed)
        return {"case": case, "A": A, "B": B, "C0": C0,
                "C": None if case["accumulate"] else torch.zeros(case["M"], case["N"], device="cuda")}
    x, w, b = _inputs(case, seed)
    Ph, Q = _out_hw(case)
    st = {"case": case, "x": x, "w": w, "b": b,
          "out": torch.empty(case["N"], case["K"], Ph, Q, device="cuda", dtype=torch.float32)}
    form = case["form"]
    if form == "tap":
        st["w_tap"] = P.filter_tap_copy(w)          # made once per filter
    elif form == "bf16_blocked":
        st["x8c"] = P.nchw_to_nchwc_bf16(x, 8)
        st["w8c"] = P.kcrs_to_kcrsck_bf16(w, 8, 1)
    elif form == "bf16":
        need = P.binding.lib.polydl_conv2d_bf16_workspace_bytes(*[case[k] for k in "NCHWKRS"])
        st["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    return st


def run(state):
    c = state["case"]
    if c["kind"] == "sgemm":
        if c["accumulate"]:
            return P.sgemm(state["A"], state["B"], state["C0"].clone())
        return P.sgemm(state["A"], state["B"], state["C"], alpha=1.0, beta=0.0)
    kw = dict(bias=state["b"], out=state["out"], stride=c["stride"], pad=c["pad"], act=c["act"])
    if c["form"] == "bf16_blocked":
        return P.conv2d_fwd_bf16_blocked(state["x8c"], state["w8c"], c["C"], **kw)
    if c["form"] == "bf16":
        return P.conv2d_fwd_bf16(state["x"], state["w"], workspace=state["ws"], **kw)
    return P.conv2d_fwd(state["x"], state["w"], w_tap=state.get("w_tap"), **kw)


def work(case):
    if case["kind"] == "sgemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 4 * (M * K + K * N + M * N * (2 if case["accumulate"] else 1)), "flops": 2 * M * N * K}
    Ph, Q = _out_hw(case)
    N, C, K, RS = case["N"], case["C"], case["K"], case["R"] * case["S"]
    el = 2 if case["form"].startswith("bf16") else 4
    return {"bytes": el * (N * C * case["H"] * case["W"] + K * C * RS) + 4 * N * K * Ph * Q + (4 * K if case["bias"] else 0),
            "flops": 2 * N * K * Ph * Q * C * RS}


def tolerance(case):
    # Sums of up to 8192 products in 32 bits (bfloat16 products are exact in 32 bits, sums are the same):
    # measured 0.1e-6 (64 terms) .. 1.2e-6 (4608 terms) against 64 bits, largest difference five times that
    return {"rel": 5e-6, "max": 5e-5}


def exact(case, seed):
    if case["kind"] == "sgemm":
        A, B, C0 = _inputs(case, seed)
        out = A.double() @ B.double()
        return out if C0 is None else out + C0.double()
    x, w, b = _inputs(case, seed)
    Ph, Q = _out_hw(case)
    p, s = case["pad"], case["stride"]
    xp = torch.nn.functional.pad(x.double(), (p, p, p, p))
    wd = w.double()
    out = torch.zeros(case["N"], case["K"], Ph * Q, dtype=torch.float64, device="cuda")
    for r in range(case["R"]):
        for t in range(case["S"]):
            tap = xp[:, :, r:r + (Ph - 1) * s + 1:s, t:t + (Q - 1) * s + 1:s].reshape(case["N"], case["C"], Ph * Q)
            f = wd[:, :, r, t].contiguous()
            for n in range(case["N"]):
                out[n] += f @ tap[n].contiguous()
    if b is not None:
        out += b.double().view(1, -1, 1)
    if case["act"] != "none":
        out.clamp_(min=0)
    if case["act"] == "relu6":
        out.clamp_(max=6)
    return out.view(case["N"], case["K"], Ph, Q)
