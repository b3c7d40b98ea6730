"""The work this library is timed on: what a program that uses it has it do, through
the package's public entry points, over the range of sizes those entry points take.

listed() holds the fixed cases, draw() further ones of the same ranges; prepare() makes
what the program has in hand before the call, run() is one pass of it, work() the bytes
and operations the pass cannot do without and exact() its results in 64 bits from plain
torch.
"""
import math

import numpy as np
import torch

import paper_2201_03611_amd as rise

DEV = "cuda"


def listed():
    return [
        # the smallest product: one call whose cost is the launch and the few workgroups
        # that share it (the library's own smallest configuration)
        {"name": "gemm_f32_128", "kind": "gemm", "mode": "f32", "stored": "f32", "M": 128, "N": 128,
         "K": 128, "ta": False, "tb": False},
        # a product of odd sizes whose rows are not 16-byte aligned, as data sets have them
        {"name": "gemm_f32_ragged", "kind": "gemm", "mode": "f32", "stored": "f32", "M": 1000,
         "N": 1531, "K": 777, "ta": False, "tb": False},
        # a training step of the FP32 product: forward, then both gradients
        {"name": "gemm_f32_step_4096", "kind": "gemm_step", "mode": "f32", "M": 4096, "N": 4096,
         "K": 4096},
        # a dense layer on bfloat16 activations and weights, the weights stored outputs x inputs
        {"name": "gemm_bf16_stored", "kind": "gemm", "mode": "bf16", "stored": "bf16", "M": 2048,
         "N": 4096, "K": 4096, "ta": False, "tb": True},
        # the compensated product at the accuracy of FP32 on badly scaled rows and columns
        {"name": "gemm_bf16x3_8192", "kind": "gemm", "mode": "bf16x3", "stored": "f32", "M": 8192,
         "N": 8192, "K": 8192, "ta": False, "tb": False},
        # one Gaussian blur of a large image
        {"name": "stencil_4096_5x5", "kind": "stencil", "H": 4096, "W": 4096, "k": 5, "pad": "clamp"},
        # a training step of a learned 7 x 7 window on an image of odd size: forward, then
        # the gradients of image and window
        {"name": "stencil_step_ragged_7x7", "kind": "stencil_step", "H": 1531, "W": 2047, "k": 7,
         "pad": "clamp"},
        # sixteen Jacobi-style steps of the blur
        {"name": "stencil_iterate_4096_5x5", "kind": "stencil_iterate", "H": 4096, "W": 4096, "k": 5,
         "pad": "clamp", "steps": 16},
        # a training step of the 64 -> 64 channel 3 x 3 layer: forward, dIn and dW
        {"name": "conv_step_32x512x512x64", "kind": "conv_step", "B": 32, "H": 512, "W": 512,
         "Cin": 64, "Cout": 64},
        # a matrix applied to a vector, then its transpose to the result (a step of a power
        # iteration or of least squares): both storage directions of the product
        {"name": "gemv_pair_4096", "kind": "gemv_pair", "M": 4096, "K": 4096},
        # the tree reduction of a long vector to one sum
        {"name": "iterate_sum_2pow26", "kind": "iterate_sum", "n": 2, "m": 1, "k": 26},
        # many products and blurs of uneven sizes in one launch of a plan
        {"name": "plan_512_256", "kind": "plan", "gemms": 512, "stencils": 256, "sizes": 1005,
         "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """Log-uniform; half of the sizes as they fall (odd ones among them), a quarter whole
    multiples of 16, a quarter of 64."""
    v = _log(rng, lo, hi)
    step = rng.choice([1, 1, 16, 64])
    return max(1, (v + step - 1) // step * step) if step > 1 else v


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "gemm_step", "stencil", "stencil_step",
                       "stencil_iterate", "conv_step", "gemv_pair", "iterate_sum", "plan"])
    if kind in ("gemm", "gemm_step"):
        mode = rng.choice(["f32", "f32", "f32", "bf16", "bf16x3", "bf16x6", "fp8"])
        # the most multiply-adds a call of this mode may cost
        most = {"f32": 4096 ** 3, "bf16": 8192 ** 3, "bf16x3": 8192 ** 3, "bf16x6": 6144 ** 3,
                "fp8": 8192 ** 3}[mode]
        if kind == "gemm_step":
            mode = mode if mode in ("f32", "bf16x3") else "f32"
            most = {"f32": 4096 ** 3, "bf16x3": 5120 ** 3}[mode]
        while True:
            M, N, K = (_size(rng, 64, 8192) for _ in range(3))
            if M * N * K <= most:
                break
        if kind == "gemm_step":
            return {"kind": kind, "mode": mode, "M": M, "N": N, "K": K}
        stored = rng.choice(["f32", "bf16"]) if mode == "bf16" else "f32"
        return {"kind": kind, "mode": mode, "stored": stored, "M": M, "N": N, "K": K,
                "ta": rng.random() < 0.25, "tb": rng.random() < 0.5}
    if kind in ("stencil", "stencil_step"):
        return {"kind": kind, "H": _size(rng, 64, 4096), "W": _size(rng, 64, 4096),
                "k": rng.choice([3, 5, 7]), "pad": rng.choice(["clamp", "zero"])}
    if kind == "stencil_iterate":
        return {"kind": kind, "H": _size(rng, 64, 4096), "W": _size(rng, 64, 4096),
                "k": rng.choice([3, 5, 7]), "pad": rng.choice(["clamp", "zero"]),
                "steps": _log(rng, 2, 16)}
    if kind == "conv_step":
        return {"kind": kind, "B": _log(rng, 1, 32), "H": _size(rng, 16, 512),
                "W": _size(rng, 16, 512), "Cin": rng.choice([32, 64]), "Cout": rng.choice([32, 64])}
    if kind == "gemv_pair":
        return {"kind": kind, "M": _size(rng, 64, 16384), "K": _size(rng, 64, 16384)}
    if kind == "iterate_sum":
        n = rng.choice([2, 2, 3, 4, 5, 8, 16])
        total = _log(rng, 1 << 12, 1 << 26)
        k = rng.randint(1, max(1, int(math.log(total) / math.log(n) + 1e-9)))
        return {"kind": kind, "n": n, "m": max(1, total // n ** k), "k": k}
    return {"kind": "plan", "gemms": _log(rng, 16, 512), "stencils": _log(rng, 8, 256),
            "sizes": rng.randrange(1 << 20), "dtype": rng.choice(["f32", "bf16"])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _uniform(g, *shape, lo=-1.0, hi=1.0):
    return torch.rand(shape, device=DEV, generator=g) * (hi - lo) + lo


def _scaled_normal(g, rows, cols, spread):
    """N(0,1) entries, row i scaled by 2^u_i with u_i ~ U(-spread, spread)."""
    x = torch.randn((rows, cols), device=DEV, generator=g)
    return x.mul_(torch.exp2(_uniform(g, rows, 1, lo=-spread, hi=spread)))


def _window(g, k):
    """A k x k window of positive weights that sum to 1."""
    w = _uniform(g, k, k, lo=0.05, hi=1.0)
    return w / w.sum()


def _plan_sizes(case):
    """(M, N, K) of every product, multiples of 32 in 64..1024, and (side, window) of every
    stencil, sides 256..2048."""
    g = np.random.default_rng(case["sizes"])
    gemms = g.choice(np.arange(64, 1025, 32), size=(case["gemms"], 3)).tolist()
    g = np.random.default_rng(case["sizes"] + 100)
    sides = g.integers(256, 2049, size=case["stencils"])
    ks = g.choice(np.array([3, 5, 7]), size=case["stencils"])
    return gemms, [(int(s), int(k)) for s, k in zip(sides, ks)]


def _slices(buf, counts, unit):
    """Consecutive 1-D pieces of buf holding counts[i] values, each starting at a multiple
    of unit values; the length used."""
    out, at = [], 0
    for n in counts:
        out.append(buf[at:at + n] if buf is not None else None)
        at += (n + unit - 1) // unit * unit
    return out, at


def _inputs(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind in ("gemm", "gemm_step"):
        M, N, K = case["M"], case["N"], case["K"]
        if case["mode"] == "f32":
            A, B = _uniform(g, M, K), _uniform(g, K, N)
        else:
            spread = 4.0 if case.get("stored", "f32") == "f32" else 1.0
            A, Bt = _scaled_normal(g, M, K, spread), _scaled_normal(g, N, K, spread)
            B = Bt.t().contiguous()
        if kind == "gemm_step":
            return {"A": A, "B": B, "dC": _uniform(g, M, N)}
        if case["stored"] == "bf16":
            A, B = A.to(torch.bfloat16), B.to(torch.bfloat16)
        return {"A": A.t().contiguous() if case["ta"] else A,
                "B": B.t().contiguous() if case["tb"] else B}
    if kind in ("stencil", "stencil_step", "stencil_iterate"):
        H, W = case["H"], case["W"]
        d = {"img": _uniform(g, H, W, lo=0.0), "w": _window(g, case["k"])}
        if kind == "stencil_step":
            d["dout"] = _uniform(g, H, W)
        return d
    if kind == "conv_step":
        B, H, W, ci, co = (case[n] for n in ("B", "H", "W", "Cin", "Cout"))
        # each image drawn by itself: no FP32 copy of the whole batch
        x = torch.empty((B, H, W, ci), device=DEV, dtype=torch.bfloat16)
        d = torch.empty((B, H, W, co), device=DEV, dtype=torch.bfloat16)
        for b in range(B):
            x[b] = torch.randn((H, W, ci), device=DEV, generator=g)
            d[b] = torch.randn((H, W, co), device=DEV, generator=g)
        return {"x": x, "w": torch.randn((co, ci, 3, 3), device=DEV, generator=g) * 0.02, "dout": d}
    if kind == "gemv_pair":
        return {"A": _uniform(g, case["M"], case["K"]), "x": _uniform(g, case["K"])}
    if kind == "iterate_sum":
        return {"x": _uniform(g, case["n"] ** case["k"] * case["m"])}
    # plan: every operand a piece of one buffer per role
    gemms, stencils = _plan_sizes(case)
    bf16 = case["dtype"] == "bf16"
    cnt = [[M * K for M, N, K in gemms], [K * N for M, N, K in gemms], [M * N for M, N, K in gemms],
           [s * s for s, k in stencils], [k * k for s, k in stencils], [s * s for s, k in stencils]]
    unit = 64
    size = [max(1, _slices(None, c, unit)[1]) for c in cnt]
    A, B = _uniform(g, size[0]), _uniform(g, size[1])
    if bf16:
        A, B = A.to(torch.bfloat16), B.to(torch.bfloat16)
    img = _uniform(g, size[3], lo=0.0)
    w = _uniform(g, size[4], lo=0.05, hi=1.0)
    for piece in _slices(w, cnt[4], unit)[0]:
        piece.div_(piece.sum())
    return {"A": A, "B": B, "C": torch.zeros(size[2], device=DEV), "img": img, "w": w,
            "out": torch.zeros(size[5], device=DEV), "cnt": cnt, "unit": unit}


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    for name in {"gemm_step": ("A", "B"), "stencil_step": ("img", "w"),
                 "conv_step": ("x", "w")}.get(case["kind"], ()):
        s[name].requires_grad_(True)
    if case["kind"] == "plan":
        gemms, stencils = _plan_sizes(case)
        piece = [_slices(s[n], c, s["unit"])[0]
                 for n, c in zip(("A", "B", "C", "img", "w", "out"), s["cnt"])]
        gp = (rise.RiseGemmProblem * max(1, len(gemms)))()
        dt = rise.RISE_BF16 if case["dtype"] == "bf16" else rise.RISE_F32
        for i, (M, N, K) in enumerate(gemms):
            gp[i] = rise.RiseGemmProblem(piece[2][i].data_ptr(), piece[0][i].data_ptr(),
                                         piece[1][i].data_ptr(), M, N, K, K, N, N, dt, 0)
        sp = (rise.RiseStencilProblem * max(1, len(stencils)))()
        for i, (side, k) in enumerate(stencils):
            sp[i] = rise.RiseStencilProblem(piece[5][i].data_ptr(), piece[3][i].data_ptr(),
                                            piece[4][i].data_ptr(), side, side, side, side, k, 0)
        torch.cuda.synchronize()
        s["plan"] = rise.Plan(gp, len(gemms), sp, len(stencils))
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "gemm":
        return rise.gemm(s["A"], s["B"], transA=case["ta"], transB=case["tb"], mode=case["mode"])
    if kind == "gemm_step":
        C = rise.RiseGemmFn.apply(s["A"], s["B"], case["mode"])
        dA, dB = torch.autograd.grad(C, (s["A"], s["B"]), s["dC"])
        return {"C": C, "dA": dA, "dB": dB}
    if kind == "stencil":
        return rise.stencil2d(s["img"], s["w"], pad=case["pad"])
    if kind == "stencil_step":
        out = rise.RiseStencil2dFn.apply(s["img"], s["w"], case["pad"])
        dimg, dw = torch.autograd.grad(out, (s["img"], s["w"]), s["dout"])
        return {"out": out, "dimg": dimg, "dw": dw}
    if kind == "stencil_iterate":
        return rise.stencil2d_iterate(s["img"], s["w"], case["steps"], pad=case["pad"])
    if kind == "conv_step":
        out = rise.RiseConv2dFn.apply(s["x"], s["w"])
        dx, dw = torch.autograd.grad(out, (s["x"], s["w"]), s["dout"])
        return {"out": out, "dx": dx, "dw": dw}
    if kind == "gemv_pair":
        y = rise.gemv(s["A"], s["x"])
        return {"y": y, "z": rise.gemv(s["A"], y, transA=True)}
    if kind == "iterate_sum":
        return rise.iterate_sum(s["x"], case["n"], case["k"])
    s["plan"].launch()
    return {"C": s["C"], "out": s["out"]}


def work(case):
    kind = case["kind"]
    if kind in ("gemm", "gemm_step"):
        M, N, K = case["M"], case["N"], case["K"]
        e = 2 if case.get("stored") == "bf16" else 4
        if kind == "gemm":
            return {"bytes": e * (M * K + K * N) + 4 * M * N, "flops": 2 * M * N * K}
        # A, B, dC in; C, dA, dB out
        return {"bytes": 8 * (M * K + K * N + M * N), "flops": 6 * M * N * K}
    if kind in ("stencil", "stencil_step", "stencil_iterate"):
        px, kk = case["H"] * case["W"], case["k"] ** 2
        if kind == "stencil":
            return {"bytes": 8 * px, "flops": 2 * kk * px}
        if kind == "stencil_step":  # img, dout in; out, dimg out
            return {"bytes": 16 * px, "flops": 6 * kk * px}
        return {"bytes": 8 * px, "flops": 2 * kk * px * case["steps"]}
    if kind == "conv_step":  # x, dout in; out, dx out
        px = case["B"] * case["H"] * case["W"]
        return {"bytes": 4 * px * (case["Cin"] + case["Cout"]),
                "flops": 3 * 18 * px * case["Cin"] * case["Cout"]}
    if kind == "gemv_pair":
        return {"bytes": 4 * case["M"] * case["K"], "flops": 4 * case["M"] * case["K"]}
    if kind == "iterate_sum":
        n = case["n"] ** case["k"] * case["m"]
        return {"bytes": 4 * n + 4 * case["m"], "flops": n}
    gemms, stencils = _plan_sizes(case)
    e = 2 if case["dtype"] == "bf16" else 4
    return {"bytes": sum(e * (M * K + K * N) + 4 * M * N for M, N, K in gemms)
            + sum(8 * s * s for s, k in stencils),
            "flops": sum(2 * M * N * K for M, N, K in gemms)
            + sum(2 * k * k * s * s for s, k in stencils)}


# ---------------------------------------------------------------------------
# the same results in 64 bits, from plain torch
# ---------------------------------------------------------------------------
def _stencil64(img, w, pad):
    k = w.shape[0]
    r = (k - 1) // 2
    H, W = img.shape
    p = torch.nn.functional.pad(img[None, None], (r, r, r, r),
                                mode="replicate" if pad == "clamp" else "constant")[0, 0]
    out = torch.zeros_like(img)
    for dy in range(k):
        for dx in range(k):
            out = out + p[dy:dy + H, dx:dx + W] * w[dy, dx]
    return out


def _conv64(x, w, dout):
    """out, dx, dw of the 3 x 3 layer with zero padding, an image at a time."""
    B, H, W, ci = x.shape
    co = w.shape[0]
    w = w.double()
    out = torch.empty((B, H, W, co), device=DEV, dtype=torch.float64)
    dx = torch.empty((B, H, W, ci), device=DEV, dtype=torch.float64)
    dw = torch.zeros((co, ci, 3, 3), device=DEV, dtype=torch.float64)
    for b in range(B):
        xp = torch.nn.functional.pad(x[b].double(), (0, 0, 1, 1, 1, 1))
        g = dout[b].double()
        gp = torch.nn.functional.pad(g, (0, 0, 1, 1, 1, 1))
        o, d = torch.zeros((H * W, co), device=DEV, dtype=torch.float64), torch.zeros(
            (H * W, ci), device=DEV, dtype=torch.float64)
        for ty in range(3):
            for tx in range(3):
                v = xp[ty:ty + H, tx:tx + W].reshape(H * W, ci)
                o += v @ w[:, :, ty, tx].t()
                dw[:, :, ty, tx] += g.reshape(H * W, co).t() @ v
                d += gp[2 - ty:2 - ty + H, 2 - tx:2 - tx + W].reshape(H * W, co) @ w[:, :, ty, tx]
        out[b], dx[b] = o.view(H, W, co), d.view(H, W, ci)
    return {"out": out, "dx": dx, "dw": dw}


def exact(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    if kind == "gemm":
        A, B = s["A"].double(), s["B"].double()
        return (A.t() if case["ta"] else A) @ (B.t() if case["tb"] else B)
    if kind == "gemm_step":
        A, B, dC = s["A"].double(), s["B"].double(), s["dC"].double()
        return {"C": A @ B, "dA": dC @ B.t(), "dB": A.t() @ dC}
    if kind == "stencil":
        return _stencil64(s["img"].double(), s["w"].double(), case["pad"])
    if kind == "stencil_step":
        img, w = (s[n].double().requires_grad_(True) for n in ("img", "w"))
        out = _stencil64(img, w, case["pad"])
        dimg, dw = torch.autograd.grad(out, (img, w), s["dout"].double())
        return {"out": out.detach(), "dimg": dimg, "dw": dw}
    if kind == "stencil_iterate":
        img, w = s["img"].double(), s["w"].double()
        for _ in range(case["steps"]):
            img = _stencil64(img, w, case["pad"])
        return img
    if kind == "conv_step":
        return _conv64(s["x"], s["w"], s["dout"])
    if kind == "gemv_pair":
        A = s["A"].double()
        y = A @ s["x"].double()
        return {"y": y, "z": A.t() @ y}
    if kind == "iterate_sum":
        return s["x"].double().view(case["m"], -1).sum(1)
    gemms, stencils = _plan_sizes(case)
    unit, cnt = s["unit"], s["cnt"]
    A, B, img, w = (_slices(s[n], c, unit)[0] for n, c in
                    (("A", cnt[0]), ("B", cnt[1]), ("img", cnt[3]), ("w", cnt[4])))
    C, out = s["C"].double(), s["out"].double()
    for (M, N, K), a, b, c in zip(gemms, A, B, _slices(C, cnt[2], unit)[0]):
        c.copy_((a.double().view(M, K) @ b.double().view(K, N)).view(-1))
    for (side, k), i, v, o in zip(stencils, img, w, _slices(out, cnt[5], unit)[0]):
        o.copy_(_stencil64(i.double().view(side, side), v.double().view(k, k), "clamp").view(-1))
    return {"C": C, "out": out}
