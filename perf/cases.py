"""The work that a user of this framework has it do, as cases that can be timed and compared.

A case is one pass of what a 4-bit pretraining step calls: the training step of one linear layer (its six operands
quantized, then fwd_y, bwd_dx and bwd_dw) under one of the recipes, dense or over the experts of an MoE layer, with
fp32 per-16 scales or power-of-two per-32 scales; the quantization of one tensor by itself; the quality statistics
of one tensor. Tensors follow the distributions of the framework's own workloads: activations N(0, 1) with 0.1% of
the channels x50 (or Student-t with 3 degrees of freedom), weights N(0, 0.02^2), gradients N(0, 1e-3^2).

listed() / draw(rng): the cases. prepare / run: one pass through the public entry points. work / tolerance: what a
pass cannot do without, and how far another correct implementation may be off. exact: the same results in 64 bits
from plain torch.
"""

from __future__ import annotations

import math

import torch

from paper_2606_20381_amd import recipe as R
from paper_2606_20381_amd import ufp4 as U
from paper_2606_20381_amd import workloads as WL

MASK = 0x6A09  # the layer's RHT sign mask


def listed():
    return [
        # one small layer, the size of the quick-start and smoke test: launches and latency count
        {"name": "step-tiny", "kind": "step", "recipe": "ufp4", "M": 256, "N": 512, "K": 256},
        # a layer with no size a multiple of a tile (a short last micro-batch, an odd hidden size)
        {"name": "step-ragged", "kind": "step", "recipe": "ufp4", "M": 1040, "N": 2064, "K": 1552},
        # an attention projection of the 2048-wide model under the comparison recipe
        {"name": "step-attn-e2m1", "kind": "step", "recipe": "e2m1", "M": 4096, "N": 2048, "K": 2048},
        # the same projection under the wider-rotation recipe of the search space
        {"name": "step-attn-rht64", "kind": "step", "recipe": "ufp4-rht64", "M": 4096, "N": 2048, "K": 2048},
        # the FFN up-projection of the 1.5B dense model, 8192 tokens
        {"name": "step-dense", "kind": "step", "recipe": "ufp4", "M": 8192, "N": 8192, "K": 2048},
        # the largest layer that the benchmark runs
        {"name": "step-square", "kind": "step", "recipe": "ufp4", "M": 16384, "N": 16384, "K": 16384},
        # the expert layer of the 7.9B MoE model: 16384 tokens routed to 6 of 64 experts
        {"name": "moe-7.9b", "kind": "moe", "G": 64, "K": 2048, "N": 1408, "routed": 98304, "cap": 16384},
        # power-of-two scales: a small layer, the dense FFN, and one GPU's experts of the 124B MoE model
        {"name": "mx-small", "kind": "mx-step", "M": 1024, "N": 3072, "K": 1024},
        {"name": "mx-dense", "kind": "mx-step", "M": 8192, "N": 8192, "K": 2048},
        {"name": "mx-moe-124b", "kind": "mx-moe", "G": 8, "K": 5120, "N": 3072, "routed": 32768, "cap": 0},
        # a gradient tensor quantized for both of its GEMMs, by itself
        {"name": "quant-sr", "kind": "quant", "form": "pair", "grid": "uniform", "sr": True, "rows": 16384,
         "cols": 16384},
        # the rotation's gain on an activation tensor (a monitoring call, which reads the numbers back)
        {"name": "stats", "kind": "stats", "grid": "uniform", "rows": 8192, "cols": 2048, "transpose": False},
    ]


def _size(rng, lo, hi, mult):
    """A multiple of `mult`, spread over the logarithm of the range."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(mult, int(round(v / mult)) * mult)


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["mx-step"] * 3 + ["moe", "mx-moe", "quant", "quant", "stats"])
    if kind in ("step", "mx-step"):
        c = {"kind": kind}
        if kind == "step":
            c["recipe"] = rng.choice(["ufp4", "ufp4", "ufp4", "e2m1", "e2m1-full-rht", "ufp4-no-sr", "ufp4-rht64"])
        mult = 64 if c.get("recipe") == "ufp4-rht64" else (32 if kind == "mx-step" else 16)
        while True:
            c.update(M=_size(rng, 128, 16384, mult), N=_size(rng, 256, 16384, mult), K=_size(rng, 256, 16384, mult))
            if c["M"] * c["N"] * c["K"] <= 1 << 38:
                return c
    if kind in ("moe", "mx-moe"):
        mult = 128 if kind == "mx-moe" else 16
        while True:
            c = {"kind": kind, "G": rng.choice([4, 8, 16, 32, 64]), "K": _size(rng, 1024, 6144, mult),
                 "N": _size(rng, 768, 4096, mult), "routed": _size(rng, 2048, 98304, 1), "cap": 0}
            if c["routed"] * c["K"] * c["N"] <= 1 << 39 and c["G"] * c["K"] * c["N"] <= 1 << 29:
                return c
    if kind == "quant":
        form = rng.choice(["rows", "cols", "dual", "pair"])
        sr = form == "pair" or (form != "dual" and rng.random() < 0.4)
        return {"kind": kind, "form": form, "grid": rng.choice(["uniform", "uniform", "e2m1"]), "sr": sr,
                "rows": _size(rng, 256, 32768, 16), "cols": _size(rng, 256, 16384, 16)}
    return {"kind": kind, "grid": rng.choice(["uniform", "e2m1"]), "rows": _size(rng, 512, 32768, 16),
            "cols": _size(rng, 512, 8192, 16), "transpose": rng.random() < 0.5}


# ---------------------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------------------


def _acts(g, rows, cols, student=False):
    x = torch.randn(rows, cols, generator=g, device="cuda")
    if student:
        chi2 = torch.zeros_like(x)
        for _ in range(3):
            chi2 += torch.randn(rows, cols, generator=g, device="cuda").square_()
        return (x / torch.sqrt(chi2 / 3.0) / math.sqrt(3.0)).bfloat16()
    ch = torch.randperm(cols, generator=g, device="cuda")[: max(1, round(0.001 * cols))]
    x[:, ch] *= 50.0
    return x.bfloat16()


def _inputs(case, seed):
    """The bf16 tensors of a case on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed * 7919 + 17)
    t = {}
    if case["kind"] in ("quant", "stats"):
        t["x"] = _acts(g, case["rows"], case["cols"])
        if case.get("sr"):
            t["x"] = (t["x"].float() * 1e-3).bfloat16()
        return t
    moe = case["kind"] in ("moe", "mx-moe")
    M = case["routed"] if moe else case["M"]
    wrows = case["G"] * case["N"] if moe else case["N"]
    t["x"] = _acts(g, M, case["K"], student=case["kind"] == "mx-moe")
    t["w"] = (torch.randn(wrows, case["K"], generator=g, device="cuda") * 0.02).bfloat16()
    t["dy"] = (torch.randn(M, case["N"], generator=g, device="cuda") * 1e-3).bfloat16()
    return t


def _counts(case):
    return WL.zipf_counts(case["routed"], case["G"], 1.1, case["cap"] or None)


def _grid(case):
    return U.UNIFORM if case["grid"] == "uniform" else U.E2M1


def prepare(case, seed):
    s = {"case": case, "seed": seed, **_inputs(case, seed)}
    kind = case["kind"]
    if kind == "step":
        s["layer"] = R.LayerStep(case["M"], case["N"], case["K"], case["recipe"])
    elif kind == "mx-step":
        M, N, K = case["M"], case["N"], case["K"]
        shapes = {"x": (M, K), "w": (N, K), "dy": (M, N), "wt": (K, N), "dyt": (N, M), "xt": (K, M)}
        s["q"] = {k: U.empty_qtensor_mx(*v) for k, v in shapes.items()}
    elif kind in ("moe", "mx-moe"):
        G, N, K, M = case["G"], case["N"], case["K"], case["routed"]
        mx = kind == "mx-moe"
        counts = _counts(case)
        s["off"], s["red"] = U.group_offsets(counts, block=32 if mx else 16)
        mr = M
        if mx:
            _, s["prow"] = U.group_offsets(counts, block=128)
            mr = s["prow"]
        shapes = {"x": (mr, K), "w": (G * N, K), "dy": (mr, N), "wt": (K, G * N), "dyt": (N, s["red"]),
                  "xt": (K, s["red"])}
        s["q"] = {k: U.empty_qtensor(*v, U.UNIFORM_MX32 if mx else U.UNIFORM) for k, v in shapes.items()}
    elif kind == "quant":
        rows, cols, f = case["rows"], case["cols"], _grid(case)
        if case["form"] != "cols":
            s["qr"] = U.empty_qtensor(rows, cols, f)
        if case["form"] != "rows":
            s["qc"] = U.empty_qtensor(cols, rows, f)
    else:
        s["rec"] = torch.empty(U.STATS_BYTES // 8, dtype=torch.float64, device="cuda")
    if kind not in ("step", "quant", "stats"):
        M = case["routed"] if "routed" in case else case["M"]
        s["y"] = torch.empty(M, case["N"], dtype=torch.bfloat16, device="cuda")
        s["dx"] = torch.empty(M, case["K"], dtype=torch.bfloat16, device="cuda")
        dw = (case["G"], case["N"], case["K"]) if "G" in case else (case["N"], case["K"])
        s["dw"] = torch.empty(dw, dtype=torch.float32, device="cuda")
    return s


# ---------------------------------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------------------------------


def _run_mx_step(s):
    q, x, w, dy, seed = s["q"], s["x"], s["w"], s["dy"], s["seed"]
    U.mx_quantize_dual(x, sign_mask_rows=MASK, sign_mask_cols=MASK, out_rows=q["x"], out_cols=q["xt"])
    U.mx_quantize_dual(w, sign_mask_rows=MASK, sign_mask_cols=MASK, out_rows=q["w"], out_cols=q["wt"])
    U.mx_quantize(dy, sign_mask=MASK, rounding=U.SR, seed=seed, stream_id=0, out=q["dy"])
    U.mx_quantize(dy, transpose=True, sign_mask=MASK, rounding=U.SR, seed=seed, stream_id=1, out=q["dyt"])
    U.mx_gemm_fwd_y(q["x"], q["w"], out=s["y"])
    U.mx_gemm_bwd_dx(q["dy"], q["wt"], out=s["dx"])
    U.mx_gemm_bwd_dw(q["dyt"], q["xt"], out=s["dw"])
    return {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}


def _run_moe(s):
    q, x, w, dy, off, red, seed = s["q"], s["x"], s["w"], s["dy"], s["off"], s["red"], s["seed"]
    U.rht_quantize(x, sign_mask=MASK, out=q["x"])
    U.quantize_dual(w, sign_mask_rows=MASK, sign_mask_cols=MASK, out_rows=q["w"], out_cols=q["wt"])
    U.rht_quantize(dy, sign_mask=MASK, rounding=U.SR, seed=seed, stream_id=0, out=q["dy"])
    U.quantize_grouped_t(dy, off, red, sign_mask=MASK, rounding=U.SR, seed=seed, stream_id=1, out=q["dyt"])
    U.quantize_grouped_t(x, off, red, sign_mask=MASK, out=q["xt"])
    U.gemm_fwd_y_grouped(q["x"], q["w"], off, out=s["y"])
    U.gemm_bwd_dx_grouped(q["dy"], q["wt"], off, out=s["dx"])
    U.gemm_bwd_dw_grouped(q["dyt"], q["xt"], off, out=s["dw"])
    return {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}


def _run_mx_moe(s):
    q, x, w, dy, off, seed = s["q"], s["x"], s["w"], s["dy"], s["off"], s["seed"]
    M = x.shape[0]
    U.mx_quantize_grouped(x, off, s["prow"], transpose=False, sign_mask=MASK, out=q["x"])
    U.mx_quantize_dual(w, sign_mask_rows=MASK, sign_mask_cols=MASK, out_rows=q["w"], out_cols=q["wt"])
    U.mx_quantize_grouped(dy, off, s["prow"], transpose=False, sign_mask=MASK, rounding=U.SR, seed=seed, stream_id=0,
                          out=q["dy"])
    U.mx_quantize_grouped(dy, off, s["red"], transpose=True, sign_mask=MASK, rounding=U.SR, seed=seed, stream_id=1,
                          out=q["dyt"])
    U.mx_quantize_grouped(x, off, s["red"], transpose=True, sign_mask=MASK, out=q["xt"])
    U.mx_gemm_fwd_y_grouped(q["x"], q["w"], off, M, out=s["y"])
    U.mx_gemm_bwd_dx_grouped(q["dy"], q["wt"], off, M, out=s["dx"])
    U.mx_gemm_bwd_dw_grouped(q["dyt"], q["xt"], off, out=s["dw"])
    return {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}


def _run_quant(s):
    c, x = s["case"], s["x"]
    if c["form"] == "dual":
        U.quantize_dual(x, fmt=_grid(c), sign_mask_rows=MASK, sign_mask_cols=MASK, out_rows=s["qr"], out_cols=s["qc"])
    else:
        fn = U.rht_quantize if c["grid"] == "uniform" else U.e2m1_quantize
        kw = {"rht": True, "sign_mask": MASK, "rounding": U.SR if c["sr"] else U.RTNE, "seed": s["seed"]}
        if "qr" in s:
            fn(x, stream_id=0, out=s["qr"], **kw)
        if "qc" in s:
            fn(x, transpose=True, stream_id=1, out=s["qc"], **kw)
    return {k: {"codes": s[k].codes, "scales": s[k].scales} for k in ("qr", "qc") if k in s}


def _run_stats(s):
    c, out = s["case"], {}
    for name, rht in (("raw", False), ("rotated", True)):
        r = U.quant_stats(s["x"], _grid(c), transpose=c["transpose"], rht=rht, sign_mask=MASK, out=s["rec"])
        out[name] = {"err2": r.err2, "ref2": r.ref2, "cross": r.cross, "hist": r.hist, "beff": r.beff}
    return out


def run(state):
    kind = state["case"]["kind"]
    if kind == "step":
        y, dx, dw = state["layer"].run(state["x"], state["w"], state["dy"], MASK, state["seed"])
        return {"y": y, "dx": dx, "dw": dw}
    return {"mx-step": _run_mx_step, "moe": _run_moe, "mx-moe": _run_mx_moe, "quant": _run_quant,
            "stats": _run_stats}[kind](state)


# ---------------------------------------------------------------------------------------------------
# What a pass cannot do without, and how far results may be apart
# ---------------------------------------------------------------------------------------------------


def work(case):
    if case["kind"] == "stats":  # both statistics of the tensor from one read
        return {"bytes": 2.0 * case["rows"] * case["cols"], "flops": 0.0}
    if case["kind"] == "quant":  # bf16 in once; half a byte of code and a fp32 scale per 16 out, per operand
        outs = 2 if case["form"] in ("dual", "pair") else 1
        return {"bytes": (2.0 + 0.75 * outs) * case["rows"] * case["cols"], "flops": 0.0}
    moe = "G" in case
    M, N, K = case["routed"] if moe else case["M"], case["N"], case["K"]
    w = (case["G"] if moe else 1) * N * K
    # X, W and dY in bf16 in, Y and dX in bf16 and dW in fp32 out; three GEMMs
    return {"bytes": 2.0 * (M * K + w + M * N) + 2.0 * (M * N + M * K) + 4.0 * w, "flops": 3 * 2.0 * M * N * K}


def tolerance(case):
    if case["kind"] == "quant":
        return "exact"  # codes and scales are defined bit for bit
    if case["kind"] == "stats":
        return {"rel": 1e-6, "max": 1e-5}  # fp64 sums, handed over as fp32 numbers; the histogram is exact
    # Y and dX are bf16: measured 1.7e-3 against 64 bits (the rounding of the store), dW 1e-7
    return {"rel": 6e-3, "max": 2e-2}


# ---------------------------------------------------------------------------------------------------
# The same results in 64 bits, from plain torch
# ---------------------------------------------------------------------------------------------------

# recipe -> (grid, rotated (fwd_y, bwd_dx, bwd_dw), SR on dY, RHT block)
_RECIPES = {"ufp4": ("uniform", (1, 1, 1), True, 16), "e2m1": ("e2m1", (0, 0, 1), True, 16),
            "e2m1-full-rht": ("e2m1", (1, 1, 1), True, 16), "ufp4-no-sr": ("uniform", (1, 1, 1), False, 16),
            "ufp4-rht64": ("uniform", (1, 1, 1), True, 64)}


def _philox16(blk, row, seed, stream):
    """Sixteen 16-bit draws per (block, row): Philox4x32-10, counter (block, row, half, stream), key = seed."""
    m32 = 0xFFFFFFFF
    out = []
    for half in range(2):
        c0, c1 = blk & m32, row & m32
        c2, c3 = torch.full_like(c0, half), torch.full_like(c0, stream)
        k0, k1 = seed & m32, (seed >> 32) & m32
        for _ in range(10):
            p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # modulo 2^64: the low 64 bits are the unsigned product's
            c0, c1, c2, c3 = ((p1 >> 32) & m32) ^ c1 ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c3 ^ k1, p0 & m32
            k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
        for c in (c0, c1, c2, c3):
            out += [c & 0xFFFF, c >> 16]
    return torch.stack(out, dim=-1)


def _rotate(a, n):
    """x S_n H_n over the n-blocks of the last axis in fp64 (the 16 signs repeated in every 16-sub-block)."""
    sign = torch.tensor([-1.0 if MASK >> (j % 16) & 1 else 1.0 for j in range(n)], dtype=torch.float64,
                        device=a.device)
    v = a.double().view(-1, n) * sign
    h = 1
    while h < n:
        v = v.view(-1, n // (2 * h), 2, h)
        v = torch.stack((v[:, :, 0] + v[:, :, 1], v[:, :, 0] - v[:, :, 1]), dim=2).reshape(-1, n)
        h *= 2
    return (v * math.sqrt(1.0 / n)).view(a.shape)


def _levels(v, grid, u):
    """Values v (fp64) onto the grid: to nearest (ties to the even code), or with the 16-bit draws u."""
    top = 7.0 if grid == "uniform" else 6.0
    v = v.clamp(-top, top)
    if grid == "uniform":
        d = torch.ones((), dtype=torch.float64, device=v.device)
    else:
        a = v.abs()
        half, one = (a < 2, a < 4) if u is None else (torch.where(v >= 0, a < 2, a <= 2),
                                                      torch.where(v >= 0, a < 4, a <= 4))
        d = torch.where(half, 0.5, torch.where(one, 1.0, 2.0)).double()
    if u is None:
        return torch.round(v / d) * d
    lo = torch.floor(v / d) * d
    return lo + d * ((lo + d * (u.double() / 65536.0)) < v)


def _operand(a, grid, rht, sr, seed, stream, block=16, rows=None):
    """A [rows, red] -> (its dequantized values in fp64, its scales, its levels). `rows`: row numbers of the draws."""
    if rows is None:
        rows = torch.arange(a.shape[0], device=a.device)
    step = max(1, (1 << 25) // max(1, a.shape[1]))
    parts = []
    for i in range(0, a.shape[0], step):
        p, r = a[i: i + step], rows[i: i + step]
        n = p.shape[0]
        y = (_rotate(p, rht) if rht else p.double()).float().double()
        B = 32 if grid == "mx" else 16
        yb = y.view(n, -1, B)
        amax = yb.abs().amax(-1, keepdim=True)
        u = None
        if sr:
            nb = a.shape[1] // 16
            u = _philox16(torch.arange(nb, device=a.device).expand(n, nb), r.view(n, 1).expand(n, nb), seed, stream)
            u = u.reshape(yb.shape)
        if grid == "mx":
            s = torch.where(amax > 0, torch.exp2(torch.frexp(amax)[1].double() - 3.0), 0.0)
            lev = _levels(torch.where(amax > 0, yb / torch.where(amax > 0, s, 1.0), 0.0), "uniform", u)
        else:
            g = 7.0 if grid == "uniform" else 6.0
            s = (amax / g).float().double()
            inv = torch.where(amax > 0, g / torch.where(amax > 0, amax, 1.0), 0.0).float().double()
            lev = _levels((yb * inv).float().double(), grid, u)
        parts.append(((lev * s).view(n, -1), s.view(n, -1), lev.view(n, -1)))
    return tuple(torch.cat(v) for v in zip(*parts)) if len(parts) > 1 else parts[0]


def _panels(s, rows):
    """Row-major scales [rows, nb] in the panel order of an operand's scale buffer."""
    p = (rows + 127) // 128
    t = torch.zeros(p * 128, s.shape[1], dtype=s.dtype, device=s.device)
    t[:rows] = s
    return t.view(p, 128, -1).transpose(1, 2).reshape(p, -1)


def _padded(t, counts, block):
    """Token rows of t with each group zero-padded to `block`, and the groups' padded ranges."""
    parts, ranges, at, pos = [], [], 0, 0
    for c in counts:
        pad = -(-c // block) * block
        z = torch.zeros(pad, t.shape[1], dtype=t.dtype, device=t.device)
        z[:c] = t[at: at + c]
        parts.append(z)
        ranges.append((pos, pos + pad))
        at, pos = at + c, pos + pad
    return torch.cat(parts), ranges


def _exact_quant(case, t, seed):
    out = {}
    for k, tr, stream in (("qr", False, 0), ("qc", True, 1)):
        if case["form"] == ("cols" if k == "qr" else "rows"):
            continue
        a = t["x"].t().contiguous() if tr else t["x"]
        s = _operand(a.float(), case["grid"], 16, case["sr"], seed, stream)[1]
        out[k] = {"codes": None, "scales": _panels(s, a.shape[0])}
    return out


def _exact_stats(case, t):
    a = (t["x"].t().contiguous() if case["transpose"] else t["x"]).float()
    out = {}
    for name, rht in (("raw", 0), ("rotated", 16)):
        q, _, lev = _operand(a, case["grid"], rht, False, 0, 0)
        ref = (_rotate(a, 16) if rht else a.double()).float().double()
        mags = [float(i) for i in range(8)] if case["grid"] == "uniform" else [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]
        hist = [int((lev.abs() == m).sum()) for m in mags]
        p = [h / lev.numel() for h in hist]
        beff = math.exp(-sum(v * math.log(v + 1e-12) for v in p)) / 8
        out[name] = {"err2": float((q - ref).square().sum()), "ref2": float(ref.square().sum()),
                     "cross": float((q * ref).sum()), "hist": hist, "beff": beff}
    return out


def exact(case, seed):
    t, kind = _inputs(case, seed), case["kind"]
    if kind == "quant":
        return _exact_quant(case, t, seed)
    if kind == "stats":
        return _exact_stats(case, t)
    mx = kind.startswith("mx")
    grid, rot, sr, n = ("mx", (1, 1, 1), True, 16) if mx else _RECIPES[case.get("recipe", "ufp4")]

    def op(a, i, noisy=False, stream=0):
        return _operand(a.float(), grid, n if rot[i] else 0, noisy and sr, seed, stream)[0]

    x, w, dy = t["x"], t["w"], t["dy"]
    if "G" not in case:
        y = op(x, 0) @ op(w, 0).t()
        dx = op(dy, 1, True, 0) @ op(w.t().contiguous(), 1).t()
        dw = op(dy.t().contiguous(), 2, True, 1) @ op(x.t().contiguous(), 2).t()
        return {"y": y, "dx": dx, "dw": dw}
    G, N, K, counts = case["G"], case["N"], case["K"], _counts(case)
    block = 32 if mx else 16
    qx, qw, qdy = op(x, 0), op(w, 0), op(dy, 1, True, 0)
    qwt = op(w.t().contiguous(), 1)
    px, ranges = _padded(x, counts, block)
    pdy, _ = _padded(dy, counts, block)
    qxt, qdyt = op(px.t().contiguous(), 2), op(pdy.t().contiguous(), 2, True, 1)
    y, dx = [], []
    dw = torch.zeros(G, N, K, dtype=torch.float64, device=x.device)
    at = 0
    for g, c in enumerate(counts):
        y.append(qx[at: at + c] @ qw[g * N: (g + 1) * N].t())
        dx.append(qdy[at: at + c] @ qwt[:, g * N: (g + 1) * N].t())
        a, b = ranges[g]
        dw[g] = qdyt[:, a:b] @ qxt[:, a:b].t()
        at += c
    return {"y": torch.cat(y), "dx": torch.cat(dx), "dw": dw}
