"""The calls this library is measured on, and their inputs.

Three kinds of work, each through the package's public calls, eagerly, as a
program that serves or prepares a quantized model makes them:

  quant   one online activation quantizer call on the activations of a layer:
          the Kronecker transform with K packed once per layer (``packed``),
          from the factor pair (``fly``), from its 15 LU parameters (``lu``),
          in the fixed fp32 order (``exact``), or a comparator (``smooth``,
          ``hadamard``, ``fwht``, ``plain``);
  linear  a W4A4 linear layer: quantize the activations, then the MXFP4 GEMM
          with the layer's prepared weight, as bf16 or fp32, or accumulated
          onto a 16-bit low-rank branch (``lora``);
  calib   one loss-and-gradient evaluation of the layer-wise calibration, the
          step that a calibration loop repeats a hundred times per layer.

Sizes are the layer shapes the benchmark and the tests use (diffusion
transformers: 256 to 18432 tokens, 1152 to 12288 features) and ranges around
them.  Inputs are drawn on the GPU from the seed: heavy-tailed values with a
few outlier channels, near-identity factors.
"""
import math

import numpy as np
import torch

import paper_2607_21446_amd as kq

LAMBDAS = (0.7, 1.3)
RANK = 32


def listed():
    return [
        # the smallest layer input: a class-token batch; launch latency is all of it
        {"name": "quant_packed_256x1152", "kind": "quant", "op": "packed", "M": 256, "d": 1152, "a": 4, "per_block": False},
        # the headline activation: one image's tokens at a 3072-wide attention projection
        {"name": "quant_packed_4608x3072", "kind": "quant", "op": "packed", "M": 4608, "d": 3072, "a": 4, "per_block": False},
        # the MLP's wide activation, K2 form, with the 16-bit output that a low-rank branch reads
        {"name": "quant_lu_y16_4608x12288", "kind": "quant", "op": "lu", "M": 4608, "d": 12288, "a": 4, "per_block": False, "y16": True},
        # a batch of four images with one factor pair per 32-column block
        {"name": "quant_fly_blocks_18432x12288", "kind": "quant", "op": "fly", "M": 18432, "d": 12288, "a": 4, "per_block": True},
        # the full-row Hadamard baseline at the size the comparison is quoted on
        {"name": "quant_fwht_4096x4096", "kind": "quant", "op": "fwht", "M": 4096, "d": 4096, "a": 4, "per_block": False},
        # a small layer on few tokens: two short launches
        {"name": "linear_256x1152x1152", "kind": "linear", "op": "packed", "M": 256, "d": 1152, "N": 1152, "a": 4, "per_block": False, "out": "bf16"},
        # a fused QKV projection on a ragged number of tokens, K built in the call
        {"name": "linear_1000x1152x3456", "kind": "linear", "op": "fly", "M": 1000, "d": 1152, "N": 3456, "a": 4, "per_block": False, "out": "bf16"},
        # attention projection of one image
        {"name": "linear_4608x3072x3072", "kind": "linear", "op": "packed", "M": 4608, "d": 3072, "N": 3072, "a": 4, "per_block": False, "out": "bf16"},
        # MLP down projection of one image: the longest contraction
        {"name": "linear_4608x12288x3072", "kind": "linear", "op": "packed", "M": 4608, "d": 12288, "N": 3072, "a": 4, "per_block": False, "out": "bf16"},
        # MLP up projection whose width is no multiple of 128, with a low-rank branch in 16 bits
        {"name": "linear_lora_4096x2240x5600", "kind": "linear", "op": "lu", "M": 4096, "d": 2240, "N": 5600, "a": 4, "per_block": True, "out": "lora"},
        # calibration of a small layer on a few samples
        {"name": "calib_2048x1152x1152", "kind": "calib", "M": 2048, "d": 1152, "N": 1152, "a": 4, "per_block": True},
        # calibration of a large layer on four images
        {"name": "calib_18432x3072x3072", "kind": "calib", "M": 18432, "d": 3072, "N": 3072, "a": 4, "per_block": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    return 32 * max(1, _log_int(rng, lo / 32, hi / 32))


def draw(rng):
    kind = rng.choice(["quant", "quant", "linear", "linear", "linear", "calib", "calib"])
    a = rng.choice([4, 4, 2, 8, 1])
    if kind == "quant":
        op = rng.choice(["packed", "packed", "fly", "lu", "exact", "smooth", "hadamard", "fwht", "plain"])
        d = _width(rng, 32, 12288)
        if op == "fwht":
            d = 1 << rng.randint(5, 14)
        c = {"kind": kind, "op": op, "M": _log_int(rng, 1, 18432), "d": d, "a": a, "per_block": False}
        if op in ("packed", "fly", "lu", "exact"):
            c["per_block"] = rng.random() < 0.4
        if op == "lu":
            c["y16"] = rng.random() < 0.5
        return c
    if kind == "linear":
        out = rng.choice(["bf16", "bf16", "fp32", "lora"])
        op = "lu" if out == "lora" else rng.choice(["packed", "fly", "lu"])
        return {"kind": kind, "op": op, "M": _log_int(rng, 16, 9216), "d": _width(rng, 256, 12288),
                "N": _log_int(rng, 64, 6144), "a": a, "per_block": rng.random() < 0.4, "out": out}
    return {"kind": kind, "M": _log_int(rng, 64, 18432), "d": _width(rng, 64, 3072), "N": _log_int(rng, 32, 3072),
            "a": a, "per_block": rng.random() < 0.6}


# ------------------------------------------------------------------ inputs

def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1009 + salt)
    return g


def _activations(M, d, seed):
    """Student-t(3) values, 0.5% of the channels times 50, bf16."""
    g = _gen(seed, 1)
    ch = torch.randperm(d, generator=g, device="cuda")[: max(1, round(0.005 * d))]
    X = torch.empty((M, d), dtype=torch.bfloat16, device="cuda")
    for r in range(0, M, 4096):
        n = min(4096, M - r)
        c = torch.randn((n, d), generator=g, device="cuda").square_()
        for _ in range(2):
            c += torch.randn((n, d), generator=g, device="cuda").square_()
        t = torch.randn((n, d), generator=g, device="cuda").mul_(c.div_(3.0).rsqrt_())
        t[:, ch] *= 50.0
        X[r:r + n] = t.to(torch.bfloat16)
    return X


def _weights(N, d, seed):
    """N(0, 1/d) entries, 1% of the input channels times 4, bf16."""
    g = _gen(seed, 2)
    W = torch.randn((N, d), generator=g, device="cuda") / math.sqrt(d)
    W[:, torch.randperm(d, generator=g, device="cuda")[: max(1, round(0.01 * d))]] *= 4.0
    return W.to(torch.bfloat16)


def _near_identity(rng, nfac, n):
    m = np.eye(n) + 0.1 * rng.standard_normal((nfac, n, n))
    bad = np.linalg.cond(m) >= 10.0
    while bad.any():
        m[bad] = np.eye(n) + 0.1 * rng.standard_normal((int(bad.sum()), n, n))
        bad = np.linalg.cond(m) >= 10.0
    return torch.from_numpy(m.astype(np.float32))


def _nfac(case):
    return case["d"] // 32 if case["per_block"] else 1


def _factors(case, seed):
    rng = np.random.default_rng([int(seed), 3])
    a = case["a"]
    return _near_identity(rng, _nfac(case), a), _near_identity(rng, _nfac(case), 32 // a)


def _lu(case, seed):
    """(a_k, b_k, c_k) of the five 2x2 factors, well away from a_k = 0."""
    rng = np.random.default_rng([int(seed), 4])
    lu = 0.15 * rng.standard_normal((_nfac(case), 5, 3))
    lu[..., 0] += 1.0
    lu[..., 1] += 0.3
    return torch.from_numpy(lu.astype(np.float32))


def _multipliers(X):
    s = X.float().abs().amax(0)
    return torch.where(s > 0, s.clamp_min(1e-30).rsqrt(), torch.ones_like(s)).contiguous()


def prepare(case, seed):
    M, d, kind, op = case["M"], case["d"], case["kind"], case.get("op")
    st = {"case": case, "X": _activations(M, d, seed)}
    if kind == "calib":
        W = _weights(case["N"], d, seed)
        st.update(W=W, Yneg=kq.calib_reference(st["X"], W), lu=_lu(case, seed).cuda(),
                  lambdas=torch.tensor(LAMBDAS, dtype=torch.float32, device="cuda"),
                  workspace=kq.calib_workspace(M, case["N"], d, case["a"], _nfac(case)))
        return st
    st["codes"] = torch.empty((M, d // 2), dtype=torch.uint8, device="cuda")
    st["scales"] = torch.empty((M, d // 32), dtype=torch.uint8, device="cuda")
    if op == "lu":
        lu = _lu(case, seed)
        st["lu"] = lu.cuda()
        A, B = kq.lu_to_factors(lu, case["a"])
        if case.get("y16") or case.get("out") == "lora":
            st["y16"] = torch.empty((M, d), dtype=torch.bfloat16, device="cuda")
    elif op in ("packed", "fly", "exact"):
        A, B = _factors(case, seed)
        st["A"], st["B"] = A.cuda(), B.cuda()
        if op == "packed":
            st["kpack"] = kq.pack_factors(st["A"], st["B"])
    elif op == "smooth":
        st["mult"] = _multipliers(st["X"])
    if kind == "linear":
        _, st["wcodes"], st["wscales"] = kq.weight_transform(_weights(case["N"], d, seed), A, B)
        if case["out"] == "lora":
            g = _gen(seed, 5)
            st["L1"] = (torch.randn((d, RANK), generator=g, device="cuda") / math.sqrt(d)).to(torch.bfloat16)
            st["L2"] = torch.randn((RANK, case["N"]), generator=g, device="cuda") / math.sqrt(RANK)
    return st


# ------------------------------------------------------------------ the calls

def _quantize(st):
    case, out = st["case"], {"codes": st["codes"], "scales": st["scales"]}
    op = case["op"]
    if op == "packed":
        return kq.quantize_packed(st["X"], st["A"], st["B"], st["kpack"], **out)
    if op == "fly":
        return kq.quantize(st["X"], st["A"], st["B"], **out)
    if op == "lu":
        return kq.quantize_lu(st["X"], st["lu"], case["a"], y16=st.get("y16"), **out)
    if op == "exact":
        return kq.quantize_exact(st["X"], st["A"], st["B"], **out)
    if op == "smooth":
        return kq.smoothquant(st["X"], st["mult"], **out)
    if op == "hadamard":
        return kq.hadamard32(st["X"], **out)
    if op == "fwht":
        return kq.fwht(st["X"], **out)
    return kq.mxfp4(st["X"], **out)


def run(st):
    case = st["case"]
    if case["kind"] == "quant":
        return _quantize(st)
    if case["kind"] == "calib":
        return kq.calib_step(st["X"], st["W"], st["Yneg"], st["lu"], st["lambdas"], a=case["a"], workspace=st["workspace"])
    codes, scales = _quantize(st)[:2]
    if case["out"] == "bf16":
        return kq.mxfp4_gemm(codes, scales, st["wcodes"], st["wscales"], out_dtype=torch.bfloat16)
    if case["out"] == "fp32":
        return kq.mxfp4_gemm(codes, scales, st["wcodes"], st["wscales"])
    C = torch.mm(torch.mm(st["y16"], st["L1"]).float(), st["L2"])
    return kq.mxfp4_gemm(codes, scales, st["wcodes"], st["wscales"], C=C, accumulate=True)


def work(case):
    M, d, kind = case["M"], case["d"], case["kind"]
    x = 2 * M * d
    if kind == "quant":
        per = {"fwht": math.log2(d), "hadamard": 5, "smooth": 1, "plain": 0}.get(case["op"], 2 * (case["a"] + 32 // case["a"]))
        return {"bytes": x + M * d // 2 + M * d // 32 + (x if case.get("y16") else 0), "flops": M * d * per}
    N = case["N"]
    if kind == "linear":
        return {"bytes": x + N * d * 17 // 32 + M * N * (2 if case["out"] == "bf16" else 4),
                "flops": 2 * M * N * d + (2 * RANK * M * (N + d) if case["out"] == "lora" else 0)}
    return {"bytes": x + 2 * N * d + 4 * M * N, "flops": 6 * M * N * d}


def tolerance(case):
    """Four times what was measured: against the 64-bit value, and for the
    quantizers against the fixed fp32 order."""
    if case["kind"] == "calib":
        return {"rel": 6e-5, "max": 4e-4}  # 1.4e-5 and 9.4e-5: a few codes at rounding ties
    if case["kind"] == "linear":
        if case["out"] == "fp32":
            return {"rel": 4e-4, "max": 0.2}  # 9.7e-5 and 0.046: codes at rounding ties, fp32 sums
        return {"rel": 7e-3, "max": 0.4 if case["out"] == "lora" else 0.12}  # 1.9e-3, 0.091 and 0.030: bf16
    if case["op"] in ("packed", "fly", "lu"):
        return {"rel": 1e-4, "max": 0.03, "differ": 1e-5}  # y16 1.9e-5 and 7.5e-3, codes 1.6e-6: ties
    return "exact"  # one fixed order


# ------------------------------------------------------------------ in 64 bits

def _blocks(case, seed):
    """K per factor pair, [nfac, 32, 32], y = K x."""
    if case["kind"] == "calib" or case["op"] == "lu":
        T = _lu_blocks(_lu(case, seed).double().cuda())
        return T.transpose(-1, -2)
    A, B = (t.double().cuda() for t in _factors(case, seed))
    return torch.einsum("fij,fkl->fikjl", A, B).reshape(-1, 32, 32)


def _lu_blocks(p):
    a, b, c = p[..., 0], p[..., 1], p[..., 2]
    G = torch.stack([torch.stack([a, b], -1), torch.stack([c * a, c * b - 1.0 / a], -1)], -2)
    T = G[:, 0]
    for k in range(1, 5):
        n = 2 * T.shape[-1]
        T = torch.einsum("fij,fkl->fikjl", T, G[:, k]).reshape(-1, n, n)
    return T


def _rows_times(x, T):
    """Every 32-column block of the rows of x times its T."""
    M, d = x.shape
    t = x.reshape(M, d // 32, 32).transpose(0, 1)
    return torch.matmul(t, T).transpose(0, 1).reshape(M, d)


def _mxfp4(y):
    """Dequantized MXFP4 of y and the clipping limit of every element."""
    v = y.reshape(y.shape[0], -1, 32)
    amax = v.abs().amax(-1, keepdim=True)
    e = torch.where(amax > 0, torch.frexp(amax)[1].double() - 3.0, torch.full_like(amax, -127.0)).clamp_min(-127.0)
    s = torch.exp2(e)
    m = v.abs() / s
    step = torch.where(m < 2, 0.5, torch.where(m < 4, 1.0, 2.0)).to(m.dtype)
    q = (torch.round(m / step) * step).clamp_max(6.0) * s * torch.sign(v)
    return q.reshape(y.shape), (6.0 * s).expand_as(v).reshape(y.shape)


def exact(case, seed):
    M, d, kind, op = case["M"], case["d"], case["kind"], case.get("op")
    if kind == "quant" and not case.get("y16"):
        return None  # whole numbers only
    x = _activations(M, d, seed).double()
    if kind == "calib":
        return _calib_exact(case, seed, x)
    K = _blocks(case, seed)
    y = _rows_times(x, K.transpose(-1, -2))
    if kind == "quant":
        return [None, None, None, y]
    w = _rows_times(_weights(case["N"], d, seed).double(), torch.linalg.inv(K))
    out = _mxfp4(y)[0] @ _mxfp4(w)[0].T
    if case["out"] == "lora":
        g = _gen(seed, 5)
        L1 = (torch.randn((d, RANK), generator=g, device="cuda") / math.sqrt(d)).to(torch.bfloat16).double()
        L2 = (torch.randn((RANK, case["N"]), generator=g, device="cuda") / math.sqrt(RANK)).double()
        out += (y @ L1) @ L2
    return out


def _calib_exact(case, seed, x):
    """The objective with the E2M1 rounding passed through, the scale held
    fixed and clipped elements passing no gradient."""
    M, d, N = case["M"], case["d"], case["N"]
    w = _weights(N, d, seed).double()
    p = _lu(case, seed).double().cuda().requires_grad_()
    T = _lu_blocks(p)
    y, v = _rows_times(x, T), _rows_times(w, torch.linalg.inv(T).transpose(-1, -2))
    (qy, ly), (qv, lv) = _mxfp4(y.detach()), _mxfp4(v.detach())
    qy = qy + (y.detach().abs() <= ly) * (y - y.detach())
    qv = qv + (v.detach().abs() <= lv) * (v - v.detach())
    out = (qy @ qv.T - x @ w.T).square().sum() / (M * N)
    la, lw = (qy - y).square().sum() / (M * d), (qv - v).square().sum() / (N * d)
    lam = torch.tensor(LAMBDAS, dtype=torch.float32).tolist()
    total = out + lam[0] * la + lam[1] * lw
    total.backward()
    return [torch.stack([out, la, lw, total]).detach(), p.grad]
