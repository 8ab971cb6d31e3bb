"""Performance cases of the sketch library, each one pass through its public entry points.

A case is a dict of plain values; ``op`` names the call it stands for:

  gen      sketch_gen_matmul: one process's share, Y = A * Omega(seed), A row-major in
           FP32, BF16 or FP8 (per-128-row scales)
  layouts  the two layouts of one product: P row-block calls, then one
           sketch_gen_matmul_reduce over P column blocks of the same A
  cm       sketch_gen_matmul_cm: A stored by columns, Y or its transpose
  tmatmul  sketch_gen_tmatmul: the second Nystrom product C = Omega^T B
  pinv     sketch_core_pinv: pseudo-inverse of the Nystrom core
  error    sketch_nystrom_error: squared norms and relative error of A - B C^+ B^T
  serve    SketchServer: a burst of requests of uneven shapes on views of one resident A

``exact`` evaluates the same products in FP64 with torch alone: Omega from its definition
(Philox4x32-10 words, u = (2 (r >> 9) + 1) 2^-24, Box-Muller in FP64).
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2603_20966_amd as sk

DEV = "cuda:0"
ESZ = {"f32": 4, "bf16": 2, "fp8": 1}
SERVED_K = (5, 16, 64)     # sketch widths of the served stream


def listed():
    return [
        # the smallest request of the served range as a call of its own: latency
        dict(name="gen_f32_1024x1024_k5", op="gen", dtype="f32", m=1024, n=1024, k=5, dist="normal"),
        # the headline step: eight 4096-row shares and the eight-block contraction split
        dict(name="layouts_f32_32768_k5", op="layouts", m=32768, n=32768, k=5, P=8, dist="normal"),
        # odd sizes (a strided A, ragged strips and row tiles), the paper's uniform entries
        dict(name="gen_f32_20011x9973_k16_uniform", op="gen", dtype="f32", m=20011, n=9973, k=16,
             dist="uniform"),
        # wide sketches of a tall A, as a range finder asks for
        dict(name="gen_f32_65536x16384_k64", op="gen", dtype="f32", m=65536, n=16384, k=64,
             dist="normal"),
        # the first Nystrom product at r = 256
        dict(name="gen_f32_32768x32768_k256", op="gen", dtype="f32", m=32768, n=32768, k=256,
             dist="normal"),
        # low-precision storage of A: a wide sketch of BF16, a narrow one of FP8
        dict(name="gen_bf16_32768x32768_k64", op="gen", dtype="bf16", m=32768, n=32768, k=64,
             dist="normal"),
        dict(name="gen_fp8_32768x32768_k5", op="gen", dtype="fp8", m=32768, n=32768, k=5,
             dist="normal"),
        # the paper's storage order
        dict(name="cm_f32_32768x32768_k64", op="cm", m=32768, n=32768, k=64, trans=False,
             dist="normal"),
        # the second Nystrom product: few columns, a long contraction
        dict(name="tmatmul_32768_r64", op="tmatmul", n=32768, p=64, k=64, dist="normal"),
        # the Nystrom core at the wider of the two usual ranks
        dict(name="pinv_r256", op="pinv", r=256),
        # the error of the approximation, as the paper's tables report it
        dict(name="error_16384_r256", op="error", n=16384, r=256),
        # requests that arrive together, m and n log-uniform in [1024, 32768]
        dict(name="serve_48_requests", op="serve", count=48, hi=32768, mix=2026),
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """Log-uniform; half of them rounded to a multiple of 64 when that stays inside."""
    v = _log_int(rng, lo, hi)
    return max(lo, v // 64 * 64) if rng.random() < 0.5 else v


def _shape(rng, k, lo=1024, hi_m=65536, hi_n=32768):
    """(m, n) within the range and below the cost of 32768 x 32768 at k = 256 (2^30 elements)."""
    while True:
        m, n = _size(rng, lo, hi_m), _size(rng, lo, hi_n)
        if m * n <= 1 << 30 and m * n * k <= 1 << 38:
            return m, n


def draw(rng: random.Random):
    op = rng.choice(["gen"] * 6 + ["layouts", "cm", "cm", "tmatmul", "tmatmul", "pinv", "error", "serve"])
    dist = rng.choice(["normal", "normal", "normal", "uniform", "rademacher"])
    if op == "gen":
        dtype = rng.choice(["f32", "f32", "f32", "bf16", "fp8"])
        k = _log_int(rng, 1, 256)
        m, n = _shape(rng, k)
        return dict(op=op, dtype=dtype, m=m, n=n, k=k, dist=dist)
    if op == "layouts":
        # block widths of whole 4096-column strips
        return dict(op=op, m=_size(rng, 8192, 32768), n=32768, k=rng.randint(2, 8), P=8, dist=dist)
    if op == "cm":
        k = _log_int(rng, 4, 128)
        m, n = _shape(rng, k, hi_m=32768)
        return dict(op=op, m=m, n=n, k=k, trans=rng.random() < 0.3, dist=dist)
    if op == "tmatmul":
        p = _log_int(rng, 4, 256)
        return dict(op=op, n=_size(rng, 4096, 65536), p=p, k=p, dist=dist)
    if op == "pinv":
        return dict(op=op, r=_log_int(rng, 24, 256))
    if op == "error":
        return dict(op=op, n=_size(rng, 2048, 16384), r=_log_int(rng, 16, 256))
    return dict(op=op, count=rng.randint(16, 48), hi=rng.choice([8192, 16384, 32768]),
                mix=rng.randrange(1 << 30))


# ---- inputs -------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(rows, cols, seed, pad=4):
    """rows x cols N(0,1) FP32 whose rows start 16-byte aligned (leading dimension padded)."""
    ld = (cols + pad - 1) // pad * pad
    A = torch.empty((rows, ld), dtype=torch.float32, device=DEV)
    A.normal_(generator=_gen(seed))
    return A[:, :cols]


def _quantised(m, n, dtype, seed):
    """(Aq, scales): BF16 by round to nearest even; FP8-E4M3 with a power-of-two scale per
    128-row block, the smallest 2^E with amax <= 448 2^E."""
    A = _normal(m, n, seed, pad=16)
    if dtype == "f32":
        return A, None
    ld = (n + 15) // 16 * 16
    if dtype == "bf16":
        Aq = torch.empty((m, ld), dtype=torch.bfloat16, device=DEV)[:, :n]
        Aq.copy_(A)
        return Aq, None
    nb = (m + 127) // 128
    rowmax = torch.zeros(nb * 128, device=DEV)
    rowmax[:m] = torch.maximum(A.amax(1), -A.amin(1))
    amax = rowmax.view(nb, 128).amax(1)
    scales = torch.exp2(torch.ceil(torch.log2(amax.double() / 448.0))).float()
    Aq = torch.empty((m, ld), dtype=torch.float8_e4m3fn, device=DEV)[:, :n]
    for b in range(0, m, 4096):
        s = scales.repeat_interleave(128)[b:min(b + 4096, m), None]
        Aq[b:b + 4096].copy_((A[b:b + 4096] / s).clamp_(-448.0, 448.0))
    return Aq, scales


def _rbf(n, seed, latent=40, dim=256):
    """n x n RBF kernel (sigma = ||X||_F / sqrt(n)) of latent-dimensional synthetic data."""
    g = _gen(seed)
    X = torch.randn((n, latent), generator=g, device=DEV) @ (
        torch.randn((latent, dim), generator=g, device=DEV) / math.sqrt(latent))
    sq = (X * X).sum(1)
    K = X @ X.t().contiguous()
    K.mul_(-2.0).add_(sq[:, None]).add_(sq[None, :]).clamp_(min=0.0)
    return K.mul_(-0.5 * n / sq.sum()).exp_()


def _core(n, r, seed):
    """(A, B, C) of a Nystrom approximation, with a test matrix drawn by torch."""
    A = _rbf(n, seed)
    Om = torch.randn((n, r), generator=_gen(seed + 7), device=DEV, dtype=torch.float64)
    B = torch.empty((n, r), dtype=torch.float64, device=DEV)
    for b in range(0, n, 2048):
        B[b:b + 2048] = A[b:b + 2048].double() @ Om
    C = Om.t().contiguous() @ B
    ld = (r + 3) // 4 * 4
    Bf = torch.empty((n, ld), device=DEV)[:, :r]
    Bf.copy_(B)
    return A, Bf, (0.5 * (C + C.t())).float()


def _pinv64(C):
    """FP64 pseudo-inverse of the symmetric C at relative tolerance 1e-12 (on the host)."""
    lam, V = np.linalg.eigh(C.double().cpu().numpy())
    keep = np.abs(lam) > 1e-12 * np.abs(lam).max()
    mu = np.where(keep, 1.0 / np.where(lam == 0, 1.0, lam), 0.0)
    return torch.from_numpy((V * mu) @ V.T).to(DEV)


def _requests(case, seed):
    """[(m, n, k, Omega seed)] of a served burst: the shapes are the case's, the seeds new."""
    rng = np.random.default_rng(case["mix"])
    out = []
    for i in range(case["count"]):
        m, n = (int(round(math.exp(rng.uniform(math.log(1024), math.log(case["hi"]))))) for _ in "mn")
        out.append((m, n, int(SERVED_K[rng.integers(0, 3)]), int(seed) * 1000 + i))
    return out


def prepare(case, seed):
    op = case["op"]
    s = dict(case, seed=int(seed))
    if op == "gen":
        s["A"], s["scales"] = _quantised(case["m"], case["n"], case["dtype"], seed)
        s["Y"] = torch.empty((case["m"], case["k"]), device=DEV)
    elif op == "layouts":
        A = _normal(case["m"], case["n"], seed)
        P, m, nb = case["P"], case["m"], case["n"] // case["P"]
        s["Yr"], s["Yc"] = (torch.empty((m, case["k"]), device=DEV) for _ in "rc")
        cut = [m * p // P for p in range(P + 1)]
        s["rows"] = [(A[a:b], s["Yr"][a:b]) for a, b in zip(cut, cut[1:])]
        s["blocks"] = [A[:, p * nb:(p + 1) * nb] for p in range(P)]
        s["row0s"] = [p * nb for p in range(P)]
    elif op == "cm":
        s["A"] = _normal(case["n"], case["m"], seed).t()
        shape = (case["k"], case["m"]) if case["trans"] else (case["m"], case["k"])
        s["Y"] = torch.empty(shape, device=DEV)
    elif op == "tmatmul":
        # B = A Omega of an n-column N(0,1) A: entries of variance n
        s["B"] = _normal(case["n"], case["p"], seed).mul_(math.sqrt(case["n"]))
        s["C"] = torch.empty((case["k"], case["p"]), device=DEV)
    elif op == "pinv":
        s["C"] = _core(4096, case["r"], seed)[2]
    elif op == "error":
        s["A"], s["B"], C = _core(case["n"], case["r"], seed)
        s["Cp"] = _pinv64(C)
    else:
        A = _normal(case["hi"], case["hi"], seed)
        s["A"], s["reqs"], s["Ys"] = A, [], []
        for m, n, k, om in _requests(case, seed):
            Y = torch.empty((m, k), device=DEV)
            s["reqs"].append(sk.make_request(k=k, seed=om, Y=Y, A=A[:m, :n]))
            s["Ys"].append(Y)
        s["server"] = sk.SketchServer(16 << 30, max_slots=32, max_batch=16, n_streams=4)
        torch.cuda.synchronize()   # the server's streams are not ordered after this one
    return s


# ---- one pass -----------------------------------------------------------------------
def run(s):
    op = s["op"]
    if op == "gen":
        return sk.sketch_gen_matmul(s["A"], s["seed"], s["k"], Y=s["Y"], a_scales=s["scales"],
                                    dist=s["dist"])
    if op == "layouts":
        for A, Y in s["rows"]:
            sk.sketch_gen_matmul(A, s["seed"], s["k"], Y=Y, dist=s["dist"])
        sk.sketch_gen_matmul_reduce(s["blocks"], s["row0s"], s["seed"], s["k"], Y=s["Yc"],
                                    dist=s["dist"])
        return s["Yr"], s["Yc"]
    if op == "cm":
        return sk.sketch_gen_matmul_cm(s["A"], s["seed"], s["k"], Y=s["Y"], y_trans=s["trans"],
                                       dist=s["dist"])
    if op == "tmatmul":
        return sk.sketch_gen_tmatmul(s["B"], s["seed"], s["k"], C=s["C"], dist=s["dist"])
    if op == "pinv":
        return sk.sketch_core_pinv(s["C"])[0]
    if op == "error":
        return sk.sketch_nystrom_error(s["A"], s["B"], s["Cp"])
    srv = s["server"]
    tickets = [srv.submit(q, s["A"], Y) for q, Y in zip(s["reqs"], s["Ys"])]
    for t in tickets:
        srv.wait(t)
    return s["Ys"]


def work(case):
    """Bytes: every input read once, every output written once (Omega is generated).  Flops:
    two per product term; the pseudo-inverse at 9 r^3 for the eigendecomposition of a symmetric
    matrix and 2 r^3 for forming it back."""
    op = case["op"]
    if op == "gen":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": m * n * ESZ[case["dtype"]] + 4 * m * k, "flops": 2 * m * n * k}
    if op == "layouts":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 2 * (4 * m * n + 4 * m * k), "flops": 4 * m * n * k}
    if op == "cm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 4 * m * n + 4 * m * k, "flops": 2 * m * n * k}
    if op == "tmatmul":
        n, p, k = case["n"], case["p"], case["k"]
        return {"bytes": 4 * n * p + 4 * k * p, "flops": 2 * n * p * k}
    if op == "pinv":
        r = case["r"]
        return {"bytes": 4 * r * r + 8 * r * r, "flops": 11 * r ** 3}
    if op == "error":
        n, r = case["n"], case["r"]
        return {"bytes": 4 * n * n + 4 * n * r + 8 * r * r + 24, "flops": 2 * n * n * r + 2 * n * r * r}
    reqs = _requests(case, 1)
    return {"bytes": sum(4 * m * n + 4 * m * k for m, n, k, _ in reqs),
            "flops": sum(2 * m * n * k for m, n, k, _ in reqs)}


# ---- the same in 64 bits ------------------------------------------------------------
def _omega64(seed, n, k, dist):
    """Omega(seed)[0:n, 0:k] in FP64 from its definition."""
    M = 0xFFFFFFFF
    q = torch.arange((n + 3) // 4, dtype=torch.int64, device=DEV)[:, None].expand(-1, k)
    x, y = (q & M).clone(), (q >> 32).clone()
    z = torch.arange(k, dtype=torch.int64, device=DEV)[None, :].expand(q.shape[0], -1).clone()
    w = torch.zeros_like(x)
    k0, k1 = seed & M, (seed >> 32) & M
    for _ in range(10):
        p0, p1 = 0xD2511F53 * x, 0xCD9E8D57 * z          # wraps modulo 2^64
        x, y, z, w = ((p1 >> 32) & M) ^ y ^ k0, p1 & M, ((p0 >> 32) & M) ^ w ^ k1, p0 & M
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    words = torch.stack([x, y, z, w], 1)                  # quads x 4 x k
    if dist == "rademacher":
        out = 1.0 - 2.0 * (words >> 31).double()
    else:
        u = (2 * (words >> 9) + 1).double() * 2.0 ** -24
        if dist == "uniform":
            out = u
        else:
            rho = torch.sqrt(-2.0 * torch.log(u[:, 0::2]))
            th = 2.0 * math.pi * u[:, 1::2]
            out = torch.stack([rho * torch.cos(th), rho * torch.sin(th)], 2).flatten(1, 2)
    return out.reshape(-1, k)[:n].contiguous()


def _product64(A, scales, Om):
    """A Om in FP64, a block of rows at a time."""
    out = torch.empty((A.shape[0], Om.shape[1]), dtype=torch.float64, device=DEV)
    for b in range(0, A.shape[0], 2048):
        rows = A[b:b + 2048]
        rows = (rows.float() if rows.dtype == torch.float8_e4m3fn else rows).double()
        if scales is not None:
            rows = rows * scales.double().repeat_interleave(128)[b:b + rows.shape[0], None]
        out[b:b + 2048] = rows @ Om
    return out


def exact(case, seed):
    op, seed = case["op"], int(seed)
    if op == "gen":
        A, sc = _quantised(case["m"], case["n"], case["dtype"], seed)
        return _product64(A, sc, _omega64(seed, case["n"], case["k"], case["dist"]))
    if op == "layouts":
        A = _normal(case["m"], case["n"], seed)
        Y = _product64(A, None, _omega64(seed, case["n"], case["k"], case["dist"]))
        return Y, Y
    if op == "cm":
        At = _normal(case["n"], case["m"], seed)
        Om = _omega64(seed, case["n"], case["k"], case["dist"])
        Y = torch.zeros((case["m"], case["k"]), dtype=torch.float64, device=DEV)
        for b in range(0, case["n"], 2048):
            Y += At[b:b + 2048].double().t().contiguous() @ Om[b:b + 2048]
        return Y.t().contiguous() if case["trans"] else Y
    if op == "tmatmul":
        B = _normal(case["n"], case["p"], seed).mul_(math.sqrt(case["n"]))
        Om = _omega64(seed, case["n"], case["k"], case["dist"])
        return Om.t().contiguous() @ B.double()
    if op == "pinv":
        return _pinv64(_core(4096, case["r"], seed)[2])
    if op == "error":
        A, B, C = _core(case["n"], case["r"], seed)
        W, Bt = B.double() @ _pinv64(C), B.double().t().contiguous()
        se = sa = 0.0
        for b in range(0, case["n"], 2048):
            a = A[b:b + 2048].double()
            se += float((a - W[b:b + 2048] @ Bt).square().sum())
            sa += float(a.square().sum())
        return torch.tensor([se, sa, math.sqrt(se / sa)], dtype=torch.float64)
    A = _normal(case["hi"], case["hi"], seed)
    return [_product64(A[:m, :n], None, _omega64(om, n, k, "normal"))
            for m, n, k, om in _requests(case, seed)]
