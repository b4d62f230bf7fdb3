"""The workloads whose speed is watched, through the package's public entry points.

Each case is what a program that uses the package runs: planned products
(`runner.FMM.matmul`) over the shapes, realizations, depths, blocks, scale
rules and options of the package's own benchmark, configurations, controls and
tests, and the error measurement (`encode_noise`, `reference_f64`,
`error_stats`).  `exact` is the same evaluation written in plain torch: the
combinations rounded in binary32 as the definition says, the e4m3 codes and
block scales, then the products and the W-combine in binary64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_26077_amd as fm
from paper_2609_26077_amd.runner import FMM, error_stats, reference_f64

# ---- realizations (U: A block 2i+j, V: B block 2j+k, W: C block 2k+i) --------
_X, _E, _Z = 0.5773502691896257, 0.8660254037844386, 0.28867513459481287   # 1/sqrt3, sqrt3/2, 1/(2 sqrt3)
_TU = [[1, 0, 0, 1], [0, 0, _X, 1], [1, 0, _X, 0], [0, 0, -_X, 1], [.5, _E, _Z, .5], [-1, 0, _X, 0], [-.5, _E, _Z, -.5]]
_TABLES = {
    "strassen": ([[1, 0, 0, 1], [0, 0, 1, 1], [1, 0, 0, 0], [0, 0, 0, 1], [1, 1, 0, 0], [-1, 0, 1, 0], [0, 1, 0, -1]],
                 [[1, 0, 0, 1], [1, 0, 0, 0], [0, 1, 0, -1], [-1, 0, 1, 0], [0, 0, 0, 1], [1, 1, 0, 0], [0, 0, 1, 1]],
                 [[1, 0, 0, 1], [0, 1, 0, -1], [0, 0, 1, 1], [1, 1, 0, 0], [-1, 0, 1, 0], [0, 0, 0, 1], [1, 0, 0, 0]]),
    "tstar": (_TU, [_TU[i - 1] for i in (1, 3, 7, 6, 4, 5, 2)], [_TU[i - 1] for i in (1, 7, 2, 5, 6, 4, 3)]),
}


def _basis_changed(seed):
    """Strassen under a random change of basis (X, Y, Z), each factor I + 0.45 N(0,1) with |det| >= 0.3."""
    rng = np.random.RandomState(seed)
    g = []
    while len(g) < 3:
        m = np.eye(2) + 0.45 * rng.standard_normal((2, 2))
        if abs(np.linalg.det(m)) >= 0.3:
            g.append(m)
    X, Y, Z = g
    U, V, W = (np.array(t, dtype=np.float64) for t in _TABLES["strassen"])
    it = lambda m: np.linalg.inv(m).T
    return U @ np.kron(X, it(Y)), V @ np.kron(Y, it(Z)), W @ np.kron(Z, it(X))


def _strassen_223():
    """<2,2,3;11>: Strassen beside the four products of a cubic <2,2,1>."""
    U, V, W = np.zeros((11, 4)), np.zeros((11, 6)), np.zeros((11, 6))
    u, v, w = (np.array(t, dtype=np.float64) for t in _TABLES["strassen"])
    U[:7] = u
    for j in range(2):
        for l in range(2):
            V[:7, 3 * j + l] = v[:, 2 * j + l]
            W[:7, 2 * l + j] = w[:, 2 * l + j]
    for i in range(2):
        for j in range(2):
            r = 7 + 2 * i + j
            U[r, 2 * i + j] = V[r, 3 * j + 2] = W[r, 4 + i] = 1.0
    return U, V, W


def _coefficients(case):
    """(grid (m, k, n), U, V, W) of the base realization, binary64."""
    name = case["realization"]
    if name == "223":
        return (2, 2, 3), *_strassen_223()
    if name == "basis":
        return (2, 2, 2), *_basis_changed(case["basis"])
    return (2, 2, 2), *(np.array(t, dtype=np.float64) for t in _TABLES[name])


def _realization(case):
    if case["realization"] in _TABLES:
        return fm.fmm_realization_builtin(case["realization"])
    shape, U, V, W = _coefficients(case)
    return fm.fmm_realization_create(U, V, W, shape=shape)


# ---- the cases ---------------------------------------------------------------
def _case(name, M, K, N, batch=1, realization="tstar", basis=0, depth=1, block=32, rule="pow2_ceil", family="gaussian",
          exact_dot=False, weights=False, kind="product"):
    c = {"kind": kind, "batch": batch, "M": M, "K": K, "N": N, "realization": realization, "basis": basis,
         "depth": depth, "block": block, "rule": rule, "family": family, "exact_dot": exact_dot, "weights": weights}
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # one small product: the latency of a call
        _case("one_256", 256, 256, 256),
        # the 256^3 configuration: a batch of a hundred trials
        _case("batch100_256", 256, 256, 256, batch=100, realization="strassen"),
        # the error controls' products: two of 1024^3, signed-uniform operands
        _case("pair_1024", 1024, 1024, 1024, batch=2, family="uniform"),
        # sizes that fit no tile: rows and columns off the 128 grid, a contracted axis off the 128-byte step
        _case("ragged_3x1000x1472x1302", 1000, 1472, 1302, batch=3, realization="strassen"),
        # the cross-shape control: eight samples at block edge 256, 1 x 128 blocks with fp32 scales, <2,2,3;11>
        _case("shape223_8x512x512x768", 512, 512, 768, batch=8, realization="223", block=128, rule="fp32_amax",
              family="uniform"),
        # the 4096^3 configuration
        _case("cube_4096", 4096, 4096, 4096),
        # the benchmark's headline product
        _case("cube_8192", 8192, 8192, 8192),
        # the two-level configuration
        _case("cube_8192_depth2", 8192, 8192, 8192, depth=2, realization="strassen", family="uniform"),
        # the basis-change sweep: 1024 small products with heavy tails on the exact-dot path
        _case("batch1024_512_exact", 512, 512, 512, batch=1024, realization="basis", basis=1, block=16,
              family="student_t3", exact_dot=True),
        # the three-level configuration: rows scaled over four decades, exact-dot path
        _case("deep_16384x8192x16384", 16384, 8192, 16384, depth=3, family="rowscaled", exact_dot=True),
        # the deployment granularity: 128 x 128 weight blocks of bfloat16-rounded combinations, fp32 amax scales
        _case("weights_8192", 8192, 8192, 8192, block=128, rule="fp32_amax", weights=True),
        # the error measurement of the controls: operand noise, fp64 reference, error sums
        _case("measure_2x2048x1024x1536", 2048, 1024, 1536, batch=2, kind="measure"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _near(x, step):
    return max(step, int(round(x / step)) * step)


def draw(rng):
    """One more case of the listed ranges."""
    what = rng.choice(["single", "single", "batch", "ragged", "ragged", "exact", "deep", "weights", "shape", "fp32", "measure"])
    fam = rng.choice(["gaussian", "uniform", "student_t3"])
    real = rng.choice(["tstar", "strassen"])
    if what == "single":       # tile-aligned single products, small to large
        s = _log(rng, 256, 8192)
        M, K, N = (min(8192, _near(s * _log(rng, 0.6, 1.6), 256)) for _ in range(3))
        depth = 1 if s < 2048 else rng.choice([1, 1, 2])
        return _case(None, M, K, N, realization=real, depth=depth, family=rng.choice(["gaussian", "uniform"]),
                     block=rng.choice([32, 32, 128]) if K % (128 << depth) == 0 else 32)
    if what == "batch":        # many small products
        M, K, N = (rng.choice([256, 512, 768]) for _ in range(3))
        return _case(None, M, K, N, batch=int(_log(rng, 8, 512)), realization=real, family=rng.choice(["gaussian", "uniform"]),
                     rule=rng.choice(["pow2_ceil", "pow2_ocp"]))
    if what == "ragged":       # odd and ragged sizes on every path
        depth, block = rng.choice([1, 1, 2]), rng.choice([16, 32, 32])
        n = 1 << depth
        s = _log(rng, 48, 2000)
        M, N = (_near(s * _log(rng, 0.5, 2.0), n) + n * rng.choice([0, 1]) for _ in range(2))
        K = _near(s * _log(rng, 0.5, 2.0), n * block)
        return _case(None, M, K, N, batch=rng.choice([1, 1, 2, 5]), realization=real, depth=depth, block=block,
                     rule=rng.choice(["pow2_ceil", "pow2_ceil", "fp32_amax"]), family="gaussian", exact_dot=rng.choice([False, True]))
    if what == "exact":        # the exact-dot path on sweeps and single products
        M, K, N = (_near(_log(rng, 256, 4096), 256) for _ in range(3))
        most = max(1, min(512, int(4e10 / (M * K * N))))
        return _case(None, M, K, N, batch=int(_log(rng, 1, most + 1)), realization="basis", basis=rng.randrange(1, 64),
                     block=rng.choice([16, 32, 128]) if K % 256 == 0 else 32, family="student_t3", exact_dot=True)
    if what == "deep":         # two and three levels
        depth = rng.choice([2, 3])
        n = 128 << depth
        M, K, N = (_near(_log(rng, 1024, 8192), n) for _ in range(3))
        return _case(None, M, K, N, realization=real, depth=depth, family=rng.choice(["gaussian", "rowscaled"]), exact_dot=True)
    if what == "weights":      # deployment granularity
        M, K, N = (_near(_log(rng, 512, 8192), 512) for _ in range(3))
        return _case(None, M, K, N, block=128, rule=rng.choice(["fp32_amax", "pow2_ceil"]), family="gaussian", weights=True)
    if what == "shape":        # another shape
        M, K = (_near(_log(rng, 512, 4096), 512) for _ in range(2))
        N = _near(_log(rng, 768, 6144), 768)
        return _case(None, M, K, N, batch=rng.choice([1, 2, 8]) if M * K * N < 3e9 else 1, realization="223",
                     block=rng.choice([32, 128]), rule=rng.choice(["pow2_ceil", "fp32_amax"]), family=fam if fam != "student_t3" else "uniform")
    if what == "fp32":         # fp32 amax scales on tile-aligned products
        M, K, N = (_near(_log(rng, 512, 4096), 512) for _ in range(3))
        return _case(None, M, K, N, realization=real, block=rng.choice([16, 32, 128]), rule="fp32_amax", family=fam)
    M, K, N = (_near(_log(rng, 256, 2048), 64) + 2 * rng.choice([0, 0, 3]) * (i != 1) for i in range(3))
    return _case(None, M, K, N, batch=rng.choice([1, 2, 4]) if M * K * N < 1e9 else 1, realization=real, kind="measure",
                 family=fam)


# ---- inputs --------------------------------------------------------------------
def _values(family, shape, gen):
    new = lambda s: torch.randn(s, generator=gen, device="cuda")
    if family == "uniform":
        return 2 * torch.rand(shape, generator=gen, device="cuda") - 1
    x = new(shape)
    if family == "student_t3":      # t with three degrees of freedom, unit variance
        chi = new(shape) ** 2
        chi += new(shape) ** 2
        chi += new(shape) ** 2
        return x / chi.div_(3).sqrt_() / math.sqrt(3.0)
    if family == "rowscaled":       # a factor over [1e-2, 1e2] per row
        return x * 10 ** (4 * torch.rand(shape[:-1] + (1,), generator=gen, device="cuda") - 2)
    return x


def _operands(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17)
    b, M, K, N = case["batch"], case["M"], case["K"], case["N"]
    A, B = _values(case["family"], (b, M, K), gen), _values(case["family"], (b, K, N), gen)
    if case["kind"] != "measure":
        return A, B, None
    # a product with the error an e4m3 product has, about 6%
    ref = torch.stack([A[i].double() @ B[i].double() for i in range(b)])
    C = ref + 0.06 * ref.square().mean().sqrt() * torch.randn((b, M, N), generator=gen, device="cuda")
    return A, B, C.float()


def prepare(case, seed):
    A, B, C = _operands(case, seed)
    flags = fm.FMM_FLAG_B_BLOCK128 | fm.FMM_FLAG_B_BF16 if case["weights"] else 0
    f = FMM(_realization(case), case["batch"], case["M"], case["K"], case["N"], case["depth"], case["block"],
            case["rule"], exact_dot=case["exact_dot"], flags=flags)
    if C is None:
        C = torch.empty((case["batch"], case["M"], case["N"]), device="cuda")
    return {"f": f, "A": A, "B": B, "C": C, "kind": case["kind"]}


def run(state):
    f, A, B, C = state["f"], state["A"], state["B"], state["C"]
    if state["kind"] == "product":
        return f.matmul(A, B, C)
    f.encode(A, B)
    noise = f.encode_noise(A, B)
    Cref = reference_f64(A, B)
    err2, ref2 = error_stats(C, Cref)
    return {"noise": noise, "reference": Cref, "err2": err2, "ref2": ref2}


# ---- what a pass needs -----------------------------------------------------------
def _grid(case):
    (m, k, n), U, _, _ = _coefficients(case)
    if case["realization"] == "223":
        return m, k, n, U.shape[0]
    g = 1 << case["depth"]
    return g, g, g, U.shape[0] ** case["depth"]


def work(case):
    b, M, K, N = case["batch"], case["M"], case["K"], case["N"]
    m, k, n, T = _grid(case)
    if case["kind"] == "measure":
        return {"bytes": b * (4 * (M * K + K * N) + 12 * M * N), "flops": 2 * b * M * K * N}
    return {"bytes": 4 * b * (M * K + K * N + M * N), "flops": 2 * b * T * (M // m) * (K // k) * (N // n)}


def tolerance(case):
    """About four times what the paths measure against `exact`: 1e-15 for binary64 sums, 1e-7 to 4e-7 (one to three
    levels) where the products are summed in binary32, 2e-5 (one level) to 6e-5 (two) on the fp8 matrix cores, whose dot
    product keeps 13 bits below each group's largest product."""
    if case["kind"] == "measure":
        return {"rel": 1e-13}
    exact = case["exact_dot"] or case["rule"] == "fp32_amax" or case["block"] == 16
    return {"rel": 2e-6} if exact else {"rel": 1.2e-4 * case["depth"]}


# ---- the same in plain torch, products and sums in binary64 -----------------------
def _flatten(base, depth):
    """Depth-l rows: column P 2^l + Q for block bits P, Q (outer level first), binary64 products left to right, rounded once."""
    out = base.reshape(-1, 2, 2)
    for _ in range(depth - 1):
        s = out.shape[1]
        out = np.einsum("rpq,sij->rspiqj", out, base.reshape(-1, 2, 2)).reshape(-1, 2 * s, 2 * s)
    return out.reshape(out.shape[0], -1).astype(np.float32)


def _combine(blocks, coef):
    x = None
    for c, a in zip(coef, blocks):
        if c != 0:
            t = a * float(c)
            x = t if x is None else x + t
    return torch.zeros_like(blocks[0]) if x is None else x


def _quantized(x, block, rule, rows=1):
    """Values that the codes of x (..., rows, contracted) stand for, binary64."""
    *lead, R, k = x.shape
    a = x.abs().reshape(*lead, R, k // block, block).amax(-1)
    if rows > 1:
        pad = -R % rows
        p = torch.nn.functional.pad(a, (0, 0, 0, pad)).reshape(*lead, (R + pad) // rows, rows, k // block).amax(-2)
        a = p.repeat_interleave(rows, dim=-2)[..., :R, :]
    a = a.clamp(min=float(np.float32(1e-12)))
    if rule == "fp32_amax":
        s = (a.double() / 448).float().double()
    else:
        m, e = torch.frexp(a)
        e = e.double() - 9
        s = torch.exp2(torch.where(m > 0.875, e + 1, e) if rule == "pow2_ceil" else e)
    s = s[..., None].expand(*a.shape, block).reshape(x.shape)
    v = (x.double() / s).float().clamp(-448, 448)
    return v.to(torch.float8_e4m3fn).double() * s


def exact(case, seed):
    A, B, C = _operands(case, seed)
    (m, k, n), U, V, W = _coefficients(case)
    if case["realization"] == "223":
        U, V, W = (t.astype(np.float32) for t in (U, V, W))
    else:
        U, V, W = (_flatten(t, case["depth"]) for t in (U, V, W))
        m = k = n = 1 << case["depth"]
    b, M, K, N = case["batch"], case["M"], case["K"], case["N"]
    mp, kp, np_ = M // m, K // k, N // n
    Ab = [A[:, i * mp:(i + 1) * mp, j * kp:(j + 1) * kp] for i in range(m) for j in range(k)]
    Bb = [B[:, j * kp:(j + 1) * kp, l * np_:(l + 1) * np_] for j in range(k) for l in range(n)]
    if case["kind"] == "measure":
        noise = torch.zeros((b, 2, U.shape[0], 2), dtype=torch.float64, device="cuda")
    else:
        out = torch.zeros((b, M, N), dtype=torch.float64, device="cuda")
    for r in range(U.shape[0]):
        x, y = _combine(Ab, U[r]), _combine(Bb, V[r]).transpose(1, 2).contiguous()
        if case["weights"]:
            y = y.bfloat16().float()
        xh = _quantized(x, case["block"], case["rule"])
        yh = _quantized(y, case["block"], case["rule"], 128 if case["weights"] else 1)
        if case["kind"] == "measure":
            for s, (v, h) in enumerate(((x, xh), (y, yh))):
                noise[:, s, r, 0] = (h - v.double()).square().sum((1, 2))
                noise[:, s, r, 1] = v.double().square().sum((1, 2))
            continue
        P = torch.bmm(xh, yh.transpose(1, 2).contiguous())
        for c in range(m * n):
            w = float(W[r, c])
            if w != 0:
                l, i = divmod(c, m)
                out[:, i * mp:(i + 1) * mp, l * np_:(l + 1) * np_] += w * P
    if case["kind"] == "product":
        return out
    ref = torch.stack([A[i].double() @ B[i].double() for i in range(b)])
    return {"noise": noise, "reference": ref, "err2": (C.double() - ref).square().sum((1, 2)), "ref2": ref.square().sum((1, 2))}
