"""The sub-product kernels of the fused plans at the sizes where their dispatch
changes: gemm_terms_kernel (one wave per inner term) on 32- and 64-edge tiles
in both layouts and all its operand forms, with the edges of tiles, steps and
blocks; and gemm_tile128_kernel / gemm_mx_kernel from the tile counts on that
they are given.  Codes, scales, every element of C against its dot-product
bound, and the relative MSE, against the oracle."""
import pytest

from tests.gpu_helpers import check_case

pytestmark = pytest.mark.gpu

ROWS, TILED = 0, 2


@pytest.mark.parametrize("bs,rule,exact", [(16, 0, False), (32, 0, False), (128, 0, False), (16, 1, False), (32, 1, False),
                                           (32, 2, False), (128, 1, False), (32, 1, True), (32, 2, True), (128, 1, True)])
@pytest.mark.parametrize("shape", [
    (1, 66, 62, 1),      # one row or column past a tile, K one block
    (3, 2, 190, 3),      # a single row of a tile
    (1, 194, 130, 9),    # K past one 128-byte step, odd number of blocks
])
def test_rows_small(bs, rule, exact, shape):
    b, M, N, kb = shape
    check_case("tstar", "gaussian", b, M, 2 * kb * bs, N, 1, bs, rule, seed=31, cfg=2, exact=exact,
               ns=exact and M * N > 16, layout=ROWS)


@pytest.mark.parametrize("bs,rule,exact", [(16, 0, False), (32, 0, False), (128, 0, False), (16, 1, False),
                                           (32, 1, False), (32, 1, True), (128, 1, False), (128, 1, True)])
def test_rows_64_edge(bs, rule, exact):
    """More than 560 tiles of 32 x 32: 25 x 24 of them, the last ones one row
    and one column wide, K one block past a step."""
    check_case("strassen", "gaussian", 1, 2 * 769, 2 * (128 + bs), 2 * 737, 1, bs, rule, seed=32, cfg=2, exact=exact,
               layout=ROWS)


@pytest.mark.parametrize("bs,exact", [(16, True), (32, False), (32, True), (128, False), (128, True)])
@pytest.mark.parametrize("shape", [
    (1, 256, 512, 512),     # 32-edge tiles, two steps
    (1, 1792, 256, 1792),   # 64-edge tiles (784 of 32), one step
    (1, 2304, 768, 2304),   # 81 tiles of 128 x 128: past a third of the chip
])
def test_tiled(bs, exact, shape):
    b, M, K, N = shape
    check_case("tstar", "gaussian", b, M, K, N, 1, bs, 1, seed=33, cfg=2, exact=exact, layout=TILED)


@pytest.mark.parametrize("depth", [2, 3])
@pytest.mark.parametrize("bs,rule,exact", [(32, 1, False), (32, 1, True), (16, 0, False)])
def test_outer_terms_and_eight_terms(depth, bs, rule, exact):
    """Eight inner terms (every wave works) and several outer ones."""
    n = 2 ** depth
    check_case("cubic8", "gaussian", 2, 33 * n, 48 * n if bs == 16 else 96 * n, 34 * n, depth, bs, rule, seed=34, cfg=2,
               exact=exact, layout=ROWS)


@pytest.mark.parametrize("bs", [32, 128])
def test_mx_rows_full_rounds(bs):
    """224 row-layout tiles of 128 x 128 fill seven eighths of the chip: the
    fp8 plan takes gemm_mx_kernel, on ragged edges of both sides."""
    check_case("strassen", "gaussian", 1, 2 * (15 * 128 + 5), 2 * (bs + 128), 2 * (13 * 128 + 7), 1, bs, 1, seed=35, cfg=2,
               layout=ROWS)


@pytest.mark.parametrize("case", [
    (1, 4096, 2048, 4096, 2),     # one full round of 128 x 128 tiles, k' = 1024: fused
    (1, 4096, 4096, 4096, 2),     # k' = 2048: fused
    (3, 2048, 2048, 2048, 2),     # 192 tiles: fused
    (1, 3072, 3072, 3072, 1),     # 144 tiles: large tiles
    (1, 4096, 8192, 4096, 1),     # k' = 4096: large tiles
])
@pytest.mark.parametrize("exact", [False, True])
def test_fused_or_large_tiles(case, exact):
    """Depth 1 from k' = 1024 on: which path a plan takes, and that C is the
    large tiles' bit for bit (both sum a term's products in the same order and
    add the terms in ascending order by one fused multiply-add)."""
    import torch
    from paper_2609_26077_amd import FMM_FLAG_LARGE_TILE, fmm_operand_views
    from paper_2609_26077_amd.runner import FMM
    b, M, K, N, layout = case
    g = torch.Generator(device="cuda").manual_seed(7)
    A = torch.randn((b, M, K), generator=g, device="cuda")
    B = torch.randn((b, K, N), generator=g, device="cuda")
    f = FMM("tstar", b, M, K, N, 1, 32, "pow2_ceil", exact_dot=exact)
    assert fmm_operand_views(f.plan, f.ws)[0].code_layout == layout
    large = FMM("tstar", b, M, K, N, 1, 32, "pow2_ceil", exact_dot=exact, flags=FMM_FLAG_LARGE_TILE)
    assert fmm_operand_views(large.plan, large.ws)[0].code_layout == 1
    assert torch.equal(f.matmul(A, B), large.matmul(A, B))


@pytest.mark.parametrize("case", [
    # (depth, bs, rule, M, K, N): one launch for both sides; uneven numbers of
    # workgroups on the two sides, tiles that end partway in rows and positions
    (1, 16, 0, 34, 160, 2), (1, 32, 1, 2, 192, 74), (1, 128, 2, 18, 768, 66), (1, 128, 0, 258, 256, 2),
    (2, 16, 1, 36, 192, 4), (2, 32, 0, 4, 384, 68), (2, 128, 1, 40, 512, 36),
])
def test_encode_one_launch(case):
    depth, bs, rule, M, K, N = case
    check_case("winograd", "gaussian", 2, M, K, N, depth, bs, rule, seed=36, cfg=2, exact=True)


def test_encode_two_launches():
    """192 MiB of operands and more go to one launch per side: the same codes
    and scales as two products of half the rows of A each (a row's codes depend
    on that row alone; half the operands of A, one launch)."""
    import torch
    from paper_2609_26077_amd.runner import FMM
    g = torch.Generator(device="cuda").manual_seed(8)
    A = torch.randn((1, 12288, 4096), generator=g, device="cuda")
    B = torch.randn((1, 4096, 512), generator=g, device="cuda")
    whole = FMM("tstar", 1, 12288, 4096, 512, 1, 32, "pow2_ceil")
    whole.encode(A, B)
    codes, scales, bcodes, bscales = whole.operands()
    h = 6144 // 2
    for i in range(2):
        # rows h i .. of both row blocks of A's grid
        Ai = torch.cat([A[:, h * i:h * (i + 1)], A[:, 6144 + h * i:6144 + h * (i + 1)]], 1).contiguous()
        half = FMM("tstar", 1, 6144, 4096, 512, 1, 32, "pow2_ceil")
        half.encode(Ai, B)
        c, s, bc, bs = half.operands()
        assert torch.equal(c, codes[:, :, h * i:h * (i + 1)]) and torch.equal(s, scales[:, :, h * i:h * (i + 1)])
        assert torch.equal(bc, bcodes) and torch.equal(bs, bscales)


@pytest.mark.parametrize("block, rule, batch", [(128, "fp32_amax", 4), (32, "pow2_ceil", 14), (16, "fp32_amax", 14)])
def test_shape_encode_launches(block, rule, batch):
    """<2,2,3;12> batches past 32 MiB (block 128) and 128 MiB of operands take
    one launch per side on the depth-1 tiles, their products alone one launch
    for both on the sixteen-wave tiles: the same codes, scales and C."""
    import numpy as np
    import torch
    import paper_2609_26077_amd as fm
    from paper_2609_26077_amd.runner import FMM
    U, V, W = np.zeros((12, 4)), np.zeros((12, 6)), np.zeros((12, 6))
    for r in range(12):
        i, j, l = r // 6, r // 3 % 2, r % 3
        U[r, 2 * i + j] = V[r, 3 * j + l] = W[r, 2 * l + i] = 1.0
    # a change of basis fills the rows, so that every block is combined
    gauge = [np.array([[1.0, 0.3], [-0.2, 0.9]]), np.array([[0.8, -0.4], [0.1, 1.1]]),
             np.array([[1.0, 0.2, -0.1], [0.3, 0.9, 0.2], [-0.2, 0.1, 1.2]])]
    real = fm.fmm_realization_transform(fm.fmm_realization_create(U, V, W, shape=(2, 2, 3)), *gauge)
    g = torch.Generator(device="cuda").manual_seed(9)
    A = torch.randn((batch, 1024, 1024), generator=g, device="cuda")
    B = torch.randn((batch, 1024, 1536), generator=g, device="cuda")
    whole = FMM(real, batch, 1024, 1024, 1536, 1, block, rule)
    C = whole.matmul(A, B)
    ops = whole.operands()
    alone = FMM(real, 1, 1024, 1024, 1536, 1, block, rule)
    for b in (0, batch - 1):
        Cb = alone.matmul(A[b:b + 1], B[b:b + 1])
        assert torch.equal(Cb[0], C[b])
        assert all(torch.equal(x[0], y[b]) for x, y in zip(alone.operands(), ops))


@pytest.mark.parametrize("depth, block", [(1, 16), (1, 128), (2, 32), (3, 32)])
@pytest.mark.parametrize("exponent", [-30, 0, 100])
def test_fp32_scale_quotients(depth, block, exponent):
    """fp32 scales, numerators within 4 ulp of every boundary between two codes
    times the scale, signed, zeros of both signs and subnormals among them:
    the codes of the correctly rounded quotient (numpy's division), exactly."""
    import numpy as np
    import torch
    from paper_2609_26077_amd.runner import FMM
    rng = np.random.RandomState(11)
    n, rows, kp = 1 << depth, 64, 1024
    nb = kp // block
    amax = np.ldexp(rng.uniform(1, 2, (rows, nb, 1)), exponent).astype(np.float32)
    s = amax / np.float32(448)
    tie = np.concatenate([np.arange(17, 32, 2) / 16 * 2.0 ** e for e in range(-6, 9)] + [np.arange(1, 16, 2) * 2.0 ** -10])
    x = (rng.choice(tie, (rows, nb, block)) * s).astype(np.float32)
    x = (x.view(np.int32) + rng.randint(-4, 5, x.shape).astype(np.int32)).view(np.float32)
    x = np.minimum(x, amax) * rng.choice([-1, 1], x.shape).astype(np.float32)
    x[:, :, 1] = 0.0
    x[:, :, 2] = -0.0
    x[:, :, 3] = np.float32(1e-45)
    x[:, :, 4] = np.float32(-1e-45)
    x[:, :, 0] = amax[:, :, 0]
    want = torch.from_numpy(np.clip(x / s, np.float32(-448), np.float32(448))).to(torch.float8_e4m3fn).view(torch.uint8)
    want = want.reshape(rows, kp).numpy()
    # the cubic algorithm's terms are the sub-blocks themselves: all alike
    A = torch.from_numpy(np.ascontiguousarray(np.tile(x.reshape(rows, kp), (n, n))))[None].cuda()
    B = torch.from_numpy(np.ascontiguousarray(np.tile(x.reshape(rows, kp).T, (n, n))))[None].cuda()
    f = FMM("cubic8", 1, n * rows, n * kp, n * rows, depth, block, "fp32_amax")
    f.encode(A, B)
    for codes, scales in (f.operands()[:2], f.operands()[2:]):
        assert (scales.cpu().numpy() == s[..., 0]).all()
        assert (codes.cpu().numpy() == want).all()


@pytest.mark.parametrize("block, rule", [(32, "pow2_ceil"), (16, "fp32_amax"), (128, "pow2_ocp")])
@pytest.mark.parametrize("change", ["none", "order", "sign", "pair", "magnitude", "half"])
@pytest.mark.parametrize("name", ["strassen", "tstar"])
def test_depth3_patterns(name, change, block, rule):
    """The depth-3 encoder by its tables' sign and magnitude pattern: T* and
    Strassen, their terms in another order, and tables that miss the patterns
    by one term's sign, two terms' signs, a magnitude, or (halved on one
    side, doubled on the other) by an exact power of two: codes and scales
    against the oracle's."""
    import numpy as np
    import torch
    import fmm_inputs as gen
    import paper_2609_26077_amd as fm
    from oracle import e4m3, fmm
    from paper_2609_26077_amd.runner import FMM
    U, V, W = fm.fmm_realization_coefficients(fm.fmm_realization_builtin(name))
    if change == "order":
        p = [4, 6, 0, 2, 1, 5, 3]
        U, V, W = U[p], V[p], W[p]
    elif change == "sign":
        U[5], W[5] = -U[5], -W[5]
    elif change == "pair":
        for r in (1, 6):
            U[r], V[r] = -U[r], -V[r]
    elif change == "magnitude":
        U[2], V[2] = 3 * U[2], V[2] / 3
    elif change == "half":
        U[0], V[0] = U[0] / 2, 2 * V[0]
    real = fm.fmm_realization_create(U, V, W)
    M, K, N = 8 * 18, 8 * 160 if block < 128 else 8 * 256, 8 * 10
    A, B = gen.operands("gaussian", 1, M, K, N, seed=0, cfg=37)
    A[0, 5] = 0.0
    f = FMM(real, 1, M, K, N, 3, block, rule)
    f.encode(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda())
    ac, asc, bc, bsc = [t.cpu().numpy()[0] for t in f.operands()]
    rules = {"fp32_amax": e4m3.RULE_FP32_AMAX, "pow2_ceil": e4m3.RULE_POW2_CEIL, "pow2_ocp": e4m3.RULE_POW2_OCP}
    tables = fm.fmm_realization_tables(real, 3)
    for side, X, T, codes, scales in (("A", A[0], tables[0], ac, asc), ("B", B[0], tables[1], bc, bsc)):
        e = fmm.encode_side(X, T, 3, block, rules[rule], side)
        assert np.array_equal(codes, e["codes"]), side
        assert np.array_equal(scales, e["scales"]), side


@pytest.mark.parametrize("case", [
    # (block, rule, bf16, M, K, N): the 128-row scale blocks' workgroups of 128
    # columns x 64 (blocks 16, 32) or 128 positions: one position run short of a
    # tile, one column in the last block, a whole block, several of each
    (16, 1, False, 34, 160, 2), (16, 0, True, 66, 96, 258), (32, 2, True, 34, 192, 256), (32, 0, False, 256, 448, 254),
    (128, 1, True, 34, 256, 130), (128, 0, False, 130, 768, 384),
])
def test_weight_blocks(case):
    bs, rule, bf16, M, K, N = case
    check_case("winograd", "student_t3", 2, M, K, N, 1, bs, rule, seed=38, cfg=2, exact=True, b_rows=128, b_bf16=bf16,
               ns=False)


def test_more_workgroups_than_one_launch_takes():
    """43691 products of 64 outer terms x three 32-edge tiles are 8388672
    workgroups of gemm_terms_kernel, whose 2^32 + 2^15 threads are more than
    one launch's axis holds: products at both ends and in between are those of
    a plan of one product, bit for bit.  (The last product is the one that two
    launches share.)"""
    import torch
    from paper_2609_26077_amd.runner import FMM
    batch, M, K, N = 43691, 8, 128, 520
    g = torch.Generator(device="cuda").manual_seed(12)
    A = torch.randn((batch, M, K), generator=g, device="cuda")
    B = torch.randn((batch, K, N), generator=g, device="cuda")
    C = FMM("cubic8", batch, M, K, N, 3, 16, "pow2_ceil").matmul(A, B)
    one = FMM("cubic8", 1, M, K, N, 3, 16, "pow2_ceil")
    for b in (0, batch // 2, batch - 2, batch - 1):
        assert torch.equal(one.matmul(A[b:b + 1], B[b:b + 1])[0], C[b]), b
    del A, B, C
    torch.cuda.empty_cache()


@pytest.mark.parametrize("case", [
    # (depth, block, rule, batch, M, K, N, cubic shape): batches past a bound on the
    # shared encode launch, whose products alone are within it
    (2, 32, "pow2_ceil", 140, 512, 512, 512, None),        # 256 MiB of 2 MiB products at depth 2
    (2, 128, "fp32_amax", 65, 1024, 2048, 1024, None),     # 1 GiB of 16 MiB products
    (1, 128, "fp32_amax", 81, 124, 512, 36, None),         # 1280 of A's tiles at block 128 (1296)
    (1, 32, "pow2_ceil", 700, 100, 64, 18, None),          # 4608 of them at blocks 16 and 32 (4900)
    (1, 128, "pow2_ocp", 7, 768, 768, 768, (3, 1, 3)),     # 1024 tiles where a side has fewer than four blocks
    (1, 16, "fp32_amax", 15, 256, 512, 1024, (1, 2, 4)),   # 1792 of them at blocks 16 and 32
])
def test_encode_launches(case):
    """Codes and scales of a batch that takes one encode launch per side are
    those of its products alone, which take one for both."""
    import numpy as np
    import torch
    import paper_2609_26077_amd as fm
    from paper_2609_26077_amd.runner import FMM
    depth, block, rule, batch, M, K, N, shape = case
    real = "winograd"
    if shape is not None:
        m, k, n = shape
        t = [(i, j, l) for i in range(m) for j in range(k) for l in range(n)]
        U, V, W = np.zeros((len(t), m * k)), np.zeros((len(t), k * n)), np.zeros((len(t), n * m))
        for r, (i, j, l) in enumerate(t):
            U[r, i * k + j] = V[r, j * n + l] = W[r, l * m + i] = 1.0
        real = fm.fmm_realization_create(U, V, W, shape=shape)
    g = torch.Generator(device="cuda").manual_seed(13)
    A = torch.randn((batch, M, K), generator=g, device="cuda")
    B = torch.randn((batch, K, N), generator=g, device="cuda")
    whole = FMM(real, batch, M, K, N, depth, block, rule)
    whole.encode(A, B)
    alone = FMM(real, 1, M, K, N, depth, block, rule)
    for b in (0, batch // 2, batch - 1):
        alone.encode(A[b:b + 1], B[b:b + 1])
        assert all(torch.equal(x[0], y[b]) for x, y in zip(alone.operands(), whole.operands()))


@pytest.mark.parametrize("M,N", [(34, 38), (1538, 1474)])
@pytest.mark.parametrize("block", [16, 32, 128])
def test_rows_exact_dot_sums_blocks_apart(block, M, N):
    """Exact-dot products in the row layout sum each block (at block 16 each
    two) by itself: beside a first sum of 2^12, forty sums of 2^-11 (the last
    bit of the whole) made of equal products.  Every partial sum is exact in
    fp32, so C is; accumulated one matrix instruction after the other, the
    products below the sum's last bit would be truncated away."""
    import torch
    from paper_2609_26077_amd.runner import FMM
    span = max(block, 32)
    kp = 41 * span
    a, b = 2.0 ** -8, 2.0 ** -3 / span
    A, B = torch.zeros((1, M, 2 * kp)), torch.zeros((1, 2 * kp, N))
    A[:, :, span:kp], B[:, span:kp] = a, b
    A[:, :, 0], B[:, 0] = 64.0, 64.0
    f = FMM("cubic8", 1, M, 2 * kp, N, 1, block, "pow2_ceil", exact_dot=True)
    C = f.matmul(A.cuda(), B.cuda())
    assert (C == 2.0 ** 12 + 40 * 2.0 ** -11).all()


@pytest.mark.parametrize("name,case", [
    # (M, K, N, block, rule, exact, flags)
    ("gemm_terms_kernel 32x32", (256, 256, 256, 32, "pow2_ceil", False, 0)),
    ("gemm_terms_kernel 64x64", (1792, 256, 1792, 32, "pow2_ceil", True, 0)),
    ("gemm_tile128_kernel 128x128", (2304, 768, 2304, 32, "pow2_ceil", False, 0)),
    ("gemm_mx_kernel 128x128", (3850, 256, 3342, 128, "pow2_ceil", False, 0)),
    ("gemm_tile256x256_kernel 256x256", (512, 512, 512, 32, "pow2_ceil", False, 8)),
    ("gemm_dq256x128_kernel 256x128", (512, 512, 512, 16, "pow2_ceil", False, 8)),
    ("gemm_exact128x128_kernel 128x128", (512, 512, 512, 32, "fp32_amax", False, 0)),
])
def test_products_kernel_is_named(name, case):
    from paper_2609_26077_amd import fmm_products_kernel
    from paper_2609_26077_amd.runner import FMM
    M, K, N, block, rule, exact, flags = case
    assert fmm_products_kernel(FMM("tstar", 1, M, K, N, 1, block, rule, exact_dot=exact, flags=flags).plan) == name


EDGE64, TILE128 = "gemm_terms_kernel 64x64", "gemm_%s_kernel 128x128"


@pytest.mark.parametrize("bs,rule,exact,case", [
    # 256 tiles of 64 x 64, the last ones one row and one column wide, K one block past a step
    (bs, rule, exact, (EDGE64, 1, 1, 1922, 2 * (128 + bs), 1922))
    for bs, rule, exact in [(16, 0, False), (32, 0, False), (128, 0, False), (16, 1, False), (32, 1, False), (32, 1, True),
                            (128, 1, False), (128, 1, True)]] + [
    # tiles of 128 x 128 that fill seven eighths of the chip, one step and three; at depth 2 one
    # tile a product, over outer terms and products
    (128, rule, exact, (TILE128 % kernel, *sizes))
    for rule, exact, kernel in [(1, False, "mx"), (1, True, "promote"), (0, False, "promote")]
    for sizes in [(1, 1, 3850, 256, 3342), (1, 1, 3850, 768, 3342), (2, 36, 500, 512, 496)]])
def test_row_layout_dispatch(bs, rule, exact, case):
    """Which kernel a row-layout plan's products take, and its results."""
    from paper_2609_26077_amd import fmm_products_kernel
    from paper_2609_26077_amd.runner import FMM
    kernel, depth, batch, M, K, N = case
    f = FMM("strassen", batch, M, K, N, depth, bs, rule, exact_dot=exact)
    assert fmm_products_kernel(f.plan) == kernel
    check_case("strassen", "gaussian", batch, M, K, N, depth, bs, rule, seed=39, cfg=2, exact=exact, layout=ROWS,
               check_every=35 if batch > 1 else None)


@pytest.mark.parametrize("case", [
    (11, 5632, 6144, 512, 16), (1, 3072, 4096, 4096, 16), (1, 5120, 2304, 4608, 32), (1, 7168, 5120, 1536, 128),
])
def test_exact_dot_takes_the_large_tiles(case):
    """Exact-dot products at depth 1 and k' >= 1024 on which the fused kernel was
    measured 15 to 26% slower than the large tiles and their W-combine pass."""
    from paper_2609_26077_amd import fmm_products_kernel
    from paper_2609_26077_amd.runner import FMM
    batch, M, K, N, block = case
    f = FMM("tstar", batch, M, K, N, 1, block, "pow2_ceil", exact_dot=True)
    assert fmm_products_kernel(f.plan) == "gemm_dq256x128_kernel 256x128"


@pytest.mark.parametrize("bs,rule,bf16", [(128, "fp32_amax", True), (32, "pow2_ceil", False)])
@pytest.mark.parametrize("batch", [30, 70, 300])
def test_weight_blocks_over_workgroups(batch, bs, rule, bf16):
    """A tile's terms over seven workgroups (one product), fewer and one (300):
    the same codes and scales."""
    import torch
    import paper_2609_26077_amd as fm
    from paper_2609_26077_amd.runner import FMM
    flags = fm.FMM_FLAG_B_BLOCK128 | (fm.FMM_FLAG_B_BF16 if bf16 else 0)
    g = torch.Generator(device="cuda").manual_seed(14)
    A = torch.randn((batch, 34, 256), generator=g, device="cuda")
    B = torch.randn((batch, 256, 70), generator=g, device="cuda")
    whole, one = (FMM("tstar", b, 34, 256, 70, 1, bs, rule, flags=flags) for b in (batch, 1))
    whole.encode(A, B)
    for b in (0, batch // 2, batch - 1):
        one.encode(A[b:b + 1], B[b:b + 1])
        assert all(torch.equal(x[0], y[b]) for x, y in zip(one.operands(), whole.operands()))


@pytest.mark.parametrize("depth,block,flags", [(1, 16, 0), (1, 128, 0), (2, 32, 0), (3, 32, 0), (1, 128, 2), (1, 32, 6)])
def test_fp32_scales_of_overflowing_combinations(depth, block, flags):
    """Finite operands whose combination overflows binary32: its block's scale
    is infinite, its finite values' codes zeros, and every other block as if
    the overflowing values were not there."""
    import torch
    from paper_2609_26077_amd.runner import FMM
    n = 1 << depth
    M, K, N = 160 * n, 384 * n, 160 * n
    g = torch.Generator(device="cuda").manual_seed(15)
    A = torch.randn((1, M, K), generator=g, device="cuda")
    B = torch.randn((1, K, N), generator=g, device="cuda")
    f = FMM("strassen", 1, M, K, N, depth, block, "fp32_amax", flags=flags)
    f.encode(A, B)
    plain = [t[0] for t in f.operands()]
    # position (row 5, k 130) of every sub-block of A, (k 130, column 5) of B
    A.view(n, 160, n, 384)[:, 5, :, 130] = 3e38
    B.view(n, 384, n, 160)[:, 130, :, 5] = 3e38
    f.encode(A, B)
    rows = {0: slice(5, 6), 1: slice(0, 128) if flags & 2 else slice(5, 6)}
    kb = 130 // block
    for side in (0, 1):
        codes, scales = (t[0] for t in f.operands()[2 * side:2 * side + 2])
        pc, ps = plain[2 * side:2 * side + 2]
        terms = torch.isinf(scales[:, 5, kb])
        assert terms.any() and not torch.isnan(scales).any()
        hit = torch.zeros_like(scales, dtype=torch.bool)
        hit[:, rows[side], kb] = True
        assert torch.equal(scales[~hit], ps[~hit])
        wide = hit.repeat_interleave(block, dim=2)
        assert torch.equal(codes[~wide], pc[~wide])
        over = codes[terms][:, rows[side], kb * block:(kb + 1) * block].clone()
        assert (scales[terms][:, rows[side], kb] == float("inf")).all()
        assert (over[:, 5 - rows[side].start, 130 - kb * block] & 0x7F == 0x7E).all()
        over[:, 5 - rows[side].start, 130 - kb * block] = 0
        assert (over & 0x7F == 0).all()


@pytest.mark.parametrize("block", [16, 32, 128])
@pytest.mark.parametrize("M,N", [(34, 38), (1538, 1474)])
def test_rows_fp32_infinite_scales(block, M, N):
    """An infinite scale of either side (a combination that overflowed) reaches
    the elements of C that the definition's sums of sA sB times block products
    give it: infinite where the sum is, NaN where an infinite product is of
    zero or meets its opposite."""
    import numpy as np
    import torch
    import paper_2609_26077_amd as fm
    from paper_2609_26077_amd.runner import FMM
    K = 2 * 3 * block
    m, n = M // 2, N // 2
    g = torch.Generator(device="cuda").manual_seed(16)
    A = torch.randn((1, M, K), generator=g, device="cuda")
    B = torch.randn((1, K, N), generator=g, device="cuda")
    A.view(2, m, 2, K // 2)[:, 3, :, 5] = 3e38
    B.view(2, K // 2, 2, n)[:, block + 2, :, 7] = 3e38
    f = FMM("strassen", 1, M, K, N, 1, block, "fp32_amax")
    C = f.matmul(A, B)[0]
    ac, asc, bc, bsc = (t[0] for t in f.operands())
    W = fm.fmm_realization_tables(f.real, 1)[2]
    want = torch.zeros((M, N), device="cuda")
    for r in range(7):
        P = torch.zeros((m, n), device="cuda")
        for k in range(3):
            x = ac[r, :, k * block:(k + 1) * block].contiguous().view(torch.float8_e4m3fn).double()
            y = bc[r, :, k * block:(k + 1) * block].contiguous().view(torch.float8_e4m3fn).double()
            S = (asc[r, :, k][:, None] * bsc[r, :, k][None]).double()
            P = (P.double() + S * (x @ y.T.contiguous())).float()        # one rounding, as a fused multiply-add
        for q in np.flatnonzero(W[r]):
            want[(q & 1) * m:(q & 1) * m + m, (q >> 1) * n:(q >> 1) * n + n] += float(W[r, q]) * P
    assert torch.isinf(want).any() and torch.isnan(want).any()
    for kind in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(kind(C), kind(want))
