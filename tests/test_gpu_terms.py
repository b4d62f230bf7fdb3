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
