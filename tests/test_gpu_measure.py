"""The error measurement at the sizes where its kernels can go wrong: the fp64
reference at the edges of its 64 x 64 tiles and 16-position steps, and the
operand-noise reduction where a term has fewer and more partials than one
workgroup has threads."""
import numpy as np
import pytest

import fmm_inputs as gen
from tests.test_gpu_noise import gpu_noise, oracle_noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 1, 1, 1), (1, 64, 16, 64), (2, 63, 15, 65), (1, 65, 17, 63), (3, 130, 33, 70), (1, 2, 200, 129),
    (2, 66, 0, 62),          # nothing to contract: zeros
    (65, 16, 48, 80),
])
def test_reference_tile_edges(shape):
    """Against numpy's binary64 product.  Both sum K products that binary64
    holds exactly (24-bit factors) with at most K roundings each, so an element
    differs by at most 2 K 2^-53 sum |a| |b|."""
    import torch
    from paper_2609_26077_amd.runner import reference_f64
    b, M, K, N = shape
    A, B = gen.operands("gaussian", b, M, K, N, seed=5, cfg=1)
    C = reference_f64(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()).cpu().numpy()
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    bound = 2 * K * 2.0 ** -53 * (np.abs(A64) @ np.abs(B64))
    assert np.all(np.abs(C - A64 @ B64) <= bound)


@pytest.mark.parametrize("case", [
    (1, 2, 32, 2, 1),           # one partial a term
    (1, 1040, 1024, 130, 1),    # 65 row tiles x 4: 260 partials on the A side
    (2, 516, 1280, 36, 2),      # two levels, ragged tiles
])
def test_noise_partials(case):
    """The sums of non-negative terms, to the relative error of as many
    binary64 additions (well inside 1e-12)."""
    b, M, K, N, depth = case
    bs = 16
    A, B, _, _, _, g = gpu_noise("strassen", "gaussian", b, M, K, N, depth, bs, 1)
    for i in range(b):
        o = oracle_noise(A[i], B[i], "strassen", depth, bs, 1)
        assert np.allclose(g[i], o, rtol=1e-12, atol=0)


def test_noise_of_many_small_products():
    """65 products of a few partials a term (one wave an output, the last
    workgroup partly idle): against the oracle."""
    b, M, K, N, bs = 65, 34, 64, 38, 32
    A, B, _, _, _, g = gpu_noise("strassen", "gaussian", b, M, K, N, 1, bs, 1)
    for i in (0, 31, 64):
        assert np.allclose(g[i], oracle_noise(A[i], B[i], "strassen", 1, bs, 1), rtol=1e-12, atol=0)
