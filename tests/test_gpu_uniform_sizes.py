"""Uniform slices at the row counts where a level's form or kernels change: small FP64 levels, FP32 levels of
27 points, restriction products; and patterns of every number of steps modulo a batch."""
import numpy as np
import pytest

import workloads as W
from gpu_util import dev, hierarchy, host, nan_vec, oracle_params, relerr, torch_cuda
from oracle import amg as OA
from oracle import smoothers as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amg():
    torch_cuda()
    import paper_2407_09848_amd as m
    return m


def line(n, half):
    """Constant band: 2 half + 1 entries per row."""
    import scipy.sparse as sp

    B = sp.diags([np.full(n - k, -1.0 / (k + 1)) for k in range(1, half + 1)], list(range(1, half + 1)))
    M = (B + B.T + sp.identity(n) * 8.0).tocsr()
    M.sort_indices()
    return W.CSR(n, M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data, (n, 1, 1))


@pytest.mark.parametrize("grid", [(47, 32, 64), (48, 32, 64), (49, 32, 64)])
def test_fp64_smoother_around_the_small_levels_limit(amg, grid):
    # 27 products per sum and a few steps of them: 1e-12 as for every other layout
    A = W.q1_27pt(*grid)
    As = A.to_scipy()
    rng = np.random.default_rng(41)
    b, x0 = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    with hierarchy(A) as h:
        assert amg.amg_level_patterns(h, 0)[1] > 0
        for zero in (True, False):
            beta, a = oracle_params(2, 4)
            x = nan_vec(A.n) if zero else dev(x0.copy())
            amg.smoother_apply(h, 0, 2, 4, dev(b), x, zero)
            assert relerr(host(x), S.smooth(As, S.l1_diagonal(As), b, None if zero else x0, 2, 4, beta, a)) <= 1e-12


@pytest.mark.parametrize("grid,patterns", [((20, 21, 22), False), ((63, 64, 64), False), ((64, 64, 64), True),
                                           ((65, 64, 64), True)])
def test_fp32_levels_of_27_points(amg, grid, patterns):
    # float32 recurrences of degree 4: 27 products and the updates, each within 2^-24, four steps
    torch = torch_cuda()
    A = W.q1_27pt(*grid)
    As = A.to_scipy()
    b = np.random.default_rng(42).uniform(-1, 1, A.n).astype(np.float32)
    with hierarchy(A, precision=amg.AMG_FP32) as h:
        assert (amg.amg_level_patterns(h, 0)[1] > 0) == patterns
        x = torch.full((A.n,), float("nan"), dtype=torch.float32, device="cuda")
        amg.smoother_apply_f32(h, 0, 2, 4, dev(b), x, True)
        beta, a = oracle_params(2, 4)
        want = S.smooth(As, S.l1_diagonal(As), b.astype(np.float64), None, 2, 4, beta, a)
        assert relerr(host(x), want) <= 4 * 40 * 2.0**-24


@pytest.mark.parametrize("grid,patterns", [((72, 72, 75), False), ((72, 72, 76), True)])
@pytest.mark.parametrize("points", [7, 27])
def test_restriction_products(amg, points, grid, patterns):
    A = (W.poisson3d_7pt if points == 7 else W.q1_27pt)(*grid)
    As = A.to_scipy()
    rng = np.random.default_rng(43)
    b, x = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    agg, _ = OA.box_aggregates(A.grid)
    with hierarchy(A) as h:
        assert amg.amg_level_transfer(h, 0)[0] == amg.AMG_TRANSFER_PRODUCT
        assert (amg.amg_level_patterns(h, 0, True)[1] > 0) == patterns
        bc = nan_vec(int(agg.max()) + 1)
        amg.amg_restrict_residual(h, 0, dev(b), dev(x), bc)
        # 64 products per row, as the tests of the products
        assert relerr(host(bc), np.bincount(agg, weights=b - As @ x)) <= 1e-12


@pytest.mark.parametrize("half", list(range(1, 14)) + [16, 20, 31])
def test_patterns_of_any_length(amg, half):
    # at most 63 products per sum
    A = line(700, half)
    As = A.to_scipy()
    x = np.random.default_rng(44).uniform(-1, 1, A.n)
    b = As @ x
    for prec in (amg.AMG_FP64, amg.AMG_FP32):
        with hierarchy(A, precision=prec, max_coarse=A.n) as h:
            padded, lanes, aligned = amg.amg_level_layout(h, 0)
            dense = prec == amg.AMG_FP32 and half in (13, 16, 31)  # 27, 33 and 63 steps: wide triples
            assert lanes == 1 and aligned and (amg.amg_level_patterns(h, 0)[1] == 0) == dense
            y = nan_vec(A.n)
            amg.amg_spmv(h, 0, dev(x), y)
            assert relerr(host(y), b) <= 1e-14
            if prec == amg.AMG_FP32:
                torch = torch_cuda()
                z = torch.full((A.n,), float("nan"), dtype=torch.float32, device="cuda")
                amg.smoother_apply_f32(h, 0, 2, 2, dev(b.astype(np.float32)), z, True)
                beta, a = oracle_params(2, 2)
                want = S.smooth(As, S.l1_diagonal(As), b.astype(np.float32).astype(np.float64), None, 2, 2, beta, a)
                assert relerr(host(z), want) <= 2 * 80 * 2.0**-24
