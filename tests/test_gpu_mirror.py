"""Mirrored diagonals (large symmetric stencil matrices of varying coefficients, half of each pair of
entries stored): products and smoothers against the oracle on whole, ragged and stacked grids, and
the matrices that have to keep dense slices."""
import numpy as np
import pytest

import workloads as W
from gpu_util import KINDS, dev, hierarchy, host, nan_vec, oracle_params, relerr, torch_cuda
from oracle import smoothers as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amg():
    torch_cuda()
    import paper_2407_09848_amd as m
    return m


def field(nx, ny, nz, seed):
    return np.exp(np.random.default_rng(seed).standard_normal((nz, ny, nx)))


def q1_varying(nx, ny, nz, seed):
    """27-point matrix D A D of varying coefficients, symmetric in every bit."""
    A = W.q1_27pt(nx, ny, nz)
    d = np.exp2(np.random.default_rng(seed).integers(-2, 3, A.n).astype(np.float64))
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    return W.CSR(A.n, A.row_ptr, A.col, A.val * d[rows] * d[A.col], A.grid)


MATRICES = {
    "whole": (lambda: W.fv_diffusion(field(128, 64, 72, 1)), 1),
    "ragged": (lambda: W.fv_diffusion(field(87, 79, 83, 2)), 1),
    "stacked": (lambda: W.stack_block_diagonal([W.fv_diffusion(field(61, 59, 60, 3 + p)) for p in range(3)]), 3),
    "plane": (lambda: W.fv_diffusion(field(811, 701, 1, 7)), 1),
    "27pt": (lambda: q1_varying(83, 80, 81, 8), 1),
}


def mirrored(amg, h):
    padded, _, aligned = amg.amg_level_layout(h, 0)
    values, patterned, _ = amg.amg_level_patterns(h, 0)
    return aligned and patterned == 0 and values < 0.66 * padded


@pytest.mark.parametrize("name", list(MATRICES))
def test_products_and_smoothers_match_oracle(amg, name):
    # at most 27 products per sum: 27 * 2^-53 of the summed magnitudes per product, a few steps of them
    make, nbatch = MATRICES[name]
    A = make()
    As = A.to_scipy()
    Minv = S.l1_diagonal(As)
    rng = np.random.default_rng(9)
    b, x0 = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    with hierarchy(A, nbatch=nbatch) as h:
        assert mirrored(amg, h)
        y = nan_vec(A.n)
        amg.amg_spmv(h, 0, dev(x0), y)
        assert relerr(host(y), As @ x0) <= 1e-14
        for kind in KINDS:
            for k in (1, 3, 4):
                beta, a = oracle_params(kind, k)
                zero = k != 3
                x = nan_vec(A.n) if zero else dev(x0.copy())
                amg.smoother_apply(h, 0, kind, k, dev(b), x, zero)
                want = S.smooth(As, Minv, b, None if zero else x0, kind, k, beta, a)
                assert relerr(host(x), want) <= 1e-12, (kind, k)


@pytest.mark.parametrize("name", ["ragged", "27pt"])
def test_fp32_smoother(amg, name):
    # float32 recurrences of degree 4: at most 27 products and the updates, each within 2^-24
    torch = torch_cuda()
    A = MATRICES[name][0]()
    As = A.to_scipy()
    b = np.random.default_rng(10).uniform(-1, 1, A.n).astype(np.float32)
    with hierarchy(A, precision=amg.AMG_FP32) as h:
        x = torch.full((A.n,), float("nan"), dtype=torch.float32, device="cuda")
        amg.smoother_apply_f32(h, 0, 2, 4, dev(b), x, True)
        beta, a = oracle_params(2, 4)
        want = S.smooth(As, S.l1_diagonal(As), b.astype(np.float64), None, 2, 4, beta, a)
        assert relerr(host(x), want) <= 4 * 40 * 2.0**-24


@pytest.mark.parametrize("change", ["one_ulp", "missing_entry", "small", "wide_pad"])
def test_other_matrices_keep_dense_slices(amg, change):
    if change == "small":
        A = W.fv_diffusion(field(64, 64, 64, 11))
    elif change == "wide_pad":  # two planes: the offsets reach half the rows
        A = W.fv_diffusion(field(700, 500, 2, 12))
    else:
        A = W.fv_diffusion(field(87, 79, 83, 13))
        row = A.n // 2
        p = A.row_ptr[row]
        while A.col[p] <= row:
            p += 1
        # 0.0: the mirror image of a stored zero is not the entry below the diagonal
        A.val[p] = np.nextafter(A.val[p], 0.0) if change == "one_ulp" else 0.0
    As = A.to_scipy()
    x0 = np.random.default_rng(14).uniform(-1, 1, A.n)
    with hierarchy(A) as h:
        assert not mirrored(amg, h)
        y = nan_vec(A.n)
        amg.amg_spmv(h, 0, dev(x0), y)
        assert relerr(host(y), As @ x0) <= 1e-14


def test_infinity_and_nan_reach_the_rows_of_a_dense_layout(amg):
    """A stacked problem without numbers leaves its neighbours alone, exactly as with dense slices
    (the same pattern with every entry scaled by its own row)."""
    A = MATRICES["stacked"][0]()
    x = np.random.default_rng(15).uniform(-1, 1, A.n)
    x[[0, 5000, A.n // 3 - 1, A.n // 3, 2 * A.n // 3 + 17, A.n - 1]] = [np.inf, np.nan, -np.inf, np.nan, np.inf, np.nan]
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    D = W.CSR(A.n, A.row_ptr, A.col, A.val * (1.0 + rows / A.n), A.grid, A.nbatch)
    got = []
    for M, expect in ((A, True), (D, False)):
        with hierarchy(M, nbatch=3) as h:
            assert mirrored(amg, h) == expect
            y = nan_vec(A.n)
            amg.amg_spmv(h, 0, dev(x), y)
            got.append(host(y))
    assert np.array_equal(np.isnan(got[0]), np.isnan(got[1]))
    assert np.array_equal(np.isinf(got[0]), np.isinf(got[1]))


def test_vectors_at_any_row(amg):
    # vectors that begin 8 bytes past a 16-byte boundary (views into a larger array)
    torch = torch_cuda()
    A = MATRICES["ragged"][0]()
    As = A.to_scipy()
    rng = np.random.default_rng(16)
    b = rng.uniform(-1, 1, A.n)
    with hierarchy(A) as h:
        bv = torch.empty(A.n + 1, dtype=torch.float64, device="cuda")[1:]
        xv = torch.full((A.n + 3,), float("nan"), dtype=torch.float64, device="cuda")[3:]
        bv.copy_(dev(b))
        assert bv.data_ptr() % 16 == 8 and xv.data_ptr() % 16 == 8
        amg.smoother_apply(h, 0, 2, 4, bv, xv, True)
        beta, a = oracle_params(2, 4)
        assert relerr(host(xv), S.smooth(As, S.l1_diagonal(As), b, None, 2, 4, beta, a)) <= 1e-12
