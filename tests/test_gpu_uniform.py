"""Uniform slices (matrices whose 64-row slices hold one value or +0 per step, kept as patterns):
the products, smoothers, transfers and cycles on them against the oracle, where slices cross grid
lines, the last slice is short, and some slices stay dense."""
import numpy as np
import pytest

import workloads as W
from gpu_util import KINDS, dev, hierarchy, host, nan_vec, oracle_params, relerr, torch_cuda
from oracle import amg as OA
from oracle import smoothers as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amg():
    torch_cuda()
    import paper_2407_09848_amd as m
    return m


def two_materials(nx, ny, nz):
    """7-point diffusion with conductivity 1 below and 8 above the middle plane: the slices that
    cross the interface's planes stay uniform or not with the shape, the diagonal has four values."""
    kappa = np.ones((nz, ny, nx))
    kappa[nz // 2:] = 8.0
    kappa[:, :, : max(1, nx // 8)] = 3.0
    return W.fv_diffusion(kappa)


MATRICES = {
    "7pt_whole_slices": lambda: W.poisson3d_7pt(64, 8, 6),
    "7pt_crossing": lambda: W.poisson3d_7pt(37, 23, 19),
    "27pt_whole_slices": lambda: W.q1_27pt(128, 6, 7),
    "27pt_crossing": lambda: W.q1_27pt(71, 13, 11),
    "27pt_short_tail": lambda: W.q1_27pt(9, 11, 13),
    "5pt": lambda: W.poisson2d_5pt(64, 64),
    "9pt_natural_ends": lambda: W.anisotropy2d_q1(300)[0],  # the line ends have values of their own
    "one_line": lambda: W.poisson3d_7pt(130, 1, 1),
    "two_materials": lambda: two_materials(256, 12, 10),
}


@pytest.mark.parametrize("name", list(MATRICES))
def test_products_and_cycles_match_oracle(amg, name):
    # sums of at most 27 products (64 in the restriction product) in double: rounding is below
    # 64 * 2^-53 of the summed magnitudes, 1e-12 as for every other layout through a whole cycle
    torch = torch_cuda()
    A = MATRICES[name]()
    As = A.to_scipy()
    Minv = S.l1_diagonal(As)
    rng = np.random.default_rng(5)
    b, x0 = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    H = OA.build_hierarchy(As, A.grid, max_coarse=100)
    with hierarchy(A, max_coarse=100) as h:
        values, patterned, steps = amg.amg_level_patterns(h, 0)
        slices = (A.n + 63) // 64
        assert 2 * patterned >= slices, (patterned, slices)
        if name == "two_materials":
            assert patterned < slices and values > 0
        assert steps <= 27 * patterned
        y = nan_vec(A.n)
        amg.amg_spmv(h, 0, dev(x0), y)
        assert relerr(host(y), As @ x0) <= 1e-14
        for kind in KINDS:
            for k in (1, 4):
                beta, a = oracle_params(kind, k)
                for zero in (True, False):
                    x = nan_vec(A.n) if zero else dev(x0.copy())
                    amg.smoother_apply(h, 0, kind, k, dev(b), x, zero)
                    want = S.smooth(As, Minv, b, None if zero else x0, kind, k, beta, a)
                    assert relerr(host(x), want) <= 1e-12, (kind, k, zero)
        z = nan_vec(A.n)
        amg.vcycle_apply(h, 2, 4, dev(b), z)
        torch.cuda.synchronize()
        beta, a = oracle_params(2, 4)
        assert relerr(host(z), OA.vcycle(H, b, 2, 4, beta)) <= 1e-12
        if len(H.levels) > 1:
            bc = nan_vec(H.levels[1].A.shape[0])
            amg.amg_restrict_residual(h, 0, dev(b), dev(x0), bc)
            assert relerr(host(bc), H.levels[0].P.T @ (b - As @ x0)) <= 1e-12


def test_few_uniform_slices_stay_dense(amg):
    rng = np.random.default_rng(6)
    A = W.fv_diffusion(np.exp(rng.standard_normal((9, 10, 64))))
    with hierarchy(A) as h:
        padded, _, aligned = amg.amg_level_layout(h, 0)
        assert aligned and amg.amg_level_patterns(h, 0) == (padded, 0, 0)


@pytest.mark.parametrize("name", ["7pt_crossing", "27pt_crossing"])
def test_infinity_and_nan_reach_the_rows_of_a_dense_layout(amg, name):
    """Entries that are no number spread through the products, the zeros of the padding included,
    exactly as from the stored values of the same pattern (every entry scaled by its own row)."""
    A = MATRICES[name]()
    rng = np.random.default_rng(7)
    x = rng.uniform(-1, 1, A.n)
    x[[0, 63, 64, 1000, A.n - 1]] = [np.nan, np.inf, -np.inf, np.nan, np.inf]
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    D = W.CSR(A.n, A.row_ptr, A.col, A.val * (1.0 + rows / A.n), A.grid)
    got = []
    for M in (A, D):
        with hierarchy(M, max_coarse=10**9 if M.n <= 4096 else 4096) as h:
            got.append(amg.amg_level_patterns(h, 0)[1])
            y = nan_vec(A.n)
            amg.amg_spmv(h, 0, dev(x), y)
            got.append(host(y))
    assert got[0] > 0 and got[2] == 0
    assert np.array_equal(np.isnan(got[1]), np.isnan(got[3]))
    assert np.array_equal(np.isinf(got[1]), np.isinf(got[3]))


@pytest.mark.parametrize("name", ["7pt_crossing", "27pt_crossing", "two_materials"])
def test_fp32_smoother(amg, name):
    # float32 recurrences of degree 4: 27 products and the updates, each within 2^-24, four steps
    A = MATRICES[name]()
    As = A.to_scipy()
    b = np.random.default_rng(8).uniform(-1, 1, A.n).astype(np.float32)
    torch = torch_cuda()
    with hierarchy(A, max_coarse=100, precision=amg.AMG_FP32) as h:
        x = torch.full((A.n,), float("nan"), dtype=torch.float32, device="cuda")
        amg.smoother_apply_f32(h, 0, 2, 4, dev(b), x, True)
        beta, a = oracle_params(2, 4)
        want = S.smooth(As, S.l1_diagonal(As), b.astype(np.float64), None, 2, 4, beta, a)
        assert relerr(host(x), want) <= 4 * 40 * 2.0**-24
