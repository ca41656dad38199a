"""Uniform slices of 128 rows, two rows per lane (large FP64 levels): products, smoothers, transfers and
dot products against the oracle where slices are whole, cross grid lines, end short (also on an odd
row), stay dense, or hold an offset that only one of their halves uses."""
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


def two_materials(nx, ny, nz):
    kappa = np.ones((nz, ny, nx))
    kappa[nz // 2:] = 8.0
    kappa[:, :, : nx // 16] = 3.0  # the first slice of every line stays dense
    return W.fv_diffusion(kappa)


MATRICES = {
    "7pt_whole": lambda: W.poisson3d_7pt(256, 128, 129),
    "7pt_odd": lambda: W.poisson3d_7pt(163, 161, 161),
    "5pt": lambda: W.poisson2d_5pt(2049, 2049),
    "two_materials": lambda: two_materials(640, 83, 80),
    "27pt": lambda: W.q1_27pt(163, 161, 161),
}


@pytest.mark.parametrize("name", list(MATRICES))
def test_products_smoothers_and_dots_match_oracle(amg, name):
    # at most 27 products per sum: 27 * 2^-53 of the summed magnitudes per product, a few steps of them
    torch = torch_cuda()
    A = MATRICES[name]()
    assert A.n >= 1 << 22
    As = A.to_scipy()
    Minv = S.l1_diagonal(As)
    rng = np.random.default_rng(11)
    b, x0 = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    with hierarchy(A) as h:
        values, patterned, _ = amg.amg_level_patterns(h, 0)
        assert 2 * patterned >= A.n // 64
        assert (values > 0) == (name == "two_materials")
        y = nan_vec(A.n)
        amg.amg_spmv(h, 0, dev(x0), y)
        assert relerr(host(y), As @ x0) <= 1e-14
        # one entry that is no number reaches the rows whose products hold it (and the padding of their
        # 64-row slices), none of another slice's
        x = x0.copy()
        nx, ny, nz = A.grid
        c = (nz // 2 * ny + ny // 2) * nx + nx // 2
        x[c] = np.nan
        amg.amg_spmv(h, 0, dev(x), y)
        got = np.isnan(host(y))
        offs = np.unique(As.indices[As.indptr[c]:As.indptr[c + 1]] - c)
        assert got[np.unique(As.indices[As.indptr[c]:As.indptr[c + 1]])].all()
        assert np.isin(np.flatnonzero(got), c - offs).all()
        cases = [(KINDS[0], 1), (KINDS[-1], 3)] if name == "27pt" else [(k, d) for k in KINDS for d in (1, 4)]
        for kind, k in cases:
            beta, a = oracle_params(kind, k)
            for zero in (True, False):
                x = nan_vec(A.n) if zero else dev(x0.copy())
                amg.smoother_apply(h, 0, kind, k, dev(b), x, zero)
                want = S.smooth(As, Minv, b, None if zero else x0, kind, k, beta, a)
                assert relerr(host(x), want) <= 1e-12, (kind, k, zero)
        # the CG's fused product and dots, and the transfers: the true residual follows the reported one
        xs = nan_vec(A.n)
        _, _, _, hist = amg.pcg_solve(h, 2, 4, dev(b), xs, True, 1e-8, 300, False, True)
        torch.cuda.synchronize()
        true = np.linalg.norm(b - As @ host(xs)) / np.linalg.norm(b)
        assert abs(true - hist[-1]) <= 1e-10 and hist[-1] <= 1e-8


def test_fp32_hierarchy_keeps_64_row_slices(amg):
    A = W.poisson3d_7pt(256, 128, 129)
    rng = np.random.default_rng(12)
    b = rng.uniform(-1, 1, A.n)
    As = A.to_scipy()
    with hierarchy(A, precision=amg.AMG_FP32) as h:
        assert 2 * amg.amg_level_patterns(h, 0)[1] >= A.n // 64
        xs = nan_vec(A.n)
        _, _, _, hist = amg.pcg_solve(h, 2, 4, dev(b), xs, True, 1e-8, 300, False, True)
        true = np.linalg.norm(b - As @ host(xs)) / np.linalg.norm(b)
        assert abs(true - hist[-1]) <= 1e-10 and hist[-1] <= 1e-8
