"""The dense coarsest factorisation (64-row tiles, inverse by doubling) at tile counts that are no
power of two, with padding, and for stacked problems."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from gpu_util import dev, hierarchy, host, nan_vec, relerr, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amg():
    torch_cuda()
    import paper_2407_09848_amd as m
    return m


@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 192, 200, 320, 333, 448, 577, 704])
@pytest.mark.parametrize("nbatch", [1, 3])
def test_coarse_solve_matches_numpy(amg, n, nbatch):
    # condition number below 20 (diagonally dominant), n <= 704: n^2 * 2^-53 * 20 < 1.2e-9 at worst,
    # and about sqrt of it in practice; the bar is the suite's 1e-12
    rng = np.random.default_rng(n)
    mats, blocks = [], []
    for p in range(nbatch):
        B = rng.uniform(-1, 1, (n, n)) * (rng.random((n, n)) < 8.0 / n)
        B = (B + B.T) / 2
        np.fill_diagonal(B, 0.0)
        np.fill_diagonal(B, np.abs(B).sum(axis=1) * 1.2 + 0.5)
        S = sp.csr_matrix(B)
        blocks.append(B)
        mats.append(W.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data, (n, 1, 1)))
    A = W.stack_block_diagonal(mats)
    b = rng.uniform(-1, 1, n * nbatch)
    with hierarchy(A, nbatch=nbatch, max_coarse=10**6) as h:
        x = nan_vec(n * nbatch)
        amg.amg_coarse_solve(h, dev(b), x)
        want = np.concatenate([np.linalg.solve(B, b[p * n:(p + 1) * n]) for p, B in enumerate(blocks)])
        assert relerr(host(x), want) <= 1e-12


@pytest.mark.parametrize("row", [3, 70, 150])
def test_indefinite_coarsest_level_is_refused(amg, row):
    # a positive diagonal with one coupling that makes the matrix indefinite in the tile of `row`
    n = 160
    B = np.eye(n) * 2.0
    B[row, row + 1] = B[row + 1, row] = 3.0
    S = sp.csr_matrix(B)
    A = W.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data, (n, 1, 1))
    with pytest.raises(amg.AmgError) as e:
        with hierarchy(A, max_coarse=10**6):
            pass
    assert e.value.code == amg.AMG_ENOTSPD


@pytest.mark.parametrize("n,sweeps,nbatch", [(1, 30, 1), (63, 8, 1), (64, 30, 1), (65, 30, 1), (700, 30, 1),
                                              (700, 7, 1), (700, 30, 2), (2048, 12, 1), (2049, 12, 1)])
def test_coarse_sweeps_match_oracle(amg, n, sweeps, nbatch):
    # the sweeps contract (every M^-1 A spectrum lies in (0, 1]): rounding adds up to at most
    # sweeps * (nonzeros per row) * 2^-53 of the result, below 1e-12
    from oracle import smoothers as S
    A = W.stack_block_diagonal([W.poisson3d_7pt(n, 1, 1) if n > 700 else W.fv_diffusion(
        np.exp(np.random.default_rng(n + p).standard_normal((1, 7 if n % 7 == 0 else 1, n // 7 if n % 7 == 0 else n))))
        for p in range(nbatch)])
    As = A.to_scipy()
    b = np.random.default_rng(17).uniform(-1, 1, A.n)
    with hierarchy(A, nbatch=nbatch, max_coarse=10**6, coarse_sweeps=sweeps) as h:
        x = nan_vec(A.n)
        amg.amg_coarse_solve(h, dev(b), x)
        assert relerr(host(x), S.smooth(As, S.l1_diagonal(As), b, None, 0, sweeps)) <= 1e-12
