"""The box levels' Galerkin products, bit by bit: every coarse entry is the sum of the fine entries of its
aggregate's rows, row by row in ascending order and within a row in ascending column order."""
import numpy as np
import pytest

import workloads as W
from gpu_util import hierarchy, host, torch_cuda
from oracle import amg as OA

pytestmark = pytest.mark.gpu


def q1_random(nx, ny, nz, seed):
    """27-point matrix D A D with random positive D: sums of up to 64 numbers that round at every step."""
    A = W.q1_27pt(nx, ny, nz)
    d = 1.0 + np.random.default_rng(seed).random(A.n)
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    return W.CSR(A.n, A.row_ptr, A.col, A.val * d[rows] * d[A.col], A.grid)


def boxes(A, grid, nbatch):
    """(row_ptr, col, val) of P^T A P, summed one fine entry after the other."""
    agg, cgrid = OA.box_aggregates(grid, nbatch)
    nc = int(agg.max()) + 1
    rows = np.repeat(np.arange(A.shape[0]), np.diff(A.indptr))
    I, J = agg[rows].astype(np.int64), agg[A.indices]
    order = np.lexsort((A.indices, rows, J, I))  # entries of (I, J) by fine row, then column
    keys, first = np.unique((I * nc + J)[order], return_index=True)
    length = np.diff(np.append(first, order.size))
    val = A.data[order]
    total = np.zeros(keys.size)
    for k in range(int(length.max())):
        on = length > k
        total[on] += val[first[on] + k]
    kept = np.abs(total) > 0.0
    ptr = np.zeros(nc + 1, dtype=np.int64)
    np.cumsum(np.bincount(keys[kept] // nc, minlength=nc), out=ptr[1:])
    return ptr, keys[kept] % nc, total[kept], cgrid


MATRICES = {
    "27pt": (lambda: q1_random(29, 22, 17, 1), 1),
    "27pt_constant": (lambda: W.q1_27pt(33, 18, 13), 1),
    "27pt_stacked": (lambda: W.stack_block_diagonal([q1_random(9, 11, 10, 2 + p) for p in range(3)]), 3),
    "7pt": (lambda: W.fv_diffusion(np.exp(np.random.default_rng(6).standard_normal((21, 30, 26)))), 1),
    "9pt": (lambda: W.anisotropy2d_q1(75)[0], 1),
    "line": (lambda: W.poisson3d_7pt(997, 1, 1), 1),
}


@pytest.mark.parametrize("name", list(MATRICES))
def test_coarse_matrices_are_the_sequential_sums(name):
    torch_cuda()
    import paper_2407_09848_amd as amg

    make, nbatch = MATRICES[name]
    A = make()
    with hierarchy(A, nbatch=nbatch, max_coarse=40) as h:
        levels = [[host(t) for t in amg.amg_level_export(h, l)[:3]] for l in range(amg.amg_num_levels(h))]
    assert len(levels) >= 3
    grid = (A.grid[0], A.grid[1], A.grid[2] // nbatch)
    import scipy.sparse as sp

    for fine, coarse in zip(levels, levels[1:]):
        M = sp.csr_matrix((fine[2], fine[1], fine[0]))
        ptr, col, val, grid = boxes(M, grid, nbatch)
        assert np.array_equal(coarse[0], ptr) and np.array_equal(coarse[1], col)
        assert np.array_equal(coarse[2], val)
