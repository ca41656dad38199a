"""What the layout of uniform slices stores, against a classification of the slices made here from the matrix:
the patterns that equal slices share, the rows per lane, and dense slices of 128 rows of which an
offset is used by one half alone or that end short."""
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


def classify(A, rows):
    """Slices of `rows` rows: per slice its number of steps, whether it is uniform and whether a step's
    offset is used by one half of 128 rows alone; and the steps of the distinct patterns."""
    n, rpl = A.n, rows // 64
    r = np.repeat(np.arange(n, dtype=np.int64), np.diff(A.row_ptr))
    off = A.col.astype(np.int64) - r
    s = r // rows
    order = np.argsort(s * (4 * n) + off + n, kind="stable")
    r, off, s = r[order], off[order], s[order]
    bits = A.val[order].view(np.uint64)
    first = np.flatnonzero(np.append(True, (np.diff(s) != 0) | (np.diff(off) != 0)))  # of every step
    top = np.maximum.reduceat(bits, first)
    low = np.minimum.reduceat(np.where(bits == 0, top[np.repeat(np.arange(first.size),
                                                               np.diff(np.append(first, bits.size)))], bits), first)
    lane = np.uint64(1) << ((r % rows) // rpl).astype(np.uint64)
    held, nonzero = [], []
    for k in range(rpl):
        own = (r % rpl) == k
        held.append(np.bitwise_or.reduceat(np.where(own, lane, np.uint64(0)), first))
        nonzero.append(np.bitwise_or.reduceat(np.where(own & (bits != 0), lane, np.uint64(0)), first))
    full = np.uint64(0xFFFFFFFFFFFFFFFF)
    whole = np.logical_and.reduce([(held[k] == full) & (nonzero[k] == nonzero[0])
                                   & ((nonzero[k] == 0) | (nonzero[k] == full)) for k in range(rpl)])
    masks = [np.where(whole, full, nonzero[k]) for k in range(rpl)]
    half = np.bitwise_or.reduceat(np.int64(1) << ((r % rows) // 64), first)
    nslices = (n + rows - 1) // rows
    at = s[first]
    steps = np.bincount(at, minlength=nslices)
    uniform = np.bincount(at, weights=top != low, minlength=nslices) == 0
    halves = (np.bincount(at, weights=half != 3, minlength=nslices) > 0) & (rows == 128)
    begin = np.append(0, np.cumsum(steps))
    record = np.stack([off[first].view(np.uint64), top, half.astype(np.uint64)] + masks, axis=1)
    if rows == 64:
        record[:, 2] = 0
    patterns = {record[begin[k]:begin[k + 1]].tobytes(): steps[k] for k in np.flatnonzero(uniform)}
    return steps, uniform, halves, sum(patterns.values())


def two_materials(nx, ny, nz, edge):
    kappa = np.ones((nz, ny, nx))
    kappa[nz // 2:] = 8.0
    kappa[:, :, :edge] = 3.0
    return W.fv_diffusion(kappa)


SMALL = {
    "7pt_whole_slices": lambda: W.poisson3d_7pt(64, 8, 6),
    "7pt_crossing": lambda: W.poisson3d_7pt(37, 23, 19),
    "27pt_whole_slices": lambda: W.q1_27pt(128, 6, 7),
    "27pt_crossing": lambda: W.q1_27pt(71, 13, 11),
    "5pt": lambda: W.poisson2d_5pt(64, 64),
    "two_materials": lambda: two_materials(256, 12, 10, 32),
}


@pytest.mark.parametrize("name", list(SMALL))
def test_equal_slices_share_their_pattern(amg, name):
    A = SMALL[name]()
    steps, uniform, _, shared = classify(A, 64)
    assert 2 * uniform.sum() >= uniform.size and shared < steps[uniform].sum()
    with hierarchy(A, max_coarse=A.n) as h:
        assert amg.amg_level_patterns(h, 0) == (64 * steps[~uniform].sum(), uniform.sum(), shared)
        assert amg.amg_level_rows_per_lane(h, 0) == 1


# 641 x 83 x 81 = 4,309,443 rows: lines and planes at every place of a slice, the last one of 67 rows
LARGE = {
    "7pt": lambda: two_materials(641, 83, 81, 40),
    "27pt": lambda: q1_islands(163, 161, 161),
}


def q1_islands(nx, ny, nz):
    A = W.q1_27pt(nx, ny, nz)
    d = np.ones(A.n)
    island = np.random.default_rng(31).choice(A.n, 9)
    island = np.append(island, A.n - 1)  # the last slice is dense
    d[island] = 2.0
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    return W.CSR(A.n, A.row_ptr, A.col, A.val * d[rows] * d[A.col], A.grid)


@pytest.mark.parametrize("name", list(LARGE))
def test_dense_slices_of_two_rows_per_lane(amg, name):
    # the bounds of the other layouts: 1e-14 for a product, 1e-12 for a few steps, 1e-10 for CG iterates
    A = LARGE[name]()
    As = A.to_scipy()
    steps, uniform, halves, shared = classify(A, 128)
    assert A.n >= 1 << 22 and A.n % 128 % 2 == 1 and 2 * uniform.sum() >= uniform.size
    assert not uniform[-1] and (~uniform & halves).sum() > 1
    rng = np.random.default_rng(32)
    b, x0 = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    Minv = S.l1_diagonal(As)
    with hierarchy(A) as h:
        assert amg.amg_level_rows_per_lane(h, 0) == 2
        values, _, stored = amg.amg_level_patterns(h, 0)
        assert (values, stored) == (128 * steps[~uniform].sum(), shared)
        y = nan_vec(A.n)
        amg.amg_spmv(h, 0, dev(x0), y)
        assert relerr(host(y), As @ x0) <= 1e-14
        for zero in (True, False):
            beta, a = oracle_params(2, 3)
            x = nan_vec(A.n) if zero else dev(x0.copy())
            amg.smoother_apply(h, 0, 2, 3, dev(b), x, zero)
            assert relerr(host(x), S.smooth(As, Minv, b, None if zero else x0, 2, 3, beta, a)) <= 1e-12, zero
        for maxit in (1, 2):
            x = nan_vec(A.n)
            rc, it, rel, _ = amg.pcg_solve_smoother(h, 2, 3, dev(b), x, True, 1e-14, maxit, True)
            want = OA.pcg(As, b, lambda r: S.smooth(As, Minv, r, None, 2, 3, beta, a), 1e-14, maxit, True)
            assert rc == amg.AMG_NOT_CONVERGED and rel == pytest.approx(want.relres, rel=1e-9)
            assert relerr(host(x), want.x) <= 1e-10
    with hierarchy(A, precision=amg.AMG_FP32) as h:
        assert amg.amg_level_rows_per_lane(h, 0) == 1


def test_infinity_and_nan_reach_the_rows_of_64_row_slices(amg):
    """Entries that are no number near dense slices of which an offset belongs to one half, against the
    same pattern in dense slices of 64 rows (every entry scaled by its own row)."""
    A = LARGE["7pt"]()
    _, uniform, halves, _ = classify(A, 128)
    x = np.random.default_rng(33).uniform(-1, 1, A.n)
    plane = A.grid[0] * A.grid[1]
    for k, s in enumerate(np.flatnonzero(~uniform & halves)[::7]):
        for at in (128 * s - 640, 128 * s - 1, 128 * s + 63, 128 * s + 130 + plane):
            x[min(max(at, 0), A.n - 1)] = (np.nan, np.inf, -np.inf)[k % 3]
    x[[0, A.n - 1]] = np.nan
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    D = W.CSR(A.n, A.row_ptr, A.col, A.val * (1.0 + rows / A.n), A.grid)
    got = []
    for M, lanes in ((A, 2), (D, 1)):
        with hierarchy(M) as h:
            assert amg.amg_level_rows_per_lane(h, 0) == lanes
            y = nan_vec(A.n)
            amg.amg_spmv(h, 0, dev(x), y)
            got.append(host(y))
    assert np.array_equal(np.isnan(got[0]), np.isnan(got[1]))
    assert np.array_equal(np.isinf(got[0]), np.isinf(got[1]))
