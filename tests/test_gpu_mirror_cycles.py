"""Mirrored diagonals inside whole cycles and CG solves, on levels that do not stream (2^19 to 3.1M rows): the
V-cycle with and without the prolongation in the post-smoothing's first kernels, the CG's directions,
products and dot products, the FP32 hierarchy, and weights per problem where a lane's two rows
belong to two problems."""
import functools

import numpy as np
import pytest

import workloads as W
from gpu_util import KINDS, dev, hierarchy, host, nan_vec, oracle_params, relerr, torch_cuda
from oracle import adjoint as AD
from oracle import amg as OA
from oracle import polynomials as P
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
    A = W.q1_27pt(nx, ny, nz)
    d = np.exp2(np.random.default_rng(seed).integers(-2, 3, A.n).astype(np.float64))
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    return W.CSR(A.n, A.row_ptr, A.col, A.val * d[rows] * d[A.col], A.grid)


PROBLEM = (61, 59, 61)  # 219,539 rows: odd
MATRICES = {
    "ragged": (lambda: W.fv_diffusion(field(87, 79, 83, 2)), 1),  # 570,459 rows
    "stacked": (lambda: W.stack_block_diagonal([W.fv_diffusion(field(*PROBLEM, 3 + p)) for p in range(3)]), 3),
    "27pt": (lambda: q1_varying(83, 80, 81, 8), 1),
    "above_fused_transfers": (lambda: W.fv_diffusion(field(115, 113, 117, 9)), 1),  # 1,520,415 rows
}


@functools.lru_cache(maxsize=4)
def problem(name):
    make, nbatch = MATRICES[name]
    A = make()
    return A, A.to_scipy(), OA.build_hierarchy(A.to_scipy(), A.grid, nbatch), nbatch


def mirrored(amg, h):
    padded, _, aligned = amg.amg_level_layout(h, 0)
    values, patterned, _ = amg.amg_level_patterns(h, 0)
    return aligned and patterned == 0 and values < 0.66 * padded


@pytest.mark.parametrize("name", list(MATRICES))
def test_vcycle_matches_oracle(amg, name):
    # as every other layout through a whole cycle: 1e-12
    A, _, H, nbatch = problem(name)
    b = np.random.default_rng(21).uniform(-1, 1, A.n)
    with hierarchy(A, nbatch=nbatch) as h:
        assert mirrored(amg, h) and amg.amg_num_levels(h) == len(H.levels)
        for kind in KINDS:
            for k in (1, 2, 4):
                beta, _ = oracle_params(kind, k)
                z = nan_vec(A.n)
                amg.vcycle_apply(h, kind, k, dev(b), z)
                assert relerr(host(z), OA.vcycle(H, b, kind, k, beta)) <= 1e-12, (kind, k)


@pytest.mark.parametrize("flexible", [False, True])
@pytest.mark.parametrize("name", list(MATRICES))
def test_cg_iterates_match_oracle(amg, name, flexible):
    # the bounds of the iterate test on dense slices: 1e-10 after 7 iterations
    A, As, H, nbatch = problem(name)
    b = W.rhs_uniform(A.n, 22)
    Minv = S.l1_diagonal(As)
    with hierarchy(A, nbatch=nbatch) as h:
        assert mirrored(amg, h)
        for kind, k in ((2, 4), (3, 3)) if name == "ragged" else ((2, 4),):
            beta, a = oracle_params(kind, k)
            preconds = {"pcg_solve": lambda r: OA.vcycle(H, r, kind, k, beta),
                        "pcg_solve_smoother": lambda r: S.smooth(As, Minv, r, None, kind, k, beta, a)}
            for call, precond in preconds.items():
                for maxit in (1, 2, 7):
                    x = nan_vec(A.n)
                    rc, it, rel, _ = getattr(amg, call)(h, kind, k, dev(b), x, True, 1e-14, maxit, flexible)
                    want = OA.pcg(As, b, precond, 1e-14, maxit, flexible)
                    assert rc == amg.AMG_NOT_CONVERGED and it == maxit == want.iters
                    assert rel == pytest.approx(want.relres, rel=1e-9), (call, kind, maxit)
                    assert relerr(host(x), want.x) <= 1e-10, (call, kind, maxit)


@pytest.mark.parametrize("name", ["ragged", "stacked", "27pt", "above_fused_transfers"])
def test_fp32_hierarchy(amg, name):
    """The FP32 V-cycle within FP32 rounding of the FP64 one, and the CG iterates those of the oracle's CG
    with the same FP32 V-cycle."""
    A, As, H, nbatch = problem(name)
    b = W.rhs_uniform(A.n, 23)
    beta, _ = oracle_params(2, 4)
    with hierarchy(A, nbatch=nbatch, precision=amg.AMG_FP32) as h:
        assert mirrored(amg, h)

        def precond(r):
            z = nan_vec(A.n)
            amg.vcycle_apply(h, 2, 4, dev(r), z)
            return host(z)

        # two smoothings of four steps per level, each of at most 28 rounded terms within 2^-24; the levels
        # together 8/7 of the finest
        assert relerr(precond(b), OA.vcycle(H, b, 2, 4, beta)) <= 8 / 7 * 8 * 28 * 2.0**-24
        for maxit in (1, 2, 7):
            x = nan_vec(A.n)
            rc, it, rel, _ = amg.pcg_solve(h, 2, 4, dev(b), x, True, 1e-14, maxit, True)
            want = OA.pcg(As, b, precond, 1e-14, maxit, True)
            assert rc == amg.AMG_NOT_CONVERGED and it == maxit
            # the two runs' residuals differ in their last bits, so a few of them round to FP32 the other way:
            # 2^-24 of single entries, with room for some growth over the iterations
            assert rel == pytest.approx(want.relres, rel=1e-6), maxit
            assert relerr(host(x), want.x) <= 1e-6, maxit


def test_weights_per_problem(amg):
    """Odd problems on top of one another: the first problem's last row shares its lane with the second
    problem's first one, whose weights are others."""
    torch = torch_cuda()
    k, count = 3, 3
    A, _, _, _ = problem("stacked")
    mats = [W.fv_diffusion(field(*PROBLEM, 3 + p)) for p in range(count)]
    Hs = [OA.build_hierarchy(m.to_scipy(), m.grid) for m in mats]
    rng = np.random.default_rng(24)
    r, c = rng.uniform(-1, 1, A.n), rng.uniform(-1, 1, A.n)
    with hierarchy(A, nbatch=count) as h:
        assert mirrored(amg, h)
        levels = amg.amg_num_levels(h)
        table = np.array(P.optimal_beta(k)[0]) * (1.0 + 0.05 * rng.standard_normal((count, levels, k)))
        beta = dev(table.ravel())
        ck = torch.empty(amg.amg_ckpt_bytes(h), dtype=torch.uint8, device="cuda")
        z, gr, gb = nan_vec(A.n), nan_vec(A.n), torch.zeros_like(beta)
        amg.vcycle_fwd_ckpt(h, k, beta, dev(r), z, ck)
        amg.vcycle_bwd(h, k, beta, ck, dev(c), gr, gb)
        z, gr, gb = host(z), host(gr), host(gb).reshape(count, levels, k)
    m0 = mats[0].n
    assert m0 % 2 == 1
    for p in range(count):
        own = slice(p * m0, (p + 1) * m0)
        betas = [table[p, l] for l in range(levels - 1)]
        assert relerr(z[own], AD.vcycle_beta(Hs[p], r[own], k, betas)) <= 1e-12
        assert relerr(gr[own], AD.vcycle_beta(Hs[p], c[own], k, betas)) <= 1e-12
        want = AD.linear_functional_grad(Hs[p], r[own], c[own], k, betas)
        assert np.allclose(gb[p, :levels - 1], want, rtol=1e-9, atol=1e-12 * np.abs(want).max())
