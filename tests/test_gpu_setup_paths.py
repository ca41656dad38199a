"""Setup paths: scans at their chunk edges, box levels whose restriction rows pass a wavefront's 64
entries, the temporary arrays' reuse, and setups on several threads at once."""
import threading

import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from gpu_util import dev, hierarchy, host, nan_vec, relerr, torch_cuda
from oracle import amg as OA

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amg():
    torch_cuda()
    import paper_2407_09848_amd as m
    return m


def banded(n, half, seed):
    """Symmetric, diagonally dominant, every entry within `half` of the diagonal nonzero."""
    rng = np.random.default_rng(seed)
    B = sp.diags([rng.uniform(-1, -0.1, n - k) for k in range(1, half + 1)], list(range(1, half + 1)))
    B = (B + B.T).tocsr()
    S = (B + sp.diags(np.asarray(np.abs(B).sum(axis=1)).ravel() + 1.0)).tocsr()
    S.sort_indices()
    return W.CSR(n, S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data, (n, 1, 1))


def check_levels(amg, A, max_coarse):
    H = OA.build_hierarchy(A.to_scipy(), A.grid, max_coarse=max_coarse)
    with hierarchy(A, max_coarse=max_coarse) as h:
        assert amg.amg_num_levels(h) == len(H.levels)
        for l, lv in enumerate(H.levels):
            rp, cl, vl, mi = (host(t) for t in amg.amg_level_export(h, l))
            ref = lv.A.tocsr()
            ref.sort_indices()
            assert np.array_equal(rp, ref.indptr) and np.array_equal(cl, ref.indices), l
            # sums of at most 8 x 81 terms of one sign class: 648 * 2^-53 of the entry, under 1e-13
            assert relerr(vl, ref.data) <= 1e-13 and relerr(mi, lv.Minv) <= 1e-13, l


@pytest.mark.parametrize("n", [4095, 4096, 4097, 8191, 8192, 8193, 8194, 16385])
def test_scans_at_chunk_edges(amg, n):
    check_levels(amg, W.poisson3d_7pt(n, 1, 1), 500)


@pytest.mark.parametrize("half", [31, 32, 40, 60])
def test_restriction_rows_around_and_beyond_a_wavefront(amg, half):
    # two rows of 2 half + 1 entries: 2 half + 2 distinct columns, 64 at half = 31
    check_levels(amg, banded(700, half, half), 100)


def test_too_many_coarse_columns_are_refused(amg):
    with pytest.raises(amg.AmgError) as e:
        with hierarchy(banded(900, 70, 1), max_coarse=100):
            pass
    assert e.value.code == amg.AMG_ECAPACITY


def test_setups_on_several_threads(amg):
    torch = torch_cuda()
    problems = [W.poisson3d_7pt(20, 21, 22), W.q1_27pt(17, 18, 16), W.fv_diffusion(
        np.exp(np.random.default_rng(3).standard_normal((18, 20, 19)))), W.poisson2d_5pt(90, 70)]
    rhs = [np.random.default_rng(p).uniform(-1, 1, A.n) for p, A in enumerate(problems)]

    def build(A, b, repeats):
        # setup and kernel-level calls: the captured graphs of vcycle_apply and pcg_solve are not for
        # threads that synchronise the device meanwhile, as releases do
        out = None
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(repeats):
                with hierarchy(A, max_coarse=300) as h:
                    out = []
                    bd = dev(b)
                    for l in range(amg.amg_num_levels(h) - 1):
                        n, nc = amg.amg_level_info(h, l)[0], amg.amg_level_info(h, l + 1)[0]
                        x, bc = nan_vec(n), nan_vec(nc)
                        amg.smoother_apply(h, l, 2, 4, bd, x, True)
                        amg.amg_restrict_residual(h, l, bd, x, bc)
                        torch.cuda.current_stream().synchronize()
                        out += [host(x), host(bc)]
                        bd = bc
                    x = nan_vec(bd.numel())
                    amg.amg_coarse_solve(h, bd, x)
                    torch.cuda.current_stream().synchronize()
                    out.append(host(x))
        return out

    want = [build(A, b, 1) for A, b in zip(problems, rhs)]
    got = [None] * len(problems)

    def work(p):
        got[p] = build(problems[p], rhs[p], 4)

    threads = [threading.Thread(target=work, args=(p,)) for p in range(len(problems))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for w, g in zip(want, got):
        assert len(w) == len(g) and all(np.array_equal(a, b) for a, b in zip(w, g))
