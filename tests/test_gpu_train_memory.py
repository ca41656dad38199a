"""The training workspace: allocated with the first differentiable V-cycle, given back with the handle."""
import numpy as np
import pytest

import workloads as W
from gpu_util import dev, hierarchy, nan_vec, torch_cuda
from oracle import polynomials as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
def test_workspace_is_given_back(precision):
    torch = torch_cuda()
    import paper_2407_09848_amd as amg

    A = W.stack_block_diagonal([W.fv_diffusion(np.exp(np.random.default_rng(p).standard_normal((40, 41, 42))))
                                for p in range(3)])
    k = 3
    b, gr, z = dev(np.random.default_rng(5).uniform(-1, 1, A.n)), nan_vec(A.n), nan_vec(A.n)

    def use():
        with hierarchy(A, nbatch=3, precision=precision) as h:
            levels = amg.amg_num_levels(h)
            beta = dev(np.tile(np.array(P.optimal_beta(k)[0]), (3, levels, 1)).ravel())
            ck = torch.empty(amg.amg_ckpt_bytes(h), dtype=torch.uint8, device="cuda")
            g = torch.zeros_like(beta)
            amg.vcycle_fwd_ckpt(h, k, beta, b, z, ck)
            amg.vcycle_bwd(h, k, beta, ck, b, gr, g)
            loss, _ = amg.amg_train_loss_grad(h, k, beta, b, g, 3)
            assert np.isfinite(loss)

    use()  # also loads what the first call of a process loads
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for _ in range(3):
        use()
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] >= free
