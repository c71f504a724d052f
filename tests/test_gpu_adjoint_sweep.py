"""GPU tests of the gradient's sweep in steps of several sites and of the states
kernel in front of it (csrc/adjoint.hip): K large enough for steps of up to four
sites, parents further back than the states kept in LDS, parentless sites, all
four states and one state only among 16 rows, partial tiles; and the row count at
which the states come from the other kernel.  FP64 against the oracle's gradient
(1e-12 of its largest entry), FP32 within 1e-4 of it, as test_gpu_adjoint_tiles.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu


def graph(K):
    """In-degrees 0..3 with parents 1, 7 and 15 sites back."""
    par = [[] if i % 6 == 0 else [j for j in (i - 15, i - 7, i - 1) if j >= 0][-(1 + i % 3):] for i in range(K)]
    return (np.cumsum([0] + [len(p) for p in par]).astype(np.int32),
            np.array([j for p in par for j in p], dtype=np.int32))


def ansatz(nqs, ctx, K, na, nb, chi):
    pp, pi = graph(K)
    prm = W.ansatz_params(K, chi, pp, pi, 0, 50 + chi)
    ans = nqs.Ansatz(ctx, K, na, nb, chi, pp, pi, 0)
    ans.bind(prm)
    return ans, pp, pi, prm


@pytest.mark.parametrize("K,na,nb,chi,N", [(24, 12, 11, 16, 33), (24, 3, 20, 7, 1), (40, 20, 20, 40, 16),
                                           (24, 12, 12, 64, 18)])
def test_against_oracle(K, na, nb, chi, N):
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    ans, pp, pi, prm = ansatz(nqs, ctx, K, na, nb, chi)
    smp = W.random_onvs(K, na, nb, N, 4, unique=False)
    cot = np.random.default_rng(5).standard_normal(N)
    ref = oracle.grad(K, chi, na, nb, pp, pi, 0, prm, smp, cot)
    for prec, tol in (("f64", 1e-12), ("f32", 1e-4)):
        g = ans.vjp(smp, torch.from_numpy(cot).cuda(), prec).cpu().numpy()
        assert np.abs(g - ref).max() <= tol * np.abs(ref).max(), prec


@pytest.mark.parametrize("prec,tol", [("f64", 1e-12), ("f32", 1e-4)])
def test_row_count_of_the_states_kernel(prec, tol):
    """16384 rows and 16385 take different kernels for the states: the gradient is
    the sum over the rows on either side."""
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    ans, _, _, _ = ansatz(nqs, ctx, 8, 4, 4, 9)
    smp = W.random_onvs(8, 4, 4, 16385, 4, unique=False)
    cot = torch.from_numpy(np.random.default_rng(6).standard_normal(16385)).cuda()
    whole = ans.vjp(smp, cot, prec).cpu().numpy()
    parts = (ans.vjp(smp[:16384], cot[:16384], prec) + ans.vjp(smp[16384:], cot[16384:], prec)).cpu().numpy()
    assert np.abs(whole - parts).max() <= tol * np.abs(whole).max()
