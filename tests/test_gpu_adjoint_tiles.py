"""GPU tests of the gradient's workgroups (csrc/adjoint.hip): a site's four
candidates on four wavefronts, its parents' cotangents split over (edge, unit
tile), column sums over 16 row phases, at sizes where these have remainders:
one unit tile (three idle wavefronts), three and four, in-degrees 0 to 3, row
counts below and past a tile and past one row split.  FP64 against the oracle's
gradient (1e-12 of its largest entry: sums of at most 2000 terms rounded at
2^-53), FP32 within 1e-4 of it (2^-24 through K sites and a few hundred rows)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chi,kind,N", [(5, "chain", 1), (16, "nnn", 17), (33, "nnn", 16), (48, "lattice", 65),
                                        (64, "lattice", 130), (20, "lattice", 2100)])
def test_against_oracle(chi, kind, N):
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    K, na, nb = 8, 4, 3
    pp, pi = {"chain": W.graph_chain, "nnn": W.graph_nn_nnn}.get(kind, lambda _: W.graph_lattice((2, 2, 2)))(K)
    prm = W.ansatz_params(K, chi, pp, pi, 3, 50 + chi)
    smp = W.random_onvs(K, na, nb, N, 4, unique=False)
    cot = np.random.default_rng(5).standard_normal(N)
    ans = nqs.Ansatz(ctx, K, na, nb, chi, pp, pi, 3)
    ans.bind(prm)
    ref = oracle.grad(K, chi, na, nb, pp, pi, 3, prm, smp, cot)
    for prec, tol in (("f64", 1e-12), ("f32", 1e-4)):
        g = ans.vjp(smp, torch.from_numpy(cot).cuda(), prec).cpu().numpy()
        assert np.abs(g - ref).max() <= tol * np.abs(ref).max(), prec
