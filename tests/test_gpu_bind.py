"""GPU tests of binding parameters (csrc/bind.hip): a bind replaces every
layout of the one before (folded and not: eta with and without zeros; both
precisions; correlator tables; the adjoint's operands), and a refused vector
leaves the old binding in force."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu
K, NA, NB, NH = 6, 3, 2, 5


@pytest.mark.parametrize("chi,ising", [(3, False), (17, True), (48, False)])
def test_rebind(chi, ising):
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    pp, pi = W.graph_nn_nnn(K)
    smp = W.random_onvs(K, NA, NB, 20, 1, unique=False)
    cot = np.random.default_rng(2).standard_normal(20)
    ans = nqs.Ansatz(ctx, K, NA, NB, chi, pp, pi, NH, ising=ising)
    eta = np.cumsum([0] + [(pp[i + 1] - pp[i]) * 4 * chi * chi + 6 * chi + 1 for i in range(K)])[:K] + 4 * chi
    eta = eta + (pp[1:K + 1] - pp[:K]) * 4 * chi * chi
    for seed, zero in ((1, False), (2, True), (3, False)):
        prm = W.ansatz_params(K, chi, pp, pi, NH, seed, ising=ising)
        assert ((prm[eta] >= 0.5) & (prm[eta] <= 1.5)).all()
        if zero:
            prm[eta[2]] = 0.0
        ans.bind(prm)
        ref = oracle.amplitudes(K, chi, NA, NB, pp, pi, NH, prm, smp, ising=ising)
        refg = oracle.grad(K, chi, NA, NB, pp, pi, NH, prm, smp, cot, ising=ising)
        for prec, tol, gtol in (("f64", 1e-12, 1e-12), ("f32", 1e-4, 1e-3), ("bf16x3", 1e-2, None)):
            la, _ = ans.logpsi(smp, prec)
            assert np.abs(la.cpu().numpy() - ref["logabs"]).max() <= tol, (prec, seed)
            if gtol:
                g = ans.vjp(smp, torch.from_numpy(cot).cuda(), prec).cpu().numpy()
                assert np.abs(g - refg).max() <= gtol * np.abs(refg).max(), (prec, seed)
    before = ans.logpsi(smp, "f64")[0]
    for bad in (-1.0, float("nan")):
        prm2 = prm.copy()
        prm2[eta[4]] = bad
        with pytest.raises(nqs.NqsError, match=r"eta\[4\]\[0\]"):
            ans.bind(prm2)
        assert torch.equal(before, ans.logpsi(smp, "f64")[0])
