"""GPU test of the Ising-RBM rows kernel's lanes (csrc/energy.hip): 16 lanes per
row over the hidden units, four rows at a time: numbers of units below, at and
past the 16 lanes, row counts with remainders of 4 and 16, both ONV words.
FP64 at the FP64 bar (1e-10); FP32 log-sums of N_h cosines rounded at 2^-24
against theta of order one: within 1e-3 of E_loc relative to its RMS."""
import numpy as np
import pytest

import oracle
from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,na,nb,nh,N", [(6, 3, 3, 1, 1), (6, 3, 3, 15, 3), (6, 2, 4, 17, 5), (35, 2, 1, 33, 2)])
def test_against_oracle(K, na, nb, nh, N):
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    h, eri = W.chain_integrals(K, 7)
    pp, pi = W.graph_chain(K)
    prm = W.ansatz_params(K, 8, pp, pi, nh, 31, ising=True)
    smp = W.random_onvs(K, na, nb, N, 4, unique=False)
    inst = nqs.Instance(ctx, K, na, nb, h, eri, 0.0)
    ans = nqs.Ansatz(ctx, K, na, nb, 8, pp, pi, nh, ising=True)
    ans.bind(prm)
    ref = oracle.eloc(K, na, nb, h, eri, 8, pp, pi, nh, prm, smp, eps=0.05, n_eps=10, seed=3, ising=True)
    rms = np.sqrt(np.mean(ref["eloc"] ** 2))
    for prec, tol in (("f64", 1e-10), ("f32", 1e-3)):
        out, _ = nqs.eloc(ctx, inst, ans, smp, eps=0.05, n_eps=10, seed=3, precision=prec)
        assert np.abs(out["eloc"].cpu().numpy() - ref["eloc"]).max() <= tol * rms, prec
