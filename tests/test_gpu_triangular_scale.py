"""GPU test of the triangular factor (csrc/psi_tri.hip) on states of very different
sizes: site i's state is multiplied by 10^g_i (its matrices by 10^(g_i - g_j) per
parent j, w by 10^-g_i), which changes no amplitude, while the matrices' entries reach
1e+-240, whose squares a double cannot hold.  Bars of the FP64 path: E_loc 1e-10
relative to max(|E|, 1e-3 RMS E), log|Psi| 1e-12 absolute."""
import numpy as np
import pytest

import oracle
from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu
K, NA, NB, N = 8, 4, 3, 21
G = (0, 140, -100, 140, -100, 0, 140, -100)


@pytest.mark.parametrize("graph,chi", [("chain", 4), ("nnn", 17), ("nnn", 48)])
def test_site_scales(graph, chi):
    from paper_2507_19276_amd import nqs
    pp, pi = W.graph_chain(K) if graph == "chain" else W.graph_nn_nnn(K)
    plain = W.ansatz_params(K, chi, pp, pi, 0, 11)
    prm, at = plain.copy(), 0
    for i in range(K):
        for j in pi[pp[i]:pp[i + 1]]:
            prm[at:at + 4 * chi * chi] *= 10.0 ** (G[i] - G[j])
            at += 4 * chi * chi
        prm[at:at + 4 * chi] *= 10.0 ** G[i]
        prm[at + 5 * chi:at + 6 * chi] *= 10.0 ** -G[i]
        at += 6 * chi + 1
    assert at == len(prm) and np.isfinite(prm).all()
    h, eri = W.chain_integrals(K, 3)
    smp = W.random_onvs(K, NA, NB, N, 5, unique=False)
    ref = oracle.eloc(K, NA, NB, h, eri, chi, pp, pi, 0, prm, smp, eps=0.0, n_eps=0)
    base = oracle.eloc(K, NA, NB, h, eri, chi, pp, pi, 0, plain, smp, eps=0.0, n_eps=0)
    tau = 1e-3 * np.sqrt(np.mean(ref["eloc"] ** 2))
    rel = lambda e: (np.abs(e - ref["eloc"]) / np.maximum(np.abs(ref["eloc"]), tau)).max()
    assert rel(base["eloc"]) <= 1e-10   # the amplitudes are the unscaled ones
    ctx = nqs.Context(0)
    inst = nqs.Instance(ctx, K, NA, NB, h, eri, 0.0)
    ans = nqs.Ansatz(ctx, K, NA, NB, chi, pp, pi, 0).bind(prm)
    out, _ = nqs.eloc(ctx, inst, ans, smp, precision="f64")
    full, _ = nqs.eloc(ctx, inst, ans, smp, precision="f64", resume=False)
    got = out["eloc"].cpu().numpy()
    assert rel(got) <= 1e-10
    la = oracle.amplitudes(K, chi, NA, NB, pp, pi, 0, prm, smp)["logabs"]
    assert np.abs(out["logabs"].cpu().numpy() - la).max() <= 1e-12
    assert np.array_equal(got, full["eloc"].cpu().numpy())
