"""GPU test of the FP64 rows' tiles per wavefront (csrc/psi_tri.h, kTriOneTileRows =
16384 rows): a call whose 21,828 rows run in one pass (two tiles per wavefront up to
two parents) against the same call with one sample of 1,819 rows per pass (one tile),
bit for bit, resumed and from site 0, real and complex; and against the FP64 oracle
at the FP64 bars (E_loc 1e-10 relative to max(|E|, 1e-3 RMS E); log|Psi| 1e-12)."""
import numpy as np
import pytest

import oracle
from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu
K, NA, NB, N = 12, 6, 6, 12


def graph(kind):
    if kind == "chain":
        return W.graph_chain(K)
    if kind == "nnn":
        return W.graph_nn_nnn(K)
    par = [[j for j in (i - 4, i - 2, i - 1) if j >= 0] for i in range(K)]   # up to three parents
    return np.cumsum([0] + [len(p) for p in par]).astype(np.int32), np.array([j for p in par for j in p], dtype=np.int32)


@pytest.mark.parametrize("kind,chi,cplx", [("chain", 7, False), ("nnn", 16, False), ("three", 9, False),
                                           ("nnn", 32, False), ("chain", 40, False), ("nnn", 64, False),
                                           ("chain", 8, True), ("nnn", 16, True), ("chain", 32, True)])
def test_passes_of_other_sizes(kind, chi, cplx):
    from paper_2507_19276_amd import nqs
    pp, pi = graph(kind)
    h, eri = W.chain_integrals(K, 3)
    prm = W.ansatz_params(K, chi, pp, pi, 0, 11, cplx=cplx)
    smp = W.random_onvs(K, NA, NB, N, 5)
    ctx = nqs.Context(0)
    inst = nqs.Instance(ctx, K, NA, NB, h, eri, 0.0)
    ans = nqs.Ansatz(ctx, K, NA, NB, chi, pp, pi, 0, cplx=cplx).bind(prm)
    eloc = nqs.eloc_complex if cplx else nqs.eloc
    out, st = eloc(ctx, inst, ans, smp, precision="f64")
    assert st["n_rows"] == N * (inst.n_conn + 1) > 16384 > inst.n_conn + 1
    got = {k: v.cpu().numpy() for k, v in out.items()}
    for kw in (dict(max_rows_per_pass=1), dict(resume=False), dict(resume=False, max_rows_per_pass=1)):
        other, st = eloc(ctx, inst, ans, smp, precision="f64", **kw)
        assert st["n_passes"] == (N if "max_rows_per_pass" in kw else 1)
        for k in got:
            assert np.array_equal(got[k], other[k].cpu().numpy()), (kw, k)
    ref = oracle.eloc(K, NA, NB, h, eri, chi, pp, pi, 0, prm, smp, eps=0.0, n_eps=0, cplx=cplx)
    e = ref["eloc"]
    tau = 1e-3 * np.sqrt(np.mean(np.abs(e) ** 2))
    assert (np.abs(got["eloc"] - e) / np.maximum(np.abs(e), tau)).max() <= 1e-10
    assert np.abs(got["logabs"] - ref["logabs"]).max() <= 1e-12
    if not cplx:   # the samples' own Phi is that of nqs_logpsi, bit for bit
        assert np.array_equal(got["logabs"], ans.logpsi(smp, "f64")[0].cpu().numpy())
