"""GPU tests of the FP32 rows in the sorted row kernel (csrc/psi_tri.h) against
the FP64 oracle at the stated FP32 bounds (bounds.py), and bit for bit between
resumed rows, rows from site 0 and other pass boundaries, whose wavefronts hold
other rows.  Sizes at the edges of its tiles, parentless sites and mixed
in-degrees, masks that bind early, partial wavefronts; the real chain at chip 16
and in-degree 4 keep the general kernel."""
import numpy as np
import pytest

import oracle
from bounds import U_F, bounds, log_bound, stated_bound
from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu


def csr(parents):
    ptr = np.cumsum([0] + [len(p) for p in parents]).astype(np.int32)
    return ptr, np.array([j for p in parents for j in p], dtype=np.int32)


def graph(kind, K):
    if kind == "chain":
        return W.graph_chain(K)
    if kind == "nnn":
        return W.graph_nn_nnn(K)
    if kind == "mixed":
        return csr([[] if i % 5 == 0 else [j for j in (i - 4, i - 2, i - 1) if j >= 0][-(1 + i % 3):] for i in range(K)])
    return csr([[j for j in range(i - 4, i) if j >= 0] for i in range(K)])   # in-degree 4


CASES = [
    # K, n_alpha, n_beta, graph, chi, N
    (8, 4, 4, "chain", 16, 9),
    (9, 4, 5, "nnn", 1, 16),
    (9, 3, 4, "mixed", 16, 5),
    (8, 4, 3, "chain", 17, 33),
    (7, 3, 3, "nnn", 32, 17),
    (7, 3, 4, "mixed", 33, 5),
    (7, 4, 3, "chain", 48, 5),
    (7, 3, 3, "nnn", 49, 3),
    (7, 3, 3, "mixed", 64, 5),
    (10, 1, 9, "nnn", 20, 6),     # few particles, few holes
    (6, 6, 2, "nnn", 16, 15),     # a full spin: one alpha state everywhere
    (40, 2, 1, "mixed", 16, 3),   # both ONV words
    (7, 3, 3, "degree4", 16, 5),
]


@pytest.mark.parametrize("K,na,nb,kind,chi,N", CASES)
def test_against_oracle(K, na, nb, kind, chi, N):
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    h, eri = W.chain_integrals(K, 11 + K)
    pp, pi = graph(kind, K)
    prm = W.ansatz_params(K, chi, pp, pi, 0, 100 + chi)
    smp = W.random_onvs(K, na, nb, N, 3, unique=False)
    inst = nqs.Instance(ctx, K, na, nb, h, eri, 0.0)
    ans = nqs.Ansatz(ctx, K, na, nb, chi, pp, pi, 0)
    ans.bind(prm)
    kw = dict(eps=0.05, n_eps=20, seed=9)
    out, _ = nqs.eloc(ctx, inst, ans, smp, precision="f32", **kw)
    full, _ = nqs.eloc(ctx, inst, ans, smp, precision="f32", resume=False, **kw)
    part, _ = nqs.eloc(ctx, inst, ans, smp, precision="f32", max_rows_per_pass=1, **kw)
    got = {k: v.cpu().numpy() for k, v in out.items()}
    for k in got:
        assert np.array_equal(got[k], full[k].cpu().numpy()) and np.array_equal(got[k], part[k].cpu().numpy()), k
    la, _ = ans.logpsi(smp, "f32")
    assert np.array_equal(got["logabs"], la.cpu().numpy())
    ref = oracle.eloc(K, na, nb, h, eri, chi, pp, pi, 0, prm, smp, bounds=bounds(K), u_f=U_F, **kw)
    assert np.all(np.abs(got["eloc"] - ref["eloc"]) <= stated_bound("f32", ref))
    assert np.abs(got["logabs"] - ref["logabs"]).max() <= log_bound("f32", K)
    assert np.array_equal(got["sign"], ref["sign"])


@pytest.mark.parametrize("chi,N", [(7, 9), (17, 5)])
def test_complex_rows(chi, N):
    """Realified: chip 16 (which real chains leave to the general kernel) and 48.
    Resumed rows and rows from site 0 are equal bit for bit; against FP64 within
    the FP32 bar of the complex path."""
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    K, na, nb = 8, 4, 4
    h, eri = W.chain_integrals(K, 21)
    pp, pi = W.graph_chain(K)
    prm = W.ansatz_params(K, chi, pp, pi, 0, 5, cplx=True)
    smp = W.random_onvs(K, na, nb, N, 3, unique=False)
    inst = nqs.Instance(ctx, K, na, nb, h, eri, 0.0)
    ans = nqs.Ansatz(ctx, K, na, nb, chi, pp, pi, 0, cplx=True)
    ans.bind(prm)
    kw = dict(eps=0.05, n_eps=20, seed=9)
    out, _ = nqs.eloc_complex(ctx, inst, ans, smp, precision="f32", **kw)
    full, _ = nqs.eloc_complex(ctx, inst, ans, smp, precision="f32", resume=False, **kw)
    ref, _ = nqs.eloc_complex(ctx, inst, ans, smp, precision="f64", **kw)
    for k in out:
        a, b, r = (x[k].cpu().numpy() for x in (out, full, ref))
        assert np.array_equal(a, b), k
        if k == "eloc":
            rms = np.sqrt(np.mean(np.abs(r) ** 2))
            assert np.abs(a - r).max() <= 1e-4 * rms
