"""GPU test of the local energies after binding other parameters to the same ansatz:
the sorted rows' buffers (triangular factor, FP64 and FP32 operand streams) are
rewritten in place, and an eta of zero switches to the four-candidate rows and back.
Every call must equal, bit for bit, that of an ansatz which was bound once."""
import numpy as np
import pytest

from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu
K, NA, NB, N = 8, 4, 3, 20


@pytest.mark.parametrize("chi,cplx", [(17, False), (32, False), (9, True)])
def test_rows_after_rebind(chi, cplx):
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    pp, pi = W.graph_nn_nnn(K)
    h, eri = W.chain_integrals(K, 3)
    inst = nqs.Instance(ctx, K, NA, NB, h, eri, 0.0)
    smp = W.random_onvs(K, NA, NB, N, 1, unique=False)
    eloc = nqs.eloc_complex if cplx else nqs.eloc
    re = 2 if cplx else 1   # doubles per entry of M, v, w, c
    site = int(pp[2]) * re * 4 * chi * chi + 2 * (re * (4 * chi + chi + 1) + chi) + (int(pp[3]) - int(pp[2])) * re * 4 * chi * chi
    eta = site + re * 4 * chi   # eta of site 2
    kept = nqs.Ansatz(ctx, K, NA, NB, chi, pp, pi, 0, cplx=cplx)
    assert kept.row_kernel("f64") is None
    for seed, zero in ((1, False), (2, False), (3, True), (4, False)):
        prm = W.ansatz_params(K, chi, pp, pi, 0, seed, cplx=cplx)
        assert 0.5 <= prm[eta] <= 1.5
        if zero:
            prm[eta] = 0.0
        kept.bind(prm)
        fresh = nqs.Ansatz(ctx, K, NA, NB, chi, pp, pi, 0, cplx=cplx).bind(prm)
        for precision, kind in (("f64", "double"), ("f32", "float")):
            assert kept.row_kernel(precision) == ("k_psi_mt<%s>" if zero else "k_psi_tri<%s>") % kind
            for resume in (True, False):
                kw = dict(eps=0.05, n_eps=16, seed=2, precision=precision, resume=resume)
                a, _ = eloc(ctx, inst, kept, smp, **kw)
                b, _ = eloc(ctx, inst, fresh, smp, **kw)
                for k in a:
                    assert np.array_equal(a[k].cpu().numpy(), b[k].cpu().numpy()), (seed, precision, resume, k)
        fresh.close()
