"""GPU tests of what a local-energy call reports to the host through pinned
memory (the mailbox in csrc/runtime.cpp): row counts of batches on either side of
the size whose row pointer is staged there, with and without drawn rows and over
several passes; a refused batch between two good ones; calls from several threads
on their own streams.  Everything compared is a count or the same computation, so
equality is exact."""
import threading

import numpy as np
import pytest
import torch

from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu
K, NA, NB, CHI = 4, 2, 2, 4


@pytest.fixture(scope="module")
def env():
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    h, eri = W.chain_integrals(K, 3)
    pp, pi = W.graph_chain(K)
    inst = nqs.Instance(ctx, K, NA, NB, h, eri, 0.0)
    ans = nqs.Ansatz(ctx, K, NA, NB, CHI, pp, pi, 0)
    ans.bind(W.ansatz_params(K, CHI, pp, pi, 0, 9))
    return nqs, ctx, inst, ans


@pytest.mark.parametrize("N,n_eps", [(1, 0), (4096, 8), (4097, 8), (4097, 0)])
def test_counts(env, N, n_eps):
    nqs, ctx, inst, ans = env
    smp = W.random_onvs(K, NA, NB, N, 5, unique=False)
    kw = dict(eps=0.05, n_eps=n_eps, seed=4)
    _, st = nqs.eloc(ctx, inst, ans, smp, **kw)
    _, sp = nqs.eloc(ctx, inst, ans, smp, max_rows_per_pass=1000, **kw)
    assert st["n_rows"] == N + st["n_det_rows"] + st["n_draw_rows"]
    assert (st["n_draw_rows"] > 0) == (n_eps > 0) or N == 1
    for k in ("n_rows", "n_det_rows", "n_draw_rows", "n_site_rows", "E", "var") if N == 1 else (
            "n_rows", "n_det_rows", "n_draw_rows", "E", "var"):
        assert st[k] == sp[k], k
    assert sp["n_passes"] >= st["n_passes"] == 1


def test_refused_batch_between(env):
    nqs, ctx, inst, ans = env
    smp = W.random_onvs(K, NA, NB, 50, 5, unique=False)
    a, sa = nqs.eloc(ctx, inst, ans, smp)
    bad = smp.copy()
    bad[17, 0] ^= 1
    with pytest.raises(Exception):
        nqs.eloc(ctx, inst, ans, bad)
    b, sb = nqs.eloc(ctx, inst, ans, smp)
    assert torch.equal(a["eloc"], b["eloc"]) and sa["E"] == sb["E"] and sa["n_site_rows"] == sb["n_site_rows"]


def test_threads(env):
    nqs, ctx, inst, ans = env
    batches = [W.random_onvs(K, NA, NB, 100 + 37 * t, 20 + t, unique=False) for t in range(4)]
    want = [nqs.eloc(ctx, inst, ans, s, eps=0.05, n_eps=8, seed=2) for s in batches]
    torch.cuda.synchronize()
    got = [[] for _ in batches]

    def run(t):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(10):
                out, st = nqs.eloc(ctx, inst, ans, batches[t], eps=0.05, n_eps=8, seed=2)
                got[t].append((out["eloc"].cpu().numpy(), st))

    ts = [threading.Thread(target=run, args=(t,)) for t in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for (w, ws), g in zip(want, got):
        assert len(g) == 10
        for e, st in g:
            assert np.array_equal(e, w["eloc"].cpu().numpy())
            for k in ("n_rows", "n_det_rows", "n_draw_rows", "n_site_rows", "E", "psi_flops"):
                assert st[k] == ws[k], k
