"""GPU test of a bind that runs out of device memory part way (allocation hook): the
work it had queued is complete when the call returns, the ansatz refuses calls, and
the next bind, on another stream, gives the results of an ansatz bound once."""
import pytest
import torch

from paper_2507_19276_amd import workloads as W

pytestmark = pytest.mark.gpu
K, CHI = 50, 64


def test_failed_bind_leaves_nothing_queued():
    from paper_2507_19276_amd import nqs
    ctx = nqs.Context(0)
    pp, pi = W.graph_nn_nnn(K)
    prm = torch.from_numpy(W.ansatz_params(K, CHI, pp, pi, 0, 3)).cuda()
    smp = W.random_onvs(K, 25, 25, 40, 1)
    once = nqs.Ansatz(ctx, K, 25, 25, CHI, pp, pi, 0).bind(prm)
    want = {p: once.logpsi(smp, p)[0] for p in ("f64", "f32", "bf16")}
    ans = nqs.Ansatz(ctx, K, 25, 25, CHI, pp, pi, 0)
    stream = torch.cuda.Stream()
    idle, failed = [], 0
    while True:
        # the buffers that the failed binds got stay: the next fails one further on
        ctx.fail_alloc_at(1 if failed == 0 else 2)
        with torch.cuda.stream(stream):
            try:
                ans.bind(prm)
                break
            except nqs.NqsError as e:
                assert e.code == nqs.NQS_ENOMEM
                idle.append(stream.query())
        failed += 1
        with pytest.raises(nqs.NqsError, match="not bound"):
            ans.logpsi(smp, "f64")
    ctx.fail_alloc_at(0)
    assert failed > 10 and all(idle)
    ans.bind(prm)
    for p in want:
        assert torch.equal(ans.logpsi(smp, p)[0], want[p]), p
