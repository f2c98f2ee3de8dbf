"""A table whose calls come on one stream, and then on several: the order between its calls holds from the first call on
another stream on, also if the first stream has been destroyed by then, with work left on it.  Gradients are small multiples of 2^-12, so that sums of them
are exact; a row that missed a push, or took another key's, is off by 10^-5 and more.  Weights and accumulators at the float32
tolerance of the oracle's, pooled sums of ten rows at ten times that of a row (|w| < 0.1)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2003_05622_amd as hps
import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


@pytest.mark.parametrize("form", ["auto", "small", "hashed", "bucket"])
@pytest.mark.parametrize("first", ["default", "torch", "destroyed"])
def test_from_one_stream_to_several(first, form, monkeypatch):
    monkeypatch.setenv("HPS_DEDUP", form)
    rng = np.random.default_rng(1)
    n, n_bags, dim, steps = 20_000, 2000, 8, 12
    keys = [synth.mix64(rng.integers(0, n, size=n).astype(np.uint64)) for _ in range(steps)]
    offsets = (np.arange(n_bags + 1, dtype=np.int64) * n // n_bags).astype(np.int32)
    dk, do = [dev(k) for k in keys], torch.from_numpy(offsets).cuda()
    pooled = [torch.empty((n_bags, dim), device="cuda") for _ in keys]
    grads = [(rng.integers(-8, 9, size=(n_bags, dim)) / 4096).astype(np.float32) for _ in keys]
    dg = [torch.from_numpy(g).cuda() for g in grads]
    gt, ot = hps.HpsTable(20 * n, dim, n, n_bags), oracle.OracleTable(20 * n, dim)
    hip, raw = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p()
    if first == "default":
        a = torch.cuda.default_stream()
    elif first == "torch":
        a = torch.cuda.Stream()
    else:
        assert hip.hipStreamCreate(ctypes.byref(raw)) == 0
        a = torch.cuda.ExternalStream(raw.value)
    b, c = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    uniq, inv = torch.zeros(n, dtype=torch.int64, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    with torch.cuda.stream(a):
        for i in range(6):
            torch.cuda._sleep(300_000)
            gt.pull(dk[i], do, n_bags, 1, pooled[i])
            gt.push(dg[i])
    if first == "destroyed":
        assert hip.hipStreamDestroy(raw) == 0
        a = torch.cuda.Stream()
    # prepared beside the last calls above, pulled and listed elsewhere
    with torch.cuda.stream(b):
        gt.prepare(dk[6], do, n_bags, 1)
    for i in range(6, steps):
        with torch.cuda.stream(c if i % 2 else a):
            torch.cuda._sleep(300_000)
            gt.pull_prepared(pooled[i])
        if i == 8:
            assert hps.lib().hps_last_unique(gt._h, uniq.data_ptr(), inv.data_ptr(), b.cuda_stream) == hps.OK
        if i + 1 < steps:
            with torch.cuda.stream(b):
                gt.prepare(dk[i + 1], do, n_bags, 1)
        with torch.cuda.stream(a if i % 2 else c):          # (the push reads what the pull on the other stream left)
            (a if i % 2 else c).wait_stream(c if i % 2 else a)
            gt.push(dg[i])
    torch.cuda.synchronize()
    assert gt.stats().error == 0
    for i in range(steps):
        want = ot.pull(keys[i], offsets)
        ou, oi = ot.last_unique()
        ot.push(grads[i])
        assert np.abs(pooled[i].cpu().numpy() - want).max() <= 2e-5, "step %d" % i
        if i == 8:
            assert np.array_equal(uniq.cpu().numpy().view(np.uint64)[: ou.size], ou) and np.array_equal(inv.cpu().numpy(), oi)
    assert gt.stats().size == ot.size
    every = np.unique(np.concatenate(keys))
    gw, ga, found = gt.get(dev(every))
    ow, oa, _ = ot.get(every)
    assert found.all()
    assert np.all(np.abs(gw.cpu().numpy() - ow) <= 1e-6 + 1e-5 * np.abs(ow)), "weights"
    assert np.all(np.abs(ga.cpu().numpy() - oa) <= 1e-6 + 1e-5 * np.abs(oa)), "accumulators"


def test_first_call_on_another_stream_while_a_third_one_is_captured():
    """It neither fails nor breaks the capture, and comes after the calls before it."""
    n, n_bags, dim = 5000, 500, 8
    gt = hps.HpsTable(4 * n, dim, n, n_bags)
    keys = synth.mix64(np.arange(n, dtype=np.uint64))
    dk, do = dev(keys), torch.from_numpy((np.arange(n_bags + 1, dtype=np.int64) * n // n_bags).astype(np.int32)).cuda()
    one, pooled = torch.ones((n_bags, dim), device="cuda"), torch.empty((n_bags, dim), device="cuda")
    x, graph, captured, other = torch.zeros(1000, device="cuda"), torch.cuda.CUDAGraph(), torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    gt.pull(dk, do, n_bags, 1, pooled)
    torch.cuda._sleep(1_000_000)
    gt.push(one)
    s = other.cuda_stream
    with torch.cuda.graph(graph, stream=captured):
        x.add_(1)
        assert hps.lib().hps_pull(gt._h, dk.data_ptr(), n, do.data_ptr(), n_bags, 1, pooled.data_ptr(), s) == hps.OK
        x.add_(1)
    torch.cuda.synchronize()
    # two orders of summing ten rows, all sums below 1: at most ten roundings of 2^-25 each way; a pull that came before its push is off by 0.4
    assert (gt.get(dk)[0].reshape(n_bags, -1, dim).sum(dim=1) - pooled).abs().max() <= 20 * 2.0**-25
    for turn in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, torch.full_like(x, 2.0 * turn + 2))
    assert gt.stats().error == 0
