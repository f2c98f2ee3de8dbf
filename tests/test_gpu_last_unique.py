"""hps_last_unique on streams of its own: beside the pull whose keys it lists, beside the push and the next
pull, after a pull that failed on the device, and replayed from a captured graph.  Keys and ranks are the oracle's bit for bit; the pushes carry zero
gradients, so the rows stay the initial ones and pooled sums stay within the float32 tolerance of the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2003_05622_amd as hps
import synth

pytestmark = pytest.mark.gpu

FORMS = ["auto", "bucket", "borders", "hashed", "radix"]


@pytest.fixture(params=FORMS)
def form(request, monkeypatch):
    monkeypatch.setenv("HPS_DEDUP", request.param)
    return request.param


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


def batch(rng, n, hot):
    keys = synth.mix64(rng.integers(0, n, size=n).astype(np.uint64))
    keys[rng.random(n) < 0.2] = synth.mix64(np.uint64(10**9 + hot))          # named by the hint from the third step on
    return keys


def even_offsets(n, n_bags):
    return (np.arange(n_bags + 1, dtype=np.int64) * n // n_bags).astype(np.int32)


@pytest.mark.parametrize("n", [5000, 200_000])
def test_beside_the_pull_and_the_next_one(form, n):
    rng = np.random.default_rng(n)
    dim, n_bags, steps = 8, n // 8, 7
    gt = hps.HpsTable(20 * n, dim, n, n_bags)
    ot = oracle.OracleTable(20 * n, dim)
    offsets = even_offsets(n, n_bags)
    keys = [batch(rng, n - 3 * i, i // 5) for i in range(steps)]
    offs = [np.minimum(offsets, k.size).astype(np.int32) for k in keys]
    dk, do = [dev(k) for k in keys], [torch.from_numpy(o).cuda() for o in offs]
    uniq = [torch.zeros(n, dtype=torch.int64, device="cuda") for _ in keys]
    inv = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in keys]
    zero = torch.zeros((n_bags, dim), device="cuda")
    side, third = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    pooled = []
    with torch.cuda.stream(side):
        gt.prepare(dk[0], do[0], n_bags, 1)
    for i in range(steps):
        torch.cuda._sleep(1_000_000)                     # the pull starts well after the calls below are enqueued
        pooled.append(gt.pull_prepared())
        # on the stream of the prepare, before the pull has run; every other time on a stream that has seen nothing
        s = third if i % 2 else side
        assert hps.lib().hps_last_unique(gt._h, uniq[i].data_ptr(), inv[i].data_ptr(), s.cuda_stream) == hps.OK
        if i + 1 < steps:
            with torch.cuda.stream(side):
                gt.prepare(dk[i + 1], do[i + 1], n_bags, 1)
        gt.push(zero)
    torch.cuda.synchronize()
    assert gt.stats().error == 0
    for i in range(steps):
        want = ot.pull(keys[i], offs[i])
        ou, oi = ot.last_unique()
        ot.push(np.zeros((n_bags, dim), np.float32))
        assert np.array_equal(uniq[i].cpu().numpy().view(np.uint64)[: ou.size], ou), "unique keys, step %d" % i
        assert np.array_equal(inv[i].cpu().numpy()[: keys[i].size], oi), "ranks, step %d" % i
        err = np.abs(pooled[i].cpu().numpy() - want) - (1e-6 + 1e-5 * np.abs(want))
        assert err.max() <= 0, "pooled, step %d: excess %g" % (i, err.max())


def test_replayed_from_a_graph(form):
    """The captured call lists whatever mini-batch of the same size is outstanding when it is replayed."""
    rng = np.random.default_rng(3)
    n, n_bags, dim = 30_000, 1000, 4
    gt = hps.HpsTable(20 * n, dim, n, n_bags)
    offsets = torch.from_numpy(even_offsets(n, n_bags)).cuda()
    uniq = torch.zeros(n, dtype=torch.int64, device="cuda")
    inv = torch.zeros(n, dtype=torch.int32, device="cuda")
    zero = torch.zeros((n_bags, dim), device="cuda")
    graph, stream = None, torch.cuda.Stream()
    for step in range(8):
        keys = batch(rng, n, 0)
        gt.pull(dev(keys), offsets, n_bags, 1)
        if step == 3:                  # (the first two dedups of a table take the plain form)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                assert hps.lib().hps_last_unique(gt._h, uniq.data_ptr(), inv.data_ptr(), stream.cuda_stream) == hps.OK
        if graph is not None:
            uniq.fill_(-1)
            inv.fill_(-1)
            graph.replay()
            torch.cuda.synchronize()
            ou, oi = oracle.dedup(keys)
            assert np.array_equal(uniq.cpu().numpy().view(np.uint64)[: ou.size], ou), "unique keys, step %d" % step
            assert np.array_equal(inv.cpu().numpy(), oi), "ranks, step %d" % step
        gt.push(zero)
    assert gt.stats().error == 0


def test_replayed_after_a_capture_by_hash(monkeypatch):
    """Raw ids crowded in a part of their range: by hash on the third dedup after a listing, when nobody is taken not to list yet.
    The mini-batches after the capture keep to that."""
    monkeypatch.delenv("HPS_DEDUP", raising=False)
    rng = np.random.default_rng(5)
    n, n_bags, dim = 30_000, 1000, 4
    gt = hps.HpsTable(20 * n, dim, n, n_bags)
    offsets = torch.from_numpy(even_offsets(n, n_bags)).cuda()
    uniq = torch.zeros(n, dtype=torch.int64, device="cuda")
    inv = torch.zeros(n, dtype=torch.int32, device="cuda")
    zero = torch.zeros((n_bags, dim), device="cuda")
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    for step in range(16):
        keys = rng.integers(0, 10**9, size=n).astype(np.uint64)
        keys[rng.random(n) < 0.4] = rng.integers(0, 5000, dtype=np.uint64) + np.uint64(7000)
        crowd = rng.random(n) < 0.5
        keys[crowd] = rng.integers(10**6, 2 * 10**6, size=int(crowd.sum())).astype(np.uint64)
        gt.pull(dev(keys), offsets, n_bags, 1)
        ou, oi = oracle.dedup(keys)
        if step == 2:
            u, i = gt.last_unique()
            assert np.array_equal(u.cpu().numpy().view(np.uint64), ou) and np.array_equal(i.cpu().numpy(), oi)
        if step == 5:
            torch.cuda.synchronize()
            with torch.cuda.graph(graph, stream=stream):
                assert hps.lib().hps_last_unique(gt._h, uniq.data_ptr(), inv.data_ptr(), stream.cuda_stream) == hps.OK
        if step >= 5:
            uniq.fill_(-1)
            inv.fill_(-1)
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(uniq.cpu().numpy().view(np.uint64)[: ou.size], ou), "unique keys, step %d" % step
            assert np.array_equal(inv.cpu().numpy(), oi), "ranks, step %d" % step
        gt.push(zero)
        gt.stats()                # (what the lookup has to report arrives)
    st = gt.stats()
    assert st.error == 0 and st.n_plain_fallbacks > 0


@pytest.mark.parametrize("n", [300, 70_000])
def test_after_a_pull_that_failed(form, n):
    """A table with no room for the mini-batch's keys, a mini-batch with the reserved key in it, and one that is pulled
    while the status is still set: keys and ranks are listed all the same."""
    rng = np.random.default_rng(n)
    n_bags, dim = 16, 4
    gt = hps.HpsTable(max(64, n // 100), dim, n, n_bags)
    offsets = torch.from_numpy(even_offsets(n, n_bags)).cuda()

    def listed(keys):
        gt.pull(dev(keys), offsets, n_bags, 1)
        uniq, inv = gt.last_unique()
        ou, oi = oracle.dedup(keys)
        assert gt.stats().last_n_unique == ou.size
        assert np.array_equal(uniq.cpu().numpy().view(np.uint64), ou) and np.array_equal(inv.cpu().numpy(), oi)
        return gt.stats().error

    few = synth.mix64(np.arange(30, dtype=np.uint64))
    for _ in range(3):              # frequent keys that the next steps' hint names
        assert listed(few[rng.integers(0, 30, size=n)]) == 0
        gt.push(torch.zeros((n_bags, dim), device="cuda"))
    full = batch(rng, n, 0)
    full[: n // 4] = few[0]
    assert listed(full) == hps.EFULL
    gt.push(torch.zeros((n_bags, dim), device="cuda"))
    assert listed(full[::-1].copy()) == hps.EFULL          # (still set: nothing is looked up)
    gt.clear_error()
    reserved = few[rng.integers(0, 30, size=n)]
    reserved[rng.integers(0, n, size=5)] = np.uint64(2**64 - 1)
    assert listed(reserved) == hps.ERESERVED
    gt.clear_error()
    assert gt.stats().size == 30
