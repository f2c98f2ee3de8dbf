"""The small form of the dedup, which looks the keys up in the same launch: around the sizes of its tiles, runs and buckets, with
keys that fill buckets, whole waves or a bucket's LDS table and more, raw and hashed; pulled in one call, prepared ahead on
another stream, and accumulated.  Keys and ranks are the oracle's bit for bit; gradients and values are small multiples of 2^-12, so
that sums of them are exact and rows differ by the rounding of the steps alone."""
import numpy as np
import pytest
import torch

import oracle
import paper_2003_05622_amd as hps
import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


def key_hash(k):
    """The hash whose leading bits name a key's bucket."""
    lo, hi = (k & np.uint64(0xFFFFFFFF)).astype(np.uint32), (k >> np.uint64(32)).astype(np.uint32)
    with np.errstate(over="ignore"):
        h = lo ^ (hi * np.uint32(0x9E3779B1))
        h = (h ^ (h >> np.uint32(16))) * np.uint32(0x85EBCA6B)
        return (h ^ (h >> np.uint32(13))) * np.uint32(0xC2B2AE35)


def close(got, want, what):
    err = np.abs(got.astype(np.float64) - want) - (1e-6 + 1e-5 * np.abs(want))
    assert err.max(initial=-1) <= 0, "%s: excess %g" % (what, err.max())


@pytest.fixture(params=["ordered", "ballot"])
def rank(request, monkeypatch):
    monkeypatch.setenv("HPS_DEDUP", "small")
    if request.param == "ballot":
        monkeypatch.setenv("HPS_RANK", "ballot")


def key_mixes(rng, n):
    crowd = synth.mix64(np.arange(400_000, dtype=np.uint64))
    crowd = crowd[key_hash(crowd) >> np.uint32(24) == 3]          # 1500 keys of one bucket: more than its table holds
    ids = lambda most: synth.mix64(rng.integers(0, most, size=n).astype(np.uint64))
    hot = lambda share: np.where(rng.random(n) < share, np.uint64(12345), ids(3 * n))
    return [ids(n), hot(0.12), np.full(n, 77, np.uint64), rng.permutation(n).astype(np.uint64) * np.uint64(5), crowd[rng.integers(0, crowd.size, size=n)],
            np.sort(hot(0.4)), synth.mix64(rng.integers(0, 30, size=n).astype(np.uint64)), rng.permutation(n).astype(np.uint64)]


@pytest.mark.parametrize("how", ["pull", "prepared"])
@pytest.mark.parametrize("n", [1, 15, 1023, 1025, 16_384, 16_385, 40_001, 65_535, 65_536, 65_537])
def test_pull_and_push(n, how, rank):
    rng = np.random.default_rng(n)
    dim, n_bags, mean = 8, max(1, n // 3), n % 2 == 0
    gt, ot = hps.HpsTable(20 * n + 100, dim, n, n_bags), oracle.OracleTable(20 * n + 100, dim)
    gt.set_pooling(mean)
    ot.set_pooling(mean)
    side = torch.cuda.Stream()
    for step, keys in enumerate(key_mixes(rng, n)):
        offsets = np.concatenate([[0], np.sort(rng.integers(0, n + 1, size=n_bags - 1)), [n]]).astype(np.int32)     # many bags empty
        dk, do = dev(keys), torch.from_numpy(offsets).cuda()
        if how == "pull":
            pooled = gt.pull(dk, do, n_bags, 1)
        else:
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                gt.prepare(dk, do, n_bags, 1)
            pooled = gt.pull_prepared()
        want = ot.pull(keys, offsets)
        ou, oi = ot.last_unique()
        st = gt.stats()
        assert st.error == 0 and st.size == ot.size and st.last_n_unique == ou.size and st.last_n_inserted == ot.n_inserted
        if step % 2 == 0:
            uniq, inv = gt.last_unique()
            assert np.array_equal(uniq.cpu().numpy().view(np.uint64), ou) and np.array_equal(inv.cpu().numpy(), oi)
        rows = gt.get(dev(ou))[0].cpu().numpy().astype(np.float64)
        total = np.concatenate([np.zeros((1, dim)), np.cumsum(rows[oi], axis=0)])
        lens = np.diff(offsets)
        close(pooled.cpu().numpy(), (total[offsets[1:]] - total[offsets[:-1]]) / (np.maximum(lens, 1)[:, None] if mean else 1), "pooled")
        if step == 0:
            close(pooled.cpu().numpy(), want, "pooled, against the oracle")
        grads = (rng.integers(-8, 9, size=(n_bags, dim)) / 4096).astype(np.float32)
        gt.push(torch.from_numpy(grads).cuda())
        ot.push(grads)
        ow, oa, _ = ot.get(ou)
        gw, ga, _ = gt.get(dev(ou))
        close(ga.cpu().numpy(), oa, "accumulators, step %d" % step)
        close(gw.cpu().numpy(), ow, "weights, step %d" % step)


@pytest.mark.parametrize("n", [1, 1025, 40_001, 65_536])
def test_accumulate(n, rank):
    rng = np.random.default_rng(n)
    dim = 8
    gt, ot = hps.HpsTable(20 * n + 100, dim, n, 1), oracle.OracleTable(20 * n + 100, dim)
    for step, keys in enumerate(key_mixes(rng, n)):
        known = np.unique(keys)[::2]
        gt.insert(dev(known))
        ot.insert(known)
        values = (rng.integers(-8, 9, size=(n, dim)) / 4096).astype(np.float32)
        gt.accumulate(dev(keys), torch.from_numpy(values).cuda())
        absent = ot.accumulate(keys, values)
        st = gt.stats()
        assert st.error == 0 and st.last_n_absent == absent
        close(gt.get(dev(known))[0].cpu().numpy(), ot.get(known)[0], "weights, step %d" % step)


def test_static_scratch_holds_the_widest_rows():
    n, dim = 1000, 1024
    gt = hps.HpsTable(4 * n, dim, n, 1)
    keys = dev(synth.mix64(np.arange(n, dtype=np.uint64)))
    gt.insert(keys)
    before = gt.get(keys)[0]
    gt.accumulate_static(keys, torch.full((n, dim), 0.5, device="cuda"))
    assert torch.equal(gt.get(keys)[0], before + 0.5) and gt.stats().error == 0


@pytest.mark.parametrize("how", ["pull", "prepared", "accumulate"])
@pytest.mark.parametrize("n", [1, 1025, 40_001])
def test_reserved_key(n, how, rank):
    """Refused by the dedup itself: nothing of the mini-batch gets into the table."""
    rng = np.random.default_rng(n)
    dim, n_bags = 8, max(1, n // 3)
    gt = hps.HpsTable(20 * n + 100, dim, n, n_bags)
    known = synth.mix64(np.arange(n, dtype=np.uint64))
    gt.insert(dev(known))
    before = gt.get(dev(known))[0]
    keys = synth.mix64(rng.integers(0, 2 * n, size=n).astype(np.uint64))
    keys[rng.integers(0, n)] = np.uint64(2**64 - 1)
    offsets = torch.from_numpy((np.arange(n_bags + 1, dtype=np.int64) * n // n_bags).astype(np.int32)).cuda()
    if how == "pull":
        gt.pull(dev(keys), offsets, n_bags, 1)
    elif how == "prepared":
        gt.prepare(dev(keys), offsets, n_bags, 1)
        gt.pull_prepared()
    else:
        gt.accumulate(dev(keys), torch.ones((n, dim), device="cuda"))
    assert gt.stats().error == hps.ERESERVED
    gt.clear_error()
    assert gt.stats().size == n and torch.equal(gt.get(dev(known))[0], before)
    keys = known[rng.integers(0, n, size=n)]
    gt.pull(dev(keys), offsets, n_bags, 1)
    assert gt.stats().error == 0 and gt.stats().size == n
