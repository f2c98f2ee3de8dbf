"""The bucket form of the dedup at the sizes where it changes shape: one tile and one more or less, the largest and
smallest mini-batch of a size class, with bags that start in the middle of tiles, empty bags, bags longer than a tile, and heavy
keys the hint names, misses, or names in vain.  Unique keys and ranks are compared bit for bit with the oracle's, rows
after the push within the float32 tolerance.  Pooled rows are compared at every step with the float64 pooling of the
rows the table itself holds, bags of up to 4096 occurrences: a bag is added up in runs of eight, so 512 additions,
off by at most 512 * 2^-24 = 3e-5 of the sum of magnitudes if all roundings went one way and by about 1.4e-6 as they
come: within 1e-6 + 1e-5 |x| for sums whose terms do not nearly cancel, and terms below 0.01 where they do."""
import numpy as np
import pytest
import torch

import paper_2003_05622_amd as hps
import oracle
import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


def close(got, want, what):
    err = np.abs(got.astype(np.float64) - want) - (1e-6 + 1e-5 * np.abs(want))
    assert err.max(initial=-1) <= 0, "%s: excess %g" % (what, err.max())


def close_pooled(gt, pooled, uniq, inverse, offsets, mean, what):
    """pooled against the bags' sums or means, in float64, of the rows the table holds (uniq: ascending, inverse: ranks)."""
    rows = gt.get(dev(uniq))[0].cpu().numpy().astype(np.float64)
    total = np.concatenate([np.zeros((1, rows.shape[1])), np.cumsum(rows[inverse], axis=0)])
    lens = np.diff(offsets)
    want = total[offsets[1:]] - total[offsets[:-1]]
    if mean:
        want /= np.maximum(lens, 1)[:, None]
    short = lens <= 4096
    close(pooled.cpu().numpy()[short], want[short], what)


# tiles of 1024 (up to 2^16 occurrences), 4096 (up to 2^20), 8192 (up to 3 * 2^20)
@pytest.mark.parametrize("n", [1, 1023, 1025, 65535, 65537, 4096 * 17 + 1, (1 << 20) + 1])
@pytest.mark.parametrize("bags", ["one", "ragged"])
def test_shapes(n, bags, monkeypatch):
    monkeypatch.setenv("HPS_DEDUP", "bucket")
    rng = np.random.default_rng(n)
    dim = 4
    n_bags = 1 if bags == "one" else max(3, n // 3)
    pool = synth.mix64(rng.integers(0, 2**40, size=max(2, n // 2)).astype(np.uint64))
    gt = hps.HpsTable(4 * n + 100, dim, n, n_bags, lr=0.05)
    ot = oracle.OracleTable(4 * n + 100, dim, lr=0.05)
    gt.set_pooling(bags == "one")            # (a bag of a million rows: its mean stays small)
    ot.set_pooling(bags == "one")
    hot = pool[:3]
    for step in range(4):
        keys = pool[rng.integers(0, pool.size, size=n)]
        # a hot key nobody has announced, the same again, another one, none
        if step < 3:
            keys[rng.random(n) < 0.3] = hot[step // 2]
        if bags == "one":
            offsets = np.array([0, n], np.int32)
        else:
            # many empty bags, a few very long ones
            cuts = np.sort(rng.integers(0, n + 1, size=n_bags - 1))
            cuts[: n_bags // 2] = cuts[n_bags // 2]
            offsets = np.concatenate([[0], np.sort(cuts), [n]]).astype(np.int32)
        pooled = gt.pull(dev(keys), torch.from_numpy(offsets).cuda(), n_bags, 1)
        ot.pull(keys, offsets)
        uniq, inv = gt.last_unique()
        ou, oi = ot.last_unique()
        assert np.array_equal(uniq.cpu().numpy().view(np.uint64), ou), "unique keys, step %d" % step
        assert np.array_equal(inv.cpu().numpy(), oi), "ranks, step %d" % step
        close_pooled(gt, pooled, ou, oi, offsets, bags == "one", "pooled, step %d" % step)
        grads = (rng.integers(-8, 9, size=(n_bags, dim)) / 4096).astype(np.float32)     # sums of these are exact
        gt.push(torch.from_numpy(grads).cuda())
        ot.push(grads)
        st = gt.stats()
        assert st.error == 0 and st.size == ot.size and st.last_n_unique == ou.size
    sample = np.unique(rng.choice(pool, size=min(2000, pool.size)))
    close(gt.get(dev(sample))[1].cpu().numpy(), ot.get(sample)[1], "accumulators")


# the sampled borders: mini-batches below and above the number of samples, both size classes that use them (up to
# 2^16 and up to 2^19 occurrences), the first size beyond; keys the equal parts of a range cannot deal out
@pytest.mark.parametrize("n", [1, 255, 8191, 20_000, 65_536, 65_537, 1 << 19, (1 << 19) + 1])
@pytest.mark.parametrize("form", ["borders", "hashed", "auto"])
def test_bunched_keys(n, form, monkeypatch):
    monkeypatch.setenv("HPS_DEDUP", form)
    rng = np.random.default_rng(n)
    gt = hps.HpsTable(8 * n + 100, 4, n, n, lr=0.05)
    ot = oracle.OracleTable(8 * n + 100, 4, lr=0.05)
    # ragged bags, half of them empty, averaged in one size of two
    n_bags, mean = n, n % 2 == 1
    gt.set_pooling(mean)
    ot.set_pooling(mean)
    # long-tailed raw ids (half of all keys within a thousandth of the range), two crowded places at the
    # ends of the 64 bits, one key over and over, all keys apart
    kinds = [lambda: np.minimum(rng.pareto(1.0, size=n) * 100.0, 1e15).astype(np.uint64),
             lambda: np.where(rng.random(n) < 0.5, rng.integers(0, n + 1, size=n), -2 - rng.integers(0, n + 1, size=n)).astype(np.int64).view(np.uint64),
             lambda: np.full(n, 77, np.uint64),
             lambda: rng.permutation(n).astype(np.uint64)]
    for step, kind in enumerate([0, 0, 0, 0, 0, 0, 1, 2, 3, 0, 1]):
        keys = kinds[kind]()
        offsets = np.concatenate([[0], np.sort(rng.choice(np.arange(0, n + 1, 2), size=n_bags - 1)), [n]]).astype(np.int32)
        pooled = gt.pull(dev(keys), torch.from_numpy(offsets).cuda(), n_bags, 1)
        ot.pull(keys, offsets)
        uniq, inv = gt.last_unique()
        ou, oi = ot.last_unique()
        assert np.array_equal(uniq.cpu().numpy().view(np.uint64), ou), "unique keys, step %d" % step
        assert np.array_equal(inv.cpu().numpy(), oi), "ranks, step %d" % step
        close_pooled(gt, pooled, ou, oi, offsets, mean, "pooled, step %d" % step)
        grads = (rng.integers(-8, 9, size=(n_bags, 4)) / 4096).astype(np.float32)
        gt.push(torch.from_numpy(grads).cuda())
        ot.push(grads)
        st = gt.stats()
        assert st.error == 0 and st.size == ot.size and st.last_n_unique == ou.size
    sample = ou[:: max(1, ou.size // 2000)]
    close(gt.get(dev(sample))[1].cpu().numpy(), ot.get(sample)[1], "accumulators")
    if form != "auto":
        assert gt.stats().n_plain_fallbacks == 0
    elif n >= 8191:
        assert gt.stats().n_plain_fallbacks > 0, "the key range was never given up"


# the borders between the two largest size classes, and between the largest and the plain form
@pytest.mark.parametrize("form", ["bucket", "hashed"])
@pytest.mark.parametrize("n", [3 << 20, (3 << 20) + 1, 12 << 20, (12 << 20) + 1])
def test_large_size_classes(n, form, monkeypatch):
    monkeypatch.setenv("HPS_DEDUP", form)
    rng = np.random.default_rng(n)
    n_bags = n // 8
    gt = hps.HpsTable(n, 4, n, n_bags)
    offsets = (np.arange(n_bags + 1, dtype=np.int64) * n // n_bags).astype(np.int32)
    for step in range(2):            # the second step with a hint
        keys = synth.mix64(rng.integers(0, n // 2, size=n).astype(np.uint64))
        keys[rng.integers(0, n, size=n // 8)] = synth.mix64(np.uint64(10**9))
        pooled = gt.pull(dev(keys), torch.from_numpy(offsets).cuda(), n_bags, 1)
        ou, oi = np.unique(keys, return_inverse=True)
        uniq, inv = gt.last_unique()
        assert np.array_equal(uniq.cpu().numpy().view(np.uint64), ou), "unique keys, step %d" % step
        assert np.array_equal(inv.cpu().numpy(), oi), "ranks, step %d" % step
        close_pooled(gt, pooled, ou, oi, offsets, False, "pooled, step %d" % step)
        gt.push(torch.zeros((n_bags, 4), device="cuda"))
    assert gt.stats().error == 0


@pytest.mark.parametrize("n", [30_000, 1_000_000])
def test_keys_in_arithmetic_progression(n, monkeypatch):
    """Multiples of a number, as ids spread by a multiplication: they fill their range evenly, so the bucket form
    suits them, whatever the number -- here the inverse of the golden ratio's 64-bit fraction (a multiplication
    by that would undo theirs), and the fraction itself with four bits less."""
    monkeypatch.setenv("HPS_DEDUP", "auto")
    rng = np.random.default_rng(n)
    n_bags = n // 8
    gt = hps.HpsTable(3 * n, 4, n, n_bags)
    offsets = (torch.arange(n_bags + 1, device="cuda") * n // n_bags).to(torch.int32)
    for factor in (pow(0x9E3779B97F4A7C15, -1, 2**64), 0x9E3779B97F4A7C1):
        gt.clear()
        for step in range(6):
            keys = rng.permutation(n).astype(np.uint64) * np.uint64(factor)
            gt.pull(dev(keys), offsets, n_bags, 1)
            uniq, inv = gt.last_unique()
            ou, oi = oracle.dedup(keys)
            assert np.array_equal(uniq.cpu().numpy().view(np.uint64), ou) and np.array_equal(inv.cpu().numpy(), oi)
            gt.push(torch.zeros((n_bags, 4), device="cuda"))
            assert gt.stats().error == 0
    assert gt.stats().n_plain_fallbacks == 0, "taken for keys that do not suit the buckets"


@pytest.mark.parametrize("listing", [False, True])
@pytest.mark.parametrize("n", [30_000, 105_000, 530_000, 1_100_000])
def test_uneven_keys_leave_the_key_range(n, listing, monkeypatch):
    """Raw ids, a tenth of the occurrences in a two-hundredth of their range: some buckets by key range overflow, though they
    hold less than an eighth of all occurrences.  Left to itself the library must give the key range up, for buckets by hash, or
    where unique keys are listed for buckets by borders (530 000: the plain form), and go on giving the same results."""
    monkeypatch.setenv("HPS_DEDUP", "auto")
    rng = np.random.default_rng(n)
    n_bags = n // 3
    gt = hps.HpsTable(10 * n, 4, n, n_bags)
    ot = oracle.OracleTable(10 * n, 4)
    offsets = (np.arange(n_bags + 1, dtype=np.int64) * n // n_bags).astype(np.int32)
    for step in range(6):
        ids = np.where(rng.random(n) < 0.1, 7 * n + rng.integers(0, n // 10, size=n), rng.integers(0, 20 * n, size=n)).astype(np.uint64)
        pooled = gt.pull(dev(ids), torch.from_numpy(offsets).cuda(), n_bags, 1)
        close(pooled.cpu().numpy(), ot.pull(ids, offsets), "pooled, step %d" % step)
        if listing or step == 5:
            uniq, inv = gt.last_unique()
            ou, oi = ot.last_unique()
            assert np.array_equal(uniq.cpu().numpy().view(np.uint64), ou), "unique keys, step %d" % step
            assert np.array_equal(inv.cpu().numpy(), oi), "ranks, step %d" % step
        gt.push(torch.zeros((n_bags, 4), device="cuda"))
        ot.push(np.zeros((n_bags, 4), np.float32))
        st = gt.stats()
        assert st.error == 0 and st.size == ot.size and st.last_n_unique == ot.n_unique
    assert gt.stats().n_plain_fallbacks >= 1, "the key range was never given up"
