"""Mini-batches with many more bags than key occurrences, in every form of the dedup: the number of bags beside a tile of
occurrences at which the bucket form stops going through all of them and searches (96 per thread: 24576 beside the 1024
occurrences of the smallest tiles, 49152 beside the next larger 4096), one less and one more, and far beyond.  Rows
and gradients are multiples of small powers of two, so every sum is exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2003_05622_amd as hps
import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


@pytest.mark.parametrize("form", ["bucket", "hashed", "radix"])
@pytest.mark.parametrize("n,n_bags", [(1, 30_000), (1000, 24_576), (1000, 24_577), (1000, 24_578), (1024, 100_000), (3000, 70_000),
                                      (3000, 300_000), (70_000, 72_000), (70_000, 840_000), (70_000, 2_000_000)])
def test_sparse_bags(n, n_bags, form, monkeypatch):
    monkeypatch.setenv("HPS_DEDUP", form)
    rng = np.random.default_rng(n + n_bags)
    dim = 4
    pool = synth.mix64(np.arange(max(2, n // 3), dtype=np.uint64))
    w = (rng.integers(-64, 65, size=(pool.size, dim)) / 64).astype(np.float32)
    gt = hps.HpsTable(4 * n + 100, dim, n, n_bags, lr=0.05)
    ot = oracle.OracleTable(4 * n + 100, dim, lr=0.05)
    for step, kind in enumerate(["apart", "clumped", "first and last"]):
        gt.clear()
        gt.insert(dev(pool), torch.from_numpy(w).cuda())
        ot = oracle.OracleTable(4 * n + 100, dim, lr=0.05)
        ot.insert(pool, w)
        keys = pool[rng.integers(0, pool.size, size=n)]
        if kind == "apart":              # bags of one here and there
            bag_of = np.sort(rng.integers(0, n_bags, size=n))
        elif kind == "clumped":          # a few bags of up to sixteen
            bag_of = np.sort(np.repeat(rng.integers(0, n_bags, size=n // 16 + 1), 16)[:n])
        else:
            bag_of = np.sort(rng.integers(0, 2, size=n) * (n_bags - 1))[:n]
        offsets = np.searchsorted(bag_of, np.arange(n_bags + 1)).astype(np.int32)
        pooled = gt.pull(dev(keys), torch.from_numpy(offsets).cuda(), n_bags, 1)
        want = ot.pull(keys, offsets)
        assert np.array_equal(pooled.cpu().numpy(), want.astype(np.float32)), "pooled, " + kind
        grads = (rng.integers(-8, 9, size=(n_bags, dim)) / 4096).astype(np.float32)
        gt.push(torch.from_numpy(grads).cuda())
        ot.push(grads)
        got, ref = gt.get(dev(pool)), ot.get(pool)
        for a, b, what in ((got[0], ref[0], "weights"), (got[1], ref[1], "accumulators")):
            err = np.abs(a.cpu().numpy() - b.reshape(a.shape)) - (1e-6 + 1e-5 * np.abs(b.reshape(a.shape)))
            assert err.max() <= 0, "%s, %s: excess %g" % (what, kind, err.max())
        assert gt.stats().error == 0
