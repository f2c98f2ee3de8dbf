"""The push at the numbers of occurrences where a key changes hands: one lane group (up to 16), one wave, one block,
several blocks whose last one adds up the partial sums.  The limits depend on the row's width and on the size of
the mini-batch.  Gradients are multiples of 2^-12 below 2^-9 and a key has at most 2^13 of them, so every float32 sum is
exact in any order, and what is left is one Adagrad step: weights and accumulators within 1e-6 + 1e-5 |x|."""
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


@pytest.mark.parametrize("dim,fill", [(4, 0), (16, 0), (32, 0), (64, 0), (100, 0), (256, 0), (260, 0), (64, 1 << 19)])
@pytest.mark.parametrize("form", ["radix", "bucket", "borders", "hashed"])
def test_piece_edges(dim, fill, form, monkeypatch):
    monkeypatch.setenv("HPS_DEDUP", form)
    rng = np.random.default_rng(dim + fill)
    edges = (1, 16, 64, 128, 256, 512, 1024, 2048, 4096)
    lens = [e + d for e in edges for d in (0, 1)] + [1025 * 3, 6000]
    keys = synth.mix64(np.arange(len(lens), dtype=np.uint64))
    occ = np.repeat(keys, lens)
    rest = synth.mix64(np.arange(1000, 1000 + max(fill, 50), dtype=np.uint64))        # keys that occur once
    n = occ.size + rest.size
    n_bags = n // 2
    gt = hps.HpsTable(2 * n, dim, n, n_bags, lr=0.05)
    ot = oracle.OracleTable(2 * n, dim, lr=0.05)
    probe = np.concatenate([keys, rest[:100]])
    for step in range(3):         # (the counters of finished chunks start anew with every mini-batch)
        batch = rng.permutation(np.concatenate([occ, rest]))
        offsets = np.sort(rng.integers(0, n + 1, size=n_bags + 1)).astype(np.int32)
        offsets[0], offsets[-1] = 0, n
        gt.pull(dev(batch), torch.from_numpy(offsets).cuda(), n_bags, 1)
        ot.pull(batch, offsets)
        grads = (rng.integers(-7, 8, size=(n_bags, dim)) / 4096).astype(np.float32)
        gt.push(torch.from_numpy(grads).cuda())
        ot.push(grads)
        w, acc = gt.get(dev(probe))[:2]
        want_w, want_acc = ot.get(probe)[:2]
        close(w.cpu().numpy(), want_w, "weights, step %d" % step)
        close(acc.cpu().numpy().reshape(want_acc.shape), want_acc, "accumulators, step %d" % step)
