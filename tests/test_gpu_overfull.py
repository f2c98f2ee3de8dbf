"""Pulls that end with more keys than the table's capacity: nothing of them stays in the table, whatever the dedup's form, and
pulls that just fit go through.  Bags of 18 to 100 initial rows |w| <= 0.01, changed by few steps: sums of at most 100 terms,
within the float32 tolerance of the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2003_05622_amd as hps
import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


@pytest.mark.parametrize("form", ["auto", "bucket", "hashed", "small", "radix"])
@pytest.mark.parametrize("n", [900, 5000, 70_000])
def test_overfull_pulls_leave_no_trace(n, form, monkeypatch):
    monkeypatch.setenv("HPS_DEDUP", form)
    dim, n_bags, cap = 4, max(50, n // 100), 5 * n - n // 3        # (n is less than a quarter of the capacity)
    rng = np.random.default_rng(n)
    gt, ot = hps.HpsTable(cap, dim, n, n_bags), oracle.OracleTable(cap, dim)
    offsets = (np.arange(n_bags + 1, dtype=np.int64) * n // n_bags).astype(np.int32)
    d_offsets = torch.from_numpy(offsets).cuda()

    def ids(first, last):
        return synth.mix64(np.arange(first, last, dtype=np.uint64))

    def pull(keys, fits):
        pooled = gt.pull(dev(keys), d_offsets, n_bags, 1)
        st = gt.stats()
        if not fits:
            assert st.error == hps.EFULL and st.size == ot.size
            gt.clear_error()
            assert gt.stats().size == ot.size
            found = gt.get(dev(keys))[2].cpu().numpy()
            assert np.array_equal(found, ot.get(keys)[2])
            return
        want = ot.pull(keys, offsets)
        assert st.error == 0 and st.size == ot.size
        assert np.all(np.abs(pooled.cpu().numpy() - want) <= 1e-6 + 1e-5 * np.abs(want))
        grads = rng.normal(size=(n_bags, dim)).astype(np.float32) * 1e-3
        gt.push(torch.from_numpy(grads).cuda())
        ot.push(grads)

    at = 0
    while ot.size + n <= cap:
        pull(ids(at, at + n), True)
        at += n
    room = cap - ot.size
    pull(rng.permutation(np.concatenate([ids(at, at + room + 1), ids(0, n - room - 1)])), False)
    pull(rng.permutation(np.resize(ids(at, at + room - 3), n)), True)
    pull(rng.permutation(np.resize(ids(at, at + room + 1), n)), False)
    pull(rng.permutation(np.resize(ids(at, at + room), n)), True)
    pull(rng.permutation(np.resize(ids(at, at + room), n)), True)
    pull(rng.permutation(np.resize(ids(at, at + room + 1), n)), False)
    k, w, a = gt.dump()
    order = np.argsort(k.cpu().numpy().view(np.uint64))
    ok, ow, oa = ot.dump()
    assert np.array_equal(k.cpu().numpy().view(np.uint64)[order], ok)
    assert np.all(np.abs(w.cpu().numpy()[order] - ow) <= 1e-6 + 1e-5 * np.abs(ow))
    assert np.all(np.abs(a.cpu().numpy()[order] - oa) <= 1e-6 + 1e-5 * np.abs(oa))


@pytest.mark.parametrize("form", ["auto", "hashed", "bucket", "radix"])
@pytest.mark.parametrize("n", [5000, 70_000])
def test_overfull_while_the_next_mini_batch_fails(n, form, monkeypatch):
    """A prepared pull ends above the capacity, or just fits, and the mini-batch prepared beside it holds the reserved key: its
    error comes before, in the midst of or after the pull's kernels, by how long either stream sleeps.  Whatever is left undone,
    no key that was in the table goes missing, and all that are in it are counted."""
    monkeypatch.setenv("HPS_DEDUP", form)
    dim, n_bags, cap = 4, n // 100, 5 * n
    rng = np.random.default_rng(n)
    gt = hps.HpsTable(cap, dim, n, n_bags)
    d_offsets = torch.from_numpy((np.arange(n_bags + 1, dtype=np.int64) * n // n_bags).astype(np.int32)).cuda()
    side, zero = torch.cuda.Stream(), torch.zeros((n_bags, dim), device="cuda")
    ids = lambda first, last: synth.mix64(np.arange(first, last, dtype=np.uint64))
    known, at = ids(0, cap - n), cap - n
    gt.insert(dev(known))
    reserved = rng.permutation(known)[:n].copy()
    reserved[::101] = np.uint64(2**64 - 1)
    d_reserved = dev(reserved)
    errors = set()
    for turn in range(30):
        room = cap - known.size
        new = room // 4 if turn % 2 else n                # fits, and leaves its marks; or does not
        keys = rng.permutation(np.concatenate([ids(at, at + new), known[: n - new]]))
        at += new
        d_keys = dev(keys)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            gt.prepare(d_keys, d_offsets, n_bags, 1)
        torch.cuda._sleep(100_000)
        gt.pull_prepared()
        with torch.cuda.stream(side):
            if turn % 3:
                torch.cuda._sleep(30_000 + 5000 * turn)
            gt.prepare(d_reserved, d_offsets, n_bags, 1)
        torch.cuda.synchronize()
        errors.add(gt.stats().error)
        gt.clear_error()
        size = gt.stats().size
        stored = gt.dump(max_rows=size)[0].cpu().numpy().view(np.uint64)
        assert size <= cap and stored.size == size and np.unique(stored).size == size
        assert np.isin(known, stored).all() and np.isin(stored, np.concatenate([known, keys])).all()
        known = stored
        # a pull beside nothing: what is stored is found, with its initial rows
        pooled = gt.pull(dev(stored[:n]), d_offsets, n_bags, 1)
        rows = gt.get(dev(stored[:n]))[0]
        gt.push(zero)
        assert gt.stats().error == 0 and gt.stats().size == size
        torch.testing.assert_close(pooled, rows.reshape(n_bags, -1, dim).sum(dim=1), rtol=1e-5, atol=1e-6)
    assert hps.ERESERVED in errors


@pytest.mark.parametrize("form", ["auto", "small", "hashed", "bucket", "radix"])
@pytest.mark.parametrize("n", [900, 5000, 70_000])
def test_marks_of_earlier_pulls_are_not_rolled_back(n, form, monkeypatch):
    """The state in which an error finds a pull whose first blocks have created more than fits, put there by hand: the error is
    set and keys are counted as created before the lookup runs, so that all its blocks stop and leave the marks and rows of the pulls
    before, which fitted.  Their keys stay."""
    monkeypatch.setenv("HPS_DEDUP", form)
    dim, n_bags, cap = 4, max(9, n // 100), 5 * n
    rng = np.random.default_rng(n)
    gt = hps.HpsTable(cap, dim, n, n_bags)
    d_offsets = torch.from_numpy((np.arange(n_bags + 1, dtype=np.int64) * n // n_bags).astype(np.int32)).cuda()
    zero = torch.zeros((n_bags, dim), device="cuda")
    ids = lambda first, last: synth.mix64(np.arange(first, last, dtype=np.uint64))
    at = cap - n + n // 10
    gt.insert(dev(ids(0, at)))
    for _ in range(4):                                    # (above the capacity if all its occurrences were new keys: marked)
        new = n // 10
        gt.pull(dev(rng.permutation(np.concatenate([ids(at, at + new), ids(0, n - new)]))), d_offsets, n_bags, 1)
        gt.push(zero)
        at += new
    stored = ids(0, at)
    # the table's state lies at the end of its storage: size, rows created last; the error after these; the counts of created rows
    state = gt.storage[-1280:].view(torch.int32)
    assert gt.stats().size == at and state[:4].tolist() == [at, 0, n // 10, 0] and state[4] == 0
    for _ in range(3):                                    # (both contexts, both sets of counts)
        gt.prepare(dev(rng.permutation(stored)[:n]), d_offsets, n_bags, 1)
        state[4] = hps.ERESERVED
        state[136] = state[200] = 2 * n
        gt.pull_prepared()
        assert gt.stats().error == hps.ERESERVED
        gt.clear_error()
        assert gt.stats().size == at and gt.get(dev(stored))[2].all()
    keys = gt.dump()[0].cpu().numpy().view(np.uint64)
    assert np.array_equal(np.sort(keys), np.sort(stored))
    keys = rng.permutation(stored)[:n]
    pooled = gt.pull(dev(keys), d_offsets, n_bags, 1)
    gt.push(zero)
    total = torch.cat([torch.zeros((1, dim), dtype=torch.float64, device="cuda"), gt.get(dev(keys))[0].double().cumsum(dim=0)])[d_offsets.long()]
    torch.testing.assert_close(pooled, (total[1:] - total[:-1]).float(), rtol=1e-5, atol=1e-6)
    assert gt.stats().error == 0 and gt.stats().size == at
