"""insert, get and dump on the GPU at the sizes where moving rows by waves of 64 keys can go wrong:
one key, a wave and one key more or less, a block, a dump's round of slots; row widths that do and do not divide a
wave; rows that exist, are new, or come twice; a table with and without room for all of them."""
import numpy as np
import pytest
import torch

import paper_2003_05622_amd as hps
import synth
from oracle import OracleTable

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


@pytest.mark.parametrize("opt", [hps.ADAGRAD_ROWWISE, hps.ADAGRAD_ELEMENTWISE])
@pytest.mark.parametrize("dim,rows", [(4, hps.ROWS_F32), (12, hps.ROWS_BF16), (100, hps.ROWS_F32_WIDE), (260, hps.ROWS_F32)])
@pytest.mark.parametrize("n", [1, 63, 65, 257, 1025])
def test_rows_in_and_out(n, dim, rows, opt):
    # values pass through unchanged (bfloat16: multiples of 2^-6 below 2 are exact), so every comparison is exact
    rng = np.random.default_rng(n + dim)
    acc_len = 1 if opt == hps.ADAGRAD_ROWWISE else dim
    kw = dict(opt=opt, init_acc=0.25, init_seed=7, row_format=rows)
    capacity = 3 * n + 2
    gt = hps.HpsTable(capacity, dim, 4 * n, 4, **kw)
    ot = OracleTable(capacity, dim, opt=opt, init_acc=0.25, init_seed=7,
                     row_format=1 if rows == hps.ROWS_BF16 else 0)
    keys = synth.mix64(np.arange(3 * n, dtype=np.uint64))
    w = (rng.integers(-127, 128, size=(2 * n, dim)) / 64).astype(np.float32)
    a = rng.integers(0, 100, size=(2 * n, acc_len)).astype(np.float32)

    def same():
        probe = np.concatenate([keys, keys[::-1], synth.mix64(np.arange(10**6, 10**6 + n, dtype=np.uint64))])
        got, want = [x.cpu().numpy() for x in gt.get(dev(probe))], ot.get(probe)
        assert np.array_equal(got[2], want[2])
        found = want[2]
        assert np.array_equal(got[0][found], want[0][found]) and np.array_equal(got[1][found], want[1][found])
        assert not got[0][~found].any() and not got[1][~found].any()         # left as they were
        k, dw, da = [x.cpu().numpy() for x in gt.dump()]
        k = k.view(np.uint64)
        order = np.argsort(k)
        ok, ow, oa = ot.dump()
        assert np.array_equal(k[order], ok) and np.array_equal(dw[order], ow) and np.array_equal(da[order], oa)
        assert gt.stats().size == ot.size and gt.stats().error == 0

    gt.insert(dev(keys[:n]), torch.from_numpy(w[:n]).cuda(), torch.from_numpy(a[:n]).cuda())
    ot.insert(keys[:n], w[:n], a[:n])
    same()
    # overwritten and new rows, accumulators at their initial value; the table has room for them as new keys
    gt.insert(dev(keys[n // 2: n // 2 + n]), torch.from_numpy(w[n:]).cuda())
    ot.insert(keys[n // 2: n // 2 + n], w[n:])
    same()
    # initial rows, every key twice (counted twice for the room check: fits) and then, without room
    # for all of them as new keys, by the second kernel
    twice = np.concatenate([keys[n: n + n // 2]] * 2)
    for more in (twice, keys):
        gt.insert(dev(more))
        ot.insert(np.unique(more))
        same()
    # a caller's arrays need no more than four-byte alignment
    out = torch.zeros(3 * n * dim + 1, device="cuda")
    acc = torch.zeros(3 * n * acc_len + 1, device="cuda")
    flags = torch.zeros(3 * n, dtype=torch.uint8, device="cuda")
    L = hps.lib()
    assert L.hps_get(gt._h, dev(keys).data_ptr(), 3 * n, out.data_ptr() + 4, acc.data_ptr() + 4, flags.data_ptr(), 0) == hps.OK
    torch.cuda.synchronize()
    want = ot.get(keys)
    # hps_get leaves absent keys' rows alone
    absent = dev(synth.mix64(np.arange(10**6, 10**6 + n, dtype=np.uint64)))
    rows, accs = torch.full((n, dim), 7.0, device="cuda"), torch.full((n, acc_len), 7.0, device="cuda")
    left = torch.ones(n, dtype=torch.uint8, device="cuda")
    assert L.hps_get(gt._h, absent.data_ptr(), n, rows.data_ptr(), accs.data_ptr(), left.data_ptr(), 0) == hps.OK
    assert (rows == 7).all() and (accs == 7).all() and not left.any()
    # while the sticky status is set nothing is found
    gt.insert(dev(np.array([2**64 - 1], dtype=np.uint64)))
    w0, a0, f0 = gt.get(dev(keys))
    assert not w0.any() and not a0.any() and not f0.any() and gt.stats().error == hps.ERESERVED
    assert np.array_equal(out[1:].cpu().numpy().reshape(3 * n, dim), want[0]) and flags.all()
    assert np.array_equal(acc[1:].cpu().numpy().reshape(3 * n, acc_len), want[1])


@pytest.mark.parametrize("opt,rows", [(hps.ADAGRAD_ROWWISE, hps.ROWS_F32), (hps.ADAGRAD_ROWWISE, hps.ROWS_F32_WIDE),
                                      (hps.ADAGRAD_ELEMENTWISE, hps.ROWS_F32)])
@pytest.mark.parametrize("capacity", [733_000, 734_100, 900_000])
def test_dump_of_many_slots(capacity, opt, rows):
    # (the slot count where a block takes several rounds at once lies between the first two.)  Marks that an emptied
    # table leaves behind in free slots do not count; every changed row goes out once.
    rng = np.random.default_rng(capacity)
    gt = hps.HpsTable(capacity, 4, 5000, 5000, opt=opt, row_format=rows, init_acc=0.25)
    ids = rng.permutation(200_000).astype(np.uint64)
    offsets = torch.arange(5001, dtype=torch.int32, device="cuda")

    def step(keys):
        gt.pull(dev(keys), offsets, 5000, 1)
        gt.push(torch.ones((5000, 4), device="cuda"))

    step(synth.mix64(ids[:5000]))
    gt.clear()
    gt.insert(dev(synth.mix64(ids[5000:])))
    changed = synth.mix64(ids[50_000:55_000])
    step(changed)
    assert gt.stats().size == 195_000
    k, w, a = [x.cpu().numpy() for x in gt.dump(dirty=True)]
    k = k.view(np.uint64)
    assert np.array_equal(np.sort(k), np.sort(changed))
    got = gt.get(dev(k))
    assert np.array_equal(got[0].cpu().numpy(), w) and np.array_equal(got[1].cpu().numpy(), a)
    assert (a >= 1.25).all()
    assert gt.dump(dirty=True)[0].numel() == 0
    k, w, a = [x.cpu().numpy() for x in gt.dump()]
    assert np.array_equal(np.sort(k.view(np.uint64)), np.sort(synth.mix64(ids[5000:])))
