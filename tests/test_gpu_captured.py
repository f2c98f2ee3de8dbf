"""Calls inside a captured graph that the header does not forbid there: the clearing of the table, and the push of a pull
that was made outside.  Counts, keys and rows are exact: gradients and learning rate are powers of two, or the rows are the ones that
were inserted."""
import numpy as np
import pytest
import torch

import paper_2003_05622_amd as hps
import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


@pytest.mark.parametrize("dirty", [False, True])
def test_dumps_around_a_captured_clear(dirty):
    dim, stream = 8, torch.cuda.Stream()
    gt = hps.HpsTable(20_000, dim, 5000, 5000)

    def load(first, n):
        keys = synth.mix64(np.arange(first, first + n, dtype=np.uint64))
        rows = torch.arange(n * dim, dtype=torch.float32, device="cuda").reshape(n, dim)
        gt.insert(dev(keys), rows)
        if dirty:
            gt.accumulate(dev(keys), rows)
            rows = rows + rows
        return keys, rows.cpu().numpy()

    def dumped(keys, rows):
        k, w, _ = gt.dump(max_rows=10_000, dirty=dirty)
        k = k.cpu().numpy().view(np.uint64)
        assert k.size == keys.size and gt.stats().size == keys.size
        a, b = np.argsort(k), np.argsort(keys)
        assert np.array_equal(k[a], keys[b]) and np.array_equal(w.cpu().numpy()[a], rows[b])

    dumped(*load(0, 1000))
    gt.clear()
    dumped(*load(2000, 3000))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        gt.clear()
    if not dirty:
        k, _, _ = gt.dump(max_rows=10_000)            # (nothing has been replayed yet)
        assert k.numel() == 3000
    for turn in range(3):
        graph.replay()
        dumped(*load(6000 + 1000 * turn, 500 + 100 * turn))


@pytest.mark.parametrize("own_stream", [False, True])
def test_captured_push_of_a_pull_made_outside(own_stream):
    """Replayed for the same outstanding mini-batch; the calls after it go on as usual.  One bag a key, the elementwise Adagrad at its
    third step: G = 3 + 1, w moves by 1/2 a step."""
    n, dim, stream = 3000, 4, torch.cuda.Stream()
    home = torch.cuda.Stream() if own_stream else torch.cuda.default_stream()
    keys = dev(synth.mix64(np.arange(n, dtype=np.uint64)))
    offsets = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    one, zero = torch.ones((n, dim), device="cuda"), torch.zeros((n, dim), device="cuda")
    gt = hps.HpsTable(4 * n, dim, n, n, opt=hps.ADAGRAD_ELEMENTWISE, lr=1.0, eps=0.0, init_acc=3.0, init_range=0.0)
    grads = zero.clone()
    torch.cuda.synchronize()
    with torch.cuda.stream(home):
        for _ in range(2):
            gt.pull(keys, offsets, n, 1)
            gt.push(zero)
        gt.pull(keys, offsets, n, 1)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            assert hps.lib().hps_push(gt._h, grads.data_ptr(), stream.cuda_stream) == hps.OK
        for g in (zero, one, zero):
            grads.copy_(g)
            graph.replay()
            torch.cuda.synchronize()
        w, a, _ = gt.get(keys)
        assert torch.equal(w, torch.full_like(w, -0.5)) and torch.equal(a, torch.full_like(a, 4.0))
        for _ in range(3):
            pooled = gt.pull(keys, offsets, n, 1)
            gt.push(zero)
            assert torch.equal(pooled, w)
        other = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            gt.pull(keys, offsets, n, 1, pooled)
            gt.push(zero)
        torch.cuda.synchronize()
        assert torch.equal(pooled, w) and gt.stats().error == 0
