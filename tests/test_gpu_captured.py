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
