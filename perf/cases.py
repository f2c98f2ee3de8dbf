"""The work this parameter server is measured by, as its users call it.

A trainer runs the paper's outer loop: mini-batches are pulled and pushed, and the rows they
touched are collected for the host tier; a serving replica reads rows by key and takes over the
rows a trainer has changed.  The kinds of cases:

  train    mini-batches on a long-lived table that holds (nearly) all ids: pull, push, and after
           the last one the rows of all touched keys read back (get);
  batch    one turn of the paper's outer loop: the table is emptied, the batch's working
           parameters are inserted with their values, mini-batches run, among them ids the table
           has never seen, and the rows are collected;
  serve    get: a replica answers for a list of keys, some of them unknown to it;
  add      accumulate: value rows are added onto the rows of their keys, then read back;
  refresh  a trainer's changed rows (after one mini-batch) go to a serving replica:
           dump of the updated rows, insert with values, read back at the replica.

Keys follow a bounded Zipf-Mandelbrot law over the resident ids, as click logs do, plus a share
of ids never seen before; ids are hashed to 64 bits or used as they are ("raw": one id space of
consecutive numbers).  Everything is drawn on the GPU from the seed.
"""
import math

import numpy as np
import torch

import paper_2003_05622_amd as hps

# Fields every case has.  dim: floats per row.  opt / rows / mean: optimizer, row format, pooling.
# examples x slots bags per mini-batch, `bag` occurrences in each on average (at least 1 unless
# `empty`, which lets bags be empty).  resident: ids in the table beforehand; zipf_s, zipf_q: the
# law their ranks follow; fresh: share of occurrences with ids never seen before.
BASE = dict(kind="train", dim=16, opt="rowwise", rows="f32", mean=False, examples=512, slots=16, bag=2.5,
            empty=False, resident=1 << 20, zipf_s=1.05, zipf_q=0.0, fresh=0.0, ids="hashed", pipelined=False, steps=4)


def _case(name, **more):
    case = dict(BASE, **more)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest mini-batches a trainer runs: 8192 short bags of narrow rows, latency above all
        _case("train_tiny", dim=8, zipf_s=1.1, steps=8),
        # few wide rows, averaged, one accumulator per element, raw ids, odd sizes, empty bags
        _case("train_ragged", dim=100, opt="elementwise", mean=True, examples=333, slots=37, bag=3.3, empty=True,
              resident=300_001, zipf_s=1.1, fresh=0.01, ids="raw"),
        # the ordinary mini-batch: 500 features per example, one id in twenty new
        _case("train_mid", examples=4096, slots=100, bag=5.0, resident=1 << 26, fresh=0.05),
        # twice that with one accumulator per element, the next mini-batch prepared beside the push
        _case("train_ahead", examples=8192, slots=100, bag=5.0, resident=1 << 25, fresh=0.05, opt="elementwise",
              pipelined=True),
        # the largest mini-batch in occurrences, on the largest table that fits three times over
        _case("train_large", examples=16384, slots=200, bag=3.0, resident=1 << 28, fresh=0.05),
        # wide rows, a few keys that make up most of the mini-batch
        _case("train_skewed", dim=64, examples=16384, slots=64, bag=8.0, resident=1 << 26, zipf_s=1.3),
        # wide rows stored as bfloat16, thousands of keys that are frequent but none that dominates
        _case("train_bf16", dim=64, rows="bf16", examples=8192, slots=64, bag=8.0, resident=1 << 26, zipf_s=1.3,
              zipf_q=222.0),
        # the paper's outer batch: a working set loaded, four mini-batches with one id in five new
        _case("outer_batch", kind="batch", examples=4096, slots=100, bag=5.0, resident=1 << 26, fresh=0.2),
        # the rows one scoring request needs: 500 features for each of 8 candidates
        _case("serve_request", kind="serve", examples=8, slots=100, bag=5.0, resident=1 << 22, fresh=0.02),
        # the rows of a bulk scoring job's mini-batch
        _case("serve_bulk", kind="serve", dim=32, examples=4096, slots=100, bag=5.0, resident=1 << 25, fresh=0.02),
        # updates computed elsewhere, added to the rows of a table
        _case("add", kind="add", examples=1024, slots=100, bag=3.0, resident=1 << 24, zipf_s=1.1, fresh=0.01),
        # a replica takes over what a mini-batch has changed
        _case("refresh", kind="refresh", dim=32, examples=2048, slots=100, bag=3.0, resident=1 << 22, steps=1),
    ]


def draw(rng):
    kind = rng.choice(["train"] * 6 + ["batch", "serve", "add", "refresh"])
    dim = rng.choice([4, 8, 16, 16, 16, 32, 64, 64, 100, 128, 260])
    # no mini-batch above the listed ones': 10^7 occurrences, 5 x 10^8 floats of gathered rows
    most = min(9_800_000, 500_000_000 // dim)
    if kind in ("add", "refresh"):
        most = min(most, 1_200_000)
    ids = rng.choice(["hashed", "hashed", "hashed", "raw"])
    if ids == "raw":
        most = min(most, 300_000)
    n = int(math.exp(rng.uniform(math.log(1000), math.log(most))))
    bag = rng.choice([1.0, rng.uniform(1.2, 4.0), rng.uniform(3.0, 9.0)])
    bags = max(1, int(n / max(bag, 1.25)))
    slots = min(bags, rng.choice([1, rng.randint(2, 40), 64, 100, 200]))
    # rows of the resident ids in at most 20 GB
    cap = min(1 << 28, int(2e10 / (6 * dim + 16)))
    if kind == "refresh":
        cap = min(cap, 1 << 22)
    resident = int(math.exp(rng.uniform(math.log(1 << 14), math.log(cap))))
    return _case(None, kind=kind, dim=dim, bag=bag, slots=slots, examples=max(1, bags // slots), resident=resident,
                 opt=rng.choice(["rowwise", "rowwise", "elementwise"]), rows=rng.choice(["f32", "f32", "f32wide", "bf16"]),
                 mean=rng.random() < 0.25, empty=rng.random() < 0.25, zipf_s=rng.choice([1.05, 1.1, 1.3]),
                 zipf_q=rng.choice([0.0, 0.0, 222.0]), fresh=rng.choice([0.0, 0.05, 0.2]),
                 ids=ids, pipelined=rng.random() < 0.25,
                 steps=1 if kind == "refresh" else rng.randint(2, 4))


# ---- inputs ------------------------------------------------------------------------------------

def _shr(x, k):
    """Logical right shift of the 64-bit patterns in an int64 tensor."""
    return (x >> k) & ((1 << (64 - k)) - 1)


def _mix64(ids):
    """The SplitMix64 output function: what hashes a feature id to its key."""
    z = ids + (0x9E3779B97F4A7C15 - (1 << 64))
    z = (z ^ _shr(z, 30)) * (0xBF58476D1CE4E5B9 - (1 << 64))
    z = (z ^ _shr(z, 27)) * (0x94D049BB133111EB - (1 << 64))
    return z ^ _shr(z, 31)


RAW_FIRST = 1 << 33         # raw ids start here
SCRAMBLE = 1_000_003        # raw ids: rank k is id k * SCRAMBLE mod resident (a prime above no divisor in use)


def _occurrences(case):
    """Key occurrences and bags of a mini-batch."""
    bags = case["examples"] * case["slots"]
    return int(round(bags * case["bag"])), bags


def _keys(case, ids):
    return _mix64(ids) if case["ids"] == "hashed" else ids + RAW_FIRST


def _head(case):
    """Weights of the most frequent ranks, and how much lies behind them (midpoint rule)."""
    s, q, n = case["zipf_s"], case["zipf_q"], case["resident"]
    k0 = min(n, 1 << 20)
    w = (np.arange(1, k0 + 1, dtype=np.float64) + q) ** -s
    tail = 0.0 if n <= k0 else ((k0 + 0.5 + q) ** (1 - s) - (n + 0.5 + q) ** (1 - s)) / (s - 1)
    return w, tail


class _Ids:
    """Draws feature ids: Zipf-Mandelbrot ranks over the resident ones, a share of fresh ones."""

    def __init__(self, case, seed):
        self.case = case
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        w, self.tail = _head(case)
        self.cum = torch.from_numpy(np.cumsum(w)).cuda()
        # fresh ids are never used twice, not by another seed either
        self.fresh_next = case["resident"] + ((1 << 36) * (1 + seed % 1000) if case["ids"] == "hashed" else 0)

    def draw(self, n):
        case, s, q = self.case, self.case["zipf_s"], self.case["zipf_q"]
        head = self.cum[-1]
        u = torch.rand(n, generator=self.gen, device="cuda", dtype=torch.float64) * (head + self.tail)
        rank = torch.searchsorted(self.cum, u, right=True).clamp_(max=self.cum.numel() - 1)
        if self.tail:
            k0 = self.cum.numel()
            v = (u - head).clamp_(min=0.0)
            far = ((k0 + 0.5 + q) ** (1 - s) + v * (1 - s)) ** (1 / (1 - s)) - q
            far = (far - 0.5).floor().to(torch.int64).clamp_(k0, case["resident"] - 1)
            rank = torch.where(u < head, rank, far)
        if case["ids"] == "raw":
            rank = rank * SCRAMBLE % case["resident"]
        if case["fresh"]:
            new = torch.rand(n, generator=self.gen, device="cuda") < case["fresh"]
            at = torch.cumsum(new, 0) - 1 + self.fresh_next
            rank = torch.where(new, at, rank)
            self.fresh_next += n
        return rank

    def offsets(self):
        # the occurrences beyond one per bag (or all of them) fall on bags at random: bag sizes
        # are Poisson-distributed, given their sum
        n, bags = _occurrences(self.case)
        least = 0 if self.case["empty"] else 1
        at = torch.randint(bags, (n - least * bags,), generator=self.gen, device="cuda")
        off = torch.zeros(bags + 1, dtype=torch.int32, device="cuda")
        torch.cumsum((torch.bincount(at, minlength=bags) + least).to(torch.int32), 0, out=off[1:])
        return off

    def touched(self, batches):
        """The distinct keys of the mini-batches in a request of fixed length: as many as are
        expected and some more, the rest of it filled with the first of them once more."""
        n, _ = _occurrences(self.case)
        keys = torch.unique(torch.cat([b["keys"] for b in batches]))
        t = _distinct(self.case, n * len(batches))
        at = torch.arange(int(1.01 * t + 5 * t ** 0.5 + 16), device="cuda")
        return keys[at % keys.numel()]

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.gen, device="cuda") * 1e-3

    def minibatch(self):
        off = self.offsets()
        ids = self.draw(_occurrences(self.case)[0])
        return dict(ids=ids, keys=_keys(self.case, ids), offsets=off,
                    grads=self.normal(off.numel() - 1, self.case["dim"]))


def _table(case, capacity, max_keys):
    n_bags = case["examples"] * case["slots"]
    return hps.HpsTable(capacity, case["dim"], max_keys, n_bags, lr=0.05,
                        opt=hps.ADAGRAD_ELEMENTWISE if case["opt"] == "elementwise" else hps.ADAGRAD_ROWWISE,
                        row_format={"f32": hps.ROWS_F32, "bf16": hps.ROWS_BF16, "f32wide": hps.ROWS_F32_WIDE}[case["rows"]])


def _fill(case, table):
    for lo in range(0, case["resident"], 1 << 24):
        table.insert(_keys(case, torch.arange(lo, min(lo + (1 << 24), case["resident"]), device="cuda")))


def prepare(case, seed):
    """A table in the middle of its training, and the next mini-batches (or keys)."""
    ids = _Ids(case, seed)
    kind, dim = case["kind"], case["dim"]
    state = dict(case=case)
    batches = [ids.minibatch() for _ in range(1 if kind in ("serve", "add") else case["steps"])]
    earlier = [ids.minibatch() for _ in range(3)]
    n_max = _occurrences(case)[0]
    n_sum = n_max * (len(batches) + len(earlier))
    if kind == "batch":
        # the working parameters: the known ids of the batch, with rows from the host tier
        known = torch.unique(torch.cat([b["ids"][b["ids"] < case["resident"]] for b in batches]))
        acc_len = dim if case["opt"] == "elementwise" else 1
        state.update(working=_keys(case, known), weights=ids.normal(known.numel(), dim) * 10,
                     acc=torch.rand(known.numel(), acc_len, generator=ids.gen, device="cuda") + 0.1)
        table = _table(case, n_sum, n_max)
    else:
        table = _table(case, case["resident"] + int(n_sum * case["fresh"] * 1.1) + 4096, n_max)
        _fill(case, table)
    table.set_pooling(case["mean"])
    for b in earlier:
        table.pull(b["keys"], b["offsets"], case["examples"], case["slots"])
        table.push(b["grads"])
    state.update(table=table, touched=ids.touched(batches), keys=batches[0]["keys"])
    if kind == "add":
        state["values"] = ids.normal(batches[0]["keys"].numel(), dim)
    if kind == "refresh":
        state["replica"] = _table(case, table.capacity, 1024)
        _fill(case, state["replica"])
        table.dump(n_sum, dirty=True)      # what the earlier mini-batches changed is already there
    if kind in ("train", "batch", "refresh"):
        state["side"] = torch.cuda.Stream() if case["pipelined"] else None
        state["batches"] = [(b["keys"], b["offsets"], b["grads"],
                             torch.empty(b["grads"].shape, device="cuda")) for b in batches]
    table.check("prepare")
    return state


# ---- one pass ----------------------------------------------------------------------------------

def _train(state):
    table, case, batches = state["table"], state["case"], state["batches"]
    shape = (case["examples"], case["slots"])
    if not case["pipelined"]:
        for keys, offsets, grads, pooled in batches:
            table.pull(keys, offsets, *shape, pooled)
            table.push(grads)
        return [b[3] for b in batches]
    # the dedup of the next mini-batch on a second stream, beside the push of this one
    table.prepare(batches[0][0], batches[0][1], *shape)
    for i, (keys, offsets, grads, pooled) in enumerate(batches):
        table.pull_prepared(pooled)
        if i + 1 < len(batches):
            with torch.cuda.stream(state["side"]):
                table.prepare(batches[i + 1][0], batches[i + 1][1], *shape)
        table.push(grads)
    return [b[3] for b in batches]


def run(state):
    case, table = state["case"], state["table"]
    kind = case["kind"]
    if kind == "train":
        pooled = _train(state)
        return dict(pooled=pooled, rows=table.get(state["touched"]))
    if kind == "batch":
        table.clear()
        table.insert(state["working"], state["weights"], state["acc"])
        pooled = _train(state)
        return dict(pooled=pooled, rows=table.get(state["touched"]))
    if kind == "serve":
        return dict(rows=table.get(state["keys"]))
    if kind == "add":
        table.accumulate(state["keys"], state["values"])
        return dict(rows=table.get(state["touched"]))
    pooled = _train(state)
    keys, weights, acc = table.dump(state["keys"].numel(), dirty=True)
    state["replica"].insert(keys, weights, acc)
    return dict(pooled=pooled, rows=state["replica"].get(state["touched"]))


# ---- what a pass cannot do without ---------------------------------------------------------------

def _distinct(case, n):
    """Expected number of distinct keys among n occurrences."""
    w, tail = _head(case)
    known = n * (1 - case["fresh"])
    total = w.sum() + tail
    u = -np.expm1(-known * w / total).sum()
    if tail:
        edge = np.unique(np.geomspace(w.size + 0.5, case["resident"] + 0.5, 4000))
        mid = np.sqrt(edge[1:] * edge[:-1])
        u += (-np.expm1(-known * (mid + case["zipf_q"]) ** -case["zipf_s"] / total) * np.diff(edge)).sum()
    return u + n * case["fresh"]


def work(case):
    dim, kind = case["dim"], case["kind"]
    n, bags = _occurrences(case)
    steps = 1 if kind in ("serve", "add") else case["steps"]
    stored = dim * (2 if case["rows"] == "bf16" else 4)
    acc = 4 * (dim if case["opt"] == "elementwise" else 1)
    u, t = _distinct(case, n), _distinct(case, n * steps)
    # get: a key and its slot's key, the row and accumulator as stored, the two and a flag out
    get = 16 + stored + acc + 4 * dim + acc + 1
    if kind == "serve":
        return dict(bytes=n * (8 + 4 * dim + acc + 1) + u * (8 + stored + acc), flops=0)
    if kind == "add":
        return dict(bytes=n * (8 + 4 * dim) + u * (8 + 2 * stored + 2 * acc) + t * get, flops=n * dim + u * dim)
    # pull: keys and offsets in, the distinct keys' slots and rows, pooled rows out;
    # push: gradients in, the distinct keys' rows and accumulators in and out
    step = 8 * n + 4 * bags + u * (8 + stored) + 4 * dim * bags + 4 * dim * bags + 2 * u * (stored + acc)
    flops = steps * (2 * n * dim + 6 * u * dim)
    more = 0
    if kind == "batch":
        known = t - n * steps * case["fresh"]
        more = known * (8 + 4 * dim + acc + 8 + stored + acc)
    if kind == "refresh":       # the changed rows out of one table and into another
        more = u * (8 + stored + acc + 2 * (8 + 4 * dim + acc) + 8 + stored + acc)
    return dict(bytes=steps * step + t * get + more, flops=flops)


def tolerance(case):
    # Four times what the same mini-batches give with bags and occurrences in reverse order, i.e.
    # with every sum taken in another order: pooled rows off by 1.8e-7 (2-norm) and single weights,
    # where frequent keys' steps cancel, by 1e-5; stored as bfloat16 a weight next to a rounding
    # border moves by a whole step (0.8 %): 2.9e-5 and 7.6e-3.
    if case["rows"] == "bf16":
        return {"rel": 1.2e-4, "max": 3e-2}
    return {"rel": 8e-7, "max": 4e-5}
