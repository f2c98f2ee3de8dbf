"""The choice of a dedup's form (csrc/form.hpp), compiled for the host: no GPU, no library."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RANGE, BORDERS, HASH, SMALL, PLAIN = range(5)
SLOW, ONE_KEY, MIXED, STAND_IN, UNEVEN, CROWDED = 2, 4, 8, 16, 32, 64

SOURCE = r"""
#include "form.hpp"
using namespace hps;
extern "C" {
FormChoice* make() { return new FormChoice(); }
void drop(FormChoice* c) { delete c; }
int next(FormChoice* c, uint32_t n, int listable, uint64_t serial, uint64_t lookups, unsigned long long range, unsigned long long other, unsigned long long small) {
  return c->next(n, listable != 0, serial, lookups, {range, other, small});
}
void listed(FormChoice* c) { c->listed(); }
void captured(FormChoice* c, uint64_t n, int form) { c->captured(n, form); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++ here")
    d = tmp_path_factory.mktemp("form")
    (d / "form.cpp").write_text(SOURCE)
    so = str(d / "libform.so")
    subprocess.check_call([gxx, "-O1", "-std=c++17", "-fPIC", "-shared", "-fsanitize=undefined", "-fsanitize-undefined-trap-on-error",
                           "-I", os.path.join(ROOT, "paper_2003_05622_amd", "csrc"), "-o", so, str(d / "form.cpp")])
    L = ctypes.CDLL(so)
    u64, vp = ctypes.c_uint64, ctypes.c_void_p
    L.listed.argtypes = [vp]
    L.make.restype = vp
    L.drop.argtypes = [vp]
    L.next.argtypes = [vp, ctypes.c_uint32, ctypes.c_int, u64, u64, u64, u64, u64]
    L.captured.argtypes = [vp, u64, ctypes.c_int]
    return L


class Caller:
    """A table's dedups, one after the other, each with its lookup, and the reports of the lookups as they arrive."""

    def __init__(self, lib):
        self.L, self.c = lib, lib.make()
        self.serial = self.lookups = self.range = self.other = self.small = 0

    def __del__(self):
        self.L.drop(self.c)

    def dedup(self, n, flags=0, listable=True):
        """The form of the next dedup.  `flags`: what its lookup reports."""
        self.serial += 1
        form = self.L.next(self.c, n, listable, self.serial, self.lookups, self.range, self.other, self.small)
        self.lookups += 1
        if form == RANGE:
            self.range = self.lookups | flags << 32
        elif form == SMALL:
            if flags & SLOW:
                self.small = self.serial
        else:
            self.other = self.lookups | (flags & (SLOW | ONE_KEY) | STAND_IN if form != PLAIN else flags & MIXED) << 32
        return form

    def list(self):
        self.L.listed(self.c)

    def capture(self, n, form):
        self.list()
        self.L.captured(self.c, n, form)


def test_captured_listing_keeps_the_form_of_uneven_keys_by_hash(lib):
    """At most 65536 occurrences by hash, the third dedup after a listing: the fourth would take the small form."""
    t, n = Caller(lib), 30_000
    assert [t.dedup(n, UNEVEN | CROWDED) for _ in range(3)] == [PLAIN, PLAIN, RANGE]
    t.list()
    assert [t.dedup(n) for _ in range(2)] == [BORDERS, BORDERS] and t.dedup(n) == HASH
    t.capture(n, HASH)
    assert {t.dedup(n, SLOW) for _ in range(300)} == {HASH}


def test_captured_listings_keep_their_forms_whatever_comes(lib):
    rng = random.Random(1)
    seen = set()
    for turn in range(300):
        t, pins = Caller(lib), {}
        sizes = rng.choice([[500, 30_000], [65_536, 65_537], [100_000, 524_288, 524_289], [30_000, 300_000, 3_000_000], [2_000_000, 13_000_000]])
        period = rng.choice([0, 1, 2, 4, 9])
        for k in range(200):
            n, listable = rng.choice(sizes), rng.random() < 0.9
            flags = rng.choice([0, 0, 0, SLOW, SLOW | ONE_KEY, UNEVEN, UNEVEN | CROWDED, MIXED])
            form = t.dedup(n, flags, listable)
            group = sum(n > most for most in (65_536, 524_288, 12 << 20))
            assert group < 3 or form == PLAIN
            if listable and group in pins:
                assert form == pins[group]
            if listable and group < 3 and rng.random() < 0.02:
                t.capture(n, form)
                pins.setdefault(group, form)
                seen.add((group, form))
            elif listable and period and k % period == 0:
                t.list()
    assert len(seen) >= 9, seen           # every form was captured, at several sizes


@pytest.mark.parametrize("n", [20_000, 65_536, 65_537, 300_000, 5_000_000])
def test_who_lists_now_and_then(lib, n):
    """Often: an order of keys once the caller is known.  Rarely: by hash from the fourth dedup after a listing on, which gains more
    in between than the listing then costs."""
    often = 10 if n <= 65_536 else 24
    for period in [1, 2, 3, 4, 5, 7, 10, 11, 12, 24, 25, 33, 64, 250]:
        t, dear, by_hash = Caller(lib), [], 0
        for k in range(6000):
            form = t.dedup(n)
            by_hash += form in (HASH, SMALL)
            for _ in range(k % 4):
                t.dedup(n, listable=False)              # accumulates in between count for nothing
            if k % period == period - 1:
                if form in (HASH, SMALL):
                    dear.append(k)
                t.list()
        if period <= often:
            assert dear == ([period - 1] if period > 3 else []) and by_hash <= max(0, period - 3)
        else:
            assert len(dear) == 6000 // period and by_hash == 6000 - 3 * -(-6000 // period)


def test_who_lists_in_no_rhythm(lib):
    """Costs in mini-batches: 20 K occurrences by range lose 20 us each, a listing of keys by hash 115 us.  Whatever the gaps between
    listings are drawn from, the choice costs no more than 1.5 times what the better of always by range and always by hash after three
    dedups does (1.0 to 1.33 for these; the losses alone, of 20 out of 46 us a step)."""
    rng = random.Random(2)
    for draw in [lambda: rng.randint(1, 6), lambda: rng.randint(1, 20), lambda: rng.choice([2, 40]), lambda: rng.choice([5, 5, 5, 14]),
                 lambda: 1 + int(rng.expovariate(1 / 8)), lambda: 1 + int(rng.expovariate(1 / 30)), lambda: rng.choice([1] * 20 + [90])]:
        t, cost, always, never, gaps = Caller(lib), 0, 0, 0, [draw() for _ in range(400)]
        for gap in gaps:
            forms = [t.dedup(20_000) for _ in range(gap)]
            t.list()
            cost += 20 * sum(f not in (HASH, SMALL) for f in forms) + 115 * (forms[-1] in (HASH, SMALL))
            always += 20 * gap
            never += 20 * min(gap, 3) + 115 * (gap > 3)
        assert cost <= 1.5 * min(always, never), (cost, always, never)


@pytest.mark.parametrize("n", [20_000, 300_000, 5_000_000])
def test_who_never_lists_goes_by_hash(lib, n):
    t, often = Caller(lib), 10 if n <= 65_536 else 24
    forms = [t.dedup(n) for _ in range(50)]
    assert RANGE in forms[:3] and set(forms[3:]) == {SMALL if n <= 65_536 else HASH}
    t.list()                                             # after many
    assert t.dedup(n, listable=False) == (SMALL if n <= 65_536 else HASH)
    assert [t.dedup(n) for _ in range(6)] == [RANGE] * 3 + [SMALL if n <= 65_536 else HASH] * 3
    t.list()                                             # after few
    assert {t.dedup(n) for _ in range(often)} == {RANGE}
    assert {t.dedup(n) for _ in range(50)} == {SMALL if n <= 65_536 else HASH}


@pytest.mark.parametrize("ahead", [1, 20, 300])
def test_mini_batches_the_small_form_does_not_suit_go_by_hash(lib, ahead):
    """The GPU is `ahead` dedups behind with what it reports.  The small form is tried again ever more rarely, one mini-batch at a
    time, and is back for good once it does well."""
    t, n, hold = Caller(lib), 20_000, 32
    written = [(0, 0)]                   # the report words after every dedup

    def dedup(suits):
        small, other = written[-1]
        seen = written[max(0, len(written) - 1 - ahead)]
        t.small, t.other = seen
        form = t.dedup(n)
        written.append((t.serial if form == SMALL and not suits else small, t.other if t.other != seen[1] else other))
        return form

    forms = [dedup(False) for _ in range(4000)]
    assert set(forms[3:]) == {SMALL, HASH}
    assert forms.count(SMALL) <= ahead + 1 + 7 and SMALL in forms[ahead + 30 : 2 * ahead + 120]
    assert set([dedup(True) for _ in range(6000)][-1000:]) == {SMALL}
    forms = [dedup(False) for _ in range(ahead + 2)] + [dedup(True) for _ in range(3 * ahead + hold + 8)]
    assert HASH in forms and forms[-1] == SMALL          # (the strikes are forgotten)


def test_mini_batches_that_suit_the_small_form_every_other_time(lib):
    """It is given up ever longer all the same."""
    t, n = Caller(lib), 20_000
    forms = [t.dedup(n, SLOW if k % 16 < 8 else 0) for k in range(8000)]
    assert forms[1000:].count(SMALL) < 400
