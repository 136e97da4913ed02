"""Table creation against the oracle, bit-exact: the supports and the root
state at the edges of the upload's words, chunks, workers and windows, of the
columns a wave stages at a time, with cells outside their domains, star cells,
initial domains with holes and empty ones, creations by several threads at
once."""
import sys
import threading

import numpy as np
import pytest

from oracle import oracle as O
from paper_2507_18413_amd import ct
from paper_2507_18413_amd import workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


CASES = [
    # columns, values, tuples, share of stars, share outside the domain, holes
    (1, 3, 1, 0.0, 0.0, False),
    (2, 70, 63, 0.0, 0.2, False),
    (3, 5, 64, 0.1, 0.1, True),
    (5, 9, 65, 0.0, 0.0, True),
    (63, 4, 4095, 0.02, 0.02, True),
    (64, 3, 4096, 0.0, 0.001, False),
    (65, 6, 4097, 0.01, 0.0, True),
    (150, 130, 900, 0.0, 0.0005, True),
    (256, 2, 300, 0.3, 0.0, False),
    (16, 2, 16_384, 0.0, 0.0, True),        # one chunk
    (16, 2, 16_385, 0.0, 0.0, True),        # and one word
    (6, 20, 87_400, 0.0, 0.01, True),       # two workers
    (4, 12, 1_100_000, 0.0, 0.3, True),     # several windows
]


def check(case, seed):
    n, d, t, star, outside, holes = case
    rng = W.rng_for(seed, 940, t)
    lo = (np.arange(n, dtype=np.int32) % 7) - 3
    ds = np.full(n, d, np.int32)
    tup = (lo + rng.integers(0, d, size=(t, n))).astype(np.int32)
    m = rng.random(tup.shape) < outside
    tup[m] = np.array([-1 << 30, 1 << 30, -4, d + 4], np.int32)[rng.integers(0, 4, size=int(m.sum()))]
    if star:
        tup[rng.random(tup.shape) < star] = ct.STAR
    lay = W.DomLayout(ds, lo)
    dom = lay.full()
    if holes:
        for i in range(0, n, max(1, n // 5)):
            if d > 2:
                lay.clear(dom, i, int(lay.values(dom, i)[int(rng.integers(0, d))]))
    g = ct.Table(tup, lo, ds, init_dom=dom)
    o = O.OracleTable(tup, lo, ds, init_dom=dom, fast=not star)
    assert g.create_status == o.create_status
    sup = g.supports()
    rows = range(g.rows) if g.rows < 200 else rng.integers(0, g.rows, size=60)
    for r in rows:
        assert (sup[r] == o.support_row(int(r))).all(), r
    gd, gc = g.state()
    od, oc = o.state()[:2]
    assert (gc == oc).all()
    assert (gd == od).all()
    if o.create_status == O.OK:
        new = W.pick_fraction_removal(rng, lay, od, frac=0.4)
        gs, gd = g.propagate(new)
        os_, od = o.propagate(new)
        assert gs == os_ and (os_ != O.OK or (gd == od).all())
    g.close()


@pytest.mark.parametrize("case", range(len(CASES)))
def test_create_edges(case):
    say("create:", CASES[case])
    check(CASES[case], case)


def test_create_empty_domain():
    say("create: a variable without a value, with and without stars")
    for star in (False, True):
        tup = np.array([[0, 1], [1, 0]], np.int32)
        if star:
            tup[0, 0] = ct.STAR
        lay = W.DomLayout(np.array([2, 2], np.int32), np.zeros(2, np.int32))
        dom = lay.full()
        dom[0] = 0
        g = ct.Table(tup, np.zeros(2, np.int32), np.array([2, 2], np.int32), init_dom=dom)
        o = O.OracleTable(tup, np.zeros(2, np.int32), np.array([2, 2], np.int32), init_dom=dom)
        assert g.create_status == o.create_status == ct.FAIL
        assert (g.state()[0] == o.state()[0]).all() and (g.state()[1] == 0).all()


def test_create_threads():
    say("create: 6 threads, 3 tables each")
    bad = []

    def work(k):
        try:
            for r in range(3):
                check(CASES[(2 * k + 3 * r + 8) % len(CASES)], 100 * k + r)
        except BaseException as e:  # noqa: BLE001
            bad.append((k, repr(e)))

    th = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not bad, bad
