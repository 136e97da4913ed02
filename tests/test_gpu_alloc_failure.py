"""Allocation failures, injected through the library's test hook
(ct_debug_fail_alloc): every allocation point of table creation, slot
allocation and batch staging returns CT_E_NOMEM, releases what it took and
leaves existing state untouched, and the library works normally after."""
import sys

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2507_18413_amd import ct
from paper_2507_18413_amd import workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def test_injected_allocation_failures():
    L = ct.lib()
    spec = W.large_table(3, t=5000, d=10, n=4)
    say("alloc failure: every allocation of ct_create in turn")
    created = None
    fired = 0
    for k in range(1, 64):
        L.ct_debug_fail_alloc(k)
        try:
            created = ct.Table(spec.tuples, spec.lo, spec.dsizes, max_depth=8)
        except ct.CTError as e:
            assert e.code == ct.E_NOMEM and "injected" in str(e), (k, str(e))
            fired += 1
            continue
        finally:
            left = L.ct_debug_fail_alloc(0)
        # the k-th allocation lies beyond those of ct_create
        assert left > 0
        break
    assert created is not None and fired >= 5
    g = created
    o = O.OracleTable(spec.tuples, spec.lo, spec.dsizes)
    say("alloc failure: slots")
    n0 = g.n_slots
    L.ct_debug_fail_alloc(1)
    with pytest.raises(ct.CTError) as e:
        g.slots_alloc(4, max_depth=8)
    L.ct_debug_fail_alloc(0)
    assert e.value.code == ct.E_NOMEM and g.n_slots == n0
    first = g.slots_alloc(4, max_depth=8)
    say("alloc failure: batch staging on a new stream")
    lay = spec.layout()
    rng = W.rng_for(3, 990, 0)
    din_h = [W.pick_fraction_removal(rng, lay, g.domains(), frac=0.2) for _ in range(4)]
    din = torch.from_numpy(np.stack(din_h).view(np.int64)).cuda()
    dout = torch.zeros_like(din)
    status = torch.full((4,), 99, dtype=torch.int32, device="cuda")
    jobs = [dict(table=g, slot=first + k, flags=ct.JOB_PROPAGATE, n_push=1, dom_in=din[k], dom_out=dout[k])
            for k in range(4)]
    stream = torch.cuda.Stream()
    for k in (1, 2, 3):
        L.ct_debug_fail_alloc(k)
        try:
            ct.propagate_batch(jobs, status, stream)
        except ct.CTError as err:
            assert err.code == ct.E_NOMEM
        finally:
            L.ct_debug_fail_alloc(0)
        torch.cuda.synchronize()
        # whether or not the batch ran, the slots are consistent: reset them
        for s in range(first, first + 4):
            while g.pop(s) == ct.OK:
                pass
    ct.propagate_batch(jobs, status, stream)
    ct.batch_status(stream)
    st = status.cpu().numpy()
    got = dout.cpu().numpy().view(np.uint64)
    for k in range(4):
        o.push()
        os_, od = o.propagate(din_h[k])
        assert st[k] == os_
        if os_ == O.OK:
            assert (got[k] == od).all()
        o.pop()
    # the table's own slot still propagates like the oracle (a level is
    # popped after every failure and every second call: the depth stays
    # within the table's 8 levels)
    for k in range(10):
        d = W.pick_fraction_removal(rng, lay, o.domains())
        assert g.push() == o.push() == 0
        gs, gd = g.propagate(d)
        os_, od = o.propagate(d)
        assert gs == os_
        if os_ == O.OK:
            assert (gd == od).all()
        if os_ != O.OK or k % 2 == 1:
            assert g.pop() == o.pop() == 0


# domain sizes, tuples, schedule
CALLS = {
    "engine": ([10, 10, 10, 10], 5000, ct.SCHED_AUTO),
    "resident split": ([640] * 8, 9000, ct.SCHED_AUTO),
    "staged": ([40, 50, 60], 9 * 4096, ct.SCHED_SPLIT),
}


@pytest.mark.parametrize("want_ct", [False, True])
@pytest.mark.parametrize("pop_first", [False, True])
@pytest.mark.parametrize("name", list(CALLS))
def test_call_without_memory_keeps_its_pushes_and_pops(name, pop_first, want_ct):
    """A synchronous call whose own allocation fails changes nothing: the
    pushes and pops before it still apply to the slot's next operation."""
    L = ct.lib()
    ds, t, schedule = CALLS[name]
    rng = W.rng_for(len(name), 991, 0)
    lo = np.zeros(len(ds), np.int32)
    d = np.array(ds, np.int32)
    tup = np.stack([rng.integers(0, x, size=t) for x in ds], 1).astype(np.int32)
    lay = W.DomLayout(d, lo)
    fired = 0
    for k in range(1, 16):
        say("call without memory:", name, "allocation", k, "pop first", pop_first, "currTable", want_ct)
        g = ct.Table(tup, lo, d, max_depth=8, schedule=schedule)
        o = O.OracleTable(tup, lo, d)
        assert (g.resident, g.resident_split) == (name == "engine", name == "resident split")
        root = o.state()[:2]
        dom = W.pick_fraction_removal(rng, lay, o.domains(), frac=0.3)
        assert g.push() == o.push() == 0
        L.ct_debug_fail_alloc(k)
        st = g.propagate(dom, want_ct=want_ct)[0]
        left = L.ct_debug_fail_alloc(0)
        if st == ct.E_NOMEM:
            fired += 1
            if pop_first:
                assert g.pop() == 0
                gd, gc = g.state()
                assert (gd == root[0]).all() and (gc == root[1]).all()
                assert g.push() == 0
            st = g.propagate(dom)[0]
        else:
            assert left > 0  # the k-th allocation lies beyond those of the call
        assert st == o.propagate(dom)[0] == O.OK
        gd, gc = g.state()
        assert (gd == o.state()[0]).all() and (gc == o.state()[1]).all()
        assert g.pop() == o.pop() == 0
        gd, gc = g.state()
        assert (gd == root[0]).all() and (gc == root[1]).all()
        # (one level down again, over the state just restored)
        dom = W.pick_fraction_removal(rng, lay, o.domains(), frac=0.1)
        assert g.push() == o.push() == 0
        gs, gd = g.propagate(dom)
        os_, od = o.propagate(dom)
        assert gs == os_ and (gs != O.OK or (gd == od).all())
        g.close()
        if left > 0:
            break
    assert fired >= 1 and left > 0
