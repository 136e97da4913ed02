"""The staged schedule (prep, update, finish launches) against the oracle,
bit-exact, at the edges of its parts: whole jobs in the prep workgroup, granule
counts around a wave of positions and a workgroup's pass, domains of one word
to more than a pass of the prep, row lists and (more than 65,536 rows) selected
bits, pushes and pops of several levels in one job, inputs without a change,
rejected and failing jobs, star cells, negative tables in the same batch,
batches of several launches, the static scratch."""
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


# domain sizes, tuples, star share, kind, branch policy
TABLES = {
    "one granule": ([5, 9, 70], 300, 0.0, 0, ct.BRANCH_AUTO),
    "4 granules": ([30, 64, 65, 3], 16384, 0.05, 0, ct.BRANCH_AUTO),
    "5 granules": ([40, 1, 20, 130], 16385, 0.0, 0, ct.BRANCH_AUTO),
    "one granule, 17 words": ([1088], 900, 0.0, 0, ct.BRANCH_AUTO),
    "64 granules": ([50, 60, 40], 64 * 4096, 0.0, 0, ct.BRANCH_INCREMENTAL),
    "65 granules": ([50, 60, 40, 9], 64 * 4096 + 1, 0.0, 0, ct.BRANCH_RESET),
    "260 granules": ([90, 7, 80, 30], 260 * 4096 - 3, 0.0, 0, ct.BRANCH_AUTO),
    "512 words": ([64 * 200, 64 * 312], 9000, 0.0, 0, ct.BRANCH_AUTO),
    "513 words": ([64 * 200, 64 * 313], 20000, 0.0, 0, ct.BRANCH_AUTO),
    "3,073 words": ([64 * 3000, 64 * 72 + 1], 5000, 0.0, 0, ct.BRANCH_INCREMENTAL),
    "selected bits": ([36000, 38000], 5000, 0.0, 0, ct.BRANCH_RESET),
    "negative": ([6, 8, 7, 5], 900, 0.0, ct.KIND_NEGATIVE, ct.BRANCH_AUTO),
    # most combinations forbidden: values go, in one to five passes of granules
    "negative, 5 granules": ([3, 2, 4000], 40000, 0.0, ct.KIND_NEGATIVE, ct.BRANCH_AUTO),
    "negative, 1 word": ([63], 62, 0.0, ct.KIND_NEGATIVE, ct.BRANCH_AUTO),
}


def make(name, rng, **kw):
    ds, t, star, kind, policy = TABLES[name]
    lo = np.arange(len(ds), dtype=np.int32) - 2
    tup = np.stack([lo[i] + rng.integers(0, ds[i], size=t) for i in range(len(ds))], 1).astype(np.int32)
    if star:
        tup[rng.random(tup.shape) < star] = ct.STAR
    if kind:
        tup = np.unique(tup, axis=0)
    ds = np.array(ds, np.int32)
    return (ct.Table(tup, lo, ds, branch_policy=policy, kind=kind, **kw),
            O.OracleTable(tup, lo, ds, kind=kind, fast=kind == 0 and not star), W.DomLayout(ds, lo))


def narrowed(rng, lay, dom):
    """The next input: a share of the values removed, or nothing, or all of
    one variable's but one, or something to reject."""
    new = dom.copy()
    r = rng.random()
    if r < 0.15:
        return new
    if r < 0.22:
        new[0] = ~np.uint64(0)
        return new
    share = rng.choice([0.02, 0.3, 0.9])
    for i in range(lay.n):
        if rng.random() < 0.4:
            continue
        vals = lay.values(new, i)
        gone = vals[rng.random(vals.size) < share]
        if gone.size == vals.size:
            gone = gone[1:]
        for a in gone:
            lay.clear(new, i, int(a))
    if r > 0.9:
        vals = lay.values(new, lay.n - 1)
        for a in vals[1:]:
            lay.clear(new, lay.n - 1, int(a))
    return new


@pytest.mark.parametrize("name", list(TABLES))
def test_staged_calls(name):
    say("staged calls:", name, TABLES[name])
    rng = W.rng_for(len(name), 930, 0)
    g, o, lay = make(name, rng, schedule=ct.SCHED_SPLIT)
    assert g.create_status == o.create_status == O.OK
    assert (g.domains() == o.domains()).all()
    depth, failed = 0, False
    for step in range(14):
        if depth and (failed or rng.random() < 0.3):
            for _ in range(int(rng.integers(1, depth + 1))):
                g.pop()
                o.pop()
                depth -= 1
        for _ in range(int(rng.integers(0, 3)) if step % 3 else 1):
            g.push()
            o.push()
            depth += 1
        dom = narrowed(rng, lay, o.domains())
        if step % 2:
            st, d, c = g.propagate(dom, want_ct=True)
        else:
            (st, d), c = g.propagate(dom), None
        os_, od, oc = o.propagate(dom, want_ct=True)
        assert st == os_, step
        failed = st in (O.FAIL, ct.E_STATE)
        if st == O.OK:
            assert (d == od).all(), step
            assert c is None or (c == oc).all(), step
        sd, sc = g.state()
        assert failed or (sd == o.state()[0]).all(), step
        assert (sc == o.state()[1]).all(), step


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("names,slots", [
    (["one granule", "4 granules", "negative"], 5),
    (["5 granules", "one granule", "64 granules", "negative", "one granule, 17 words"], 4),
    (["260 granules", "513 words", "4 granules", "65 granules"], 3),
    (["selected bits", "512 words"], 30),  # the static scratch takes several launches
])
def test_staged_batches(names, slots, noalloc):
    say("staged batches:", names, slots, "slots each, noalloc", noalloc)
    rng = W.rng_for(len(names), 931, slots)
    tabs = [make(n, rng) for n in names]
    first = [g.slots_alloc(slots, max_depth=8) for g, _, _ in tabs]
    steps = 6 if slots < 10 else 2
    stacks = [[[] for _ in range(slots)] for _ in tabs]  # the levels' domains, per slot
    cur = [[o.domains() for _ in range(slots)] for _, o, _ in tabs]
    for step in range(steps):
        jobs, want = [], []
        for s in range(slots):
            for k, (g, o, lay) in enumerate(tabs):
                stack = stacks[k][s]
                flags, n_pop, n_push = ct.JOB_PROPAGATE, 0, 0
                r = rng.random()
                dead = cur[k][s] is None
                if r < 0.15 or (dead and not stack):
                    flags |= ct.JOB_FROM_ROOT
                    del stack[:]
                    cur[k][s] = tabs[k][1].domains()
                else:
                    if stack and (dead or r < 0.5):
                        n_pop = int(rng.integers(1, len(stack) + 1))
                        cur[k][s] = stack[-n_pop]
                        del stack[len(stack) - n_pop:]
                    n_push = min(int(rng.integers(0, 3)), 8 - len(stack))
                    stack.extend([cur[k][s]] * n_push)
                    if r > 0.93:
                        flags = 0  # pops and pushes only
                dead = cur[k][s] is None
                dom = narrowed(rng, lay, tabs[k][1].domains() if dead else cur[k][s])
                din = torch.from_numpy(dom.view(np.int64).copy()).cuda()
                dout = torch.full_like(din, -1)
                cout = torch.full((g.W,), -1, dtype=torch.int64, device="cuda") if rng.random() < 0.4 else None
                jobs.append(dict(table=g, slot=first[k] + s, flags=flags, n_pop=n_pop, n_push=n_push, dom_in=din,
                                 dom_out=dout, ct_out=cout))
                want.append((k, s, flags, dom))
        status = torch.full((len(jobs),), 99, dtype=torch.int32, device="cuda")
        ct.propagate_batch(jobs, status, noalloc=noalloc)
        ct.batch_status()
        st = status.cpu().numpy()
        for j, (k, s, flags, dom) in enumerate(want):
            o = tabs[k][1]
            if flags == 0:
                assert st[j] == ct.OK, (step, j)
                continue
            if cur[k][s] is None:  # a failed slot
                assert st[j] == ct.E_STATE, (step, j)
                continue
            # the slot's domains from the root, then this input: the closure
            # does not depend on the path, so the slots share one oracle
            o.push()
            o.propagate(cur[k][s])
            os_, od, oc = o.propagate(dom, want_ct=True)
            if os_ == O.OK:
                wd, wc = o.state()[:2]
            o.pop()
            assert st[j] == os_, (step, j, names[k])
            job = jobs[j]
            if os_ == O.OK:
                sd, sc = tabs[k][0].state(job["slot"])
                assert (job["dom_out"].cpu().numpy().view(np.uint64) == od).all(), (step, j, names[k])
                assert (sd == wd).all() and (sc == wc).all(), (step, j, names[k])
                if job["ct_out"] is not None:
                    assert (job["ct_out"].cpu().numpy().view(np.uint64) == oc).all(), (step, j, names[k])
                cur[k][s] = od
            elif os_ == O.FAIL:
                cur[k][s] = None
            elif job["ct_out"] is not None:
                assert (job["ct_out"] == -1).all(), (step, j, names[k])


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("ds,tuples", [
    ([95], 100), ([96], 5000), ([40, 55], 4096), ([191], 300), ([192], 20_000),  # one, two, four waves a granule
    ([7, 90, 2, 100, 3], 9000), ([200, 1, 200], 40_000), ([60] * 10, 17_000),    # segments across the parts' ends
    ([1, 2, 3], 70), ([64 * 200, 64 * 313], 6000), ([36_000, 38_000], 5000),     # a long list, selected bits
])
def test_staged_roots(ds, tuples, noalloc):
    say("staged roots: domains", ds, tuples, "tuples, noalloc", noalloc)
    rng = W.rng_for(len(ds), 933, tuples)
    lo = np.zeros(len(ds), np.int32)
    d = np.array(ds, np.int32)
    tup = np.stack([rng.integers(0, x, size=tuples) for x in ds], 1).astype(np.int32)
    if len(ds) > 3:
        tup[rng.random(tup.shape) < 0.02] = ct.STAR
    g = ct.Table(tup, lo, d)
    lay = W.DomLayout(d, lo)
    doms = [lay.full()]
    for share in (0.02, 0.5, 0.97):
        dom = lay.full()
        for i in range(lay.n):
            keep = rng.random(ds[i]) >= share
            keep[int(rng.integers(0, ds[i]))] = True
            for a in np.nonzero(~keep)[0]:
                lay.clear(dom, i, int(a))
        doms.append(dom)
    doms.append(lay.full())
    doms[-1][0] = 0  # a variable without a value
    first = g.slots_alloc(len(doms), max_depth=0)
    din = torch.from_numpy(np.stack(doms).view(np.int64).copy()).cuda()
    dout, cts = torch.zeros_like(din), torch.full((len(doms), g.W), -1, dtype=torch.int64, device="cuda")
    status = torch.full((len(doms),), 99, dtype=torch.int32, device="cuda")
    for _ in range(2):
        ct.propagate_batch([dict(table=g, slot=first + k, flags=ct.JOB_PROPAGATE | ct.JOB_ROOT, dom_in=din[k],
                                 dom_out=dout[k], ct_out=None if k % 2 else cts[k]) for k in range(len(doms))],
                           status, noalloc=noalloc)
    ct.batch_status()
    for k, dom in enumerate(doms):
        o = O.OracleTable(tup, lo, d, init_dom=dom)
        assert int(status[k]) == o.create_status, k
        sd, sc = g.state(first + k)
        od, oc = o.state()[:2]
        assert (sc == oc).all(), k
        if o.create_status == O.OK:
            assert (sd == od).all() and (dout[k].cpu().numpy().view(np.uint64) == od).all(), k
            assert k % 2 or (cts[k].cpu().numpy().view(np.uint64) == oc).all(), k


@pytest.mark.parametrize("n_tables,n_pool,dom,tuples,negatives,hub", [
    (3, 4, (2, 130), (20, 400), 1, False),
    (40, 30, (2, 20), (30, 20_000), 6, True),
    (300, 500, (2, 9), (20, 300), 20, False),     # more tables than compute units
    (6, 5, (36_000, 36_000), (2000, 4000), 0, True),  # wide domains
])
def test_model_rounds(n_tables, n_pool, dom, tuples, negatives, hub):
    say("model rounds:", n_tables, "tables over", n_pool, "variables, domains", dom, "negatives", negatives, "hub", hub)
    rng = W.rng_for(n_tables, 932, 0)
    ds = rng.integers(dom[0], dom[1] + 1, size=n_pool).astype(np.int32)
    lay = W.DomLayout(ds, np.zeros(n_pool, np.int32))
    M = ct.Model(np.zeros(n_pool, np.int32), ds)
    gts, ots, scopes = [], [], []
    for c in range(n_tables):
        k = int(rng.integers(2, 4))
        sc = rng.choice(n_pool, size=k, replace=False).astype(np.int32)
        if hub and 0 not in sc:
            sc[0] = 0  # every table has this variable
        d = ds[sc]
        t = int(rng.integers(tuples[0], tuples[1] + 1))
        tup = np.unique(np.stack([rng.integers(0, d[i], size=t) for i in range(k)], 1).astype(np.int32), axis=0)
        kind = ct.KIND_NEGATIVE if c < negatives else 0
        if kind:
            tup = tup[: max(1, int(np.prod(d.astype(np.float64)) // 4))]
        lo = np.zeros(k, np.int32)
        gts.append(ct.Table(tup, lo, d, kind=kind))
        ots.append(O.OracleTable(tup, lo, d, kind=kind, fast=kind == 0))
        M.add(gts[-1], sc)
        scopes.append(sc)
    out = torch.zeros(lay.D, dtype=torch.int64, device="cuda")
    pool, stack, total = lay.full(), [], 0
    for step in range(9):
        if stack and step % 4 == 3:
            for _ in range(int(rng.integers(1, len(stack) + 1))):
                M.pop()
                for o in ots:
                    o.pop()
                pool = stack.pop()
        for _ in range(2 if step % 3 == 1 else 1):
            M.push()
            for o in ots:
                o.push()
            stack.append(pool.copy())
        new = pool if step == 0 else W.pick_fraction_removal(rng, lay, pool, frac=0.02 if step % 2 else 0.3)
        st, props, rounds = M.fixpoint(torch.from_numpy(new.view(np.int64).copy()).cuda(), out)
        os_, opool, _ = O.fixpoint(ots, scopes, lay, new)
        assert st == os_, step
        assert props >= 0 and rounds >= 1
        total += props
        if st == ct.OK:
            pool = out.cpu().numpy().view(np.uint64).copy()
            assert (pool == opool).all(), step
            for c in range(0, n_tables, max(1, n_tables // 5)):  # (waits for the model's stream)
                assert (gts[c].state()[0] == ots[c].state()[0]).all(), (step, c)
                assert (gts[c].state()[1] == ots[c].state()[1]).all(), (step, c)
        else:
            M.pop()
            for o in ots:
                o.pop()
            pool = stack.pop()
    assert total > 0


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("ds,tuples,slots", [
    ([110_000, 100_000], 3000, 10),  # selected bits, domains of more than a prep pass, one update item
    ([130, 70], 400, 900),           # smallest prep workgroup
])
def test_staged_jobs_without_row_lists(ds, tuples, slots, noalloc):
    """Jobs whose prep passes no barrier between reading |dom| and noting its
    items: selected bits, inputs without a change, an emptied variable."""
    say("staged jobs without row lists: domains", ds, tuples, "tuples", slots, "slots, noalloc", noalloc)
    rng = W.rng_for(len(ds), 934, tuples)
    lo, d = np.zeros(len(ds), np.int32), np.array(ds, np.int32)
    tup = np.stack([rng.integers(0, x, size=tuples) for x in ds], 1).astype(np.int32)
    g = ct.Table(tup, lo, d)
    lay = W.DomLayout(d, lo)
    root = g.domains()
    most = lay.full()
    for i, n in enumerate(ds):
        for a in rng.choice(n, size=n // 5, replace=False):
            lay.clear(most, i, int(a))
    gone = root.copy()
    gone[lay.off[1]:] = 0  # the second variable has no value left
    P = ct.JOB_PROPAGATE
    kinds = [(P | ct.JOB_ROOT, lay.full()), (P | ct.JOB_ROOT, most), (P, root), (P | ct.JOB_FROM_ROOT, root), (P, gone)]
    want = []
    for flags, dom in kinds:
        if flags & ct.JOB_ROOT:
            o = O.OracleTable(tup, lo, d, init_dom=dom)
            want.append((o.create_status, o.state()[0], o.state()[1]))
        else:
            o = O.OracleTable(tup, lo, d)
            st = o.propagate(dom)[0]
            want.append((st, o.state()[0], o.state()[1]))
    assert [w[0] for w in want] == [O.OK] * 4 + [O.FAIL]
    first = g.slots_alloc(slots, max_depth=0)
    of = [k % len(kinds) for k in range(slots)]
    din = torch.from_numpy(np.stack([kinds[k][1] for k in of]).view(np.int64).copy()).cuda()
    dout = torch.zeros_like(din)
    status = torch.full((slots,), 99, dtype=torch.int32, device="cuda")
    ct.propagate_batch([dict(table=g, slot=first + s, flags=kinds[k][0], dom_in=din[s], dom_out=dout[s])
                        for s, k in enumerate(of)], status, noalloc=noalloc)
    ct.batch_status()
    st, got = status.cpu().numpy(), dout.cpu().numpy().view(np.uint64)
    for s, k in enumerate(of):
        assert st[s] == want[k][0], (s, k)
        if want[k][0] == O.OK:
            assert (got[s] == want[k][1]).all(), (s, k)
            if s < 10:
                sd, sc = g.state(first + s)
                assert (sd == want[k][1]).all() and (sc == want[k][2]).all(), (s, k)


@pytest.mark.parametrize("sizes", [[40] * 60, [1] * 40 + [700] * 3 + [40] * 40, [300, 310, 320, 330] * 4])
def test_queued_batches_keep_their_descriptors(sizes):
    """Batches queued ahead of the GPU: the descriptors of each are its own
    until it has run, over several turns of the staging buffers and a growth."""
    say("queued batches:", len(sizes), "of", sorted(set(sizes)), "jobs")
    rng = W.rng_for(len(sizes), 935, max(sizes))
    g, o, lay = make("one granule", rng)
    first = g.slots_alloc(max(sizes), max_depth=0)
    doms, want = [], []
    for _ in range(7):
        dom = W.pick_fraction_removal(rng, lay, o.domains(), frac=0.2)
        o.push()
        st, od = o.propagate(dom)
        doms.append(dom)
        want.append(od if st == O.OK else None)
        o.pop()
    assert any(w is not None for w in want)
    din = torch.from_numpy(np.stack(doms).view(np.int64).copy()).cuda()
    batches = []
    for b, n in enumerate(sizes):
        dout = torch.full((n, g.D), -1, dtype=torch.int64, device="cuda")
        status = torch.full((n,), 99, dtype=torch.int32, device="cuda")
        # (push and propagate would do as well; a second job kind changes the
        # descriptors' flags from batch to batch)
        flags = ct.JOB_PROPAGATE | (ct.JOB_FROM_ROOT if b % 3 else ct.JOB_ROOT)
        batches.append((ct.Batch([dict(table=g, slot=first + k, flags=flags, dom_in=din[(b + k) % 7], dom_out=dout[k])
                                  for k in range(n)]), dout, status))
    torch.cuda.synchronize()
    torch.cuda._sleep(20_000_000)  # the GPU starts some 10 ms after the first batch is queued
    for batch, _, status in batches:
        ct.propagate_batch(batch, status)
    ct.batch_status()
    for b, (_, dout, status) in enumerate(batches):
        st, got = status.cpu().numpy(), dout.cpu().numpy().view(np.uint64)
        for k in range(sizes[b]):
            w = want[(b + k) % 7]
            assert st[k] == (O.FAIL if w is None else O.OK), (b, k)
            assert w is None or (got[k] == w).all(), (b, k)


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("extra", [0, 1])
def test_large_root_batches(extra, noalloc):
    """Root batches of about as many granules as the streaming update takes up
    (4,096 on 256 compute units): just below it, and above with rejected jobs,
    emptied variables and tables of every size among the others."""
    names = {"64 granules": 63 + 2 * extra, "5 granules": 6, "one granule": 9, "260 granules": extra,
             "one granule, 17 words": 3, "513 words": 2}
    say("large root batch:", names, "noalloc", noalloc)
    rng = W.rng_for(len(names), 936, extra)
    jobs, want, tabs = [], [], []
    for name, slots in names.items():
        ds, t, star, _, _ = TABLES[name]
        lo, d = np.zeros(len(ds), np.int32), np.array(ds, np.int32)
        tup = np.stack([rng.integers(0, x, size=t) for x in ds], 1).astype(np.int32)
        if name == "5 granules":
            tup[rng.random(tup.shape) < 0.03] = ct.STAR
        g = ct.Table(tup, lo, d, max_depth=0)
        tabs.append(g)
        lay = W.DomLayout(d, lo)
        doms = [lay.full(), W.pick_fraction_removal(rng, lay, lay.full(), frac=0.6, nvars=(1, 2)), lay.full(), lay.full()]
        doms[2][0] = 0 if lay.words[0] == 1 else doms[2][0]  # a variable without a value
        doms[3][-1] = ~np.uint64(0)  # values beyond the domain, if its last word has room for them
        ref = []
        for k, dom in enumerate(doms):
            if k == 3 and ds[-1] % 64:
                ref.append((ct.E_INVALID,) + O.OracleTable(tup, lo, d).state()[:2])
            else:
                o = O.OracleTable(tup, lo, d, init_dom=dom)
                ref.append((o.create_status,) + o.state()[:2])
        first = g.slots_alloc(slots, max_depth=0) if slots else 0
        for s in range(slots):
            k = int(rng.integers(0, 4)) if s > 1 else s
            din = torch.from_numpy(doms[k].view(np.int64).copy()).cuda()
            dout = torch.full_like(din, -1)
            cout = torch.full((g.W,), -1, dtype=torch.int64, device="cuda") if s % 3 == 0 else None
            jobs.append(dict(table=g, slot=first + s, flags=ct.JOB_PROPAGATE | ct.JOB_ROOT, dom_in=din, dom_out=dout,
                             ct_out=cout))
            want.append((name, s, ref[k]))
    turn = rng.permutation(len(jobs))
    jobs, want = [jobs[k] for k in turn], [want[k] for k in turn]
    assert (sum(j["table"].granules for j in jobs) >= 4096) == bool(extra)
    status = torch.full((len(jobs),), 99, dtype=torch.int32, device="cuda")
    for _ in range(2):
        ct.propagate_batch(jobs, status, noalloc=noalloc)
    ct.batch_status()
    st = status.cpu().numpy()
    for j, (name, s, (ws, wd, wc)) in enumerate(want):
        assert st[j] == ws, (name, s)
        sd, sc = jobs[j]["table"].state(jobs[j]["slot"])
        assert (sc == wc).all(), (name, s)
        if ws != O.FAIL:
            assert (sd == wd).all(), (name, s)
        if ws == O.OK:
            assert (jobs[j]["dom_out"].cpu().numpy().view(np.uint64) == wd).all(), (name, s)
            c = jobs[j]["ct_out"]
            assert c is None or (c.cpu().numpy().view(np.uint64) == wc).all(), (name, s)
