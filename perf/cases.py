"""The workloads whose speed this library is measured by.

Each case is one thing that a program using the library does: a search's
synchronous propagate / push / pop calls on one table, the creation of a
table, a batch of search nodes, a batch of root recomputations, the search
steps of a model of many tables, the rounds of many concurrent searches.
Sizes follow the shapes of ``workloads.py`` and of the tests.

``listed()`` names the cases, ``draw(rng)`` gives others of the same ranges,
``prepare(case, seed)`` makes inputs and handles, ``run(state)`` is one pass,
``work(case)`` the bytes a pass cannot do without.  Every output is a whole
number (statuses and bit patterns), so there is nothing to compare within a
tolerance: ``exact`` has no value for any case.
"""
import math

import numpy as np
import torch

from paper_2507_18413_amd import ct
from paper_2507_18413_amd import workloads as W
from paper_2507_18413_amd.solver import GpuTables


def listed():
    return [
        # a search over one small constraint: every call is pure latency
        dict(name="calls tiny", what="calls", kind="positive", n=3, dlo=8, dhi=8, t=200, calls=100, cut=0.125),
        # a search over one large table (200,000 tuples, 3,125 words a row)
        dict(name="calls large", what="calls", kind="positive", n=5, dlo=50, dhi=50, t=200_000, calls=100, cut=0.05),
        # one constraint over 100 variables (linear-constraint instances)
        dict(name="calls wide", what="calls", kind="positive", n=100, dlo=64, dhi=160, t=10_000, calls=60, cut=0.05),
        # one constraint over 150 variables with up to 2,000 values each
        dict(name="calls paper shape", what="calls", kind="positive", n=150, dlo=2, dhi=2000, t=15_000, calls=30,
             cut=0.05),
        # the largest table of the serving mix, searched with plain calls
        dict(name="calls 2M tuples", what="calls", kind="positive", n=8, dlo=8, dhi=128, t=2_000_000, calls=40,
             cut=0.05),
        # forbidden combinations: a conflict table
        dict(name="calls negative", what="calls", kind="negative", n=5, dlo=7, dhi=9, t=12_000, calls=40, cut=0.12),
        # loading a table: supports and root propagation from its tuples and
        # initial domains with holes
        dict(name="create 1M", what="create", n=6, dlo=20, dhi=20, t=1_000_000, zipf=True),
        # a frontier of search nodes on one skewed table
        dict(name="nodes 4096", what="nodes", n=6, dlo=20, dhi=20, t=1_000_000, zipf=True, nodes=4096, cut=0.6,
             tables_out=False),
        # a smaller frontier on a table with more values, currTables wanted
        dict(name="nodes 500 long rows", what="nodes", n=8, dlo=8, dhi=128, t=300_000, zipf=False, nodes=500, cut=0.3,
             tables_out=True),
        # restarting a model: the roots of its tables from changed domains
        dict(name="roots 400", what="roots", tables=400, tlo=100, thi=500_000),
        # search steps of a model of many tables that share variables
        dict(name="model 400 tables", what="model", tables=400, pool=1000, tlo=100, thi=500_000, steps=6),
        # many searches over a mix of tables, one request of each per batch
        dict(name="searches 128", what="searches", tables=48, searches=128, tlo=1_000, thi=2_000_000, rounds=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["calls", "calls", "calls", "calls", "calls", "calls", "create", "nodes", "nodes", "roots",
                       "model", "searches"])
    if what == "calls":
        shape = rng.choice(["small", "large", "large", "wide", "negative", "short"])
        c = dict(what="calls", kind="positive", cut=round(rng.uniform(0.04, 0.13), 3))
        if shape == "small":
            c.update(n=rng.randint(2, 8), dlo=rng.randint(3, 8), dhi=rng.randint(9, 40), t=_log_int(rng, 50, 16_000),
                     calls=rng.randint(60, 110))
        elif shape == "large":
            c.update(n=rng.randint(3, 10), dlo=rng.randint(8, 40), dhi=rng.randint(50, 128),
                     t=_log_int(rng, 20_000, 1_900_000), calls=rng.randint(30, 60))
        elif shape == "wide":
            c.update(n=rng.randint(40, 150), dlo=rng.randint(2, 64), dhi=_log_int(rng, 100, 1_900),
                     t=rng.randint(3_000, 15_000), calls=rng.randint(20, 40))
        elif shape == "negative":
            c.update(kind="negative", n=rng.randint(3, 6), dlo=rng.randint(6, 8), dhi=rng.randint(9, 14),
                     t=_log_int(rng, 100, 20_000), calls=rng.randint(30, 50))
        else:
            c.update(kind="short", n=rng.randint(4, 30), dlo=rng.randint(4, 12), dhi=rng.randint(13, 40),
                     t=_log_int(rng, 300, 60_000), calls=rng.randint(40, 70))
        return c
    if what == "create":
        return dict(what="create", n=rng.randint(3, 10), dlo=rng.randint(8, 30), dhi=rng.randint(31, 128),
                    t=_log_int(rng, 20_000, 1_000_000), zipf=rng.random() < 0.5)
    if what == "nodes":
        if rng.random() < 0.5:
            return dict(what="nodes", n=rng.randint(3, 7), dlo=rng.randint(5, 15), dhi=rng.randint(16, 30),
                        t=_log_int(rng, 20_000, 900_000), zipf=rng.random() < 0.5, nodes=_log_int(rng, 40, 4_000),
                        cut=round(rng.uniform(0.2, 0.6), 2), tables_out=False)
        return dict(what="nodes", n=rng.randint(5, 10), dlo=rng.randint(8, 60), dhi=rng.randint(61, 128),
                    t=_log_int(rng, 10_000, 400_000), zipf=rng.random() < 0.5, nodes=_log_int(rng, 40, 700),
                    cut=round(rng.uniform(0.1, 0.4), 2), tables_out=rng.random() < 0.5)
    if what == "roots":
        return dict(what="roots", tables=rng.randint(20, 390), tlo=rng.randint(100, 3_000),
                    thi=rng.randint(50_000, 500_000))
    if what == "model":
        tables = rng.randint(20, 390)
        return dict(what="model", tables=tables, pool=int(2.5 * tables), tlo=rng.randint(100, 2_000),
                    thi=rng.randint(30_000, 500_000), steps=rng.randint(4, 8))
    return dict(what="searches", tables=rng.randint(8, 48), searches=rng.randint(16, 128), tlo=rng.randint(1_000, 5_000),
                thi=rng.randint(100_000, 1_900_000), rounds=5)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _shape_rng(case):
    """The table's shape belongs to the case, its contents to the seed."""
    key = [int(v) if not isinstance(v, str) else sum(map(ord, v)) for k, v in sorted(case.items())
           if k not in ("name", "cut")]
    return np.random.default_rng(key)


def _dsizes(case):
    return _shape_rng(case).integers(case["dlo"], case["dhi"] + 1, size=case["n"]).astype(np.int32)


def _tuples(rng, dsizes, t, zipf=False, distinct=False):
    """t tuples, uniform or with truncated Zipf(1.1) columns.  In a large
    product of domains repeated tuples are rare and are left in."""
    space = math.prod(int(d) for d in dsizes)
    t = max(1, min(t, space // 2))
    if distinct or space < 4_000_000 and not zipf:
        return W.distinct_uniform_tuples(rng, dsizes, t)
    out = np.empty((t, len(dsizes)), np.int32)
    for i, d in enumerate(dsizes):
        if zipf:
            cdf = np.cumsum(W.zipf_probs(int(d), 1.1))
            out[:, i] = np.minimum(np.searchsorted(cdf, rng.random(t, dtype=np.float32)), d - 1)
        else:
            out[:, i] = rng.integers(0, d, size=t, dtype=np.int32)
    return out


def _n_tuples(dsizes, t):
    return max(1, min(t, math.prod(int(d) for d in dsizes) // 2))


def _keep(rng, dsizes, cut, nvars):
    """A domain bitmap with every value but ceil(cut x d) values of nvars
    random variables."""
    lay = W.DomLayout(dsizes, np.zeros_like(dsizes))
    out = lay.full()
    for i in rng.choice(lay.n, size=min(nvars, lay.n), replace=False):
        d = int(dsizes[i])
        for a in rng.choice(d, size=min(d, math.ceil(cut * d)), replace=False):
            lay.clear(out, int(i), int(a))
    return out


def _node_domains(rng, dsizes, root, n_nodes, cut):
    """Per node and variable, f ~ U[0, cut] of the root's values removed."""
    lay = W.DomLayout(dsizes, np.zeros_like(dsizes))
    out = np.zeros((n_nodes, lay.D), np.uint64)
    for i in range(lay.n):
        vals = lay.values(root, i)
        gone = np.floor(rng.random(n_nodes) * cut * vals.size).astype(np.int64)
        rank = rng.random((n_nodes, vals.size)).argsort(axis=1).argsort(axis=1)
        bits = np.zeros((n_nodes, int(lay.words[i]) * 64), np.uint8)
        bits[:, vals] = rank >= gone[:, None]
        o, w = int(lay.off[i]), int(lay.words[i])
        out[:, o:o + w] = np.packbits(bits, axis=1, bitorder="little").view(np.uint64)
    return out


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def _many(case):
    """Shapes of a model's or a serving mix's tables: arity, domain sizes and
    tuple counts drawn as in ``workloads``; (scope or None, dsizes, t)."""
    r = _shape_rng(case)
    out = []
    if case["what"] == "searches":
        for _ in range(case["tables"]):
            ds = r.integers(8, 129, size=int(r.integers(3, 11))).astype(np.int32)
            out.append((None, ds, _n_tuples(ds, _log_int_np(r, case))))
        return None, out
    pool = r.integers(4, 65, size=case.get("pool", int(2.5 * case["tables"]))).astype(np.int32)
    for _ in range(case["tables"]):
        scope = r.choice(pool.size, size=int(r.integers(2, 9)), replace=False).astype(np.int32)
        out.append((scope, pool[scope], _n_tuples(pool[scope], _log_int_np(r, case))))
    return pool, out


def _log_int_np(r, case):
    return int(round(math.exp(r.uniform(math.log(case["tlo"]), math.log(case["thi"])))))


# ---------------------------------------------------------------------------
# prepare
# ---------------------------------------------------------------------------
def prepare(case, seed):
    rng = np.random.default_rng([seed, 71])
    return {"calls": _prepare_calls, "create": _prepare_create, "nodes": _prepare_nodes, "roots": _prepare_roots,
            "model": _prepare_model, "searches": _prepare_searches}[case["what"]](case, rng)


def _prepare_calls(case, rng):
    ds = _dsizes(case)
    negative, short = case["kind"] == "negative", case["kind"] == "short"
    tup = _tuples(rng, ds, case["t"], distinct=negative)
    if short:
        tup[rng.random(tup.shape) < 0.15] = ct.STAR
    t = ct.Table(tup, np.zeros_like(ds), ds, kind=ct.KIND_NEGATIVE if negative else ct.KIND_POSITIVE)
    # a level before every call, U{1..depth} levels back after every tenth
    script = [(_keep(rng, ds, case["cut"], int(rng.integers(1, 4))), rng.random() if k % 10 == 9 else None)
              for k in range(case["calls"])]
    return dict(run=_run_calls, table=t, root=t.domains(), script=script)


def _prepare_create(case, rng):
    ds = _dsizes(case)
    return dict(run=_run_create, tuples=_tuples(rng, ds, case["t"], case["zipf"]), lo=np.zeros_like(ds), dsizes=ds,
                init=_keep(rng, ds, 0.1, len(ds)))


def _prepare_nodes(case, rng):
    ds = _dsizes(case)
    t = ct.Table(_tuples(rng, ds, case["t"], case["zipf"]), np.zeros_like(ds), ds)
    n = case["nodes"]
    first = t.slots_alloc(n, max_depth=0)
    din = _cuda(_node_domains(rng, ds, t.domains(), n, case["cut"]))
    dout = torch.zeros_like(din)
    cts = torch.zeros((n, t.W), dtype=torch.int64, device="cuda") if case["tables_out"] else None
    status = torch.zeros(n, dtype=torch.int32, device="cuda")
    batch = ct.Batch([dict(table=t, slot=first + k, flags=ct.JOB_PROPAGATE | ct.JOB_FROM_ROOT, dom_in=din[k],
                           dom_out=dout[k], ct_out=cts[k] if cts is not None else None) for k in range(n)])
    out = dict(domains=dout, status=status)
    if cts is not None:
        out["tables"] = cts
    return dict(run=_run_batch, batch=batch, status=status, out=out)


def _prepare_roots(case, rng):
    _, shapes = _many(case)
    tabs = [ct.Table(_tuples(rng, ds, t), np.zeros_like(ds), ds, max_depth=0) for _, ds, t in shapes]
    off = np.cumsum([0] + [t.D for t in tabs])
    off_ct = np.cumsum([0] + [t.W for t in tabs])
    din = np.concatenate([_keep(rng, ds, float(rng.random() * 0.2), len(ds)) for _, ds, _ in shapes])
    din = _cuda(din)
    dout = torch.zeros_like(din)
    cts = torch.zeros(int(off_ct[-1]), dtype=torch.int64, device="cuda")
    status = torch.zeros(len(tabs), dtype=torch.int32, device="cuda")
    batch = ct.Batch([dict(table=t, slot=t.slots_alloc(1, max_depth=0), flags=ct.JOB_PROPAGATE | ct.JOB_ROOT,
                           dom_in=din[off[k]:], dom_out=dout[off[k]:], ct_out=cts[off_ct[k]:])
                      for k, t in enumerate(tabs)])
    return dict(run=_run_batch, batch=batch, status=status, out=dict(domains=dout, tables=cts, status=status))


def _prepare_model(case, rng):
    pool, shapes = _many(case)
    hidden = (rng.random(pool.size) * pool).astype(np.int32)  # a solution: the root never fails
    m = ct.Model(np.zeros_like(pool), pool)
    tabs = []
    for scope, ds, t in shapes:
        tup = _tuples(rng, ds, t)
        tup[0] = hidden[scope]
        tabs.append(ct.Table(tup, np.zeros_like(ds), ds, max_depth=16))
        m.add(tabs[-1], scope)
    keep = np.stack([_keep(rng, pool, 0.05, int(rng.integers(1, 4))) for _ in range(case["steps"])])
    lay = W.DomLayout(pool, np.zeros_like(pool))
    model = GpuTables(m, lay.D)
    failed, root = model.fixpoint(lay.full())
    if failed:
        raise RuntimeError("the planted model has no root")
    return dict(run=_run_model, model=model, tables=tabs, keep=keep, root=root)


def _prepare_searches(case, rng):
    _, shapes = _many(case)
    tabs = [ct.Table(_tuples(rng, ds, t, zipf=k % 2 == 1), np.zeros_like(ds), ds, max_depth=8)
            for k, (_, ds, t) in enumerate(shapes)]
    n, rounds = case["searches"], case["rounds"]
    of = rng.integers(0, len(tabs), size=n)
    first = {int(c): tabs[c].slots_alloc(int((of == c).sum()), max_depth=8) for c in sorted(set(of.tolist()))}
    slot = []
    for c in of.tolist():
        slot.append(first[c])
        first[c] += 1
    width = max(t.D for t in tabs)
    keep = np.zeros((rounds, n, width), np.uint64)
    start = np.zeros((n, width), np.uint64)
    for j, c in enumerate(of.tolist()):
        start[j, :tabs[c].D] = tabs[c].domains()
        for r in range(rounds):
            keep[r, j, :tabs[c].D] = _keep(rng, shapes[c][1], 0.05, int(rng.integers(1, 5)))
    keep, start = _cuda(keep), _cuda(start)
    din, dout = torch.zeros_like(keep), torch.zeros_like(keep)
    status = torch.zeros((rounds, n), dtype=torch.int32, device="cuda")
    batches, before = [], []
    for r in range(rounds):
        # the first request starts at the root, each next one pushes a level;
        # the last backtracks two levels first
        last = r == rounds - 1
        how = dict(flags=ct.JOB_PROPAGATE | ct.JOB_FROM_ROOT) if r == 0 else \
            dict(flags=ct.JOB_PROPAGATE, n_pop=2 if last else 0, n_push=1)
        batches.append(ct.Batch([dict(table=tabs[c], slot=slot[j], dom_in=din[r, j], dom_out=dout[r, j], **how)
                                 for j, c in enumerate(of.tolist())]))
        before.append(start if r == 0 else dout[r - 3] if last else dout[r - 1])
    return dict(run=_run_searches, batches=batches, before=before, keep=keep, din=din, dout=dout, status=status)


# ---------------------------------------------------------------------------
# run
# ---------------------------------------------------------------------------
def run(state):
    return state["run"](state)


def _run_calls(s):
    t, cur, stack = s["table"], s["root"], []
    status, domains = [], []
    for keep, back in s["script"]:
        t.push()
        stack.append(cur)
        st, dom = t.propagate(cur & keep)
        status.append(st)
        domains.append(dom)
        if st == ct.OK:
            cur = dom
        else:
            t.pop()
            cur = stack.pop()
        if back is not None and stack:
            for _ in range(1 + int(back * len(stack))):
                if stack:
                    t.pop()
                    cur = stack.pop()
    while stack:
        t.pop()
        stack.pop()
    return dict(status=np.array(status, np.int32), domains=np.stack(domains).view(np.int64))


def _run_create(s):
    t = ct.Table(s["tuples"], s["lo"], s["dsizes"], init_dom=s["init"])
    domains, table = t.state()
    t.close()
    return dict(domains=domains.view(np.int64), table=table.view(np.int64))


def _run_batch(s):
    ct.propagate_batch(s["batch"], s["status"])
    return s["out"]


def _run_model(s):
    m, cur, depth, status, pools = s["model"], s["root"], 0, [], []
    for keep in s["keep"]:
        m.push()
        failed, pool = m.fixpoint(cur & keep)
        status.append(failed)
        pools.append(pool)
        if failed:
            m.pop()
        else:
            cur = pool
            depth += 1
    for _ in range(depth):
        m.pop()
    return dict(status=np.array(status, np.int32), pools=np.stack(pools).view(np.int64))


def _run_searches(s):
    for r, b in enumerate(s["batches"]):
        torch.bitwise_and(s["before"][r], s["keep"][r], out=s["din"][r])
        ct.propagate_batch(b, s["status"][r])
    return dict(domains=s["dout"], status=s["status"])


# ---------------------------------------------------------------------------
# work and exact values
# ---------------------------------------------------------------------------
def _call_bytes(ds, t, cut, nvars=2.0):
    """One call: the support words of the removed values, currTable read and
    written, the domains in and out, one residue word for each value."""
    words = -(-_n_tuples(ds, t) // 64)
    rows = nvars * math.ceil(cut * float(np.mean(ds)))
    return 8 * words * (rows + 2) + 16 * float(np.sum(-(-ds // 64))) + 8 * float(np.sum(ds))


def work(case):
    what = case["what"]
    if what in ("calls", "create", "nodes"):
        ds = _dsizes(case)
        rows, words = int(ds.sum()), -(-_n_tuples(ds, case["t"]) // 64)
        if what == "calls":
            b = case["calls"] * _call_bytes(ds, case["t"], case["cut"])
        elif what == "create":
            b = 4 * _n_tuples(ds, case["t"]) * case["n"] + 8 * rows * words + 8 * words
        else:
            # supports once; per node its currTable and domains
            per = 8 * words * (2 if case["tables_out"] else 1) + 16 * float(np.sum(-(-ds // 64)))
            b = 8 * rows * words + case["nodes"] * per
        return dict(bytes=b, flops=0)
    _, shapes = _many(case)
    if what == "roots":
        # every support row of a kept value (on average 0.9 of them), the new currTables twice
        b = sum(8 * -(-t // 64) * (0.9 * float(ds.sum()) + 2) for _, ds, t in shapes)
    elif what == "model":
        # a step reaches the tables of two or so variables
        per = float(np.mean([_call_bytes(ds, t, 0.05, 1.0) for _, ds, t in shapes]))
        b = case["steps"] * (4 * per + 16 * case["pool"])
    else:
        per = float(np.mean([_call_bytes(ds, t, 0.05, 2.5) for _, ds, t in shapes]))
        b = case["rounds"] * case["searches"] * per
    return dict(bytes=b, flops=0)


def exact(case, seed):
    return None  # statuses and bit patterns: whole numbers, compared as they are
