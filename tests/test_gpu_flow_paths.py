"""Runs by cash flows (test_gpu_flows.py) in the situations that need a size, a
graph or a change of curves of their own: graphs that the caller captured,
the library's own graphs with a second branch, curves whose products leave the
FP64 range, books whose rows take several tiles, flows that are kept a batch of
nodes or of tiles at a time, both sides of the rules between the kernels."""
import sys

import numpy as np
import pytest

import oracle
import synth
from tests._helpers import RTOL, assert_reserves_close, to_np
from tests.test_gpu_flows import every_kind, upload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def rr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1401_1757_amd as rr
    return rr


@pytest.mark.parametrize("frac", [False, True])
def test_caller_graph_follows_regenerated_curves(rr, frac):
    """A graph that the caller captured from the allocation-free call reads the
    curves of the last regeneration, within the bounds that the discount
    products need, past them (a slow mean reversion: the bound is passed, the
    products are not large), and where products overflow (long policies with
    them; those that end before keep their reserves)."""
    rng = np.random.default_rng(60)
    w = synth.random_small(rng, n=200, n_steps=120, n_scen=1, n_nodes=1, products=(0, 1, 4, 5))
    pf = w.portfolio
    if frac:
        pf.timing = np.where(np.isin(pf.product, (0, 1)), synth.FRACTIONAL, pf.timing).astype(np.int32)
    base = dict(a=0.1, b=0.03, sigma=0.01, dt=1.0 / 12.0)
    models = [base, dict(base, a=0.01, sigma=0.3), dict(base, b=-200.0), base]
    stream = torch.cuda.Stream()
    ctx = rr.Context(0, stream=stream)
    try:
        ctx.basis_generate_vasicek(w.basis.q, 70, 120, [0.03], key=(1, 2), frac=0.25 if frac else 0.0, **base)
        ctx.portfolio_upload(pf)
        out = ctx.alloc_outputs(1, 70, stats=True)
        torch.cuda.synchronize()
        ctx.reserve_recurrence_noalloc(0, 1, 0, 70, 12, out)
        assert ctx.get_option(rr.OPT_LAST_K) == 0
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ctx.reserve_recurrence_noalloc(0, 1, 0, 70, 12, out)
        for rep, m in enumerate(models):
            key = (7, 8 + rep)
            _say(f"replay after regeneration {m}")
            ctx.curves_generate_vasicek([0.03], key=key, **m)
            torch.cuda.synchronize()
            for x in out.values():
                x.fill_(float("nan"))
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            v, _ = oracle.vasicek_curves(r0=[0.03], n_scen=70, n_steps=120, key=key, **m)
            b = synth.Basis(q=w.basis.q, v=np.asarray(v).reshape(1, 70, 120))
            b.frac = 0.25 if frac else 0.0
            with np.errstate(over="ignore", invalid="ignore"):
                ref = oracle.reserves(b, pf, 0, 1, 0, 70)
                worst = np.log(v).cumsum(axis=-1).max(axis=-1).max()
            # 700: the log of what FP64 holds, with room for the amounts (at most 1e12)
            short = pf.term_m < 1 + np.argmax(np.append(np.log(v).cumsum(axis=-1).reshape(70, 120).max(axis=0), 1e9) > 670.0)
            assert short.all() == (worst <= 670.0) and short.any()
            got, want, gross = (x[:, short] for x in (to_np(out["r0"]), ref["r_all"][..., 0], ref["gross"]))
            assert_reserves_close(got, want, gross)
            if short.all():
                err = np.abs(to_np(out["totals"]) - ref["totals"])
                assert np.all(err <= RTOL * ref["gross_totals"])
                assert np.array_equal(to_np(out["stats"])[:, 1], oracle.node_stats(to_np(out["totals"]))[1])
    finally:
        torch.cuda.synchronize()
        ctx.close()


def test_two_branch_graphs_over_many_output_sets(rr):
    """Runs large enough for the graph's second branch (more than 40,000 tiles x
    scenarios), on more output sets than graphs are kept, without a wait
    between them and with other work on the stream: every set is that of the
    direct launches, bit for bit, and no graph goes while it runs."""
    rng = np.random.default_rng(61)
    n, scen, sets = 9_000, 300, 14
    assert (n // 64) * scen > 40_000
    w = synth.random_small(rng, n=n, n_steps=60, n_scen=scen, n_nodes=1, products=(0, 1, 4, 5))
    ctx = rr.Context(0)
    try:
        ctx.basis_upload(w.basis.q, w.basis.v)
        ctx.portfolio_upload(w.portfolio)
        ctx.set_option(rr.OPT_USE_GRAPH, 0)
        _say("direct launches")
        ref = ctx.reserve_recurrence(0, 1, 0, scen, 12, ctx.alloc_outputs(1, scen, stats=True))
        assert ctx.get_option(rr.OPT_LAST_K) == 0
        torch.cuda.synchronize()
        ctx.set_option(rr.OPT_USE_GRAPH, 1)
        outs = [ctx.alloc_outputs(1, scen, stats=True) for _ in range(sets)]
        for rep in range(3):
            _say(f"round {rep}")
            for o in outs:
                for x in o.values():
                    x.fill_(float("nan"))
            kept = []
            for i, o in enumerate(outs):
                for _ in range(2):   # launched directly, then captured
                    ctx.reserve_recurrence(0, 1, 0, scen, 12, o)
                if i % 3 == 0:   # a replay of the graph just made, and a read behind it
                    for x in o.values():
                        x.fill_(float("nan"))
                    ctx.reserve_recurrence(0, 1, 0, scen, 12, o)
                    kept.append({k: x.clone() for k, x in o.items()})
            torch.cuda.synchronize()
            for o in outs + kept:
                assert all(torch.equal(o[k], ref[k]) for k in ref)
    finally:
        torch.cuda.synchronize()
        ctx.close()


@pytest.mark.parametrize("log10,flows", [(4.0, True), (25.0, True), (27.0, False)])
def test_totals_on_both_sides_of_the_chunk_range(rr, log10, flows):
    """Factors 10^x and 10^-x by turns, then 10^-x: products over all months leave
    the FP64 range; those of a time chunk (ten of 160 months) stay within e^600
    up to x = 26."""
    rng = np.random.default_rng(62)
    w = synth.random_small(rng, n=300, n_steps=160, n_scen=66, n_nodes=1, products=(0, 1, 2, 3, 4, 5))
    big = 10.0 ** log10
    v = w.basis.v
    v[:, :, :60] = np.where(np.arange(60) % 2 == 0, big, 1.0 / big)
    v[:, :, 60:] = 1.0 / big
    chunk = -(-int(w.portfolio.term_m.max()) // 16)
    assert (chunk * log10 * np.log(10.0) <= 600.0) == flows
    ctx = rr.Context(0)
    try:
        ctx.basis_upload(w.basis.q, v)
        ctx.portfolio_upload(w.portfolio)
        ref = oracle.reserves(w.basis, w.portfolio, 0, 1, 0, 66)
        for call in (ctx.reserve_recurrence, ctx.reserve_recurrence_noalloc):
            _say(f"totals, factors 1e{log10:g}, {call.__name__}")
            out = ctx.alloc_outputs(1, 66, r0=False, stats=True)
            call(0, 1, 0, 66, 12, out)
            torch.cuda.synchronize()
            assert (ctx.get_option(rr.OPT_LAST_K) == 0) == flows
            err = np.abs(to_np(out["totals"]) - ref["totals"])
            assert np.all(err <= RTOL * ref["gross_totals"]), err.max()
    finally:
        ctx.close()


def kinds(seed, n, n_steps, n_scen, n_nodes, frac=True, **more):
    """Every kind of policy (levels alone without `frac`) on Gompertz-Makeham
    tables, so that the flows of late months count."""
    w = every_kind(seed, n, n_steps, n_scen, n_nodes, special=frac, **more)
    w.basis.q = synth.mortality_tables(w.basis.q.shape[1], [1.0, 1.2])
    return w


class Book:
    """A workload uploaded to a context; runs of it are checked against one oracle
    run over all nodes and scenarios, or (`sample`) over some of the policies, with
    the totals against the sum of the run's own reserves."""

    def __init__(self, rr, ctx, w, sample=None):
        self.rr, self.ctx, self.w = rr, ctx, w
        upload(ctx, w)
        pf = w.portfolio
        self.pick = np.arange(pf.n)
        if sample is not None:
            self.pick = np.sort(np.random.default_rng(sample).choice(pf.n, sample, replace=False))
            pf = pf.subset(self.pick)
        self.sampled = sample is not None
        self.ref = oracle.reserves(w.basis, pf, 0, w.basis.n_nodes, 0, w.basis.n_scen, w.node_step_m)

    def run(self, noalloc=False, node0=0, nnode=None, scen0=0, nscen=None, flows=True, **which):
        w, ctx = self.w, self.ctx
        nnode = w.basis.n_nodes - node0 if nnode is None else nnode
        nscen = w.basis.n_scen - scen0 if nscen is None else nscen
        out = ctx.alloc_outputs(nnode, nscen, **which)
        for x in out.values():
            x.fill_(float("nan"))
        call = ctx.reserve_recurrence_noalloc if noalloc else ctx.reserve_recurrence
        call(node0, nnode, scen0, nscen, w.node_step_m, out)
        torch.cuda.synchronize()
        assert (ctx.get_option(self.rr.OPT_LAST_K) == 0) == flows
        at = np.s_[node0:node0 + nnode, scen0:scen0 + nscen]
        if "r0" in out:
            assert bool(torch.isfinite(out["r0"]).all())
            of = lambda x: x[node0:node0 + nnode, :, scen0:scen0 + nscen]
            assert_reserves_close(to_np(out["r0"])[:, self.pick], of(self.ref["r_all"][..., 0]), of(self.ref["gross"]))
        if self.sampled:
            tot, bar = to_np(out["r0"].sum(dim=1)), RTOL * to_np(out["r0"].abs().sum(dim=1))
        else:
            tot, bar = self.ref["totals"][at], RTOL * np.maximum(self.ref["gross_totals"][at], 1e-300)
        if "totals" in out:
            assert np.all(np.abs(to_np(out["totals"]) - tot) <= bar)
        if "stats" in out:
            st = to_np(out["stats"])
            mean, tail = oracle.node_stats(tot)
            assert np.all(np.abs(st[:, 0] - mean) <= bar.max(axis=1)) and np.all(np.abs(st[:, 1] - tail) <= bar.max(axis=1))
        return out


@pytest.fixture()
def ctx(rr):
    c = rr.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


ROWS = 48 << 20   # bytes of the rows of summed flows, all nodes of a launch together


@pytest.mark.parametrize("frac", [False, True])
def test_totals_with_several_tiles_a_row(rr, ctx, frac):
    """More tiles x nodes than rows: a row's wavefronts add each tile to what the
    last one left, another length and another cut of the months, with a second
    row for flows within the month; late nodes with most of the book expired."""
    n, steps, nodes, scen = 20_000, 400, 60, 2
    assert ROWS // ((steps // 8 + 1) * 64 * (2 if frac else 1)) // nodes < n // 64
    b = Book(rr, ctx, kinds(63, n, steps, scen, nodes, frac=frac, node_step=9,
                            products=tuple(range(7)) if frac else (0, 1, 2, 4, 5)))
    for noalloc in (False, True):
        _say(f"totals {n} x {nodes} x {scen}, frac={frac}, noalloc={noalloc}")
        b.run(noalloc, r0=False, stats=True)
    b.run(node0=1, nnode=nodes - 3, r0=False, totals=False, stats=True)


def test_totals_with_more_nodes_than_rows(rr, ctx):
    """Nodes in several launches (two rows of 4,000 months a node)."""
    n, steps, nodes = 70, 4000, 800
    assert ROWS // ((steps // 8 + 1) * 64 * 2) < nodes
    b = Book(rr, ctx, kinds(64, n, steps, 2, nodes, node_step=5))
    for noalloc in (False, True):
        _say(f"totals {n} x {nodes} x 2, {steps} steps, noalloc={noalloc}")
        b.run(noalloc, r0=False, stats=True)


@pytest.mark.parametrize("frac", [False, True])
def test_reserves_with_flows_a_batch_of_nodes_at_a_time(rr, ctx, frac):
    """The allocation-free call keeps the flows of as many nodes as its 64 MiB
    hold; the other call those of all: the same bits."""
    n, steps, nodes, scen = 640, 1200, 14 if frac else 24, 20
    # flows of a node: its tiles' months (half of `steps` on average, tiles sorted by term)
    assert nodes * (n // 64) * 64 * (steps // 2 - 8) * 8 * (2 if frac else 1) > 64 << 20
    b = Book(rr, ctx, kinds(65, n, steps, scen, nodes, frac=frac, node_step=5,
                            products=tuple(range(7)) if frac else (0, 1, 2, 4, 5)))
    for which in (dict(totals=False), dict(stats=True), dict(totals=False, stats=True)):
        _say(f"reserves {n} x {nodes} x {scen}, frac={frac}, {which}")
        assert torch.equal(b.run(True, **which)["r0"], b.run(False, **which)["r0"])
    b.run(True, node0=1, scen0=2, totals=False)


@pytest.mark.parametrize("frac", [False, True])
def test_reserves_with_flows_a_batch_of_tiles_at_a_time(rr, ctx, frac):
    """One node's flows do not fit the allocation-free call's 64 MiB."""
    n, steps, scen = 25_000, 700, 45
    assert (n // 64) * 64 * (steps // 2 - 8) * 8 > 64 << 20
    b = Book(rr, ctx, kinds(66, n, steps, scen, 1, frac=frac, products=tuple(range(7)) if frac else (0, 1, 2, 4, 5)),
             sample=900)
    a = b.run(stats=True)
    for which in (dict(totals=False), dict(stats=True)):
        _say(f"reserves {n} x {scen}, frac={frac}, {which}")
        assert torch.equal(b.run(True, **which)["r0"], a["r0"])


def test_reserves_with_more_flows_than_are_kept(rr, ctx):
    """Past 256 MiB of flows the ordinary call takes a batch of tiles at a time too,
    launched directly and from a graph with a second branch."""
    n, steps, scen = 40_000, 1000, 70
    w = kinds(67, n, steps, scen, 1, frac=False, products=(0,))
    w.portfolio.term_m[:] = np.maximum(w.portfolio.term_m, 900)
    assert (n // 64) * 64 * 900 * 8 > 256 << 20 and (n // 64) * scen > 40_000
    b = Book(rr, ctx, w, sample=300)
    a = b.run(stats=True)
    first = {k: x.clone() for k, x in a.items()}
    for call in ("captured", "replayed"):
        _say(f"reserves {n} x {scen}, {call}")
        for x in a.values():
            x.fill_(float("nan"))
        ctx.reserve_recurrence(0, 1, 0, scen, w.node_step_m, a)
        torch.cuda.synchronize()
        assert all(torch.equal(a[k], first[k]) for k in a)


@pytest.mark.parametrize("n,scen,flows", [(4096, 2, True), (4160, 4, False), (4160, 5, True), (64, 1, False)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_which_kernel_a_reserve_run_takes(rr, ctx, n, scen, flows, noalloc):
    """Up to 64 tiles, past them sixteen level tiles a scenario: cash flows from
    two scenarios on."""
    _say(f"reserves {n} x {scen}")
    Book(rr, ctx, kinds(68 + n + scen, n, 20, scen, 1, frac=False, products=(0,))).run(noalloc, flows=flows, stats=True)


@pytest.mark.parametrize("n,nodes,scen,flows", [(512 * 64, 1, 1, True), (512 * 64 + 1, 1, 1, False), (256 * 64, 2, 1, True),
                                                (256 * 64 + 1, 2, 1, False), (512 * 64 + 1, 1, 2, True)])
def test_which_kernel_a_totals_run_takes(rr, ctx, n, nodes, scen, flows):
    """One scenario of more than 512 tiles keeps the policies' own chains."""
    _say(f"totals {n} x {nodes} x {scen}")
    Book(rr, ctx, kinds(69 + n + nodes + scen, n, 20, scen, nodes, frac=False, products=(0,))).run(flows=flows, r0=False,
                                                                                                 stats=True)


def test_pinned_options_ask_for_the_recurrence_kernel(rr, ctx):
    """The launch options are the recurrence kernel's; its results with them and
    the cash flows' without agree within the bar."""
    b = Book(rr, ctx, kinds(70, 900, 150, 40, 2))
    a = b.run(stats=True)
    for opt, value, back in ((rr.OPT_BLOCK_K, 8, 0), (rr.OPT_BLOCK_J, 1, 0), (rr.OPT_WG_PER_CU, 2, 0), (rr.OPT_XCD_QUEUES, 0, 1)):
        ctx.set_option(opt, value)
        _say(f"option {opt} = {value}")
        b.run(flows=False, stats=True)
        ctx.set_option(opt, back)
    again = b.run(stats=True)
    assert all(torch.equal(a[k], again[k]) for k in a)


@pytest.mark.parametrize("frac", [False, True])
def test_reserve_product_shapes_give_the_same_bits(rr, ctx, frac):
    """The four shapes of a workgroup's part, chosen by their number: every one
    against the oracle, and the scenarios they share bit for bit."""
    n, scen = 30_080, 345    # 470 tiles and more
    b = Book(rr, ctx, kinds(71, n, 24, scen, 1, frac=frac, products=tuple(range(7)) if frac else (0,)), sample=700)
    _say(f"reserves {n} x {scen}, frac={frac}")
    a = b.run(stats=True)["r0"]                     # 64 policies x 128 scenarios
    for scen0, nscen in ((0, 31), (7, 33), (9, 64), (3, 65), (281, 64), (0, 344)):
        _say(f"scenarios {scen0} .. {scen0 + nscen - 1}")
        part = b.run(scen0=scen0, nscen=nscen, totals=False)["r0"]
        assert torch.equal(part, a[:, :, scen0:scen0 + nscen])
    small = kinds(72, 200, 100, scen, 2, frac=frac)   # 64 x 16
    b = Book(rr, ctx, small)
    a = b.run(totals=False)["r0"]
    for scen0, nscen in ((0, 2), (5, 15), (1, 16), (328, 17)):
        part = b.run(scen0=scen0, nscen=nscen, totals=False)["r0"]
        assert torch.equal(part, a[:, :, scen0:scen0 + nscen])
