"""Runs by cash flows (test_gpu_flows.py) in the situations that need a size, a
graph or a change of curves of their own: graphs that the caller captured,
the library's own graphs with a second branch, curves whose products leave the
FP64 range."""
import sys

import numpy as np
import pytest

import oracle
import synth
from tests._helpers import RTOL, assert_reserves_close, to_np

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
