"""GPU parity of the calls that go by summed expected cash flows (a policy's
flows are formed once, forward in time, and meet the scenarios as one
multiply-add per month) against the CPU oracle's backward recurrence.

Bar: totals within 1e-10 of the summed gross PV, reserves within 1e-10 of
max(|r|, gross PV).  Sizes sit at the edges of the kernels' tiles: 64 policies
per tile, 8 steps per block, 64 scenarios per workgroup, more rows than one
workgroup adds up, several tiles per wavefront."""
import sys

import numpy as np
import pytest

import oracle
import synth
from tests._helpers import RTOL, assert_reserves_close, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EVERY_LIFE_PRODUCT = tuple(range(7)) + (synth.JL_ENDOW, synth.JL_ASSUR1, synth.JL_ASSUR2,
                                        synth.JL3_ANN, synth.LS3_ANN)


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def rr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1401_1757_amd as rr
    return rr


@pytest.fixture()
def ctx(rr):
    c = rr.Context(0)
    yield c
    c.close()


def random_markov(rng, n_models, n_ages, m):
    w = rng.dirichlet(np.full(m, 0.4), size=(n_models, n_ages, m))
    return w, rng.uniform(-0.1, 0.3, (n_models, m))


def every_kind(seed, n, n_steps, n_scen, n_nodes, n_tables=2, states=3, node_step=7, frac=0.3,
               products=EVERY_LIFE_PRODUCT, special=True, shock=True):
    """Every kind of policy the library has (level products only without
    `special`), on random tables and curves."""
    rng = np.random.default_rng(seed)
    w = synth.random_small(rng, n=n, n_steps=n_steps, n_scen=n_scen, n_nodes=n_nodes, shock=shock,
                           products=products, n_tables=n_tables)
    pf = w.portfolio
    if special:
        pf = synth.with_cash_flow_tables(rng, pf, frac=0.1, n_rows=4)
        pf = synth.with_payment_patterns(rng, pf, 0.4, 0.3)
        n_ages = w.basis.q.shape[1]
        models = synth.phi_models(n_ages) if states == 3 else random_markov(rng, 2, n_ages, states)
        pf = synth.with_markov_policies(rng, pf, models, frac=0.1)
        level = np.isin(pf.product, (synth.SL_ANN, synth.JL_ANN)) & (pf.escalation == 0) & (pf.annual == 0)
        pick = level & (rng.uniform(size=n) < 0.5)
        pf.timing = np.where(pick, synth.FRACTIONAL, pf.timing).astype(np.int32)
        w.basis.frac = frac
    return synth.Workload("every kind", w.basis, pf, node_step_m=node_step)


def upload(ctx, w):
    b, pf = w.basis, w.portfolio
    ctx.basis_upload(b.q, b.v, b.shock, frac=b.frac)
    if pf.markov is not None:
        ctx.markov_upload(*pf.markov)
    ctx.portfolio_upload(pf)


def check_totals(ctx, w, node0=0, nnode=None, scen0=0, nscen=None, noalloc=False):
    b = w.basis
    nnode = b.n_nodes - node0 if nnode is None else nnode
    nscen = b.n_scen - scen0 if nscen is None else nscen
    out = ctx.alloc_outputs(nnode, nscen, r0=False, stats=True)
    for x in out.values():
        x.fill_(float("nan"))
    call = ctx.reserve_recurrence_noalloc if noalloc else ctx.reserve_recurrence
    call(node0, nnode, scen0, nscen, w.node_step_m, out)
    torch.cuda.synchronize()
    ref = oracle.reserves(b, w.portfolio, node0, nnode, scen0, nscen, w.node_step_m)
    tot = to_np(out["totals"])
    err = np.abs(tot - ref["totals"])
    assert np.all(err <= RTOL * np.maximum(ref["gross_totals"], 1e-300)), err.max()
    mean, q = oracle.node_stats(tot)
    st = to_np(out["stats"])
    assert np.all(np.abs(st[:, 0] - mean) <= 1e-12 * np.abs(tot).max(axis=1))
    assert np.array_equal(st[:, 1], q)
    return out


@pytest.mark.parametrize("n,steps,scen,nodes", [(1, 1, 1, 1), (63, 7, 64, 1), (64, 8, 1, 2), (65, 9, 65, 3),
                                                (700, 16, 130, 2), (450, 90, 37, 3), (900, 260, 5, 2)])
@pytest.mark.parametrize("special", [False, True])
def test_totals_every_kind(ctx, n, steps, scen, nodes, special):
    w = every_kind(n + steps + scen, n, steps, scen, nodes, special=special)
    upload(ctx, w)
    _say(f"totals {n} policies x {nodes} x {scen}, {steps} steps, special={special}")
    check_totals(ctx, w)
    if nodes > 1:
        check_totals(ctx, w, node0=1, scen0=scen // 2)


@pytest.mark.parametrize("products", [(0,), (1, 8, 9), (2,), (3, 10), (12,), (13,)])
def test_totals_of_one_model(ctx, products):
    """Each state model alone: the kernel instances without the others."""
    w = every_kind(50 + products[0], 200, 100, 20, 2, products=products, special=False)
    upload(ctx, w)
    _say(f"totals, products {products}")
    check_totals(ctx, w)


def test_totals_large_markov_and_device_tables(ctx):
    """Nine-state models, tables too large for LDS."""
    w = every_kind(77, 600, 80, 70, 2, n_tables=12, states=9)
    assert w.basis.q.size > 8192
    upload(ctx, w)
    _say("totals, nine-state models, tables in device memory")
    check_totals(ctx, w)
    check_totals(ctx, w, noalloc=True)


def test_totals_many_tiles_per_row(ctx):
    """More tiles than rows (several tiles per wavefront, rows added in
    chunks), terms that differ between the tiles of a row, at a node where
    part of the book has expired; the allocation-free call gives the same
    bits."""
    w = every_kind(5, 300_000, 40, 3, 2, special=False, products=(0, 1, 2, 4, 5), node_step=19)
    upload(ctx, w)
    _say("totals, 300,000 policies")
    a = check_totals(ctx, w)
    b = check_totals(ctx, w, noalloc=True)
    assert torch.equal(a["totals"], b["totals"]) and torch.equal(a["stats"], b["stats"])


def test_totals_replayed_after_other_work(ctx):
    """Graph replays with fresh outputs and other calls between them."""
    w = every_kind(9, 500, 60, 90, 2)
    upload(ctx, w)
    first = check_totals(ctx, w)
    for rep in range(3):
        _say(f"replay {rep}")
        ctx.reserve_recurrence(0, 2, 0, 7, w.node_step_m)
        again = ctx.alloc_outputs(2, 90, r0=False, stats=True)
        ctx.reserve_recurrence(0, 2, 0, 90, w.node_step_m, again)
        torch.cuda.synchronize()
        assert torch.equal(again["totals"], first["totals"])
        assert torch.equal(again["stats"], first["stats"])


@pytest.mark.parametrize("big", [1.0e4, 1.0e-4])
def test_totals_on_curves_whose_products_leave_the_range(ctx, big):
    """Alternating factors big and 1/big, then ones of one size: products of a
    hundred factors overflow or vanish, the reserves of short policies do not."""
    w = every_kind(31, 300, 160, 66, 1, special=False, shock=False)
    v = w.basis.v
    v[:, :, :60] = np.where(np.arange(60) % 2 == 0, big, 1.0 / big)
    v[:, :, 60:] = 1.0 / big if big > 1 else big
    upload(ctx, w)
    _say(f"totals, factors {big}")
    check_totals(ctx, w)


def check_reserves(ctx, w, node0=0, nnode=None, scen0=0, nscen=None, noalloc=False, totals=True):
    b = w.basis
    nnode = b.n_nodes - node0 if nnode is None else nnode
    nscen = b.n_scen - scen0 if nscen is None else nscen
    out = ctx.alloc_outputs(nnode, nscen, totals=totals, stats=True)
    for x in out.values():
        x.fill_(float("nan"))
    call = ctx.reserve_recurrence_noalloc if noalloc else ctx.reserve_recurrence
    call(node0, nnode, scen0, nscen, w.node_step_m, out)
    torch.cuda.synchronize()
    ref = oracle.reserves(b, w.portfolio, node0, nnode, scen0, nscen, w.node_step_m)
    assert_reserves_close(to_np(out["r0"]), ref["r_all"][..., 0], ref["gross"])
    if totals:
        err = np.abs(to_np(out["totals"]) - ref["totals"])
        assert np.all(err <= RTOL * np.maximum(ref["gross_totals"], 1e-300)), err.max()
    return out


@pytest.mark.parametrize("n,steps,scen,nodes", [(1, 1, 2, 1), (63, 31, 16, 1), (64, 32, 17, 2), (65, 33, 32, 3),
                                                (200, 64, 33, 1), (700, 16, 130, 2), (450, 90, 64, 3),
                                                (300, 140, 65, 2), (900, 260, 5, 2), (130, 100, 129, 1)])
@pytest.mark.parametrize("special", [False, True])
def test_reserves_every_kind(ctx, n, steps, scen, nodes, special):
    w = every_kind(3 * n + steps + scen, n, steps, scen, nodes, special=special)
    upload(ctx, w)
    _say(f"reserves {n} policies x {nodes} x {scen}, {steps} steps, special={special}")
    a = check_reserves(ctx, w)
    b = check_reserves(ctx, w, noalloc=True)
    assert all(torch.equal(a[k], b[k]) for k in a)
    if nodes > 1:
        check_reserves(ctx, w, node0=1, scen0=scen // 2, totals=False)


@pytest.mark.parametrize("products", [(0,), (1, 8, 9), (2,), (3, 10), (12,), (13,)])
def test_reserves_of_one_model(ctx, products):
    w = every_kind(70 + products[0], 200, 100, 70, 2, products=products, special=False)
    upload(ctx, w)
    _say(f"reserves, products {products}")
    check_reserves(ctx, w)


def test_reserves_large_markov_and_device_tables(ctx):
    w = every_kind(78, 600, 80, 70, 2, n_tables=12, states=9)
    upload(ctx, w)
    _say("reserves, nine-state models, tables in device memory")
    check_reserves(ctx, w)


def test_reserves_follow_regenerated_curves(ctx):
    """The discount products kept beside the curves are those of the last
    generation, through graph replays and a change of the start rates."""
    rng = np.random.default_rng(12)
    w = synth.random_small(rng, n=300, n_steps=120, n_scen=1, n_nodes=1)
    vas = dict(a=synth.VAS_A, b=synth.VAS_B, sigma=synth.VAS_SIGMA, dt=1.0 / 12.0)
    ctx.basis_generate_vasicek(w.basis.q, 70, 120, [0.03], key=(5, 6), **vas)
    ctx.portfolio_upload(w.portfolio)
    out = ctx.alloc_outputs(1, 70)
    for r0, key in ((0.03, (5, 6)), (0.03, (5, 7)), (0.01, (9, 7)), (0.03, (5, 6))):
        _say(f"generation {r0} {key}")
        ctx.curves_generate_vasicek([r0], key=key, **vas)
        ctx.reserve_recurrence(0, 1, 0, 70, 12, out)
        torch.cuda.synchronize()
        v, _ = oracle.vasicek_curves(r0=[r0], n_scen=70, n_steps=120, key=key, **vas)
        ref = oracle.reserves(synth.Basis(q=w.basis.q, v=np.asarray(v).reshape(1, 70, 120)), w.portfolio, 0, 1, 0, 70)
        assert_reserves_close(to_np(out["r0"]), ref["r_all"][..., 0], ref["gross"])


@pytest.mark.parametrize("big", [1.0e4, 1.0e-4])
def test_reserves_on_curves_whose_products_leave_the_range(ctx, big):
    w = every_kind(32, 300, 160, 66, 1, special=False, shock=False)
    v = w.basis.v
    v[:, :, :60] = np.where(np.arange(60) % 2 == 0, big, 1.0 / big)
    v[:, :, 60:] = 1.0 / big if big > 1 else big
    upload(ctx, w)
    _say(f"reserves, factors {big}")
    check_reserves(ctx, w)


@pytest.mark.parametrize("steps,scen,big", [(1, 1, 0.0), (15, 63, 0.0), (16, 64, 0.0), (17, 65, 0.0), (33, 257, 0.0),
                                            (160, 70, 1.0e4)])
def test_node_means_from_the_discount_products(ctx, steps, scen, big):
    """Sixteen months a workgroup, 256 scenarios a round; a part of the
    scenarios; curves without kept products (`big`)."""
    w = every_kind(steps + scen, 150, steps, scen, 2, special=False, shock=big == 0.0)
    if big:
        w.basis.v[:, :, :60] = np.where(np.arange(60) % 2 == 0, big, 1.0 / big)
        w.basis.v[:, :, 60:] = 1.0 / big
    upload(ctx, w)
    for s0, ns in ((0, scen), (scen // 3, scen - scen // 3)):
        _say(f"node means {steps} steps, scenarios {s0}..{s0 + ns - 1}")
        out = ctx.node_expected_reserves(0, 2, s0, ns, w.node_step_m)
        torch.cuda.synchronize()
        ref = oracle.reserves(w.basis, w.portfolio, 0, 2, s0, ns, w.node_step_m)
        mean = ref["r_all"][..., 0].mean(axis=2)
        assert np.all(np.abs(to_np(out["r0"]) - mean) <= RTOL * np.maximum(np.abs(mean), ref["gross"].mean(axis=2)))
        total = ref["totals"].mean(axis=1)
        assert np.all(np.abs(to_np(out["totals"]) - total) <= RTOL * np.maximum(ref["gross_totals"].mean(axis=1), 1e-300))


@pytest.mark.parametrize("n,scen", [(4096, 2), (4160, 4), (4160, 5)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_reserves_both_sides_of_the_tile_rule(ctx, n, scen, noalloc):
    """64 tiles, and 65 at more and fewer than sixteen a scenario."""
    w = every_kind(n + scen, n, 20, scen, 1, special=False, products=(0,))
    upload(ctx, w)
    _say(f"reserves {n} policies x {scen}")
    check_reserves(ctx, w, noalloc=noalloc)
