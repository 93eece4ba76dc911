"""The calls whose speed this library is measured by: inputs, one pass through
the public binding, the work it cannot do without, and its results in plain
64-bit torch.

Every case values a synthetic book of life policies (Gompertz-Makeham
mortality) on synthetic interest scenarios (flat or Vasicek), at sizes taken
from this repository's own workloads (1,000 annuities on one curve; 100,000
mixed policies on one curve and with whole reserve paths; 10,000 policies on
1,000 scenarios, once and at 60 outer nodes; the representative annuity
portfolio) and at odd sizes between them.  `kind` says which call a pass makes:

  reserves    reserve_recurrence: per-policy reserves, portfolio totals and,
              with more than one scenario, the 1-in-200 statistic
  totals      reserve_recurrence asked for totals and statistics only
  path        reserve_recurrence in path mode (every step of every policy)
  noalloc     reserve_recurrence_noalloc (serving code that may not allocate)
  generated   curves_generate_vasicek, then reserve_recurrence on them
  node_means  node_expected_reserves (scenario average per policy and node)
  surrogate   surrogate_infer (bfloat16 network, exact rows outside its box)
  train_step  surrogate_gradients, then surrogate_adam_step
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1401_1757_amd as rr

LIMIT_AGE = 1440                                   # months; q = 1 from here on
VAS_A, VAS_B, VAS_SIGMA, VAS_R0, DT = 0.1, 0.03, 0.01, 0.03, 1.0 / 12.0
NODE_STEP = 12
TAIL = 0.005
TWO_LIFE = (rr.JL_ANN, rr.REV_ANN, rr.LS_ANN, rr.JL_ENDOW, rr.JL_ASSUR1, rr.JL_ASSUR2)
THREE_LIFE = (rr.JL3_ANN, rr.LS3_ANN)
F64 = torch.float64


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # A quotation or a small scheme valued on one flat curve: latency.
        dict(name="scheme_one_curve", kind="reserves", book="annuities", policies=1000, nodes=1,
             scenarios=1, steps=300, all_states=False),
        # A serving process that revalues a block on a few stressed curves, without allocating.
        dict(name="stress_curves_noalloc", kind="noalloc", book="mixed", policies=5003, nodes=1,
             scenarios=13, steps=600, all_states=False),
        # A whole mixed book on the best-estimate curve.
        dict(name="book_one_curve", kind="reserves", book="mixed", policies=100_000, nodes=1,
             scenarios=1, steps=600, all_states=False),
        # The same book's reserve at every future month (projections, profit testing).
        dict(name="book_paths", kind="path", book="mixed", policies=100_000, nodes=1, scenarios=1,
             steps=600, all_states=False),
        # The headline workload: every policy on every inner scenario.
        dict(name="inner_scenarios", kind="reserves", book="mixed", policies=10_000, nodes=1,
             scenarios=1000, steps=600, all_states=False),
        # Monte Carlo with fresh scenarios drawn on the device for each valuation.
        dict(name="fresh_scenarios", kind="generated", book="mixed", policies=10_000, nodes=1,
             scenarios=1000, steps=600, all_states=False),
        # Nested valuation: the capital figure of every outer node.
        dict(name="outer_nodes_totals", kind="totals", book="mixed", policies=10_000, nodes=60,
             scenarios=500, steps=600, all_states=False),
        # The representative annuity portfolio (escalating and annual payments, reversions).
        dict(name="annuity_portfolio_totals", kind="totals", book="representative",
             policies=200_000, nodes=1, scenarios=1000, steps=756, all_states=False),
        # Expected reserve of every policy at every outer node.
        dict(name="node_means", kind="node_means", book="mixed", policies=10_000, nodes=60,
             scenarios=500, steps=600, all_states=False),
        # Every product the library has, odd sizes, shocked nodes.
        dict(name="every_product", kind="reserves", book="products", policies=4001, nodes=2,
             scenarios=333, steps=420, all_states=False),
        # The learned surrogate over the headline workload.
        dict(name="surrogate_inner_scenarios", kind="surrogate", book="mixed", policies=10_000,
             nodes=1, scenarios=1000, steps=600, all_states=False),
        # One Adam step of the surrogate's training loop.
        dict(name="surrogate_train_step", kind="train_step", book="none", policies=8192, nodes=1,
             scenarios=1, steps=600, all_states=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["reserves", "reserves", "reserves", "totals", "totals", "path", "noalloc",
                       "generated", "node_means", "surrogate", "train_step"])
    if kind == "train_step":
        return dict(kind=kind, book="none", policies=64 * rng.randint(4, 128), nodes=1, scenarios=1,
                    steps=600, all_states=False)
    book = "mixed"
    if kind == "path":
        book = rng.choice(["mixed", "annuities"])
    elif kind in ("reserves", "totals", "noalloc"):
        book = rng.choice(["mixed", "mixed", "annuities", "representative", "products"])
    steps = {"annuities": rng.randint(60, 480), "representative": 756,
             "products": rng.randint(120, 480)}.get(book, rng.randint(300, 600))
    nodes = 1 if kind in ("path", "generated") or book in ("annuities", "representative") \
        else rng.choice([1, 1, _log_int(rng, 2, 60)])
    policies = _log_int(rng, 300, 100_000 if book != "products" else 8000)
    scenarios = 1 if kind == "path" else _log_int(rng, 1, 1000)
    if kind == "surrogate":
        policies, nodes = _log_int(rng, 300, 10_000), 1
    if kind == "path":
        policies = min(policies, 60_000)
    if kind != "totals":           # per-policy reserves: at most ten million a pass
        while policies * nodes * scenarios > 10_000_000:
            if nodes > 4:
                nodes //= 2
            elif scenarios > 40:
                scenarios = scenarios * 2 // 3
            else:
                policies = policies * 2 // 3
    while nodes * scenarios > 30_000 or (kind == "totals" and policies * nodes * scenarios > 150_000_000):
        scenarios = max(1, scenarios * 2 // 3)
        policies = max(300, policies * 2 // 3)
    if kind == "noalloc":          # the static scratch takes up to 64 MiB of per-tile totals
        while (policies // 64 + 8) * nodes * scenarios > 7_000_000:
            scenarios = scenarios * 2 // 3
    states = kind in ("reserves", "noalloc") and policies * nodes * scenarios <= 2_000_000 and rng.random() < 0.25
    return dict(kind=kind, book=book, policies=policies, nodes=nodes, scenarios=scenarios,
                steps=steps, all_states=states)


# ---------------------------------------------------------------------------
# Inputs (host arrays, from the seed alone)
# ---------------------------------------------------------------------------
def _gm_q(n_ages, loading):
    x = np.arange(n_ages) / 12.0
    h = 5e-4 / 12.0 + (7.5e-5 / math.log(1.1)) * 1.1 ** x * (1.1 ** DT - 1.0)
    q = np.minimum(1.0, -np.expm1(-h) * loading)
    q[LIMIT_AGE:] = 1.0
    return q


def _vas_consts():
    a, s, e = VAS_A, VAS_SIGMA, math.exp(-VAS_A * DT)
    var_r = s * s * (1.0 - e * e) / (2.0 * a)
    var_y = s * s / (a * a) * (DT - 2.0 * (1.0 - e) / a + (1.0 - e * e) / (2.0 * a))
    cov = s * s / (2.0 * a * a) * (1.0 - e) ** 2
    rho = cov / math.sqrt(var_r * var_y)
    return e, (1.0 - e) / a, math.sqrt(var_r), rho * math.sqrt(var_y), math.sqrt(var_y * (1.0 - rho * rho))


def _vas_curves(z0, z1, r0):
    """One-step discount factors [scenario][step] from two normals per step."""
    e, om, sd_r, ry, py = _vas_consts()
    v = np.empty(z0.shape)
    r = np.full(z0.shape[0], float(r0))
    for t in range(z0.shape[1]):
        v[:, t] = np.exp(-(VAS_B * DT + (r - VAS_B) * om + ry * z0[:, t] + py * z1[:, t]))
        r = VAS_B + (r - VAS_B) * e + sd_r * z0[:, t]
    return v


def _lognormal(rng, mean, sd_log, n):
    return rng.lognormal(math.log(mean) - 0.5 * sd_log * sd_log, sd_log, n)


def _book(case, rng):
    """Policies as host arrays; q tables; Markov models or None."""
    n, steps, book = case["policies"], case["steps"], case["book"]
    i32 = lambda x: np.asarray(x).astype(np.int32)
    pf = SimpleNamespace(escalation=None, anniv_m=None, annual=None, cf_row=None, cf=None,
                         age3_m=None, table3=None)
    markov, frac = None, 0.0
    pf.timing = np.full(n, rr.ARREARS, np.int32)
    pf.premium = np.zeros(n)
    if book == "annuities":
        pf.product = np.full(n, rr.SL_ANN, np.int32)
        pf.age1_m = i32(rng.integers(720, 961, n))
        pf.age2_m = np.zeros(n, np.int32)
        pf.term_m = np.full(n, steps, np.int32)
        pf.table1 = pf.table2 = np.zeros(n, np.int32)
        pf.amount = _lognormal(rng, 1e4, 0.5, n)
        loadings = (1.0,)
    elif book == "representative":
        pf.product = i32(rng.choice([rr.SL_ANN, rr.JL_ANN, rr.REV_ANN, rr.LS_ANN], n, p=[0.6, 0.1, 0.2, 0.1]))
        two = np.isin(pf.product, TWO_LIFE)
        pf.age1_m = i32(rng.integers(684, 805, n))
        pf.age2_m = i32(np.where(two, rng.integers(684, 805, n), 0))
        male = rng.uniform(size=n) < 0.75
        pf.table1 = i32(~male)
        pf.table2 = i32(np.where(two, male, ~male))
        pf.term_m = i32(LIMIT_AGE - np.where(two, np.minimum(pf.age1_m, pf.age2_m), pf.age1_m))
        pf.annual = i32(rng.uniform(size=n) < 0.2)
        pay = _lognormal(rng, 5.0, math.sqrt(math.log1p(0.09)), n)
        pf.amount = np.where(pf.annual == 1, pay, 12.0 * pay)
        pf.escalation = np.where(rng.uniform(size=n) < 0.05, rng.choice([0.03, 0.0425, 0.05], n), 0.0)
        pf.anniv_m = i32(rng.integers(1, 13, n))
        loadings = (1.0, 0.6)
    elif book == "products":
        pf.product = i32(rng.integers(0, 14, n))
        life2, life3 = np.isin(pf.product, TWO_LIFE + THREE_LIFE), np.isin(pf.product, THREE_LIFE)
        pf.age1_m = i32(rng.integers(240, 961, n))
        pf.age2_m = i32(np.where(life2, rng.integers(240, 961, n), 0))
        pf.age3_m = i32(np.where(life3, rng.integers(240, 961, n), 0))
        pf.term_m = i32(rng.integers(1, steps + 1, n))
        pf.table1 = i32(rng.integers(0, 2, n))
        pf.table2, pf.table3 = i32(rng.integers(0, 2, n)), i32(rng.integers(0, 2, n))
        ann = np.isin(pf.product, (rr.SL_ANN, rr.JL_ANN, rr.REV_ANN, rr.LS_ANN))
        pf.amount = np.where(ann | (pf.product >= rr.MARKOV), _lognormal(rng, 1e4, 0.5, n),
                             _lognormal(rng, 1e5, 0.8, n))
        pf.timing = i32(np.where(ann | life3, rng.integers(0, 2, n), rr.ARREARS))
        pf.escalation = np.where(ann & (rng.uniform(size=n) < 0.2), 0.03, 0.0)
        pf.annual = i32(ann & (rng.uniform(size=n) < 0.2))
        pf.anniv_m = i32(rng.integers(1, 13, n))
        level = (pf.escalation == 0) & (pf.annual == 0)
        frac = 0.5
        f = np.isin(pf.product, (rr.SL_ANN, rr.JL_ANN)) & level & (rng.uniform(size=n) < 0.1)
        pf.timing[f] = rr.FRACTIONAL
        pf.premium = np.where(level & (rng.uniform(size=n) < 0.6), pf.amount * 1e-3, 0.0)
        pf.cf_row = i32(rng.integers(0, 3, n))
        pf.cf = rng.uniform(0.0, 0.2, (3, steps))
        # Permanent health insurance: healthy, sick, dead; benefit while sick.
        qh = np.stack([_gm_q(961 + steps + 1, x) for x in (1.0, 1.3)])
        inc, qs = np.minimum(0.3 * np.sqrt(qh), 0.5), np.minimum(2.0 * qh, 1.0)
        w = np.zeros(qh.shape + (3, 3))
        w[..., 0, 2], w[..., 0, 1] = qh, (1.0 - qh) * inc
        w[..., 1, 2], w[..., 1, 0] = qs, (1.0 - qs) * 0.08
        w[..., 0, 0], w[..., 1, 1] = 1.0 - w[..., 0, 1] - w[..., 0, 2], 1.0 - w[..., 1, 0] - w[..., 1, 2]
        w[..., 2, 2] = 1.0
        markov = (w, np.tile([0.0, 1.0 / 12.0, 0.0], (2, 1)))
        loadings = (0.8, 1.2)
    else:
        pf.product = i32(rng.choice([rr.SL_ANN, rr.JL_ANN, rr.TERM, rr.ENDOW], n, p=[0.4, 0.2, 0.2, 0.2]))
        pf.age1_m = i32(rng.integers(240, 1021, n))
        pf.age2_m = i32(np.where(pf.product == rr.JL_ANN, rng.integers(240, 1021, n), 0))
        lo = min(60, steps)            # every term equally often: path buffers have one length
        pf.term_m = i32(rng.permutation(lo + np.arange(n) % (steps + 1 - lo)))
        term, endow = pf.product == rr.TERM, pf.product == rr.ENDOW
        pf.table1 = i32(term + 2 * endow)
        pf.table2 = pf.table1.copy()
        pf.amount = np.where(term | endow, _lognormal(rng, 1e5, 0.8, n), _lognormal(rng, 1e4, 0.5, n))
        mid = (pf.age1_m + 0.5 * pf.term_m) / 12.0
        rate = (5e-4 + 7.5e-5 * 1.1 ** mid) * 1.2 / 12.0
        u = rng.uniform(size=n)
        pf.premium = np.where(term, pf.amount * rate * (0.9 + 0.4 * u), 0.0) + \
            np.where(endow, pf.amount / pf.term_m * (0.6 + 0.35 * u), 0.0)
        loadings = (0.8, 1.2, 1.0)
    ages = pf.age1_m if pf.age3_m is None else np.maximum(pf.age1_m, pf.age3_m)
    q = np.stack([_gm_q(int((np.maximum(ages, pf.age2_m) + pf.term_m).max()) + 1, x) for x in loadings])
    return pf, q, markov, frac


def _inputs(case, seed, curves=True):
    """Everything a case is about, as host arrays made from the seed."""
    rng = np.random.default_rng([int(seed), 1401])
    x = SimpleNamespace(case=case, key=(int(seed) % (1 << 62) + 1, 1757))
    if case["book"] == "none":
        return x
    x.pf, x.q, x.markov, x.frac = _book(case, rng)
    k, s, t = case["nodes"], case["scenarios"], case["steps"]
    x.shock = rng.normal(1.0, 0.05, k) if k > 1 else None
    x.r0 = VAS_R0 + 0.01 * rng.standard_normal(k) if k > 1 else np.array([VAS_R0])
    x.v = None
    if case["kind"] == "generated":
        if curves:
            x.v = np.stack([_vas_curves(*_philox_normals(x.key, j, s, t), x.r0[j]) for j in range(k)])
    elif s == 1 and k == 1:
        x.v = np.full((1, 1, t), (1.0 + rng.uniform(0.02, 0.04)) ** -DT)
    else:
        x.v = np.stack([_vas_curves(*rng.standard_normal((2, s, t)), x.r0[j]) for j in range(k)])
    return x


def _philox_normals(key, node, n_scen, n_steps):
    """The two normals of every (scenario, step) of a node: Box-Muller on the
    Philox4x64-10 block of counter (step, scenario, node, 0)."""
    u64 = lambda v: np.uint64(v & ((1 << 64) - 1))

    def mul(m, x):      # high and low words of a 64 x 64 bit product
        lo32, s32 = u64(0xFFFFFFFF), u64(32)
        mh, ml, xh, xl = u64(m >> 32), u64(m & 0xFFFFFFFF), x >> s32, x & lo32
        mid = ml * xh + ((ml * xl) >> s32)
        mid2 = mh * xl + (mid & lo32)
        return mh * xh + (mid >> s32) + (mid2 >> s32), u64(m) * x

    with np.errstate(over="ignore"):
        t, s = np.meshgrid(np.arange(n_steps, dtype=np.uint64), np.arange(n_scen, dtype=np.uint64))
        c = [t, s, np.full(t.shape, node, np.uint64), np.zeros(t.shape, np.uint64)]
        k0, k1 = key
        for _ in range(10):
            h0, l0 = mul(0xD2E7470EE14C6C93, c[0])
            h1, l1 = mul(0xCA5A826395121157, c[2])
            c = [h1 ^ c[1] ^ u64(k0), l1, h0 ^ c[3] ^ u64(k1), l0]
            k0, k1 = k0 + 0x9E3779B97F4A7C15, k1 + 0xBB67AE8584CAA73B
    u = [((w >> np.uint64(11)).astype(np.float64) + 0.5) * 2.0 ** -53 for w in c[:2]]
    rad = np.sqrt(-2.0 * np.log(u[0]))
    return rad * np.cos(2.0 * math.pi * u[1]), rad * np.sin(2.0 * math.pi * u[1])


# -- surrogate model ---------------------------------------------------------
def _zero_rates(v):
    """Zero rates at tenors 1..50 years of curves [..., step]."""
    lv = np.cumsum(np.log(v), axis=-1)
    m = np.minimum(12 * np.arange(1, rr.SG_TENORS + 1), v.shape[-1])
    return -12.0 * lv[..., m - 1] / m


def _mlp_params(seed):
    """Weights of the size a fitted network has (FP32 vector of the blob)."""
    rng = np.random.default_rng([int(seed), 256])
    h, f = rr.SG_HIDDEN, rr.SG_FEATURES
    w1 = np.zeros((rr.SG_INPUTS, h))
    w1[:f] = rng.normal(0.0, 1.0 / math.sqrt(f), (f, h))
    parts = [w1, rng.normal(0.0, 0.1, h), rng.normal(0.0, 1.0 / 16.0, (h, h)), rng.normal(0.0, 0.1, h),
             rng.normal(0.0, 1.0 / 16.0, h), rng.normal(0.0, 0.1, 1)]
    return np.concatenate([p.reshape(-1) for p in parts]).astype(np.float32)


def _model(x, seed):
    """A model whose training box holds all but about one policy in 500 and
    one scenario in 500, as a network fitted to such a book has it."""
    raw_p, raw_s, zbar, evec = _features(x)
    s = raw_s.shape[0]
    mu, sd, lo, hi = np.zeros(17), np.ones(17), np.zeros(17), np.ones(17)
    for cols, data in ((list(range(8)) + [16], raw_p), (range(8, 13), raw_s)):
        for j, c in enumerate(cols):
            mu[c], sd[c] = data[:, j].mean(), max(data[:, j].std(), 1e-3)
            lo[c], hi[c] = data[:, j].min(), data[:, j].max()
    lo[13:16], hi[13:16], mu[13], sd[13:16] = 0.0, 1.0, 0.8, 0.4
    edge = 1e-7 * (1.0 + np.abs(lo) + np.abs(hi))     # no row lies on the box's faces
    lo, hi = lo - edge, hi + edge
    hi[6] = np.quantile(raw_p[:, 6], 1.0 - 1.0 / 500.0)
    if s > 10:
        hi[9] = np.quantile(raw_s[:, 1], 1.0 - 1.0 / 500.0)
    return dict(params=_mlp_params(seed), mu=mu, sd=sd, lo=lo, hi=hi,
                tmu=np.array([9.0, 7.0, 0.02, 0.3]), tsd=np.array([4.0, 4.0, 0.05, 0.25]),
                zbar=zbar, evec=evec,
                signature=np.array([[0, -1, 1], [0, 0, 1], [1, -1, -1], [2, -1, -1]], np.int32))


def _features(x):
    """Raw policy features [n][9] (0-7 and 16) and scenario features [s][5]."""
    pf = x.pf
    slot = np.stack([pf.product == p for p in (rr.SL_ANN, rr.JL_ANN, rr.TERM, rr.ENDOW)], 1)
    raw_p = np.concatenate([np.stack([pf.age1_m / 12.0, pf.term_m / 12.0], 1), slot,
                            np.stack([np.log(pf.amount), 12.0 * pf.premium / pf.amount,
                                      np.where(slot[:, 1], pf.age2_m / 12.0, 0.0)], 1)], 1)
    z = _zero_rates(x.v[0])
    zbar = z.mean(0)
    val, vec = np.linalg.eigh(np.cov(z, rowvar=False, bias=True) if z.shape[0] > 1 else np.eye(50))
    evec = vec[:, ::-1][:, :3].T
    evec = evec * np.sign(evec[np.arange(3), np.abs(evec).argmax(1)])[:, None]
    raw_s = np.concatenate([-12.0 * np.log(x.v[0][:, :1]), (z - zbar) @ evec.T, np.ones((z.shape[0], 1))], 1)
    return raw_p, raw_s, zbar, evec


# ---------------------------------------------------------------------------
# State and pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    x = _inputs(case, seed, curves=False)
    ctx = rr.Context(0)
    st = SimpleNamespace(case=case, ctx=ctx)
    if case["kind"] == "train_step":
        g = torch.Generator().manual_seed(int(seed) % (1 << 60))
        z = torch.zeros(case["policies"], rr.SG_INPUTS)
        z[:, :rr.SG_FEATURES] = torch.randn(case["policies"], rr.SG_FEATURES, generator=g)
        st.z, st.t = z.cuda(), torch.randn(case["policies"], generator=g).cuda()
        ones = np.ones(17)
        ctx.surrogate_set_weights(rr.pack_surrogate_blob(
            _mlp_params(seed), 0 * ones, ones, -9 * ones, 9 * ones, np.zeros(4), np.ones(4),
            np.zeros(50), np.zeros((3, 50)), np.zeros((4, 3))))
        return st
    if x.markov is not None:
        ctx.markov_upload(*x.markov)
    if case["kind"] == "generated":
        st.vas = dict(r0=x.r0, a=VAS_A, b=VAS_B, sigma=VAS_SIGMA, dt=DT, key=x.key)
        ctx.basis_generate_vasicek(x.q, case["scenarios"], case["steps"], shock=x.shock, frac=x.frac, **st.vas)
    else:
        ctx.basis_upload(x.q, x.v, x.shock, frac=x.frac)
    ctx.portfolio_upload(x.pf)
    k, s = case["nodes"], case["scenarios"]
    if case["kind"] == "path":
        st.out = ctx.alloc_outputs(1, 1, r0=False, totals=False, path_node=0)
    elif case["kind"] != "node_means":
        st.out = ctx.alloc_outputs(k, s, r0=case["kind"] != "totals", all_states=case["all_states"],
                                   stats=s > 1)
    if case["kind"] == "surrogate":
        ctx.surrogate_set_weights(rr.pack_surrogate_blob(**_model(x, seed)))
    return st


def run(st):
    c, ctx = st.case, st.ctx
    k, s = c["nodes"], c["scenarios"]
    if c["kind"] == "train_step":
        grad, loss = ctx.surrogate_gradients(st.z, st.t)
        ctx.surrogate_adam_step(grad, 1e-3)
        return {"grad": grad, "loss": loss}
    if c["kind"] == "node_means":
        return ctx.node_expected_reserves(0, k, 0, s, NODE_STEP)
    if c["kind"] == "surrogate":
        return ctx.surrogate_infer(0, k, 0, s, NODE_STEP, st.out, tail=TAIL, report=False)
    if c["kind"] == "noalloc":
        return ctx.reserve_recurrence_noalloc(0, k, 0, s, NODE_STEP, st.out, tail=TAIL)
    if c["kind"] == "generated":
        ctx.curves_generate_vasicek(**st.vas)
    return ctx.reserve_recurrence(0, k, 0, s, NODE_STEP, st.out, tail=TAIL)


# ---------------------------------------------------------------------------
# Work
# ---------------------------------------------------------------------------
def _live_steps(case):
    """Expected policy-months summed over the nodes."""
    lo, hi = {"annuities": (case["steps"], case["steps"]), "representative": (640, 756),
              "products": (1, case["steps"])}.get(case["book"], (min(60, case["steps"]), case["steps"]))
    terms = np.arange(lo, hi + 1)
    return case["policies"] * float(sum(np.maximum(terms - NODE_STEP * k, 0).mean()
                                        for k in range(case["nodes"])))


def work(case):
    """A reserve is a sum over the policy's months of expected cash flow times
    discount: two operations per policy, month and scenario where per-policy
    reserves are asked for.  Totals need the policies' cash flows (about eight
    operations a policy-month) and the curves once."""
    n, k, s, t = case["policies"], case["nodes"], case["scenarios"], case["steps"]
    if case["kind"] == "train_step":
        return dict(bytes=4.0 * (n * (rr.SG_INPUTS + 1) + 8 * rr.SG_PARAMS),
                    flops=6.0 * n * (17 * 256 + 256 * 256 + 256))
    curves = 0.0 if case["kind"] == "generated" else 8.0 * k * s * t
    book, months = 72.0 * n, _live_steps(case)
    if case["kind"] == "path":
        return dict(bytes=book + curves + 8.0 * (months + n), flops=12.0 * months)
    if case["kind"] == "totals":
        return dict(bytes=book + curves + 8.0 * k * s, flops=8.0 * months + 2.0 * k * s * t)
    if case["kind"] == "node_means":
        return dict(bytes=book + curves + 8.0 * k * n, flops=10.0 * months + 2.0 * k * s * t)
    if case["kind"] == "surrogate":
        return dict(bytes=book + curves + 8.0 * n * s, flops=2.0 * n * s * (17 * 256 + 256 * 256 + 256))
    width = 4 if case["all_states"] else 1
    return dict(bytes=book + curves + 8.0 * width * k * n * s, flops=8.0 * months + 2.0 * months * s)


# ---------------------------------------------------------------------------
# Results in 64 bits
# ---------------------------------------------------------------------------
def _dev(a, dt=F64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda" if torch.cuda.is_available() else "cpu")


def _flows(x, idx, node, start=0):
    """Expected cash flows at months 0..steps of policies idx seen from a node,
    for the reserve of state slot `start`: (flows paid at month starts and
    ends [n][steps + 1], flows paid within the month [n][steps + 1] or None)."""
    pf, case = x.pf, x.case
    shift, steps = node * NODE_STEP, case["steps"]
    col = lambda a, dt=F64: None if a is None else _dev(np.asarray(a)[idx], dt)
    prod, S = col(pf.product, torch.long), col(pf.term_m, torch.long) - shift
    amount, prem, timing = col(pf.amount), col(pf.premium), col(pf.timing, torch.long)
    q = _dev(x.q)
    if x.shock is not None:
        q = torch.clamp(q * x.shock[node], max=1.0)
    n, top = prod.shape[0], q.shape[1] - 1
    lives = []
    for age, tab in ((pf.age1_m, pf.table1), (pf.age2_m, pf.table2),
                     (pf.age3_m if pf.age3_m is not None else pf.age2_m,
                      pf.table3 if pf.table3 is not None else pf.table2)):
        t = torch.clamp(col(tab, torch.long), max=q.shape[0] - 1)
        lives.append((q, t, col(age, torch.long) + shift))
    is_in = lambda *p: torch.isin(prod, torch.tensor(p, device=prod.device))
    two, three = is_in(*TWO_LIFE), is_in(*THREE_LIFE)
    n_l = 1 + two.long() + 2 * three.long()
    # alive[l]: probability that life l + 1 lives; slots 1-3 start with some dead
    ones = torch.ones(n, dtype=F64, device=prod.device)
    alive = [ones.clone(), torch.where(n_l > 1, ones, 0 * ones), torch.where(n_l > 2, ones, 0 * ones)]
    has = start == 0
    if start:
        has = (is_in(rr.LS_ANN, rr.JL_ASSUR2) & (start < 3)) | (is_in(rr.REV_ANN) & (start == 2)) | \
            is_in(rr.LS3_ANN) | is_in(rr.MARKOV)
        for who, l, slots in ((two, 1, (1,)), (two, 0, (2,)), (three, 2, (1, 3)), (three, 1, (2, 3))):
            if start in slots:
                alive[l] = torch.where(who, 0 * ones, alive[l])
        has = has.to(F64)
    mk = is_in(rr.MARKOV)
    if x.markov is not None:
        w, c = _dev(x.markov[0]), _dev(x.markov[1])
        m = w.shape[-1]
        model = torch.where(mk, col(pf.table1, torch.long), 0)
        pi = torch.zeros(n, m, dtype=F64, device=prod.device)
        if start < m:
            pi[:, start] = 1.0
    esc = col(pf.escalation) if pf.escalation is not None else 0 * ones
    annual = col(pf.annual, torch.long) if pf.annual is not None else torch.zeros_like(prod)
    anniv = col(pf.anniv_m, torch.long) if pf.anniv_m is not None else torch.full_like(prod, 12)
    patterned = (esc > 0) | (annual == 1)
    cf = None if pf.cf is None else _dev(pf.cf)
    row = None if cf is None else col(pf.cf_row, torch.long)
    ann = is_in(rr.SL_ANN, rr.JL_ANN, rr.REV_ANN, rr.LS_ANN, *THREE_LIFE)
    sl, jl, rev, ls = (is_in(p) for p in (rr.SL_ANN, rr.JL_ANN, rr.REV_ANN, rr.LS_ANN))
    jl3, ls3, tabp = is_in(rr.JL3_ANN), is_in(rr.LS3_ANN), is_in(rr.CF_TABLE)
    death1, death2 = is_in(rr.TERM, rr.ENDOW_ASSUR, rr.JL_ASSUR1), is_in(rr.JL_ASSUR2)
    matur = is_in(rr.ENDOW, rr.ENDOW_ASSUR, rr.JL_ENDOW)
    out = torch.zeros(n, steps + 1, dtype=F64, device=prod.device)
    mid = torch.zeros_like(out) if x.frac > 0 and bool((timing == rr.FRACTIONAL).any()) else None

    def every(a):       # all lives of the policy alive
        return torch.where(three, a[0] * a[1] * a[2], torch.where(two, a[0] * a[1], a[0]))

    def any_(a):        # some life alive
        return a[0] + (1.0 - a[0]) * (a[1] + (1.0 - a[1]) * a[2])

    def paying(a, e):   # probability that the annuity is in payment
        return torch.where(sl | jl | jl3, e, torch.where(rev, (1.0 - a[0]) * a[1], any_(a)))

    def factor(T):
        cnt = torch.div(T + 12 - anniv, 12, rounding_mode="floor")
        lev = (1.0 + esc) ** cnt
        at = (cnt > 0) & ((T - anniv) % 12 == 0)
        return torch.where(patterned, torch.where(annual == 1, torch.where(at, 12.0 * lev, 0 * lev), lev), ones)

    e_now = every(alive)
    no_dead = torch.where(death2, (1.0 - alive[0]) * (1.0 - alive[1]), 0 * ones)
    for t in range(steps + 1):
        on = (t < S)
        if not bool((t <= S).any()):
            break
        if t > 0:   # arrears part of month t - 1 was added below; maturity values here
            out[:, t] += torch.where((t == S) & matur, e_now * amount, 0 * ones)
        if t == steps:
            break
        f_adv, f_arr = factor(shift + t), factor(shift + t + 1)
        adv = ann & (timing == rr.ADVANCE) & on
        prem_p = torch.where(mk, pi[:, 0], e_now) if x.markov is not None else e_now
        out[:, t] += torch.where(adv, paying(alive, e_now) * amount / 12.0 * f_adv, 0 * ones)
        out[:, t] -= torch.where(on, prem_p * prem, 0 * ones)
        if mid is not None:
            fr = (timing == rr.FRACTIONAL) & on
            pf_ = ones.clone()
            for l, (qq, tab, age) in enumerate(lives):
                g = 1.0 - x.frac * qq[tab, torch.clamp(age + t, max=top)]
                pf_ = torch.where(n_l > l, pf_ * g, pf_)
            mid[:, t] += torch.where(fr, e_now * pf_ * amount / 12.0, 0 * ones)
        nxt = [a * (1.0 - qq[tab, torch.clamp(age + t, max=top)]) for a, (qq, tab, age) in zip(alive, lives)]
        e_nxt = every(nxt)
        both_dead = torch.where(death2, (1.0 - nxt[0]) * (1.0 - nxt[1]), 0 * ones)
        arr = torch.where(ann & (timing == rr.ARREARS), paying(nxt, e_nxt) * amount / 12.0 * f_arr, 0 * ones)
        arr += torch.where(death1, (e_now - e_nxt) * amount, 0 * ones) + (both_dead - no_dead) * amount
        if cf is not None:
            arr += torch.where(tabp, e_nxt * amount * cf[row, min(shift + t, cf.shape[1] - 1)], 0 * ones)
        if x.markov is not None:
            W = w[model, torch.clamp(lives[0][2] + t, max=w.shape[1] - 1)]
            pi = (pi[:, :, None] * W).sum(1)
            arr = torch.where(mk, (pi * c[model]).sum(1) * amount, arr)
        out[:, t + 1] += torch.where(on, arr, 0 * ones)
        alive, e_now, no_dead = nxt, e_nxt, both_dead
    out[S <= 0] = 0.0
    if start:
        out, mid = out * has[:, None], None if mid is None else mid * has[:, None]
    return out, mid


def _discounts(x, node):
    """Discount to month t [steps + 1][scenario] and to month t + frac."""
    v = _dev(x.v[node]).T
    D = torch.cat([torch.ones_like(v[:1]), torch.cumprod(v, 0)])
    Df = None
    if x.frac > 0:
        Df = torch.cat([D[:-1] * v ** x.frac, torch.zeros_like(D[:1])])
    return D, Df


def _stats(tot):
    s = tot.shape[1]
    rank = max(1, min(s, math.ceil(TAIL * s - 1e-9)))
    return torch.stack([tot.mean(1), torch.sort(tot, 1, descending=True).values[:, rank - 1]], 1)


def exact(case, seed):
    if case["kind"] == "train_step":
        return _exact_step(case, seed)
    x = _inputs(case, seed)
    n, k, s = case["policies"], case["nodes"], case["scenarios"]
    kind = case["kind"]
    if kind == "path":
        return {"path": _exact_path(x)}
    slots = 4 if case["all_states"] else 1
    r0, tot = [], []
    for j in range(k):
        D, Df = _discounts(x, j)
        Db = D.mean(1, keepdim=True) if kind == "node_means" else None
        rows, sums = [], 0.0
        for i in range(0, n, 50_000):
            idx = np.arange(i, min(n, i + 50_000))
            per_slot = []
            for a in range(slots):
                f, m = _flows(x, idx, j, a)
                if kind == "totals":
                    sums = sums + f.sum(0, keepdim=True) @ D + (0.0 if m is None else m.sum(0, keepdim=True) @ Df)
                else:
                    r = f @ (D if Db is None else Db)
                    per_slot.append(r if m is None else r + m @ Df)
            if kind != "totals":
                rows.append(torch.stack(per_slot, -1) if slots > 1 else per_slot[0])
                sums = sums + per_slot[0].sum(0, keepdim=True)
        tot.append(sums.reshape(1, -1))
        r0.append(torch.cat(rows) if rows else None)
    tot = torch.cat(tot)
    if kind == "node_means":
        return {"r0": torch.stack([r.reshape(-1) for r in r0]), "totals": tot.reshape(-1)}
    if kind == "surrogate":
        r = _exact_network(x, seed, r0[0])
        tot = r.sum(0, keepdim=True)
        r0 = [r]
    out = {"totals": tot}
    if kind != "totals":
        out["r0"] = torch.stack(r0)
    if s > 1:
        out["stats"] = _stats(tot)
    return out


def _exact_path(x):
    """The state-0 reserve at every month of every policy (policies of the
    single- and joint-life books), by the backward recurrence."""
    case, pf = x.case, x.pf
    steps = case["steps"]
    v = _dev(x.v[0][0])
    q = _dev(x.q)
    i64 = lambda a: _dev(a, torch.long)
    S, prod, amount, prem = i64(pf.term_m), i64(pf.product), _dev(pf.amount), _dev(pf.premium)
    two = prod == rr.JL_ANN
    pay = torch.where((prod == rr.SL_ANN) | two, amount / 12.0, 0.0 * amount)
    death = torch.where(prod == rr.TERM, amount, 0.0 * amount)
    r = torch.where(prod == rr.ENDOW, amount, 0.0 * amount)
    off = torch.cumsum(S + 1, 0) - (S + 1)
    path = torch.empty(int((S + 1).sum()), dtype=F64, device=v.device)
    path[off + S] = r
    top = q.shape[1] - 1
    for t in range(steps - 1, -1, -1):
        p = 1.0 - q[i64(pf.table1), torch.clamp(i64(pf.age1_m) + t, max=top)]
        p = torch.where(two, p * (1.0 - q[i64(pf.table2), torch.clamp(i64(pf.age2_m) + t, max=top)]), p)
        on = t < S
        r = torch.where(on, v[t] * (p * (r + pay) + (1.0 - p) * death) - prem, r)
        path[(off + t)[on]] = r[on]
    return path


def _exact_network(x, seed, reserves):
    """Rows inside the model's box through the network in 64 bits, the others
    from the exact reserves."""
    m = _model(x, seed)
    raw_p, raw_s, _, _ = _features(x)
    prm, at = _dev(m["params"]), 0
    parts = []
    for shape in ((32, 256), (256,), (256, 256), (256,), (256,), (1,)):
        size = int(np.prod(shape))
        parts.append(prm[at:at + size].reshape(shape))
        at += size
    w1, b1, w2, b2, w3, b3 = parts
    pc, sc = list(range(8)) + [16], list(range(8, 13))
    box = lambda raw, c: np.all((raw >= m["lo"][c]) & (raw <= m["hi"][c]), axis=1)
    zp, zs = (raw_p - m["mu"][pc]) / m["sd"][pc], (raw_s - m["mu"][sc]) / m["sd"][sc]
    zst = (np.array([1.0, 0.0, 0.0]) - m["mu"][13:16]) / m["sd"][13:16]
    hp = _dev(zp) @ torch.cat([w1[:8], w1[16:17]])
    hs = _dev(zs) @ w1[8:13] + _dev(zst) @ w1[13:16] + b1
    slot = raw_p[:, 2:6].argmax(1)
    scale, offset = _dev(x.pf.amount * m["tsd"][slot]), _dev(x.pf.amount * m["tmu"][slot])
    okp, oks = _dev(box(raw_p, pc), torch.bool), _dev(box(raw_s, sc), torch.bool)
    gelu = lambda a: torch.nn.functional.gelu(a, approximate="tanh")
    r = reserves.clone()
    for i in range(0, r.shape[0], 400):
        a = gelu(hp[i:i + 400, None, :] + hs[None])
        y = gelu(a.reshape(-1, 256) @ w2 + b2) @ w3 + b3
        y = y.reshape(a.shape[:2]) * scale[i:i + 400, None] + offset[i:i + 400, None]
        r[i:i + 400] = torch.where(okp[i:i + 400, None] & oks[None], y, r[i:i + 400])
    return r


def _exact_step(case, seed):
    g = torch.Generator().manual_seed(int(seed) % (1 << 60))
    z = torch.zeros(case["policies"], rr.SG_INPUTS)
    z[:, :rr.SG_FEATURES] = torch.randn(case["policies"], rr.SG_FEATURES, generator=g)
    t = _dev(torch.randn(case["policies"], generator=g).numpy())
    prm = _dev(_mlp_params(seed)).requires_grad_(True)
    parts = torch.split(prm, [32 * 256, 256, 256 * 256, 256, 256, 1])
    gelu = lambda a: torch.nn.functional.gelu(a, approximate="tanh")
    h = gelu(_dev(z.numpy()) @ parts[0].reshape(32, 256) + parts[1])
    h = gelu(h @ parts[2].reshape(256, 256) + parts[3])
    loss = ((h @ parts[4] + parts[5] - t) ** 2).mean()
    loss.backward()
    return {"grad": prm.grad, "loss": loss.detach().reshape(1)}
