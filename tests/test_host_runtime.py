"""The library's host code on a stand-in for the HIP runtime (hip_double.cpp; no
GPU, no kernel runs): which kernels a call launches, what it does when device
memory runs out, and what may be destroyed while the GPU is still at work.
Each test is a program of its own, in a child process that loads the stand-in
before the library."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, sys
import numpy as np
hd = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
hd.hd_log.restype = hd.hd_faults.restype = ctypes.c_char_p
hd.hd_used.restype = hd.hd_buffer_end.restype = ctypes.c_uint64
for f, a in ((hd.hd_set_memory, [ctypes.c_uint64]), (hd.hd_buffer_end, [ctypes.c_uint64]),
             (hd.hd_set_capturing, [ctypes.c_uint64, ctypes.c_int])):
    f.argtypes = a
import paper_1401_1757_amd as rr
import synth
lib = rr.load_library()
STREAM = 0x51000          # the caller's stream (a name: the stand-in never looks behind it)
SAFE, WIDE = dict(a=0.1, b=0.03, sigma=0.01), dict(a=0.02, b=0.03, sigma=0.01)


class Ctx:
    def __init__(self):
        self.h = ctypes.c_void_p()
        assert lib.rr_create(ctypes.byref(self.h), 0, STREAM) == 0

    def ok(self, rc):
        assert rc == 0, (rc, lib.rr_last_error(self.h))

    def generate(self, q, n_scen, n_steps, nodes=1, frac=0.0, **vs):
        keep = []
        q = np.ascontiguousarray(q)
        b = rr.Basis(q.shape[0], q.shape[1], q.ctypes.data, nodes, n_scen, n_steps, None, None, rr.HOST, frac)
        self.ok(lib.rr_basis_generate_vasicek(self.h, ctypes.byref(b), ctypes.byref(self.vas(nodes, keep, vs))))

    def vas(self, nodes, keep, vs):
        return rr.vasicek_struct(vs["a"], vs["b"], vs["sigma"], 1.0 / 12.0, [0.03] * nodes, (3, 4), keep)

    def regenerate(self, nodes=1, **vs):
        keep = []
        self.ok(lib.rr_curves_generate_vasicek(self.h, ctypes.byref(self.vas(nodes, keep, vs))))

    def portfolio(self, pf):
        keep = []
        self.ok(lib.rr_portfolio_upload(self.h, ctypes.byref(rr.portfolio_struct(pf, keep))))
        self.n = pf.n

    def run(self, nodes, scen, mask, noalloc=False, at=1):
        # output buffers are never touched: made-up addresses, another set per `at`
        r = rr.Run(0, nodes, 0, scen, 12, mask, 0.005)
        base = at << 40
        o = rr.Outputs(base, base + (1 << 38), None, 0, base + (1 << 39))
        f = lib.rr_reserve_recurrence_noalloc if noalloc else lib.rr_reserve_recurrence
        return f(self.h, ctypes.byref(r), ctypes.byref(o))


def log():
    s = hd.hd_log().decode()
    hd.hd_clear()
    return s


def book(n, n_steps, products=(0, 1, 4, 5), seed=1, scen=2):
    w = synth.random_small(np.random.default_rng(seed), n=n, n_steps=n_steps, n_scen=scen, products=products)
    return w.basis.q, w.portfolio
"""


@pytest.fixture(scope="module")
def double(tmp_path_factory):
    import paper_1401_1757_amd as rr
    if not os.path.exists(rr.LIB_PATH):
        from paper_1401_1757_amd import build
        build.build()
    so = str(tmp_path_factory.mktemp("hip") / "libhip_double.so")
    subprocess.check_call(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-I", "/opt/rocm/include", "-o", so,
                           os.path.join(ROOT, "tests", "hip_double.cpp")])
    return so


def run(double, program):
    code = PRELUDE + textwrap.dedent(program)
    res = subprocess.run([sys.executable, "-c", code, double], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-3000:]


@pytest.mark.parametrize("model", ["SAFE", "WIDE"])
def test_discount_products_follow_every_regeneration(double, model):
    """A graph that the caller captured reads the kept discount products, so
    curves regenerated in place renew them whatever the model's range, also
    where runs made afterwards go by the recurrence kernel."""
    run(double, f"""
    q, pf = book(300, 120)
    c = Ctx()
    c.generate(q, 70, 600, **SAFE)
    first = log()
    D = [int(l.split(" D ")[1]) for l in first.splitlines() if "k_vas_scan" in l]
    assert len(D) == 1 and D[0], first
    c.portfolio(pf)
    hd.hd_set_capturing(STREAM, 1)
    c.ok(c.run(1, 70, rr.OUT_R0 | rr.OUT_TOTALS, noalloc=True))
    hd.hd_set_capturing(STREAM, 0)
    assert "k_reserve_mm" in log() and not hd.hd_faults()
    c.regenerate(**{model})
    again = log()
    assert [int(l.split(" D ")[1]) for l in again.splitlines() if "k_vas_scan" in l] == D, again
    c.ok(c.run(1, 70, rr.OUT_R0, noalloc=True))
    assert ("k_reserve_mm" in log()) == ({model} is SAFE)
    """)


def test_graphs_are_destroyed_after_their_launches(double):
    """More output sets than graphs are kept, a larger run, another stream, other
    options, other uploads: no executable graph is destroyed while a launch of
    it may still run, nothing waits on the way, and those set aside stay few."""
    run(double, """
    q, pf = book(3000, 60)
    c = Ctx()
    c.generate(q, 1000, 60, **SAFE)
    c.portfolio(pf)
    mask = rr.OUT_R0 | rr.OUT_TOTALS | rr.OUT_STATS
    for at in range(1, 40):
        c.ok(c.run(1, 1000, mask, at=at))
        c.ok(c.run(1, 1000, mask, at=at))
        assert hd.hd_live_execs() <= 8 * 6, hd.hd_live_execs()
    assert "graph: " in log()
    c.ok(lib.rr_set_option(c.h, rr.OPT_BLOCK_K, 8))
    c.ok(lib.rr_set_option(c.h, rr.OPT_BLOCK_J, 1))
    c.ok(lib.rr_set_option(c.h, rr.OPT_WG_PER_CU, 1))
    for at in range(1, 12):
        for rep in range(2):
            c.ok(c.run(1, 1000, mask, at=at))
    runs = lambda scen: [c.ok(c.run(1, scen, mask)) for rep in range(3)]
    c.ok(lib.rr_set_option(c.h, rr.OPT_CURVE_SHARE, 0))
    runs(1000)
    c.ok(lib.rr_set_stream(c.h, STREAM + 0x100))
    runs(1000)
    c.regenerate(**WIDE)
    runs(1000)
    c.portfolio(book(5000, 60, seed=2)[1])
    runs(1000)
    c.generate(q, 2000, 60, **SAFE)
    runs(2000)
    assert not hd.hd_faults(), hd.hd_faults()
    lib.rr_destroy(c.h)
    assert not hd.hd_faults() and hd.hd_live_execs() == 0, hd.hd_faults()
    """)


def test_dropping_graphs_does_not_wait(double):
    run(double, """
    q, pf = book(300, 60)
    c = Ctx()
    c.generate(q, 70, 60, **SAFE)
    c.portfolio(pf)
    c.ok(c.run(1, 70, rr.OUT_R0 | rr.OUT_TOTALS))
    waits = hd.hd_waits()
    for at in range(1, 20):
        for rep in range(2):
            c.ok(c.run(1, 70, rr.OUT_R0 | rr.OUT_TOTALS, at=at))
    c.ok(lib.rr_set_stream(c.h, STREAM + 0x100))
    assert hd.hd_waits() == waits and hd.hd_last_error() == 0
    """)


@pytest.mark.parametrize("sigma,steps,flows", [(0.01, 600, True), (0.3, 600, True), (8.0, 600, False), (8.0, 16, True)])
def test_totals_route_by_the_range_of_a_time_chunk(double, sigma, steps, flows):
    """Totals by summed flows need the products of a sixteenth of the months
    only; where those too could leave the range, the policies' own chains."""
    run(double, f"""
    q, pf = book(300, {min(steps, 120)})
    c = Ctx()
    c.generate(q, 70, {steps}, a=0.02, b=0.03, sigma={sigma})
    c.portfolio(pf)
    log()
    for noalloc in (False, True):
        c.ok(c.run(1, 70, rr.OUT_TOTALS | rr.OUT_STATS, noalloc=noalloc))
        names = log()
        assert ("k_flow_totals" in names) == {flows} and ("k_recurrence" in names) != {flows}, names
        assert "k_flow_totalsILi" not in names   # one form of the kernel
    """)


def test_a_run_is_captured_on_its_second_call(double):
    """The first call of a run launches directly, the second captures, later ones
    replay; more output sets in turn than are kept are always launched directly."""
    run(double, """
    q, pf = book(300, 60)
    c = Ctx()
    c.generate(q, 70, 60, **SAFE)
    c.portfolio(pf)
    mask = rr.OUT_R0 | rr.OUT_TOTALS
    log()
    kinds = []
    for rep in range(3):
        c.ok(c.run(1, 70, mask))
        lines = log().splitlines()
        kinds.append((all(l.startswith("graph: ") for l in lines), hd.hd_live_execs()))
    assert kinds == [(False, 0), (True, 1), (True, 1)], kinds
    for rep in range(3):
        for at in range(2, 11):
            c.ok(c.run(1, 70, mask, at=at))
    assert hd.hd_live_execs() == 1 and "graph: " not in log()
    for rep in range(3):
        for at in range(2, 10):
            c.ok(c.run(1, 70, mask, at=at))
    assert "graph: " in log() and not hd.hd_faults()
    """)


@pytest.mark.parametrize("mask", ["rr.OUT_R0", "rr.OUT_R0 | rr.OUT_TOTALS | rr.OUT_STATS", "rr.OUT_TOTALS"])
def test_runs_without_room_for_flows_take_the_recurrence_kernel(double, mask):
    run(double, f"""
    q, pf = book(20000, 120)
    c = Ctx()
    c.generate(q, 30, 120, **SAFE)
    c.portfolio(pf)
    log()
    hd.hd_set_memory(hd.hd_used() + (2 << 20))   # the flows of 313 tiles take 20 MiB, their rows 0.3
    for rep in range(4):
        c.ok(c.run(1, 30, {mask}))
        names = log()
        if {mask} & rr.OUT_R0:
            assert "k_recurrence" in names and "k_flow" not in names and "k_reserve_mm" not in names, names
            assert ("graph: " in names) == (rep > 0), (rep, names)   # nothing is captured anew
    hd.hd_set_memory(1 << 36)
    c.ok(c.run(1, 30, {mask}))
    assert "k_flow_sums" in log() and not hd.hd_faults()
    """)


def test_discount_products_leave_the_memory_to_others(double):
    """The kept products take at most an eighth of what is free; a basis that leaves
    less is valued by the recurrence kernel as if there were none."""
    run(double, """
    q, pf = book(300, 120)
    for room, kept in ((40, True), (6, False)):     # in curve arrays, which take one; the generator three more
        c = Ctx()
        hd.hd_set_memory(1 << 36)
        base = hd.hd_used()
        curves = 120 * 1056 * 8
        hd.hd_set_memory(base + room * curves)
        c.generate(q, 1024, 120, **SAFE)
        c.portfolio(pf)
        log()
        c.ok(c.run(1, 1024, rr.OUT_R0, noalloc=True))
        assert ("k_reserve_mm" in log()) == kept
        c.regenerate(**SAFE)
        c.ok(c.run(1, 1024, rr.OUT_R0, noalloc=True))
        assert ("k_reserve_mm" in log()) == kept
        lib.rr_destroy(c.h)
    """)


def test_a_portfolio_that_found_no_room_is_not_valued(double):
    run(double, """
    q, pf = book(300, 60)
    c = Ctx()
    c.generate(q, 70, 60, **SAFE)
    c.portfolio(pf)
    c.ok(c.run(1, 70, rr.OUT_R0))
    keep = []
    big = rr.portfolio_struct(book(20000, 60, seed=2)[1], keep)
    used = hd.hd_used()
    for extra in range(0, 3 << 20, 100 << 10):
        hd.hd_set_memory(used + extra)
        rc = lib.rr_portfolio_upload(c.h, ctypes.byref(big))
        log()
        if rc == 0:
            break
        assert rc == rr.RR_ENOMEM and c.run(1, 70, rr.OUT_R0) == rr.RR_ESTATE and log() == ""
    assert rc == 0 and extra > 0
    """)


def test_a_failed_regeneration_keeps_the_present_curves_bound(double):
    run(double, """
    q, pf = book(300, 160)
    c = Ctx()
    v = np.full((1, 70, 160), 1e-27)
    keep = []
    c.ok(lib.rr_basis_upload(c.h, ctypes.byref(rr.basis_struct(q, v, None, keep))))
    c.portfolio(pf)
    c.ok(c.run(1, 70, rr.OUT_TOTALS, noalloc=True))
    assert "k_recurrence" in log()
    hd.hd_set_memory(hd.hd_used())
    assert lib.rr_curves_generate_vasicek(c.h, ctypes.byref(c.vas(1, keep, SAFE))) == rr.RR_ENOMEM
    log()
    c.ok(c.run(1, 70, rr.OUT_TOTALS, noalloc=True))
    assert "k_recurrence" in log()
    hd.hd_set_memory(1 << 36)
    c.regenerate(**SAFE)
    log()
    c.ok(c.run(1, 70, rr.OUT_TOTALS, noalloc=True))
    assert "k_flow_totals" in log()
    """)


def test_a_failed_call_is_reported_once(double):
    """The launches' check of the runtime's last error does not find the error that
    an earlier call has reported already."""
    run(double, """
    q, pf = book(300, 60)
    c = Ctx()
    c.generate(q, 70, 60, **SAFE)
    c.portfolio(pf)
    c.ok(c.run(1, 70, rr.OUT_R0 | rr.OUT_TOTALS))
    hd.hd_set_memory(hd.hd_used())
    big = rr.Basis(q.shape[0], q.shape[1], np.ascontiguousarray(q).ctypes.data, 1, 4000, 60, None, None, rr.HOST, 0.0)
    v = np.ones((1, 4000, 60))
    big.v = v.ctypes.data
    other = Ctx.__new__(Ctx)
    other.h = ctypes.c_void_p()
    hd.hd_set_memory(hd.hd_used() + 100000)
    assert lib.rr_create(ctypes.byref(other.h), 0, STREAM) == 0
    assert lib.rr_basis_upload(other.h, ctypes.byref(big)) == rr.RR_ENOMEM
    c.ok(c.run(1, 70, rr.OUT_R0 | rr.OUT_TOTALS, at=2))
    c.ok(c.run(1, 70, rr.OUT_TOTALS, noalloc=True))
    """)


def test_markov_models_that_found_no_room_leave_no_portfolio_on_them(double):
    run(double, """
    q, pf = book(300, 60, products=(0,))
    c = Ctx()
    c.generate(q, 70, 60, **SAFE)
    w, ben = synth.phi_models(q.shape[1])

    def markov(w, ben):
        keep = [np.ascontiguousarray(w), np.ascontiguousarray(ben)]
        m = rr.Markov(w.shape[0], w.shape[2], w.shape[1], keep[0].ctypes.data, keep[1].ctypes.data, rr.HOST)
        return lib.rr_markov_upload(c.h, ctypes.byref(m))

    c.ok(markov(w, ben))
    c.portfolio(synth.with_markov_policies(np.random.default_rng(1), pf, (w, ben), 0.5))
    c.ok(c.run(1, 70, rr.OUT_R0))
    hd.hd_set_memory(hd.hd_used())
    log()
    assert markov(np.concatenate([w] * 40), np.concatenate([ben] * 40)) == rr.RR_ENOMEM
    assert c.run(1, 70, rr.OUT_R0) == rr.RR_ESTATE and log() == ""
    hd.hd_set_memory(1 << 36)
    c.portfolio(pf)
    c.ok(c.run(1, 70, rr.OUT_R0))
    """)


@pytest.mark.parametrize("captured", ["STREAM", "STREAM + 0x100"])
def test_another_stream_while_the_caller_captures(double, captured):
    """Changing to a stream that the caller is capturing, or away from one, drops
    the captured runs without an operation on any stream."""
    run(double, f"""
    q, pf = book(300, 60)
    c = Ctx()
    c.generate(q, 70, 60, **SAFE)
    c.portfolio(pf)
    for rep in range(2):
        c.ok(c.run(1, 70, rr.OUT_R0 | rr.OUT_TOTALS))
    assert hd.hd_live_execs() == 1
    waits = hd.hd_waits()
    hd.hd_set_capturing({captured}, 1)
    c.ok(lib.rr_set_stream(c.h, STREAM + 0x100))
    assert hd.hd_waits() == waits and not hd.hd_faults(), hd.hd_faults()
    hd.hd_set_capturing({captured}, 0)
    for rep in range(3):
        c.ok(c.run(1, 70, rr.OUT_R0 | rr.OUT_TOTALS))
    lib.rr_destroy(c.h)
    assert hd.hd_live_execs() == 0 and not hd.hd_faults(), hd.hd_faults()
    """)
