"""The propagator applied by its series (qme_set_products(ctx, 1)) against the
dense products (0) and the oracle: the edges of the row passes' shapes, ragged
sizes, components of H with different shifts, long and empty rows of H, the
choice between the forms, and batches that mix them."""
import numpy as np
import pytest

import workloads as W
from oracle import evolve as ev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2403_07042_amd")
from paper_2403_07042_amd import _lib as L  # noqa: E402

# the suite's tolerances against the oracle, relative to the largest element;
# two forms that each meet it differ by at most twice as much
TOL = {"fp64": 1e-12, "fp32": 1e-5, "bf16x3": 1e-4}


def cavity_chain(n, dt=0.25, gamma=0.01):
    """n cavities in a row with one photon among them, leaking at the ends."""
    return dict(W.photon_lattice(n, 1, mu=0.2, g=0.0, gamma=0.0, dt=dt, atoms_per_site=0),
                jumps=[(W.PHOTON_LEAK, 0, -1, gamma), (W.PHOTON_LEAK, n - 1, -1, gamma)])


def random_model(n, degree, seed, dt=0.02, isolated=0):
    """A general model: a random symmetric H with rows of about `degree` entries
    (the first state coupled to many more) in two components of different
    frequency, the last `isolated` states coupled to nothing, and a lowering
    operator (the next state, the last one leaving the basis)."""
    rng = np.random.default_rng(seed)
    h = np.zeros((n, n))
    half = n // 2
    for lo, hi in ((0, half), (half, n - isolated)):
        for _ in range((hi - lo) * degree // 2):
            a, b = rng.integers(lo, hi, 2)
            if a != b:
                h[a, b] = h[b, a] = rng.uniform(0.02, 0.2)
    h[0, 1:20] = h[1:20, 0] = 0.05
    h += np.diag(np.where(np.arange(n) < half, 1.0, 3.0) + rng.uniform(0.0, 0.1, n))
    r, c = np.nonzero(h)
    src = list(range(n))
    return {"general": True, "name": f"random_{n}", "n": n,
            "h": (r.astype(np.int32), c.astype(np.int32), h[r, c]),
            "jumps": [(0.01, src, src[1:] + [-1], [1.0] * n)], "dt": dt}


def run(wl, precision, form, calls, rho0, fold=True):
    sol = P.Solver(wl, precision)
    sol.set_products(form)
    sol.set_fold(fold)
    sol.set_rho(rho0, sink=0.125)
    for k in calls:
        sol.step(k)
    rho, sink = sol.get_rho()
    _, trace, _ = sol.observe()
    sol.close()
    return rho, sink, trace


def check(got, ref, precision):
    tol = 2 * TOL[precision]
    assert np.abs(got[0] - ref[0]).max() < tol * np.abs(ref[0]).max()
    assert np.array_equal(got[0], got[0].conj().T)
    assert abs(got[1] - ref[1]) < tol and abs(got[2] - (1.0 - got[1])) < max(1e-12, 0.1 * tol)


SIZES = [33, 64, 65, 255, 256, 257, 511, 513, 1023, 1025, 2047, 2049]


@pytest.mark.parametrize("fold", [True, False])
@pytest.mark.parametrize("precision", ["fp32", "fp64", "bf16x3"])
@pytest.mark.parametrize("n", SIZES)
def test_shape_edges_against_dense(n, precision, fold):
    wl = cavity_chain(n)
    psi = W.haar_psi(n, 3)
    rho0 = np.outer(psi, psi.conj())
    print(f"series N={n} {precision} fold={fold}", flush=True)
    check(run(wl, precision, 1, (3, 4), rho0, fold), run(wl, precision, 0, (3, 4), rho0, fold), precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [33, 256, 257, 1025, 2049, 4097, 5121])
def test_one_pass_steps_equal_profiled_steps(n, precision):
    """A step in one pass is the arithmetic of its two passes (which a profiled
    call runs): the same bits, over odd and even counts of steps."""
    wl = cavity_chain(n)
    psi = W.haar_psi(n, 3)
    print(f"one-pass steps N={n} {precision}", flush=True)
    got = []
    for profiled in (False, True):
        sol = P.Solver(wl, precision)
        sol.set_products(1)
        sol.set_rho(np.outer(psi, psi.conj()), sink=0.125)
        if profiled:
            sol.profile(True)
        for k in (1, 2, 3):
            sol.step(k)
        got.append((*sol.get_rho(), sol.observe()[1]))
        sol.close()
    assert np.array_equal(got[0][0], got[1][0])
    assert got[0][1:] == got[1][1:]


@pytest.mark.parametrize("n,precision", [(4095, "fp32"), (4097, "fp32"), (5120, "fp32"), (5121, "fp32"),
                                         (4097, "fp64")])
def test_large_shapes_against_dense(n, precision):
    wl = cavity_chain(n)
    psi = W.haar_psi(n, 3)
    rho0 = np.outer(psi, psi.conj())
    print(f"series N={n} {precision}", flush=True)
    check(run(wl, precision, 1, (2, 1), rho0), run(wl, precision, 0, (2, 1), rho0), precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64", "bf16x3"])
@pytest.mark.parametrize("n,degree,isolated", [(130, 3, 0), (300, 9, 70), (700, 14, 1)])
def test_general_models_against_oracle(n, degree, isolated, precision):
    """Rows of H of very different length (a state coupled to twenty others,
    states coupled to none), two components of H with different shifts, a
    decoherence operator inside the basis."""
    wl = random_model(n, degree, n, isolated=isolated)
    psi = W.haar_psi(n, 5)
    rho0 = np.outer(psi, psi.conj())
    s = ev.GeneralSystem(wl)
    ref, sink = ev.evolve(s, rho0, 20, sink0=0.125)
    print(f"series general N={n} {precision}", flush=True)
    got = run(wl, precision, 1, (20,), rho0)
    check(got, (ref, sink), precision)


def test_products_knob():
    """The series is the default where H is sparse enough, asking for split
    products or form 0 selects the dense ones, small systems have none."""
    sol = P.Solver(W.photon_lattice(16, 16, gamma=0.05), "fp32")
    psi = W.haar_psi(sol.n, 7)
    rho0 = np.outer(psi, psi.conj())

    def state():
        sol.set_rho(rho0)
        sol.step(5)
        return sol.get_rho()[0]

    default = state()
    sol.set_products(1)
    series = state()
    sol.set_products(0)
    dense = state()
    sol.set_products(-1)
    sol.set_split(True)
    split = state()
    sol.set_split(False)
    again = state()
    assert np.array_equal(default, series) and np.array_equal(again, series)
    assert np.array_equal(dense, split) and not np.array_equal(dense, series)
    for form in (-2, 2):
        with pytest.raises(L.QmeError) as e:
            sol.set_products(form)
        assert e.value.status == L.QME_E_ARG
    sol.close()
    small = P.Solver(W.jc_single(), "fp32")
    with pytest.raises(L.QmeError) as e:
        small.set_products(1)
    assert e.value.status == L.QME_E_UNSUPPORTED
    small.close()


@pytest.mark.parametrize("sizes", [(40, 200), (40, 600), (200, 1100), (40, 2100)])
def test_batch_of_both_forms_equals_solo(sizes):
    """Batches of series instances in every shape of their passes, beside
    instances with dense products: each bitwise as alone."""
    wls = [cavity_chain(n, dt=0.1 + 0.05 * k) for n in sizes for k in range(2)]
    sols = []
    for k, wl in enumerate(wls):
        sol = P.Solver(wl, "fp32")
        sol.set_products(1 if k % 4 != 1 else 0)
        psi = W.haar_psi(sol.n, k)
        sol.set_rho(np.outer(psi, psi.conj()))
        sols.append(sol)
    b = P.Batch(sols)
    print(f"batch of both forms, N = {sizes}", flush=True)
    b.step(3)
    b.step(4)
    torch.cuda.synchronize()
    for k, (wl, sol) in enumerate(zip(wls, sols)):
        alone = P.Solver(wl, "fp32")
        alone.set_products(1 if k % 4 != 1 else 0)
        alone.set_fold(False)
        if k % 4 == 1:
            alone.set_split(False)
        psi = W.haar_psi(alone.n, k)
        alone.set_rho(np.outer(psi, psi.conj()))
        alone.step(7)
        assert np.array_equal(sol.get_rho()[0], alone.get_rho()[0]), (sizes, k)
        alone.close()
    b.close()
    for sol in sols:
        sol.close()


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-4), ("fp64", 1e-9)])
@pytest.mark.parametrize("make", [lambda: W.photon_lattice(27, 21, gamma=0.05),      # N = 1134, ld = 1152
                                  lambda: W.photon_lattice(9, 7, mu=0.1, g=0.1, dt=0.1, gamma=0.05),
                                  W.tch_2x2, lambda: random_model(300, 5, 8, isolated=40)])
def test_adjoint_against_dense(make, precision, tol):
    """Gradients by the series (rotations by row passes, the sum of rho X on
    the tiles that reach the gradient only) against the dense products',
    recomputed and whole segments."""
    wl = make()
    sol = P.Solver(wl, precision)
    psi = W.haar_psi(sol.n, 4)
    sol.set_rho(np.outer(psi, psi.conj()))
    obs = np.random.default_rng(6).uniform(0.0, 1.0, sol.n)
    out = {}
    for form in (0, 1):
        sol.set_products(form)
        print(f"adjoint N={sol.n} {precision} form={form}", flush=True)
        out[form] = [sol.adjoint(7, obs, checkpoint_every=every) for every in (3, 16)]
    sol.close()
    for (f0, g0), (f1, g1) in zip(out[0], out[1]):
        assert abs(f0 - f1) < tol * abs(f0)
        assert np.linalg.norm(g0 - g1) < tol * np.linalg.norm(g0)
    assert np.array_equal(out[1][0][1], out[1][1][1])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [33, 256, 257, 1025, 2049, 3073, 4097, 5121])
def test_pure_against_dense(n, precision):
    """Pure-state steps in one launch per call (a workgroup per vector)
    against one launch per step over dU, at the edges of the shapes; the
    vectors of a call and the split of a run into calls change no bit."""
    wl = dict(cavity_chain(n), jumps=[])
    sol = P.Solver(wl, precision)
    psi = np.stack([W.haar_psi(n, 9), W.haar_psi(n, 10)])
    out = {}
    for form, calls in ((1, (9,)), ("split", (4, 1, 4)), (0, (9,))):
        sol.set_products(0 if form == 0 else 1)
        sol.set_psi(psi)
        print(f"pure N={n} {precision} form={form}", flush=True)
        for k in calls:
            sol.step_pure(k)
        out[form] = sol.get_psi()
    sol.set_products(1)
    sol.set_psi(psi[1])
    sol.step_pure(9)
    assert np.array_equal(sol.get_psi(), out[1][1])
    sol.close()
    assert np.array_equal(out["split"], out[1])
    tol = 2 * {"fp32": 1e-5, "fp64": 1e-12}[precision]
    assert np.abs(out[1] - out[0]).max() < tol * np.abs(out[0]).max()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,degree", [(140, 3), (400, 14)])
def test_pure_general_models_against_oracle(n, degree, precision):
    """Rows of H longer than the entries kept in registers, and components
    whose phases differ (a pure state keeps its phase)."""
    wl = dict(random_model(n, degree, n), jumps=[])
    psi = W.haar_psi(n, 5)
    sol = P.Solver(wl, precision)
    sol.set_products(1)
    sol.set_psi(psi)
    print(f"pure general N={n} {precision}", flush=True)
    sol.step_pure(50)
    got = sol.get_psi()
    sol.close()
    ref = ev.evolve_pure(ev.GeneralSystem(wl), psi, 50)
    assert np.abs(got - ref).max() < {"fp32": 1e-5, "fp64": 1e-11}[precision] * np.abs(ref).max()


def many_channels():
    """Two cavities (one and two atoms, cap 1), every decay and dephasing: N = 32
    with eight channels inside the basis."""
    jumps = [(W.PHOTON_LEAK, c, -1, 0.02 + 0.01 * c) for c in range(2)]
    for kind in (W.ATOM_DECAY, W.ATOM_DEPHASE):
        jumps += [(kind, c, k, 0.01) for c, k in ((0, 0), (1, 0), (1, 1))]
    return {"name": "channels", "atoms": [1, 2], "photon_cap": [1, 1], "exc_min": 0, "exc_max": -1,
            "omega_c": [1.0, 1.05], "omega_a": [0.9, 1.0, 1.1], "g": [0.1, 0.08, 0.12],
            "hops": [(0, 1, 0.05)], "jumps": jumps, "dt": 0.05}


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("make", [
    W.jc_single, lambda: W.jc_single(cap=6),                       # N = 8, 14: two entries a row of dU
    lambda: W.jc_single(cap=15),                                   # N = 32
    lambda: W.photon_lattice(4, 3, mu=0.1, gamma=0.05, dt=0.1, atoms_per_site=0, g=0.0),   # N = 12: series
    lambda: W.photon_lattice(17, 1, mu=0.1, gamma=0.05, dt=0.1, atoms_per_site=0, g=0.0),
    lambda: W.photon_lattice(4, 4, mu=0.1, g=0.1, gamma=0.05, dt=0.1),                     # N = 32
    many_channels,                                                 # the general kernel
    lambda: dict(random_model(24, 4, 2)),                          # a row of H past eight entries
])
def test_single_workgroup_kernels_against_oracle(make, precision):
    wl = make()
    general = wl.get("general", False)
    s = ev.GeneralSystem(wl) if general else ev.System(wl)
    psi = W.haar_psi(s.n, 13)
    rho0 = np.outer(psi, psi.conj())
    ref, sink = ev.evolve(s, rho0, 60, sink0=0.125)
    sol = P.Solver(wl, precision)
    sol.set_rho(rho0, sink=0.125)
    print(f"single workgroup N={s.n} {precision}", flush=True)
    sol.step(41)
    sol.step(19)
    rho, got_sink = sol.get_rho()
    _, trace, _ = sol.observe()
    sol.close()
    check((rho, got_sink, trace), (ref, sink), precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("make", [
    lambda: W.photon_lattice(16, 1, mu=0.1, gamma=0.05, dt=0.1, atoms_per_site=0, g=0.0),   # 256 threads
    lambda: W.photon_lattice(22, 1, mu=0.1, gamma=0.05, dt=0.1, atoms_per_site=0, g=0.0),   # 512
    lambda: W.photon_lattice(23, 1, mu=0.1, gamma=0.05, dt=0.1, atoms_per_site=0, g=0.0),   # 1024
    lambda: W.jc_single(cap=8), lambda: W.jc_single(cap=11),       # N = 18: series; 24: rows of dU
    # N = 20, |H dt| past the series: the rows of dU with 512 threads
    lambda: dict(W.jc_single(cap=9), omega_c=[0.0], omega_a=[0.0], dt=60.0, g=[0.02]),
])
def test_single_workgroup_widths_against_oracle(make, precision):
    test_single_workgroup_kernels_against_oracle(make, precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64", "bf16x3"])
@pytest.mark.parametrize("n", [128, 513, 2048])
def test_profiled_series_runs_the_callers_launches(n, precision):
    """After qme_set_products(ctx, 1) a profiled call of folded steps records the
    launches of an unprofiled one: the call's first pass, one pass per step and
    the last trace; a stride samples the steps; the state's bits are the same, and
    those of the two passes per step that a profiled call runs by default."""
    wl = cavity_chain(n)
    psi = W.haar_psi(n, 3)
    out = []
    for form, every in ((1, 0), (1, 1), (1, 3), (-1, 1)):
        sol = P.Solver(wl, precision)
        sol.set_products(form)
        sol.set_rho(np.outer(psi, psi.conj()), sink=0.125)
        sol.profile(every)
        print(f"profiled series N={n} {precision} form={form} every={every}", flush=True)
        for k in (1, 2, 4):
            sol.step(k)
        torch.cuda.synchronize()
        counts = [c for _, c in sol.profile_read().values()]
        # steps 0, 3 and 6 are sampled; of the calls' first ones 0 and 3, of the last ones 0 and 6
        if form == 1:
            assert counts == {0: [0, 0, 0, 0], 1: [3, 7, 3, 0], 3: [2, 3, 2, 0]}[every]
        else:
            assert counts[:2] == [7, 7]
        out.append((*sol.get_rho(), sol.observe()[1]))
        sol.close()
    for got in out[1:]:
        assert np.array_equal(got[0], out[0][0]) and got[1:] == out[0][1:]


@pytest.mark.parametrize("n,precision,theta,one", [
    (4096, "fp32", 0.2, True), (4097, "fp32", 0.004, True), (4097, "fp32", 0.2, False),
    (5121, "fp32", 0.04, True), (5121, "fp32", 0.2, False),
    (4097, "fp64", 0.2, True), (5121, "fp64", 0.2, False)])
def test_large_folded_steps_one_pass_or_two(n, precision, theta, one):
    """Past N = 4096 a long series steps in two passes (its one-pass body spills),
    a short one in one; the bits are those of the other form, which a profiled
    call runs by default."""
    wl = cavity_chain(n, dt=theta / 0.4)      # |H dt| = 2 mu dt
    psi = W.haar_psi(n, 3)
    out = []
    for form in (1, -1):
        sol = P.Solver(wl, precision)
        sol.set_products(form)
        sol.set_rho(np.outer(psi, psi.conj()), sink=0.125)
        sol.profile(True)
        print(f"one pass or two N={n} {precision} |H dt|={theta} form={form}", flush=True)
        for k in (1, 2):
            sol.step(k)
        torch.cuda.synchronize()
        counts = [c for _, c in sol.profile_read().values()]
        if form == 1:
            assert counts == ([2, 3, 2, 0] if one else [3, 3, 2, 0])
        out.append((*sol.get_rho(), sol.observe()[1]))
        sol.close()
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]
