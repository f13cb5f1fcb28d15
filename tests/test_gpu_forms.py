"""Which form of the propagator the steps take by default (qme_set_products -1):
never the series where H has rows so long that its passes are the slower form,
on both sides of the line.  The forms round differently, so a state tells which
one ran."""
import numpy as np
import pytest

import workloads as W
from oracle import evolve as ev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2403_07042_amd")


def general(n, rows, cols, dt=0.3, row_sum=1.0):
    """A closed general model: couplings of one value, |H|_1 = row_sum."""
    r, c = np.concatenate([rows, cols]), np.concatenate([cols, rows])
    longest = np.bincount(r, minlength=n).max()
    return {"general": True, "name": f"general_{n}", "n": n, "jumps": [], "dt": dt,
            "h": (r.astype(np.int32), c.astype(np.int32), np.full(r.size, row_sum / longest))}


def star(n):
    """State 0 coupled to all others (one cavity with many atoms, one excitation)."""
    return general(n, np.zeros(n - 1, int), np.arange(1, n))


def ring(n, degree):
    """Every state coupled to its degree / 2 next and to as many before."""
    i = np.arange(n)
    return general(n, np.tile(i, degree // 2), np.concatenate([(i + k) % n for k in range(1, degree // 2 + 1)]))


def tavis_cummings(atoms):
    """One cavity with `atoms` atoms and at most one excitation: the photon's
    state is coupled to every atom's."""
    return {"name": f"tc_{atoms}", "atoms": [atoms], "photon_cap": [1], "exc_min": 0, "exc_max": 1,
            "omega_c": [1.0], "omega_a": [1.0] * atoms, "g": [0.05] * atoms, "hops": [],
            "jumps": [(W.PHOTON_LEAK, 0, -1, 0.01)], "dt": 0.05}


def states(wl, precision, forms):
    sol = P.Solver(wl, precision)
    psi = W.haar_psi(sol.n, 3)
    rho0 = np.outer(psi, psi.conj())
    out = []
    for form in forms:
        print(f"{wl['name']} N={sol.n} {precision} form={form}", flush=True)
        sol.set_products(form)
        sol.set_rho(rho0)
        sol.step(2)
        out.append(sol.get_rho()[0])
    sol.close()
    return out


@pytest.mark.parametrize("precision", ["fp32", "fp64", "bf16x3"])
@pytest.mark.parametrize("make", [lambda: star(129), lambda: star(501), lambda: star(2048),
                                  lambda: tavis_cummings(64), lambda: ring(513, 32), lambda: ring(2048, 128)])
def test_long_rows_take_dense_products(make, precision):
    default, dense = states(make(), precision, (-1, 0))
    assert np.array_equal(default, dense)


@pytest.mark.parametrize("precision", ["fp32", "fp64", "bf16x3"])
@pytest.mark.parametrize("make", [lambda: ring(129, 2), lambda: ring(513, 4), lambda: ring(2048, 16)])
def test_short_rows_take_the_series(make, precision):
    default, dense, series = states(make(), precision, (-1, 0, 1))
    assert np.array_equal(default, series) and not np.array_equal(default, dense)


def vectors(wl, precision, forms):
    sol = P.Solver(wl, precision)
    psi = W.haar_psi(sol.n, 3)
    out = []
    for form in forms:
        print(f"pure {wl['name']} N={sol.n} {precision} form={form}", flush=True)
        sol.set_products(form)
        sol.set_psi(psi)
        sol.step_pure(3)
        out.append(sol.get_psi())
    sol.close()
    return out


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("make", [lambda: star(65), lambda: star(501), lambda: star(2048), lambda: ring(257, 32),
                                  lambda: ring(2048, 32), lambda: ring(4097, 32)])
def test_pure_long_rows_take_dense(make, precision):
    default, dense = vectors(make(), precision, (-1, 0))
    assert np.array_equal(default, dense)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("make", [lambda: ring(64, 2), lambda: ring(2048, 2), lambda: ring(4097, 4)])
def test_pure_short_rows_take_the_series(make, precision):
    default, dense, series = vectors(make(), precision, (-1, 0, 1))
    assert np.array_equal(default, series) and not np.array_equal(default, dense)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("make", [
    lambda: W.photon_lattice(4, 3, mu=0.02, gamma=0.05, dt=0.01, atoms_per_site=0, g=0.0),  # N = 12
    lambda: W.photon_lattice(18, 1, mu=0.02, gamma=0.05, dt=0.01, atoms_per_site=0, g=0.0),
    lambda: W.photon_lattice(4, 4, mu=0.1, g=0.1, gamma=0.05, dt=0.1)])                     # N = 32
def test_small_systems_obey_form_zero(make, precision):
    """Systems that step by the series in their single workgroup by default: form
    0 multiplies by dU instead, and both agree with the oracle."""
    wl = make()
    s = ev.System(wl)
    psi = W.haar_psi(s.n, 13)
    rho0 = np.outer(psi, psi.conj())
    ref, sink = ev.evolve(s, rho0, 60)
    sol = P.Solver(wl, precision)
    out = []
    for form in (-1, 0, -1):
        print(f"single workgroup N={sol.n} {precision} form={form}", flush=True)
        sol.set_products(form)
        sol.set_rho(rho0)
        sol.step(60)
        out.append(sol.get_rho())
    sol.close()
    assert np.array_equal(out[0][0], out[2][0]) and not np.array_equal(out[0][0], out[1][0])
    tol = {"fp32": 1e-5, "fp64": 1e-12}[precision]
    for rho, got in out:
        assert np.abs(rho - ref).max() < tol * np.abs(ref).max() and abs(got - sink) < tol


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("cap", [7, 8, 10, 11])
def test_short_rows_of_du_in_one_workgroup(cap, precision):
    """One cavity and one atom, N = 16, 18, 22, 24: dU's rows have two entries, so
    its products are the faster form and the default at every N."""
    wl = W.jc_single(cap=cap)
    default, dense = states(wl, precision, (-1, 0))
    assert np.array_equal(default, dense)


def test_batch_takes_the_forms_at_config():
    """An instance's form is read when the batch is made and by config()."""
    wl = ring(200, 4)
    sol = P.Solver(wl, "fp32")
    psi = W.haar_psi(sol.n, 3)
    rho0 = np.outer(psi, psi.conj())
    solo = P.Solver(wl, "fp32")
    solo.set_fold(False)
    ref = {}
    for form in (-1, 0):
        solo.set_products(form)
        if form == 0:
            solo.set_split(False)
        solo.set_rho(rho0)
        solo.step(2)
        ref[form] = solo.get_rho()[0]
    solo.close()
    assert not np.array_equal(ref[-1], ref[0])
    b = P.Batch([sol])
    for form, config, expected in ((-1, False, -1), (0, False, -1), (0, True, 0), (-1, True, -1)):
        sol.set_products(form)
        if config:
            b.config()
        sol.set_rho(rho0)
        b.step(2)
        torch.cuda.synchronize()
        assert np.array_equal(sol.get_rho()[0], ref[expected]), (form, config)
    assert sol.products == 1
    b.close()
    sol.close()


def solo_unfolded(wl, form, tiles, steps, rho0):
    sol = P.Solver(wl, "fp32")
    sol.set_products(form)
    sol.set_fold(False)
    if form == 0:
        sol.set_split(False)
    sol.set_tiles(*tiles)
    sol.set_rho(rho0)
    sol.step(steps)
    out = sol.get_rho()
    sol.close()
    return out


@pytest.mark.parametrize("dense,series", [([40], [64]), ([24, 60], [63, 64]), ([200, 130], [65, 128]),
                                          ([250], [129, 256, 40]), ([40], [257, 64]), ([], [64, 33]),
                                          ([], [65, 128, 40]), ([], [129])])
@pytest.mark.parametrize("tiles", [(32, 32), (64, 64)])
def test_batches_of_small_systems_equal_solo(dense, series, tiles):
    """The launches of a batch by its sizes and forms (both forms' workgroups in one
    launch up to N = 256, workgroups of 64, 128 and 256 threads for the series
    alone): every instance bitwise as alone, unfolded."""
    sols, refs = [], []
    for k, (n, form) in enumerate([(n, 0) for n in dense] + [(n, 1) for n in series]):
        wl = dict(ring(n, 4), dt=0.02 + 0.05 * k)
        psi = W.haar_psi(n, k)
        rho0 = np.outer(psi, psi.conj())
        if n > 32:
            refs.append(solo_unfolded(wl, form, tiles, 7, rho0))
        else:
            refs.append(None)         # (alone it takes its single workgroup)
        sol = P.Solver(wl, "fp32")
        if n > 32:
            sol.set_products(form)
        sol.set_tiles(*tiles)
        sol.set_rho(rho0)
        sols.append(sol)
    b = P.Batch(sols)
    print(f"batch dense {dense} series {series} tiles {tiles}", flush=True)
    b.step(3)
    b.step(4)
    torch.cuda.synchronize()
    for sol, ref in zip(sols, refs):
        rho, sink = sol.get_rho()
        if ref is not None:
            assert np.array_equal(rho, ref[0]) and sink == ref[1], sol.n
        assert abs(np.trace(rho).real - 1.0) < 1e-6
    b.close()
    for sol in sols:
        sol.close()


def test_unfolded_steps_have_a_rule_of_their_own():
    """Where the steps do not fold (fold off, batches), the series saves less: a
    model on the line steps by it folded and by dense products unfolded."""
    found = []
    for n in (64, 100, 120, 200):
        sol = P.Solver(ring(n, 4), "fp32")
        folded = sol.products
        sol.set_fold(False)
        found.append((folded, sol.products))
        sol.close()
    assert found == [(0, 0), (1, 0), (1, 0), (1, 1)]
