"""The autotuner and the form of the step (no GPU): the tiles and splits it tunes
are knobs of the dense products, so it leaves a solver that steps by the series
alone, and no cached entry of another form or an older version is applied."""
import pytest

from paper_2403_07042_amd import autotune as A

KEY = A.solver_key("gfx950", "fp32", 512, 512)
OLD = {"tiles": [128, 128], "split": True}          # as versions before the forms wrote it


class FakeTensor:
    def clone(self):
        return self


class FakeSolver:
    """The knobs of a context whose default form is the series or dense; asking
    for split products selects the dense ones, as qme_set_split does."""
    torch, precision, n, ld, state = None, "fp32", 512, 512, FakeTensor()

    def __init__(self, series, asked=False):
        self.series, self.asked, self.tiles, self.split, self.steps = series, asked, (32, 32), True, 0

    @property
    def products(self):
        return 1 if self.series and not self.asked else 0

    @property
    def tile1(self):
        return self.tiles[0]

    @property
    def tile2(self):
        return self.tiles[1]

    def set_tiles(self, a, b):
        self.tiles = (a, b)

    def set_split(self, enable):
        self.split = self.asked = bool(enable)

    def step(self, n, state=None):
        self.steps += n


@pytest.fixture
def tuner(monkeypatch):
    monkeypatch.setattr(A, "_arch", lambda torch: "gfx950")

    def timed(torch, fn, trials):
        fn()
        return 1.0
    monkeypatch.setattr(A, "_time", timed)


@pytest.mark.parametrize("entry", [None, OLD, dict(OLD, form=0)])
def test_series_solver_is_left_alone(tuner, tmp_path, entry):
    path = str(tmp_path / "tune.json")
    if entry:
        A.save_cache({KEY: entry}, path)
    sol = FakeSolver(series=True)
    for _ in range(2):
        assert A.tune_solver(sol, path=path) == (32, 32, False)
    assert sol.products == 1 and sol.tiles == (32, 32) and sol.split and sol.steps == 0
    # a dense model's entry of the same size stays for that model
    assert A.load_cache(path)[KEY]["form"] == (0 if entry and "form" in entry else 1)


def test_asked_split_does_not_keep_the_slower_form(tuner, tmp_path):
    sol = FakeSolver(series=True, asked=True)
    assert A.tune_solver(sol, path=str(tmp_path / "tune.json")) == (32, 32, False)
    assert sol.products == 1 and sol.steps == 0


@pytest.mark.parametrize("entry", [None, OLD, {"tiles": [64, 64], "split": False, "form": 1}])
def test_dense_solver_is_tuned_and_cached(tuner, tmp_path, entry):
    path = str(tmp_path / "tune.json")
    if entry:
        A.save_cache({KEY: entry}, path)
    sol = FakeSolver(series=False)
    best = A.tune_solver(sol, path=path)
    assert sol.steps > 0 and best[:2] in A.candidates("fp32", 512)
    assert A.load_cache(path)[KEY]["form"] == 0
    again = FakeSolver(series=False)
    assert A.tune_solver(again, path=path) == best and again.steps == 0
    assert again.tiles == best[:2] and again.split == best[2]


def test_batch_sizes_by_the_series_keep_their_tiles(tuner):
    class FakeBatch:
        torch = None

        def __init__(self, solvers):
            self.solvers, self.steps = solvers, 0

        def config(self, use_graph, largest_first):
            pass

        def step(self, n):
            self.steps += 1
    series, dense = FakeSolver(series=True), FakeSolver(series=False)
    dense.n = 64
    b = FakeBatch([series, dense])
    best, results = A.tune_batch(b)
    assert best[2][512] == (32, 32) == series.tiles
    assert len([k for k in results if k[0] == "tiles"]) == 8
    assert b.steps == 2 * (1 + 4 + 3)         # one time for the series' size, four for the dense one's
