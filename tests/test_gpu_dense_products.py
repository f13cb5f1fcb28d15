"""The dense products' kernels (tile bodies, splits, whole panels, direct loads,
the folded epilogues, the trace in the first product, the batched tiles, the
dense adjoint and pure step) under the tests that were written for them.  Sparse
models step by the series by default, so those tests run them no longer by
themselves; here the same tests run with every solver on form 0."""
import inspect
import itertools

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2403_07042_amd")
from paper_2403_07042_amd import api  # noqa: E402

import test_gpu_adjoint as adjoint  # noqa: E402
import test_gpu_autotune as autotune  # noqa: E402
import test_gpu_batch as batch  # noqa: E402
import test_gpu_direct_loads as loads  # noqa: E402
import test_gpu_general as general  # noqa: E402
import test_gpu_general_operators as operators  # noqa: E402
import test_gpu_graph as graph  # noqa: E402
import test_gpu_pure as pure  # noqa: E402
import test_gpu_resume as resume  # noqa: E402
import test_gpu_selection as selection  # noqa: E402
import test_gpu_step as step  # noqa: E402

TESTS = [
    step.test_fused_trace_scalars_across_calls, step.test_folded_trace_in_first_product_scalars,
    step.test_whole_panel_folded_trace_scalars, step.test_bf16x3_wide_first_product_bitwise,
    step.test_tch_n144, step.test_lattice_small_with_sink, step.test_lattice_2048_closed_form,
    step.test_lattice_2048_fp64_against_oracle_steps, step.test_tail_split_of_the_lower_product,
    step.test_tail_split_in_two_reduce_groups, step.test_folded_steps_match_unfolded,
    step.test_tch_chain3_n1728_against_oracle, step.test_leaking_lattice_folded_against_oracle,
    step.test_profile_sampling_stride, step.test_small_launch_split,
    loads.test_tile_bodies_bitwise_equal, loads.test_whole_panel_body_bitwise_equal,
    loads.test_adjoint_bitwise_equal,
    autotune.test_tile_choice_is_bitwise_neutral_and_tuner_picks_valid, autotune.test_batch_tuner,
    batch.test_batch_equals_solo_bitwise, batch.test_batch_per_instance_tiles_bitwise,
    batch.test_graph_replays_with_eager_work_between, batch.test_batch_against_oracle,
    batch.test_full_sweep_256_instances,
    graph.test_graph_replays_match_eager,
    general.test_exported_model_is_bitwise_the_structured_one, general.test_hydrogen_bond_64_against_oracle,
    operators.test_tch_collective_decay_n144_against_oracle,
    operators.test_tch_collective_decay_n1024_against_oracle,
    operators.test_batch_of_collective_contexts_equals_solo,
    adjoint.test_adjoint_matches_tangent_linear, adjoint.test_checkpoint_interval_does_not_change_the_gradient,
    adjoint.test_lattice_2048_adjoint_against_closed_form_gradient,
    resume.test_resume_from_host_checkpoint_is_bitwise, resume.test_split_calls_equal_one_call,
    selection.test_eps_zero_changes_nothing,
    pure.test_pure_matches_oracle, pure.test_pure_photon_plane_4131_against_closed_form,
    pure.test_pure_equals_density_path_on_gpu, pure.test_vectors_independent_and_runs_split_bitwise,
]


def calls(test):
    """(test, arguments) for every combination of the test's own parameters."""
    axes = []
    for mark in getattr(test, "pytestmark", []):
        if mark.name == "parametrize":
            names = [n.strip() for n in mark.args[0].split(",")]
            axes.append([dict(zip(names, v if len(names) > 1 else (v,))) for v in mark.args[1]])
    for combo in itertools.product(*axes):
        kw = {k: v for part in combo for k, v in part.items()}
        ident = "-".join([test.__name__[5:]] + [getattr(v, "__name__", str(v)) for v in kw.values()])
        yield pytest.param(test, kw, id=ident)


class DenseSolver(api.Solver):
    def __init__(self, *args, **kwargs):
        super().__init__(*args, **kwargs)
        self.set_products(0)
        assert self.products == 0


@pytest.mark.parametrize("test,kw", [c for t in TESTS for c in calls(t)])
def test_on_dense_products(test, kw, monkeypatch, tmp_path):
    monkeypatch.setattr(P, "Solver", DenseSolver)
    monkeypatch.setattr(api, "Solver", DenseSolver)
    have = {"tmp_path": tmp_path, "monkeypatch": monkeypatch}
    fixtures = {n: have[n] for n in inspect.signature(test).parameters if n not in kw}
    test(**kw, **fixtures)
