"""The parity cases of small problems on 256 x 256 tiles: the rule for the tile edge gives nearly all of them 128 x 128 ones, so
the chunked and sliced forms, the per-row gradients, the vocabulary slices and the degenerate extents of the large tiles are
asked for here."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import test_gpu_parity as P                               # noqa: E402
from paper_2511_17599_amd import inputs as I              # noqa: E402
from conftest import set_plan, tile_edges                 # noqa: E402


@pytest.fixture(autouse=True)
def _large_tiles(monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    set_plan(monkeypatch, FLCE_TILE=256)


def cases_of(test):
    """The argument lists of a parametrised test."""
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize" and m.args[0] != "dtype,generic")


@pytest.mark.parametrize("wl", [w for w in cases_of(P.test_ragged_and_small_shapes) if w.dtype == "bf16"], ids=lambda w: w.name)
def test_ragged_and_small_shapes(wl):
    assert tile_edges(wl.N, wl.d, wl.V) == (256, 256)
    P.check_against_oracle(wl, I.make_inputs(wl), grad_loss=-0.75)


@pytest.mark.parametrize("windows,vc,nc", cases_of(P.test_chunk_and_window_splits))
def test_chunk_and_window_splits(monkeypatch, windows, vc, nc):
    P.test_chunk_and_window_splits(monkeypatch, "bf16", 0, windows, vc, nc)
    assert tile_edges(700, 160, 1500) == (256, 256)


@pytest.mark.parametrize("sdh,sdw,vc,nc", cases_of(P.test_split_k_contractions))
def test_split_k_contractions(monkeypatch, sdh, sdw, vc, nc):
    P.test_split_k_contractions(monkeypatch, "bf16", 0, sdh, sdw, vc, nc)
    assert tile_edges(1100, 288, 1800) == (256, 256)


@pytest.mark.parametrize("d", cases_of(P.test_tuned_loop_short_and_odd_k))
def test_short_and_odd_k(d):
    P.test_tuned_loop_short_and_odd_k(d)


@pytest.mark.parametrize("eps", [0.0, 0.1])
@pytest.mark.parametrize("knobs", [{}, {"FLCE_SPLITK_DH": 3, "FLCE_SPLITK_DW": 2}], ids=["plain", "slices"])
def test_per_row_losses_and_gradients(monkeypatch, eps, knobs):
    set_plan(monkeypatch, **knobs)
    P.test_per_row_losses_and_gradients(monkeypatch, "bf16", eps, 0)
    assert tile_edges(900, 160, 1700) == (256, 256)


def test_vocabulary_slices():
    P.test_vocabulary_slices_merge_to_the_whole("bf16", "mean")


def test_partial_gradients():
    P.test_partial_gradients_then_scaling("bf16", "sum", -0.5)


def test_no_row_counts():
    P.test_all_rows_ignored()


@pytest.mark.parametrize("case", [c for c in P._random_cases(24, 2024) if c["wl"].dtype == "bf16"], ids=lambda c: c["wl"].name)
def test_seeded_random_shapes_and_plans(monkeypatch, case):
    P.test_seeded_random_shapes_and_plans(monkeypatch, case)
    assert tile_edges(case["wl"].N, case["wl"].d, case["wl"].V) == (256, 256)
