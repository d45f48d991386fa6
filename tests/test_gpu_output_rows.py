"""The contractions' rounded output, written 32 rows x 128 columns (64 with 128-row tiles) per wavefront through LDS: hidden sizes that end inside a
wavefront's columns or leave one without any, vocabularies that end inside its rows, rows of dH scattered between ignored
ones, and no K slice or running sum in the way (one chunk each)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import inputs as I              # noqa: E402
from conftest import set_plan, tile_edges                             # noqa: E402
from test_gpu_parity import check_against_oracle          # noqa: E402


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("N,d,V", [(300, 32, 257), (129, 128, 700), (257, 160, 511), (90, 416, 97), (513, 288, 290)])
def test_rounded_output_rows(monkeypatch, N, d, V, tile):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    set_plan(monkeypatch, FLCE_SPLITK_DH=1, FLCE_SPLITK_DW=1, FLCE_TILE=tile)
    assert tile_edges(N, d, V) == (tile, tile)
    wl = I.Workload(f"rows_{N}_{d}_{V}", N, d, V, "bf16", "zipf", zipf_s=1.1, ignore_frac=0.3, seed=500 + d)
    check_against_oracle(wl, I.make_inputs(wl))
