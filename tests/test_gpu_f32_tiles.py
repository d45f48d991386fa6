"""The fp32 main loop at the edges of its tiles: 64-row tiles below 320 tiles of 128 x 128 logits, 128-row tiles from there
on, in both directions; K tails shorter than a 16-byte chunk row, K longer than one block of partial sums, rows and columns past the end."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import inputs as I              # noqa: E402
from conftest import set_plan, tile_edges                             # noqa: E402
from test_gpu_parity import check_against_oracle          # noqa: E402


@pytest.mark.parametrize("tile,N,d,V,ignore", [
    (64, 64, 32, 64, 0.0), (64, 65, 8, 129, 0.1), (64, 63, 72, 257, 0.0), (64, 300, 1064, 200, 0.3), (64, 5, 256, 2100, 0.0),
    (128, 1300, 72, 3800, 0.1), (128, 1281, 8, 3713, 0.5), (128, 130, 200, 20500, 0.0), (128, 20500, 40, 130, 0.02),
    (128, 1409, 1032, 3650, 0.0),
    (64, 1401, 72, 3701, 0.1), (64, 1408, 40, 3712, 0.0), (128, 1280, 40, 4096, 0.0), (128, 1153, 72, 3969, 0.1),   # 319, 319, 320, 320
    (64, 1170, 96, 2500, 0.0), (64, 2000, 264, 2400, 0.1),
], ids=str)
def test_f32_tiles(tile, N, d, V, ignore):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert tile_edges(N, d, V, "f32") == (tile, tile)
    wl = I.Workload(f"f32_{N}_{d}_{V}", N, d, V, "f32", "uniform", ignore_frac=ignore, seed=700 + N + d)
    check_against_oracle(wl, I.make_inputs(wl))


@pytest.mark.parametrize("tile,N,V", [(64, 700, 1500), (64, 1100, 2900), (128, 1300, 3800)])
def test_f32_chunks_and_slices(monkeypatch, tile, N, V):
    """Several chunks with running sums and K slices, at both tile sizes."""
    set_plan(monkeypatch, FLCE_VC_TILES=3, FLCE_NC_TILES=2, FLCE_SPLITK_DH=3, FLCE_SPLITK_DW=2, FLCE_WINDOWS=3)
    assert tile_edges(N, 136, V, "f32") == (tile, tile)
    wl = I.Workload(f"f32_chunks_{N}_{V}", N, 136, V, "f32", "zipf", zipf_s=1.1, ignore_frac=0.1, seed=710)
    check_against_oracle(wl, I.make_inputs(wl), grad_loss=-0.5)
