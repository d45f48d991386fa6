"""Contractions whose K extent ends inside a tile: counted rows and vocabulary one K step (32) and one element to either side of
a multiple of 32 and of 256, with both tile edges of either type, K whole, cut in 5 slices (some of them empty) and as
the plan has it (dW and dH in one launch)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import inputs as I              # noqa: E402
from conftest import set_plan, tile_edges                             # noqa: E402
from test_gpu_parity import check_against_oracle          # noqa: E402


@pytest.mark.parametrize("dtype,tile,N,d,V", [("bf16", 256, 1300, 264, 2100), ("bf16", 128, 700, 64, 1000),
                                              ("f32", 64, 700, 64, 1000), ("f32", 128, 1300, 72, 4000)])
@pytest.mark.parametrize("counted,over", [(1, 0), (31, 1), (32, 31), (33, 32), (256, 33), (257, 255), (289, 256)])
@pytest.mark.parametrize("slices", [None, 1, 5])
def test_k_ends(monkeypatch, dtype, tile, N, d, V, counted, over, slices):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if slices:
        set_plan(monkeypatch, FLCE_SPLITK_DH=slices, FLCE_SPLITK_DW=slices)
    if dtype == "bf16":
        set_plan(monkeypatch, FLCE_TILE=tile)
    V = V // 256 * 256 + over
    assert tile_edges(N, d, V, dtype) == (tile, tile)
    wl = I.Workload(f"kends_{N}_{counted}_{over}", N, d, V, dtype, "uniform", seed=1300 + counted)
    x = I.make_inputs(wl)
    x["y"][counted:] = wl.ignore_index
    check_against_oracle(wl, x)
