"""The tuned bf16 loop with 128 x 128 tiles (problems with few 256-row tiles, and short hidden sizes), at the edges of its
tiles: one row or column more or less than a tile, halves of the 256-row blocks the operands are packed in, hidden sizes
that end inside a K step or inside a half of the 256-column blocks, one K step; chunks, K slices and per-row gradients."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import flce_oracle as O                       # noqa: E402
from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd import inputs as I              # noqa: E402
from paper_2511_17599_amd.runner import session_for, to_device   # noqa: E402
from conftest import set_plan                             # noqa: E402
from test_gpu_parity import check_against_oracle, nerr    # noqa: E402


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def wl_of(N, d, V, ignore=0.1, **kw):
    return I.Workload(f"small_{N}_{d}_{V}", N, d, V, "bf16", "zipf", zipf_s=1.1, ignore_frac=ignore, seed=1100 + N + d, **kw)


@pytest.mark.parametrize("N,d,V,ignore", [
    (127, 32, 129, 0.0), (128, 64, 128, 0.1), (129, 96, 127, 0.1), (1, 256, 2000, 0.0), (257, 128, 383, 0.5),
    (385, 416, 385, 0.02), (130, 1032, 700, 0.1), (640, 40, 640, 0.3), (300, 2080, 520, 0.1), (2200, 136, 3000, 0.1),
    (511, 8, 257, 0.0),
])
def test_small_tiles(N, d, V, ignore):
    plan = B.flce_plan_describe(N, d, V, B.FLCE_DTYPE_BF16)
    print(plan, flush=True)
    assert "tiles=128/128" in plan
    wl = wl_of(N, d, V, ignore)
    x = I.make_inputs(wl)
    got, f, _ = check_against_oracle(wl, x, grad_loss=2.0)
    s = got["session"]                                       # the forward that reads H where it lies, fewer windows
    lse = torch.empty_like(s.lse)
    assert B.flce_forward_static(s.H, s.W, s.y, N, d, V, s.ignore_index, s.red, s.dt, s.loss, lse, None, None,
                                 s.stream()) == B.FLCE_OK
    assert np.abs(lse.double().cpu().numpy() - f["lse"]).max() <= 2e-6 * np.abs(f["lse"]).max()


@pytest.mark.parametrize("sdh,sdw", [(1, 1), (3, 2)])
def test_small_tiles_chunks_slices_and_rows(monkeypatch, sdh, sdw):
    set_plan(monkeypatch, FLCE_VC_TILES=2, FLCE_NC_TILES=1, FLCE_SPLITK_DH=sdh, FLCE_SPLITK_DW=sdw, FLCE_WINDOWS=3)
    wl = wl_of(700, 200, 1100)
    assert "tiles=128/128" in B.flce_plan_describe(wl.N, wl.d, wl.V, B.FLCE_DTYPE_BF16)
    x = I.make_inputs(wl)
    check_against_oracle(wl, x)
    gr = np.linspace(-1, 2, wl.N).astype(np.float32)
    s = session_for(wl, x)
    rows = torch.empty(wl.N, device=s.device)
    assert s.forward_rows(rows, 0.1) == B.FLCE_OK and s.backward_rows(to_device(gr, s.device), 0.1) == B.FLCE_OK
    b = O.backward_per_row(I.to_f64(x["H"]), I.to_f64(x["W"]), x["y"], gr.astype(np.float64), wl.ignore_index, 0.1)
    assert nerr(s.dH.double().cpu().numpy(), b["dH"]) <= 2e-2 and nerr(s.dW.double().cpu().numpy(), b["dW"]) <= 2e-2


def test_both_tile_sizes_agree_bit_for_bit_in_the_logits():
    """The K order of a logit does not depend on the tile, so the per-row target logits of a sliced call are the same bits
    as a 256-row plan's on the same rows (N and V large enough for that plan, the small call a part of it)."""
    big, small = wl_of(6000, 320, 20000, 0.0), (300, 700)
    x = I.make_inputs(big)
    assert "tiles=256" in B.flce_plan_describe(big.N, big.d, big.V, B.FLCE_DTYPE_BF16)
    H, W = to_device(x["H"], "cuda").view(torch.bfloat16), to_device(x["W"], "cuda").view(torch.bfloat16)
    y = torch.from_numpy(x["y"] % small[1]).cuda()
    st = torch.cuda.current_stream()

    def target_logits(N, V):
        assert ("tiles=128" if N == small[0] else "tiles=256") in B.flce_plan_describe(N, big.d, V, B.FLCE_DTYPE_BF16)
        m, a, z = (torch.empty(N, device="cuda") for _ in range(3))
        nb = B.flce_workspace_bytes(N, big.d, V, B.FLCE_DTYPE_BF16, 0)
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
        assert B.flce_forward_partial(H, W, y, N, big.d, V, 0, big.V, -100, B.FLCE_DTYPE_BF16, m, a, z, ws, nb, st) == B.FLCE_OK
        return z
    assert torch.equal(target_logits(big.N, big.V)[:small[0]], target_logits(*small))
