"""bf16 with a hidden size that is a multiple of 8 but not of 32: the tuned loop with a last K step that ends inside its 32
elements (1, 2 or 3 chunks of 8 left, alone or after whole steps), with both tile edges, against the oracle and against the
general loop."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd import inputs as I              # noqa: E402
from paper_2511_17599_amd.runner import run_workload, session_for, to_device   # noqa: E402
from conftest import set_plan, tile_edges                             # noqa: E402
from test_gpu_parity import check_against_oracle, nerr    # noqa: E402


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def wl_of(N, d, V, ignore=0.1, **kw):
    return I.Workload(f"ragged_{N}_{d}_{V}", N, d, V, "bf16", "uniform", ignore_frac=ignore, seed=800 + N + d, **kw)


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("N,d,V", [(1, 8, 1), (255, 16, 257), (257, 24, 255), (600, 40, 700), (520, 104, 1030),
                                   (300, 200, 2100), (1030, 248, 513), (70, 520, 5000), (513, 1048, 600)])
def test_ragged_hidden_sizes(monkeypatch, N, d, V, tile):
    set_plan(monkeypatch, FLCE_TILE=tile)
    assert "loop=tuned" in B.flce_plan_describe(N, d, V, B.FLCE_DTYPE_BF16) and tile_edges(N, d, V) == (tile, tile)
    wl = wl_of(N, d, V)
    x = I.make_inputs(wl)
    got, _, _ = check_against_oracle(wl, x)
    s = got["session"]                                       # the forward that reads H where it lies
    lse = torch.empty_like(s.lse)
    assert B.flce_forward_static(s.H, s.W, s.y, N, d, V, s.ignore_index, s.red, s.dt, s.loss, lse, None, None,
                                 s.stream()) == B.FLCE_OK
    assert torch.equal(lse, s.lse) or (lse - s.lse).abs().max() <= 2e-6 * s.lse.abs().max()
    set_plan(monkeypatch, FLCE_GENERIC=1)
    g = run_workload(wl, x)
    assert np.abs(g["lse"] - got["lse"]).max() <= 4e-6 * np.abs(g["lse"]).max()
    if got["n_valid"]:
        assert nerr(got["dH"], g["dH"]) < 1e-2 and nerr(got["dW"], g["dW"]) < 1e-2


@pytest.mark.parametrize("tile", [128, 256])
def test_ragged_hidden_chunks(monkeypatch, tile):
    """Chunks with running sums, K slices and the per-row gradients at a ragged hidden size."""
    set_plan(monkeypatch, FLCE_VC_TILES=2, FLCE_NC_TILES=2, FLCE_SPLITK_DH=2, FLCE_SPLITK_DW=2, FLCE_WINDOWS=3,
             FLCE_TILE=tile)
    wl = wl_of(900, 280, 1800)
    assert tile_edges(wl.N, wl.d, wl.V) == (tile, tile)
    x = I.make_inputs(wl)
    check_against_oracle(wl, x)
    from oracle import flce_oracle as O
    gr = np.linspace(-1, 2, wl.N).astype(np.float32)
    s = session_for(wl, x)
    rows = torch.empty(wl.N, device=s.device)
    assert s.forward_rows(rows, 0.1) == B.FLCE_OK and s.backward_rows(to_device(gr, s.device), 0.1) == B.FLCE_OK
    b = O.backward_per_row(I.to_f64(x["H"]), I.to_f64(x["W"]), x["y"], gr.astype(np.float64), wl.ignore_index, 0.1)
    assert nerr(s.dH.double().cpu().numpy(), b["dH"]) <= 2e-2 and nerr(s.dW.double().cpu().numpy(), b["dW"]) <= 2e-2


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("static", [False, True])
def test_what_lies_behind_a_row_does_not_reach_it(monkeypatch, static, tile):
    """The element after a row's last is the next row's first: an infinity there must not turn this row's logit into NaN."""
    N, d, V = 300, 72, 512
    set_plan(monkeypatch, FLCE_TILE=tile)
    assert tile_edges(N, d, V) == (tile, tile)
    wl = wl_of(N, d, V, ignore=0.0)
    x = I.make_inputs(wl)
    H, W = torch.from_numpy(x["H"].view(np.int16)).view(torch.bfloat16).clone(), torch.from_numpy(x["W"].view(np.int16)).view(torch.bfloat16).clone()
    H = H.abs() + 0.5                                        # every product with the infinities below is -inf, none is NaN
    W[1::2] = float("-inf")                                  # every other vocabulary entry gets probability 0
    x["y"] = (x["y"] // 2) * 2
    s = session_for(wl, dict(H=H.cuda(), W=W.cuda(), y=x["y"]))
    if static:
        assert B.flce_forward_static(s.H, s.W, s.y, N, d, V, s.ignore_index, s.red, s.dt, s.loss, s.lse, None, None,
                                     s.stream()) == B.FLCE_OK
    else:
        assert s.forward() == B.FLCE_OK
    want = torch.logsumexp(H.double() @ W[0::2].double().t(), 1)
    assert torch.isfinite(s.lse).all() and (s.lse.cpu().double() - want).abs().max() <= 1e-5 * want.abs().max()
