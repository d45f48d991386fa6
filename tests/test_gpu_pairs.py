"""Problems whose dW and dH tiles go out as one launch (pair=1 in the plan line), with K slices in neither, one or both of
them and with every tile edge; the compaction inside the row preparation up to 2048 rows and on its own beyond; forwards
with and without a pre-tiled copy of H."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd import inputs as I              # noqa: E402
from paper_2511_17599_amd.runner import session_for       # noqa: E402
from conftest import set_plan, tile_edges                 # noqa: E402
from test_gpu_parity import check_against_oracle          # noqa: E402


BF16 = [(300, 600, 500, 0.1), (700, 256, 4845, 0.3), (5000, 64, 700, 0.02), (2048, 64, 2000, 0.1), (2049, 64, 2000, 0.1),
        (1, 32, 300, 0.0), (1500, 72, 1500, 0.97), (300, 64, 500, 1.0)]
F32 = [(300, 600, 500, 0.1), (2048, 72, 600, 0.2), (2049, 72, 600, 0.2), (100, 264, 1500, 0.0)]


@pytest.mark.parametrize("dtype,tile,N,d,V,ignore", [("bf16", t, *c) for t in (128, 256) for c in BF16] +
                         [("f32", 64, *c) for c in F32])
def test_pair_launches(monkeypatch, dtype, tile, N, d, V, ignore):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if dtype == "bf16":
        set_plan(monkeypatch, FLCE_TILE=tile)
    assert tile_edges(N, d, V, dtype) == (tile, tile)
    dt = {"bf16": B.FLCE_DTYPE_BF16, "f32": B.FLCE_DTYPE_F32}[dtype]
    assert " pair=1 " in B.flce_plan_describe(N, d, V, dt)
    wl = I.Workload(f"pair_{N}_{d}_{V}", N, d, V, dtype, "zipf", zipf_s=1.1, ignore_frac=ignore, seed=1000 + N + d)
    check_against_oracle(wl, I.make_inputs(wl), grad_loss=0.5)


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("N,d,V,copy", [(600, 384, 240000, 1), (600, 384, 200000, 0), (600, 392, 240000, 1), (585, 384, 20040, 0)])
def test_forward_copy_of_h_where_it_pays(monkeypatch, N, d, V, copy, tile):
    """Shapes on either side of the rule (4.6e10 + 9300 N d products), one with a ragged hidden size: the plan line says whether
    the forward makes the copy, and the log-sum-exps are those of a product in 64 bits."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    set_plan(monkeypatch, FLCE_TILE=tile)
    assert tile_edges(N, d, V) == (tile, tile)
    assert f" h_copy={copy}/1 " in B.flce_plan_describe(N, d, V, B.FLCE_DTYPE_BF16)
    g = torch.Generator(device="cuda").manual_seed(N + V)
    H = torch.randn(N, d, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, d, device="cuda", generator=g) * 0.05).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g)
    wl = I.Workload(f"copy_{N}_{d}_{V}_{tile}", N, d, V, "bf16", "uniform", seed=1)
    s = session_for(wl, dict(H=H, W=W, y=y))
    s.lse.fill_(float("nan"))
    assert s.forward() == B.FLCE_OK
    want, zt = torch.empty(N, dtype=torch.float64, device="cuda"), torch.empty(N, dtype=torch.float64, device="cuda")
    W64 = W.double()
    for i in range(0, N, 200):
        z = H[i:i + 200].double() @ W64.t()
        want[i:i + 200] = torch.logsumexp(z, 1)
        zt[i:i + 200] = z.gather(1, y[i:i + 200, None])[:, 0]
    # fp32 logits (|z| < 10) and sums of exponentials: about 1e-6 of lse ~ 13
    assert (s.lse.double() - want).abs().max() <= 2e-6 * want.abs().max()
    assert abs(s.loss.item() - (want - zt).mean().item()) <= 2e-6 * want.abs().max()
