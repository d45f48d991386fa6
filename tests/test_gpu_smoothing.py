"""The mean logit of label smoothing (column sums of W, one dot product per row) at the edges of its blocks: 1024-row
chunks of W taken 256 rows at a time, 16 lanes of 16 bytes across the hidden size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import flce_oracle as O                       # noqa: E402
from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd import inputs as I              # noqa: E402
from paper_2511_17599_amd.runner import session_for       # noqa: E402


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,d,N", [(1, 8, 1), (15, 64, 5), (257, 136, 6), (1024, 128, 7), (1279, 136, 9), (3000, 1048, 4)])
def test_mean_logit(dtype, V, d, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = I.Workload(f"smooth_{dtype}_{V}_{d}", N, d, V, dtype, "uniform", seed=400 + V + d, w_std=1.0)
    x = I.make_inputs(wl)
    print(f"[case] {wl.name}", flush=True)
    s = session_for(wl, x)
    rows = torch.empty(N, dtype=torch.float32, device=s.device)
    assert s.forward_rows(rows, 0.9) == B.FLCE_OK            # nine tenths of the loss is lse - mean logit
    f = O.forward_per_row(I.to_f64(x["H"]), I.to_f64(x["W"]), x["y"], wl.ignore_index, 0.9)
    # fp32 sums: logits of standard deviation sqrt(d) <= 33, the mean of V of them and lse each to about 1e-6 of that
    assert np.abs(rows.double().cpu().numpy() - f["loss_rows"]).max() <= 1e-5 * max(np.sqrt(d), np.abs(f["loss_rows"]).max())
