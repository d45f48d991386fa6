"""Problems whose dW and dH tiles go out as one launch (pair=1 in the plan line), with K slices in neither, one or both of
them; the compaction inside the row preparation up to 2048 rows and on its own beyond; forwards with and without a
pre-tiled copy of H."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd import inputs as I              # noqa: E402
from test_gpu_parity import check_against_oracle          # noqa: E402


@pytest.mark.parametrize("N,d,V,dtype,ignore", [
    (300, 600, 500, "bf16", 0.1), (700, 256, 4845, "bf16", 0.3), (5000, 64, 700, "bf16", 0.02), (2048, 64, 2000, "bf16", 0.1),
    (2049, 64, 2000, "bf16", 0.1), (1, 32, 300, "bf16", 0.0), (1500, 72, 1500, "bf16", 0.97), (300, 64, 500, "bf16", 1.0),
    (300, 600, 500, "f32", 0.1), (2048, 72, 600, "f32", 0.2), (2049, 72, 600, "f32", 0.2), (100, 264, 1500, "f32", 0.0),
])
def test_pair_launches(N, d, V, dtype, ignore):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt = {"bf16": B.FLCE_DTYPE_BF16, "f32": B.FLCE_DTYPE_F32}[dtype]
    plan = B.flce_plan_describe(N, d, V, dt)
    print(plan, flush=True)
    assert "pair=1" in plan
    wl = I.Workload(f"pair_{N}_{d}_{V}", N, d, V, dtype, "zipf", zipf_s=1.1, ignore_frac=ignore, seed=1000 + N + d)
    check_against_oracle(wl, I.make_inputs(wl), grad_loss=0.5)


def test_forward_copy_of_h_where_it_pays():
    """The same shape family on either side of the rule, results checked by the per-row sums of the other cases' kind."""
    assert B.flce_workspace_bytes(8192, 4096, 128256, B.FLCE_DTYPE_BF16, 0) > 8192 * 4096 * 2
    assert B.flce_workspace_bytes(1024, 512, 20000, B.FLCE_DTYPE_BF16, 0) < 1024 * 512 * 2 + (1 << 20)
