"""Contraction launches cut into more K slices than a batch of loads of the slice sum (default plan: few output tiles over
a long K extent), with the last batch full and ragged."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd import inputs as I              # noqa: E402
from test_gpu_parity import check_against_oracle          # noqa: E402


@pytest.mark.parametrize("N,d,V,key,least", [
    (200, 64, 20000, "splitk_dH", 17),                     # one output tile, 79 K tiles of the vocabulary
    (5000, 64, 300, "splitk_dW", 9),                       # two output tiles, 20 K tiles of tokens
    (300, 520, 7000, "splitk_dH", 9),                      # six output tiles (d in three), rows beyond the first tile
])
def test_many_k_slices(N, d, V, key, least):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    plan = dict(kv.split("=") for kv in B.flce_plan_describe(N, d, V, B.FLCE_DTYPE_BF16).split()[2:])
    print(plan, flush=True)
    assert int(plan[key]) >= least
    wl = I.Workload(f"slices_{N}_{d}_{V}", N, d, V, "bf16", "uniform", ignore_frac=0.1, seed=600 + d)
    check_against_oracle(wl, I.make_inputs(wl))
