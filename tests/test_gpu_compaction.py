"""The backward's compaction of the counted rows at the edges of its ranges (16 wavefronts, groups of 64 rows, 8 groups at a
time): rows that count in order, the rest of the map -1, seen through dH of a problem small in everything else."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import inputs as I              # noqa: E402
from test_gpu_parity import check_against_oracle          # noqa: E402


@pytest.mark.parametrize("N", [1, 63, 64, 65, 1023, 1024, 1025, 8191, 8193, 17000])
@pytest.mark.parametrize("which", ["most", "few", "head", "tail"])
def test_counted_rows(N, which):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = I.Workload(f"compact_{N}_{which}", N, 32, 40, "bf16", "uniform", seed=900 + N)
    x = I.make_inputs(wl)
    r = np.random.default_rng(N)
    dead = {"most": r.random(N) < 0.1, "few": r.random(N) < 0.97, "head": np.arange(N) >= N // 3,
            "tail": np.arange(N) < N // 2}[which]
    x["y"][dead] = wl.ignore_index
    check_against_oracle(wl, x)
