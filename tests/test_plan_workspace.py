"""Host-only: what the launch plan adds to the workspace for speed is bounded, at the sizes where it would grow largest."""
import pytest

from paper_2511_17599_amd import binding as B
from conftest import set_plan

CAP = 512 << 20
BF16 = B.FLCE_DTYPE_BF16


@pytest.mark.parametrize("N,d,V", [(103047, 7824, 22916), (131072, 4104, 128256), (300000, 1000, 50000)])
def test_ragged_hidden_sizes_run_the_forward_in_words_per_row(N, d, V):
    """d % 32 != 0: partials of at most 8 rounds of 256 rows, column sums, a word per row; the copy of H past 512 MiB is not
    made.  Below that size it is."""
    items = 8 * 256 * 256 + 4 * (N + 256)
    words = 12 * items + 4 * (-(-V // 1024) * d + d + N) + 16 * -(-N // 256) + 4096
    assert B.flce_workspace_bytes(N, d, V, BF16, 0) <= words
    n = CAP // 2 // (2 * d)
    assert B.flce_workspace_bytes(n, d, V, BF16, 0) >= n * d * 2


@pytest.mark.parametrize("N,d,V,dt", [(6232, 8040, 106136, BF16), (32116, 2064, 23705, BF16), (3830, 4880, 136110, B.FLCE_DTYPE_F32),
                                      (1500, 16384, 60000, BF16), (2, 1024, 159101, BF16), (2682, 6080, 72653, BF16)])
def test_k_slices_take_a_bounded_share_of_the_workspace(N, d, V, dt):
    f = dict(kv.split("=") for kv in B.flce_plan_describe(N, d, V, dt).split()[2:])
    rows = {k: 256 * int(f[k].split("x")[1]) for k in ("row_chunks", "vocab_chunks")}
    print(f)
    for slices, chunk in (("splitk_dH", "row_chunks"), ("splitk_dW", "vocab_chunks")):
        n = int(f[slices])
        assert n <= 64 and (n == 1 or n * rows[chunk] * d * 4 <= CAP)


@pytest.mark.parametrize("slices", [1, 17, 64])
def test_every_number_of_slices_the_plan_takes_can_be_asked_for(monkeypatch, slices):
    set_plan(monkeypatch, FLCE_SPLITK_DH=slices, FLCE_SPLITK_DW=slices)
    line = B.flce_plan_describe(20000, 64, 20000, BF16)
    assert f"splitk_dH={slices} splitk_dW={slices} " in line
