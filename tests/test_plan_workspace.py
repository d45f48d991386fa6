"""Host-only: what the launch plan adds to the workspace for speed is bounded, at the sizes where it would grow largest."""
import pytest

from paper_2511_17599_amd import binding as B

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
