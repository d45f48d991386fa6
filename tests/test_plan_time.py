"""Host-only: a launch plan costs little beside the call it is made in (an autograd step makes four).  Timed in turn with a call
that is refused at its first check, the least of many batches each, so that neither a busy machine nor its clock decides."""
import time

from paper_2511_17599_amd import binding as B


def _least_seconds(calls, batches=80, n=60):
    best = [float("inf")] * len(calls)
    for _ in range(batches):
        for k, call in enumerate(calls):
            t = time.perf_counter()
            for _ in range(n):
                call()
            best[k] = min(best[k], time.perf_counter() - t)
    return best


def test_sizing_a_workspace():
    """At 1030 x 200 x 20011 a search over 63 numbers of slices of both contractions at both tile edges made this 4 refused calls
    long, in either direction; it is 1.2 (forward, which needs no such search) and 1.9 (backward)."""
    size = B.lib().flce_workspace_bytes
    N, d, V = 1030, 200, 20011
    assert size(N, d + 1, V, 0, 0) == 0
    refused, forward, backward = _least_seconds([lambda: size(N, d + 1, V, 0, 0), lambda: size(N, d, V, 0, 0),
                                                 lambda: size(N, d, V, 0, 1)])
    assert forward <= 2.4 * refused and backward <= 3.3 * refused, (refused, forward, backward)
