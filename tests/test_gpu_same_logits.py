"""GPU: the backward's recomputed logit is the forward's.  In a confident row exp(logit - lse) - 1 is zero but for the rounding of
the exponent; a logit that the two directions add up differently shows there with its own rounding error, tens of times larger."""
import math

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd.runner import Session           # noqa: E402
from conftest import tile_edges                           # noqa: E402

IGNORE = -100


def confident(N, d, V, dtype, logit, seed):
    """Rows whose target logit is about `logit` and whose other logits are below a third of it."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn(V, d, device="cuda", generator=g)
    y = torch.randint(0, V, (N,), device="cuda", generator=g)
    H = W[y] * (logit / (W[y] ** 2).sum(1, keepdim=True))
    t = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    return H.to(t), W.to(t), y


def check(s, y, logit):
    rows = y != IGNORE
    Wy = s.W[y[rows]].double()
    # dH of a confident row is its one large g, times W's target row; the others' g are below exp(-2/3 logit)
    g = (s.dH[rows].double() * Wy).sum(1) / (Wy ** 2).sum(1) * int(rows.sum())
    # the exponent is z log2(e) - (lse log2(e) rounded), half a unit in the last place (bf16 logits are off by at most 1 %)
    bound = math.log(2) * 2.0 ** (math.floor(math.log2(1.02 * logit * math.log2(math.e))) - 24) + 3e-7
    print(f"       largest g {g.abs().max().item():.2e}, bound {bound:.2e}", flush=True)
    assert g.abs().max().item() <= 1.02 * bound


@pytest.mark.parametrize("logit", [40.0, 165.0])
@pytest.mark.parametrize("dtype,edges,N,d,V", [
    ("f32", (64, 64), 250, 520, 4100), ("f32", (64, 64), 1024, 512, 4096), ("f32", (64, 64), 601, 512, 6200),
    ("f32", (128, 128), 1300, 512, 4000), ("bf16", (128, 128), 268, 512, 1029), ("bf16", (256, 128), 919, 256, 8257),
    ("bf16", (128, 256), 270, 672, 11116), ("bf16", (256, 256), 2060, 1032, 20011)])
def test_confident_rows(dtype, edges, N, d, V, logit):
    H, W, y = confident(N, d, V, dtype, logit, 60 + d)
    y[5::9] = IGNORE
    assert tile_edges(N, d, V, dtype) == edges
    print(f"[case] confident {dtype} N={N} d={d} V={V} logit={logit}", flush=True)
    s = Session(N, d, V, dtype, "mean", IGNORE, H, W, y)
    assert s.forward() == B.FLCE_OK and s.backward() == B.FLCE_OK
    check(s, y, logit)


@pytest.mark.parametrize("logit", [40.0, 165.0])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 1e30])
def test_confident_rows_beside_rows_left_out(value, logit):
    """fp32 with bf16 parts: ignored rows hold values that have none, so the forward computes their tiles both ways; the backward
    leaves those rows out and has tiles without them."""
    N, d, V = 1300, 512, 4000
    H, W, y = confident(N, d, V, "f32", logit, 71)
    H[3::70] = value
    y[3::70] = IGNORE
    assert tile_edges(N, d, V, "f32") == (128, 128)
    print(f"[case] confident beside {value} logit={logit}", flush=True)
    s = Session(N, d, V, "f32", "mean", IGNORE, H, W, y)
    assert s.forward() == B.FLCE_OK and s.backward() == B.FLCE_OK
    check(s, y, logit)
    assert not s.dH[3::70].any()
