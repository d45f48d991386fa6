"""fp32 on 128-row tiles, whose products are taken from bf16 parts of the operands: the error against 64 bits stays that of fp32
sums, and values that have no such parts (infinities, values next to the largest) give what fp32 products give."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd.runner import Session           # noqa: E402
from conftest import tile_edges                           # noqa: E402


def _run(N, d, V, seed, change=None, reduction="mean"):
    g = torch.Generator(device="cuda").manual_seed(seed)
    H = torch.randn(N, d, device="cuda", generator=g)
    W = torch.randn(V, d, device="cuda", generator=g) * 0.05
    y = torch.randint(0, V // 2, (N,), device="cuda", generator=g)
    if change:
        change(H, W)
    assert tile_edges(N, d, V, "f32") == (128, 128)
    print(f"[case] f32 parts N={N} d={d} V={V} seed={seed}", flush=True)
    s = Session(N, d, V, "f32", reduction, -100, H, W, y)
    assert s.forward() == B.FLCE_OK and s.backward() == B.FLCE_OK
    z = H.double() @ W.double().t()
    lse = torch.logsumexp(z, 1)
    G = torch.exp(z - lse[:, None])
    G[torch.arange(N, device="cuda"), y] -= 1
    if reduction == "mean":
        G /= N
    return s, lse, G, H.double(), W.double()


def _rel(a, b):
    return ((a.double() - b).norm() / b.norm()).item()


@pytest.mark.parametrize("N,d,V", [(1300, 72, 3800), (1409, 1032, 3650), (1281, 8, 3713), (2100, 136, 2600)])
def test_error_against_64_bits(N, d, V):
    s, lse, G, H, W = _run(N, d, V, 40 + d)
    # a rounding to 32 bits is 3e-8 on average, sums of a thousand of them with random signs stay below 1e-6
    assert _rel(s.lse, lse) < 2e-7
    assert _rel(s.dH, G @ W) < 1e-6 and _rel(s.dW, G.t() @ H) < 1e-6


def test_masked_vocabulary_rows():
    """A column of ones in H and minus infinity in W: logits of minus infinity, probabilities of zero.  (Whole K steps of
    counted rows: a padding row's logits are 0 * inf.)"""
    def mask(H, W):
        H[:, 0] = 1.0
        W[2000:, 0] = float("-inf")
    s, lse, G, H, W = _run(1408, 72, 3800, 51, mask)
    assert torch.isfinite(s.lse).all() and _rel(s.lse, lse) < 2e-7
    assert _rel(s.dH[:, 1:], (G @ W[:, 1:])) < 1e-6       # column 0 is 0 * inf
    assert _rel(s.dW, G.t() @ H) < 1e-6 and not s.dW[2000:].any()


def test_values_next_to_the_largest():
    """3.4e38 rounds past the largest bf16 number."""
    def big(H, W):
        H[:, 3] *= 1e-38
        W[:, 3] = 3.4e38 * torch.sign(W[:, 3])
    s, lse, G, H, W = _run(1300, 72, 3800, 52, big)
    assert _rel(s.lse, lse) < 2e-7
    keep = [c for c in range(72) if c != 3]
    assert _rel(s.dW[:, keep], (G.t() @ H)[:, keep]) < 1e-6
    assert _rel(s.dH[:, keep], (G @ W)[:, keep]) < 1e-6


@pytest.mark.parametrize("factor", [1e-30, 2.0 ** -112, 1e-36])
def test_small_values(factor):
    """Columns whose parts would lie below the smallest normal bf16 number.  (Summed loss: the gradients of the last ones are
    mostly normal numbers still, half a step of 2^-149 on 1e-38 is 7e-8.)"""
    def small(H, W):
        W[:, 5] *= factor
        H[:, 6] *= factor
    s, lse, G, H, W = _run(1300, 72, 3800, 53, small, reduction="sum")
    assert _rel(s.dH[:, 5].double() / factor, (G @ W)[:, 5] / factor) < 2e-6
    assert _rel(s.dW[:, 6].double() / factor, (G.t() @ H)[:, 6] / factor) < 2e-6


@pytest.mark.parametrize("factor", [1e-30, 1e-34])
def test_small_upstream_gradients(factor):
    """One loss per row: G holds the rows' upstream gradients."""
    from paper_2511_17599_amd.torch_api import linear_cross_entropy
    g = torch.Generator(device="cuda").manual_seed(55)
    H = torch.randn(1300, 72, device="cuda", generator=g).requires_grad_()
    W = (torch.randn(3800, 72, device="cuda", generator=g) * 0.05).requires_grad_()
    y = torch.randint(0, 3800, (1300,), device="cuda", generator=g)
    print(f"[case] f32 row gradients of {factor}", flush=True)
    rows = linear_cross_entropy(H, W, y, reduction="none")
    one = torch.autograd.grad(rows, (H, W), torch.ones_like(rows), retain_graph=True)
    few = torch.autograd.grad(rows, (H, W), torch.full_like(rows, factor))
    for a, b in zip(few, one):
        assert _rel(a.double() / factor, b.double()) < 1e-6


def test_nan_stays_in_its_row():
    def nan(H, W):
        H[7, 9] = float("nan")
    s, lse, *_ = _run(1300, 72, 3800, 54, nan)
    other = torch.arange(1300, device="cuda") != 7
    assert not torch.isfinite(s.lse[7]) and _rel(s.lse[other], lse[other]) < 2e-7


def test_logits_are_off_to_both_sides():
    """The bf16 instruction's sums round down: 0.33 of sqrt(d) 2^-24 on average at d = 512, against an error of 2.8 a logit, the same for
    all logits and therefore not averaged out in a log-sum-exp.  Half of the vocabulary is added up negated: over both
    halves nothing stays.  (Every row has one logit that counts, in one half or the other; the others lie 10^4 below.)"""
    N, d, V = 128 * 320, 512, 64
    g = torch.Generator(device="cuda").manual_seed(56)
    H = torch.randn(N, d, device="cuda", generator=g)
    W = torch.randn(V, d, device="cuda", generator=g)
    first = torch.arange(N, device="cuda") % 2 == 0
    H[:, 0], H[:, 1], H[:, 2] = 1.0, first.float(), 1.0 - first.float()
    W[:, :3] = 0.0
    W[:, 0] = -1e4
    W[10, 0] = W[40, 0] = 0.0
    W[40, 1], W[10, 2] = -1e4, -1e4
    y = torch.full((N,), 10, dtype=torch.int64, device="cuda")
    assert tile_edges(N, d, V, "f32") == (128, 128)
    print("[case] f32 parts, sign of the error", flush=True)
    s = Session(N, d, V, "f32", "mean", -100, H, W, y)
    assert s.forward() == B.FLCE_OK
    z = torch.where(first, H.double() @ W[10].double(), H.double() @ W[40].double())
    e = (s.lse.double() - z) / (d ** 0.5 * 2.0 ** -24)
    print(f"       {e[first].mean().item():+.3f} {e[~first].mean().item():+.3f} rms {e.pow(2).mean().sqrt().item():.3f}", flush=True)
    # the mean of N such errors is off by 2.8 / sqrt(N) = 0.014
    assert abs(e.mean().item()) < 0.07 and e.pow(2).mean().sqrt().item() < 4.0
