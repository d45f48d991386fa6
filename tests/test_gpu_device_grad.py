"""The upstream gradient as a device word: the same bits as the host value, for both reductions, both types and every way the
contractions write out (one chunk, several with running sums, K slices); through autograd, on another stream; and its
lifetime there."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd import inputs as I              # noqa: E402
from paper_2511_17599_amd.runner import session_for       # noqa: E402
from paper_2511_17599_amd.torch_api import linear_cross_entropy   # noqa: E402
from conftest import set_plan                             # noqa: E402


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("reduction,grad", [("mean", -0.75), ("sum", 0.3), ("mean", 0.0)])
@pytest.mark.parametrize("env", [{}, {"FLCE_VC_TILES": 2, "FLCE_NC_TILES": 2, "FLCE_SPLITK_DH": 2}], ids=["plain", "chunks"])
def test_device_gradient(monkeypatch, dtype, reduction, grad, env):
    set_plan(monkeypatch, **env)
    wl = I.Workload("devgrad", 700, 136, 1500, dtype, "uniform", ignore_frac=0.1, reduction=reduction, seed=1200)
    s = session_for(wl, I.make_inputs(wl), grad_loss=grad)
    assert s.forward() == B.FLCE_OK and s.backward() == B.FLCE_OK
    want = s.dH.clone(), s.dW.clone()
    s.dH.fill_(7.0), s.dW.fill_(7.0)
    g = torch.full((1,), grad, device=s.device)
    assert B.flce_backward_device_grad(s.H, s.W, s.y, s.lse, s.N, s.d, s.V, s.ignore_index, s.red, s.dt, g, s.dH, s.dW,
                                       s.ws, s.bwd_bytes, s.stream()) == B.FLCE_OK
    assert torch.equal(s.dH, want[0]) and torch.equal(s.dW, want[1])


class _FillDuringBackward(torch.autograd.Function):
    """Adds nothing; its backward, on the stream of its forward, takes small blocks of memory and fills them with NaN."""
    during = None

    @staticmethod
    def forward(ctx, x):
        return x.sum() * 0.0

    @staticmethod
    def backward(ctx, g):
        junk = [torch.full((1,), float("nan"), device="cuda") for _ in range(64)]
        _FillDuringBackward.during({t.data_ptr() for t in junk})
        return torch.zeros(1, device="cuda")


def test_the_gradient_outlives_the_kernels_that_read_it(monkeypatch):
    """The gradient word is made on the default stream and dropped by autograd as soon as the kernels that read it are enqueued.
    Where those run on a side stream that is busy for a while, the default stream takes and overwrites blocks of that size
    inside the same backward pass and before they run: the word's block must not be among them.  (On one stream it is.)"""
    H0 = torch.randn(300, 128, device="cuda").bfloat16()
    W0 = (torch.randn(2000, 128, device="cuda") * 0.02).bfloat16()
    y = torch.randint(0, 2000, (300,), device="cuda")
    x = torch.ones(1, device="cuda", requires_grad=True)
    A = torch.randn(4096, 4096, device="cuda")
    side = torch.cuda.Stream()
    call, enqueued, seen = B.flce_backward_device_grad, [], []

    def busy_then_call(*args):
        if torch.cuda.current_stream() == side:
            for _ in range(30):                              # tens of milliseconds
                A @ A
        rc = call(*args)
        enqueued.append((args[10].data_ptr(), torch.cuda.Event()))
        enqueued[-1][1].record()
        return rc

    def step(on_side):
        H, W = H0.clone().requires_grad_(), W0.clone().requires_grad_()
        fill = _FillDuringBackward.apply(x)                  # made before the loss: its backward runs after the loss's
        if on_side:
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                A @ A
                loss = linear_cross_entropy(H, W, y)
            torch.cuda.current_stream().wait_stream(side)
        else:
            loss = linear_cross_entropy(H, W, y)
        (loss * 0.5 + fill).backward()
        torch.cuda.synchronize()
        word, waiting, taken = seen.pop()
        return H.grad, W.grad, waiting, word in taken

    monkeypatch.setattr(B, "flce_backward_device_grad", busy_then_call)
    monkeypatch.setattr(_FillDuringBackward, "during",
                        lambda taken: seen.append((enqueued[-1][0], not enqueued[-1][1].query(), taken)))
    want = step(False)
    assert want[3]                                           # blocks of the word's size do come back at once
    for _ in range(3):
        dH, dW, waiting, reused = step(True)
        assert waiting and not reused                        # the fills were there while the kernels were not
        assert torch.equal(dH, want[0]) and torch.equal(dW, want[1])


def test_autograd_on_a_side_stream():
    """Forward on a side stream, backward called from the default one, the gradient made there."""
    H0 = torch.randn(300, 128, device="cuda").bfloat16()
    W0 = (torch.randn(2000, 128, device="cuda") * 0.02).bfloat16()
    y = torch.randint(0, 2000, (300,), device="cuda")
    ref = None
    side = torch.cuda.Stream()
    for rep in range(4):
        H, W = H0.clone().requires_grad_(), W0.clone().requires_grad_()
        if rep == 0:
            loss = linear_cross_entropy(H, W, y)
        else:
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                loss = linear_cross_entropy(H, W, y)
            torch.cuda.current_stream().wait_stream(side)
        (loss * 0.5).backward()
        torch.cuda.synchronize()
        if ref is None:
            ref = H.grad, W.grad
        assert torch.equal(H.grad, ref[0]) and torch.equal(W.grad, ref[1])
