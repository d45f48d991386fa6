"""The upstream gradient as a device word: the same bits as the host value, for both reductions, both types and every way the
contractions write out (one chunk, several with running sums, K slices); and through autograd, on another stream."""
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


def test_autograd_on_a_side_stream():
    """Forward on a side stream, backward called from the default one, the gradient made there: repeated with freed memory
    reused in between."""
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
        junk = [torch.full((64,), float("nan"), device="cuda") for _ in range(64)]
        torch.cuda.synchronize()
        del junk
        if ref is None:
            ref = H.grad, W.grad
        assert torch.equal(H.grad, ref[0]) and torch.equal(W.grad, ref[1])
