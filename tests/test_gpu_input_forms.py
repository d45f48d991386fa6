"""GPU: whatever form the operands come in (more dimensions, strides, a narrower type of targets), the autograd front end
gives the bits that it gives for plain two-dimensional operands and int64 targets, and hands back the caller's shapes."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

FORMS = {
    "three_dims": lambda H, y: (H.reshape(6, 11, -1), y.reshape(6, 11)),
    "columns": lambda H, y: (H.t().contiguous().t(), y),
    "strided_targets": lambda H, y: (H, torch.stack([y, y], 1)[:, 0]),
    "int32_targets": lambda H, y: (H, y.int()),
    "targets_of_two_dims": lambda H, y: (H, y.reshape(11, 6)),
    "row_slice": lambda H, y: (torch.cat([H, H], 1)[:, :H.shape[1]], y),
}


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("reduction", ["mean", "none"])
def test_same_bits(form, reduction):
    from paper_2511_17599_amd.torch_api import linear_cross_entropy

    g = torch.Generator().manual_seed(5)
    H0 = torch.randn(66, 40, generator=g).bfloat16().cuda()
    W0 = torch.randn(130, 40, generator=g).bfloat16().cuda()
    y0 = torch.randint(0, 130, (66,), generator=g).cuda()
    y0[7] = -100

    def run(H, y):
        H, W = H.detach().requires_grad_(), W0.clone().requires_grad_()
        loss = linear_cross_entropy(H, W, y, reduction=reduction)
        loss.backward(torch.ones_like(loss))
        assert loss.shape == (() if reduction == "mean" else y.shape) and loss.dtype == torch.float32
        assert H.grad.shape == H.shape and W.grad.shape == W.shape
        return loss.detach().reshape(-1), H.grad.reshape(66, 40), W.grad

    want = run(H0, y0)
    got = run(*FORMS[form](H0, y0))
    for a, b in zip(got, want):
        assert torch.equal(a, b)
