"""Host-only: the word that the autograd front end hands to the library as the upstream gradient holds the gradient's value,
also where torch only marks it: a lazily negated view (the gradient of a complex expression), a zero tensor without storage,
another type.  The library's calls are replaced by one that reads that word as the kernels do, through its address."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

from paper_2511_17599_amd import torch_api as T           # noqa: E402


@pytest.fixture
def word_read(monkeypatch):
    read = []

    def backward(H, W, y, lse, N, d, V, ignore_index, reduction, dt, grad_loss, dH, dW, *rest):
        assert grad_loss.dtype == torch.float32
        address = grad_loss.data_ptr()
        read.append(ctypes.c_float.from_address(address).value if address else None)
        dH.zero_(), dW.zero_()
        return T.B.FLCE_OK

    monkeypatch.setattr(T, "_prepare", lambda H, W, y: (H, W, y))
    monkeypatch.setattr(T, "_stream", lambda device: 0)
    monkeypatch.setattr(T, "_workspace", lambda *a: (None, 0))
    monkeypatch.setattr(T.B, "flce_forward", lambda H, W, y, N, d, V, i, r, dt, loss, *rest: loss.fill_(2.0) and T.B.FLCE_OK)
    monkeypatch.setattr(T.B, "flce_backward_device_grad", backward)
    return read


def _loss():
    H, W = torch.zeros(4, 8, requires_grad=True), torch.zeros(3, 8, requires_grad=True)
    return T.linear_cross_entropy(H, W, torch.zeros(4, dtype=torch.int64))


@pytest.mark.parametrize("use,value", [
    (lambda loss: loss * 0.5, 0.5),
    (lambda loss: torch.view_as_real(torch.complex(torch.zeros(()), loss).conj().resolve_conj()).sum(), -1.0),
    (lambda loss: (torch.complex(loss, loss) * (1 + 3j)).imag, 4.0),
    (lambda loss: loss.double() * 0.25, 0.25),
], ids=["plain", "negated", "complex", "double"])
def test_through_autograd(word_read, use, value):
    use(_loss()).backward()
    assert word_read == [value]


@pytest.mark.parametrize("gradient,value", [
    (lambda: torch.tensor(3 + 4j).conj().imag, -4.0),
    (lambda: torch._efficientzerotensor(()), 0.0),
    (lambda: torch.arange(6.0)[4], 4.0),
], ids=["negated", "zero", "element"])
def test_given_gradient(word_read, gradient, value):
    _loss().backward(gradient=gradient())
    assert word_read == [value]
