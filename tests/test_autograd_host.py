"""CPU tests of the autograd layer's host decisions (no kernel runs)."""
import pytest
import torch

from paper_1701_01748_amd import autograd as A


def test_transforms_are_seen():
    seen = []

    def f(x):
        seen.append(A._transforms_active())
        return (x * x).sum()
    torch.func.grad(f)(torch.ones(3))
    assert seen == [True] and A._transforms_active() is False


def test_a_torch_without_the_query_takes_the_pieces(monkeypatch):
    """Where torch does not say whether a function transform is active, calls
    still work: they take the composed operations, which serve both."""
    monkeypatch.delattr(torch._C, "_are_functorch_transforms_active")
    assert A._transforms_active() is True


class _CudaLike(torch.Tensor):
    is_cuda = True


def test_fidelity_decision_without_the_query(monkeypatch):
    monkeypatch.delattr(torch._C, "_are_functorch_transforms_active")
    x = torch.zeros(4, 4).as_subclass(_CudaLike)
    assert A._one_node((object(),), x, (torch.zeros(3, dtype=torch.complex64),)) is False


@pytest.mark.parametrize("make", [lambda c: c, lambda c: c.conj(), lambda c: c.conj().imag, lambda c: c[::2], lambda c: c.real,
                                  lambda c: c.to(torch.complex128), lambda c: c.clone().requires_grad_(True),
                                  lambda c: c.clone().requires_grad_(True).conj(), lambda c: c[:0]])
def test_dense_is_plain_memory(make):
    t = make(torch.randn(8, dtype=torch.complex64))
    for dtype in (t.dtype, torch.complex128 if t.is_complex() else torch.float64):
        d = A._dense(t, dtype)
        assert d.dtype == dtype and d.is_contiguous() and not (d.is_conj() or d.is_neg() or d.requires_grad)
        assert torch.equal(d, t.detach().to(dtype))
        plain = torch.view_as_real(d) if d.is_complex() else d   # what the memory holds
        ref = t.detach().resolve_conj().resolve_neg().to(dtype)
        assert torch.equal(plain, torch.view_as_real(ref) if d.is_complex() else ref)
