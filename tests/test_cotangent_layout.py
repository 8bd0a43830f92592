"""A cotangent that is a column-major FP64 matrix on the device is read in
place; every other form is copied into one."""
import pytest

torch = pytest.importorskip("torch")


def forms():
    g = torch.Generator().manual_seed(0)
    base = torch.randn(6, 10, dtype=torch.float64, generator=g)
    cm = base[:4, :5].t().contiguous().t()
    wide = torch.randn(5, 8, dtype=torch.float64, generator=g)
    yield "column-major", cm, True
    yield "longer column stride", wide.t()[:4], True
    yield "odd offset", wide.t()[1:5], False
    yield "row-major", cm.contiguous(), False
    yield "every second row", wide.t()[::2], False
    yield "broadcast", torch.ones((), dtype=torch.float64).expand(4, 5), False
    yield "repeated column", cm[:, :1].expand(4, 5), False
    yield "float32", cm.float().t().contiguous().t(), False
    yield "negated view", torch.view_as_complex(torch.stack([cm, cm], -1)).conj().imag, False
    yield "zero tensor", torch._efficientzerotensor((4, 5), dtype=torch.float64), False


@pytest.mark.parametrize("name,t,same", forms(), ids=lambda v: v if isinstance(v, str) else "")
def test_read_in_place_or_copied(name, t, same):
    from paper_2311_11943_amd import autograd
    out = autograd._colmajor(t, 4, 5, torch.device("cpu"))
    assert (out is t) == same
    assert out.dtype == torch.float64 and tuple(out.shape) == (4, 5) and out.stride(0) == 1 and out.stride(1) >= 4
    assert not out.is_neg() and out.data_ptr() % 16 == 0
    assert torch.equal(out, t.to(torch.float64) + 0)


def test_none_is_zero():
    from paper_2311_11943_amd import autograd
    out = autograd._colmajor(None, 4, 5, torch.device("cpu"))
    assert out.stride() == (1, 4) and not out.any()
