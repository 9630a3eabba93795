"""gwq.linear and gwq.linear_bf16 called the plain way (csrc/gwq_call.cpp) against the same calls through ctypes, which a
stream or a workspace of the caller's takes: the library call is the same, so the results are the same bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2411_00850_amd as gwq


def _layer(n, k, bits=4, group=128, ppm=10000, with_index=True):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + k + bits)
    w = torch.randn((n, k), generator=gen, device="cuda").mul_(0.02).half()
    return gwq.pack(w, torch.rand((n, k), generator=gen, device="cuda"), bits, ppm, group=group, with_index=with_index)


@pytest.mark.parametrize("m", [1, 5, 16, 17, 130])
@pytest.mark.parametrize("n, k, bits, group, with_index", [(257, 1024, 4, 128, True), (1000, 4096, 3, 16, True), (256, 256, 4, 32, False)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_same_as_through_ctypes(m, n, k, bits, group, with_index, dtype):
    if dtype is torch.bfloat16 and group != 128:
        group = 128
    fn = gwq.linear if dtype is torch.float16 else gwq.linear_bf16
    p = _layer(n, k, bits, group, with_index=with_index)
    x = torch.randn((m, k), device="cuda").to(dtype)
    want = fn(p, x, stream=torch.cuda.current_stream())
    got = fn(p, x)
    assert got.dtype is dtype and got.shape == (m, n) and got.is_contiguous() and not got.requires_grad
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    out = torch.empty_like(got)
    assert fn(p, x, out=out) is out and torch.equal(out.view(torch.int16), want.view(torch.int16))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                      # the stream that is current, and its memory
        on_side = fn(p, x)
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(on_side.view(torch.int16), want.view(torch.int16))


def test_what_is_not_the_plain_case_goes_the_other_way():
    p = _layer(64, 256)
    x = torch.randn((3, 256), device="cuda").half()
    want = gwq.linear(p, x)
    for bad in (x.float(), x[:, :128], x.t().contiguous().t(), x.cpu(), torch.randn((3, 128), device="cuda").half()):
        with pytest.raises(AssertionError):
            gwq.linear(p, bad)
    with pytest.raises(AssertionError):
        gwq.linear_bf16(p, x)

    class Sub(torch.Tensor):
        pass
    assert torch.equal(gwq.linear(p, x.as_subclass(Sub)), want)
    out = torch.empty((3, 64), dtype=torch.int16, device="cuda")     # never checked: 16-bit words are what is written
    assert gwq.linear(p, x, out=out) is out and torch.equal(out.view(torch.float16), want)
    assert torch.equal(gwq.linear(p, torch.nn.Parameter(x)), want)


def test_errors_are_the_library_s():
    p = _layer(64, 256)
    with pytest.raises(gwq.GwqError) as e:
        gwq.linear(p, torch.empty((0, 256), dtype=torch.float16, device="cuda"))
    assert "gwq_linear:" in str(e.value)
    p.bits = 5
    for m in (1, 40):
        with pytest.raises(gwq.GwqError):
            gwq.linear(p, torch.zeros((m, 256), dtype=torch.float16, device="cuda"))
    p.bits = 4
    keep, p.qweight = p.qweight, None
    with pytest.raises(AttributeError):
        gwq.linear(p, torch.zeros((1, 256), dtype=torch.float16, device="cuda"))
    p.qweight = keep                                   # fields are read at every call
    with pytest.raises(gwq.GwqError):                  # groups of 128 alone take bfloat16
        gwq.linear_bf16(_layer(64, 256, group=32), torch.zeros((1, 256), dtype=torch.bfloat16, device="cuda"))
    a, b = _layer(64, 256), _layer(64, 256, bits=3)
    x = torch.randn((2, 256), device="cuda").half()
    want = gwq.linear(b, x)
    for f in ("bits", "qweight", "scales", "zeros", "row_ptr", "col_idx", "out_val", "index"):
        setattr(a, f, getattr(b, f))
    assert torch.equal(gwq.linear(a, x), want)
