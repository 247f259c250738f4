"""spconv_ew and spconv_copy_cols at sizes around the 16-byte vectors they move, aligned and not."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DTS = [torch.float32, torch.float16, torch.bfloat16]


@pytest.mark.parametrize("dtype", DTS)
@pytest.mark.parametrize("n", [1, 7, 8, 9, 2051, 70_001])
@pytest.mark.parametrize("shift", [0, 1])
def test_ew(dtype, n, shift):
    import paper_2311_12862_amd as sp
    g = torch.Generator(device="cuda").manual_seed(n)
    a, b = (torch.randn(n + 1, generator=g, device="cuda").to(dtype)[shift:shift + n] for _ in range(2))
    out = torch.full((n + 2,), 7.0, dtype=dtype, device="cuda")
    want = {sp.EW_RELU: a.float().clamp(min=0), sp.EW_ADD: a.float() + b.float(),
            sp.EW_ADD_RELU: (a.float() + b.float()).clamp(min=0), sp.EW_RELU_BWD: torch.where(b > 0, a, torch.zeros_like(a)).float()}
    for op, w in want.items():
        out.fill_(7.0)
        sp.ew(op, a, None if op == sp.EW_RELU else b, out[1:n + 1] if shift else out[:n])
        assert torch.equal(out[1:n + 1] if shift else out[:n], w.to(dtype)), (op, n, shift)
        assert (out[n + 1:] == 7).all() and (not shift or out[0] == 7)   # nothing beside the tensor is written
    sp.ew(sp.EW_ADD, a, b, a)   # in place
    assert torch.equal(a, want[sp.EW_ADD].to(dtype))


@pytest.mark.parametrize("dtype", DTS)
@pytest.mark.parametrize("shape", [(1, 8, 0, 16, 8, 8), (301, 24, 8, 40, 16, 16), (77, 7, 1, 9, 2, 5), (1000, 6, 2, 10, 4, 4),
                                   (129, 12, 4, 36, 28, 8)])
def test_copy_cols(dtype, shape):
    import paper_2311_12862_amd as sp
    rows, sld, so, dld, do, cols = shape
    src = torch.randn(rows, sld, device="cuda").to(dtype)
    dst = torch.randn(rows, dld, device="cuda").to(dtype)
    want = dst.clone()
    want[:, do:do + cols] = src[:, so:so + cols]
    sp.copy_cols(src, so, dst, do, cols)
    assert torch.equal(dst, want)
