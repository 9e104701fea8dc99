"""Weight gradients of tensors that do not start on 16 bytes (GPU): the tiled
kernel fetches 16-byte chunks by DMA, so such tensors take the GEMM.  Against
torch in FP64 on the CPU, with the bound of an FP32 sum of K exact products in
any order, (K + 2) 2^-24 sum|terms|."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _at(t, elements):
    """A device copy of t that starts `elements` past an allocation's start."""
    buf = torch.empty(t.numel() + elements, dtype=t.dtype, device="cuda")
    v = buf[elements:].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("c,co,stride,up", [(16, 32, 1, 0), (32, 16, 1, 1), (64, 64, 2, 0), (40, 72, 1, 0)])
@pytest.mark.parametrize("xo,dyo", [(4, 0), (0, 4), (2, 6)])
def test_weight_gradient_of_shifted_tensors(c, co, stride, up, xo, dyo):
    from paper_2507_01152_amd import sonosim as sg
    from paper_2507_01152_amd.session import Session
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, h, w = 2, 12, 35
    g = torch.Generator().manual_seed(c + co)
    ho, wo = (((2 if up else 1) * d - 1) // stride + 1 for d in (h, w))
    x, dy = torch.randn((n, h, w, c), generator=g).bfloat16(), torch.randn((n, ho, wo, co), generator=g).bfloat16()

    def exact(x, dy):
        x = x.permute(0, 3, 1, 2)
        if up:
            x = x.repeat_interleave(2, 2).repeat_interleave(2, 3)
        return torch.nn.grad.conv2d_weight(x, (co, c, 3, 3), dy.permute(0, 3, 1, 2), stride=stride, padding=1).permute(0, 2, 3, 1)

    ref, mag = exact(x.double(), dy.double()), exact(x.double().abs(), dy.double().abs())
    m = n * ho * wo
    with Session(0) as sess:
        dw, db = torch.empty((co, 3, 3, c), device="cuda"), torch.empty(co, device="cuda")
        sg.sg_conv_backward_weight(sess.ctx, sg.conv_desc(n, h, w, c, co, 3, stride, 1, up), _at(x, xo), _at(dy, dyo), dw, db)
        assert bool(((dw.cpu().double() - ref).abs() <= (m + 8) * 2.0 ** -24 * mag + 1e-30).all())
        s = dy.double()
        assert bool(((db.cpu().double() - s.sum((0, 1, 2))).abs() <= (m + 8) * 2.0 ** -24 * s.abs().sum((0, 1, 2)) + 1e-30).all())
