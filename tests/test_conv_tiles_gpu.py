"""Conv products at the edges of the kernels' tiles and of the rules that
choose them (GPU), against torch in FP64 on the CPU.

Bars: bf16 products are exact in FP32, so an FP32 sum of K terms lies within
(K + 2) u sum|terms| of the exact sum (u = 2^-24, any order); a bf16 store
adds at most 2^-8 of the stored magnitude.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
U, BF = 2.0 ** -24, 2.0 ** -8


@pytest.fixture(scope="module")
def sess():
    from paper_2507_01152_amd.session import Session
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    s = Session(0)
    yield s
    s.close()


def _conv(x, w, stride, up):
    """NHWC x, [Co][k][k][C] w, FP64, pad k // 2."""
    x = x.permute(0, 3, 1, 2)
    if up:
        x = x.repeat_interleave(2, 2).repeat_interleave(2, 3)
    return torch.nn.functional.conv2d(x, w.permute(0, 3, 1, 2), stride=stride, padding=w.shape[1] // 2).permute(0, 2, 3, 1)


def _check(got, exact, bound, what):
    err = (got.cpu().double() - exact).abs()
    assert bool((err <= bound).all()), (what, float((err / bound.clamp_min(1e-300)).max()))


def _layer(sess, n, h, w, c, co, k=3, stride=1, up=0, seed=0):
    """Forward (bf16 and FP32), data gradient (written and added into) and weight gradient of one layer."""
    from paper_2507_01152_amd import sonosim as sg
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((n, h, w, c), generator=g).bfloat16()
    wt = (torch.randn((co, k, k, c), generator=g) * 0.1).bfloat16()
    b = torch.randn(co, generator=g)
    x64, w64 = x.double().requires_grad_(True), wt.double().requires_grad_(True)
    v = _conv(x64, w64, stride, up)
    dy = torch.randn(v.shape, generator=g).bfloat16()
    dx, dw = torch.autograd.grad(v, (x64, w64), dy.double())
    xa, wa = x.double().abs().requires_grad_(True), wt.double().abs().requires_grad_(True)
    va = _conv(xa, wa, stride, up)
    dxa, dwa = torch.autograd.grad(va, (xa, wa), dy.double().abs())
    v, va = v.detach(), va.detach()
    d = sg.conv_desc(n, h, w, c, co, k, stride, k // 2, up)
    X, Wt, B, DY = (t.cuda() for t in (x, wt, b, dy))
    y, y32 = torch.empty_like(DY), torch.empty(DY.shape, device="cuda")
    sg.sg_conv_forward(sess.ctx, d, X, Wt, B, True, y=y, y_f32=y32)
    exact = torch.relu(v + b.double())
    bound = (k * k * c + 3) * U * (va + b.double().abs())
    _check(y32, exact, bound + 1e-30, "y_f32")
    _check(y, exact, bound + BF * (exact + bound) + 1e-30, "y")
    old = torch.randn(x.shape, generator=g).cuda()
    D = torch.full(x.shape, 7.0, device="cuda")
    sg.sg_conv_backward_data(sess.ctx, d, DY, Wt, D)
    kd = (4 if up else 1) * k * k * co
    _check(D, dx, (kd + 6) * U * dxa + 1e-30, "dx")
    D = old.clone()
    sg.sg_conv_backward_data(sess.ctx, d, DY, Wt, D, accumulate=True)
    _check(D, dx + old.cpu().double(), (kd + 8) * U * (dxa + old.cpu().double().abs()) + 1e-30, "dx added")
    dW, dB = torch.empty(wt.shape, device="cuda"), torch.empty(co, device="cuda")
    sg.sg_conv_backward_weight(sess.ctx, d, X, DY, dW, dB)
    m = dy.numel() // co
    _check(dW, dw, (m + 8) * U * dwa + 1e-30, "dw")
    _check(dB, dy.double().sum((0, 1, 2)), (m + 8) * U * dy.double().abs().sum((0, 1, 2)) + 1e-30, "db")


# few rows: the smallest tiles (64 x 16, 64 x 32, 32 x 64), rows around their edges, columns past one tile
@pytest.mark.parametrize("m", [1, 31, 33, 64, 65, 129])
@pytest.mark.parametrize("c,co", [(40, 8), (40, 16), (64, 24), (32, 40), (96, 64), (64, 72), (32, 136)])
def test_smallest_gemm_tiles(sess, m, c, co):
    _layer(sess, 1, 1, m, c, co, seed=m + co)


# enough blocks for the next larger tiles (64 x 64, 128 x 64, 128 x 32, 256 x 16), ragged in rows
@pytest.mark.parametrize("h,w,c,co", [(127, 131, 40, 128), (257, 129, 40, 72), (255, 259, 40, 32), (259, 509, 40, 8)])
def test_larger_gemm_tiles(sess, h, w, c, co):
    _layer(sess, 1, h, w, c, co, seed=h)


# stride 2 (four parity classes, one of them without rows on a side of one pixel) and 1 x 1
@pytest.mark.parametrize("n,h,w,c,co,k,stride", [(1, 2, 3, 40, 64, 3, 2), (3, 17, 16, 64, 40, 3, 2), (2, 33, 7, 128, 136, 3, 2),
                                                (2, 9, 11, 64, 72, 1, 1)])
def test_stride_and_pointwise(sess, n, h, w, c, co, k, stride):
    _layer(sess, n, h, w, c, co, k, stride, seed=n)


# inputs read upsampled: the data gradient's quads of fine pixels, over every tile of the GEMM
@pytest.mark.parametrize("n,h,w,c,co,k,stride", [(1, 1, 1, 40, 40, 3, 1), (3, 5, 7, 64, 64, 3, 1), (1, 3, 11, 24, 40, 3, 1),
                                                (2, 9, 8, 16, 64, 3, 1), (2, 7, 5, 136, 72, 3, 1), (1, 65, 63, 72, 40, 3, 1),
                                                (1, 129, 65, 40, 64, 3, 1), (2, 91, 93, 136, 40, 3, 1),
                                                (1, 181, 182, 24, 40, 3, 1), (1, 182, 183, 8, 40, 3, 1), (2, 6, 5, 48, 40, 5, 1),
                                                (2, 6, 5, 48, 40, 3, 2)])
def test_upsampled_layers(sess, n, h, w, c, co, k, stride):
    _layer(sess, n, h, w, c, co, k, stride, up=1, seed=h)


# the tiled weight gradient: every channel group, each way of reading the input, tiles of 8 (stride 2: 4)
# x 32 output pixels cut at each side, more tiles than blocks (the last shapes)
@pytest.mark.parametrize("c,co", [(8, 16), (16, 32), (24, 16), (24, 32), (32, 32), (64, 96), (96, 16)])
@pytest.mark.parametrize("n,h,w,stride,up", [(2, 1, 17, 1, 0), (1, 9, 33, 1, 0), (3, 8, 64, 1, 0), (2, 17, 31, 2, 0), (1, 10, 67, 2, 0),
                                            (1, 32, 66, 2, 0), (2, 1, 9, 1, 1), (1, 5, 17, 1, 1), (1, 12, 32, 1, 1)])
def test_tiled_weight_gradient(sess, n, h, w, c, co, stride, up):
    _layer(sess, n, h, w, c, co, 3, stride, up, seed=c + h)


@pytest.mark.parametrize("n,h,w,c,co,stride,up", [(9, 67, 250, 16, 16, 1, 0), (70, 33, 65, 32, 32, 2, 0), (40, 18, 33, 32, 32, 1, 1)])
def test_tiled_weight_gradient_many_tiles(sess, n, h, w, c, co, stride, up):
    _layer(sess, n, h, w, c, co, 3, stride, up, seed=n)


# 64 and more channels with the input tile and its halo in LDS (from 256 blocks of 16 x 16 pixels x 64
# channels on): tiles cut at each side, several channel groups, upsampled inputs (the stored halo), and the
# shapes next to the rule's lines
@pytest.mark.parametrize("n,h,w,c,co,up", [(64, 17, 31, 64, 64, 0), (32, 33, 18, 64, 128, 0), (65, 18, 16, 128, 128, 0),
                                          (256, 16, 16, 128, 64, 0), (255, 16, 16, 64, 64, 0), (1030, 16, 16, 128, 64, 0),
                                          (256, 8, 8, 64, 64, 1), (33, 17, 13, 128, 64, 1), (70, 9, 9, 256, 64, 1), (64, 8, 16, 256, 128, 1)])
def test_halo_layers(sess, n, h, w, c, co, up):
    _layer(sess, n, h, w, c, co, up=up, seed=h + w)


# inference passes two layers at a time where nothing stores the tensor between them: the frames are the training
# forward's outputs clamped to [0, 1] (same K order and roundings: equal bits), their bf16 the rounded frames,
# also where audited frames were replaced; one image tile, ragged tiles, several
@pytest.mark.parametrize("n,h,w", [(1, 16, 16), (2, 32, 48), (3, 112, 80)])
def test_inference_passes(sess, n, h, w):
    from paper_2507_01152_amd import sonosim as sg
    from test_surrogate_gpu import _pairs
    wl = _pairs(n, h, w, seed=n)
    vids = sess.load(wl)
    sid = sg.sg_surr_create(sess.ctx, h, w, seed=5)
    out = torch.empty((n, h, w), dtype=torch.float32, device="cuda")
    out16 = torch.empty((n, h, w), dtype=torch.bfloat16, device="cuda")
    sg.sg_surr_infer(sess.ctx, sid, vids, wl.probes, wl.poses, out, [], 30.0)
    sg.sg_surr_infer_bf16(sess.ctx, sid, vids, wl.probes, wl.poses, out16, [], 30.0)
    assert torch.equal(out.bfloat16(), out16)
    sg.sg_surr_train_step(sess.ctx, sid, vids, wl.probes, wl.poses, 0.0)
    yhat = sg.sg_surr_tensor(sess.ctx, sid, sg.SURR_T_YHAT, 0).reshape(n, h, w)
    assert np.array_equal(np.clip(yhat, 0, 1), out.cpu().numpy())
    for audit, frac in (([n - 1], 1.0), (list(range(n)), 0.0)):   # one frame replaced; all of them
        _, nf = sg.sg_surr_infer(sess.ctx, sid, vids, wl.probes, wl.poses, out, audit, np.inf, frac)
        _, nf16 = sg.sg_surr_infer_bf16(sess.ctx, sid, vids, wl.probes, wl.poses, out16, audit, np.inf, frac)
        assert nf == nf16 == len(audit) and torch.equal(out.bfloat16(), out16)
    sg.sg_surr_destroy(sess.ctx, sid)
