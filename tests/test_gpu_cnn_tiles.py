"""Implicit-GEMM convolutions at the sizes where the block tile changes (ragged
rows and columns in every tile, several launches of parity classes) and the
two-channel layer's kernels.

Bars: a BF16 result within one rounding (2^-8 relative) plus the FP32
accumulation, an FP32 one within the accumulation, 1e-5 of the sum of the
products' magnitudes (K <= 1e5 terms in partial sums of at most a few thousand)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# (batch, hw, ci, co, stride): forward tiles of 128x128, 128x64, 128x32 and 64x64;
# stride 4 has 16 parity classes, some without taps
CASES = [(9, 61, 8, 136, 1), (9, 61, 40, 72, 1), (18, 61, 16, 24, 1), (5, 33, 24, 40, 2),
         (64, 64, 72, 8, 2), (70, 61, 32, 64, 2), (6, 30, 16, 16, 4)]


def im2col(x, s):
    N, H, W, C = x.shape
    ho, wo = (H - 1) // s + 1, (W - 1) // s + 1
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    return torch.cat([p[:, ky:ky + (ho - 1) * s + 1:s, kx:kx + (wo - 1) * s + 1:s]
                      for ky in range(3) for kx in range(3)], dim=3).reshape(N * ho * wo, 9 * C)


def col2im(dcol, shape, s):
    N, H, W, C = shape
    ho, wo = (H - 1) // s + 1, (W - 1) // s + 1
    p = torch.zeros((N, H + 2, W + 2, C), dtype=torch.float64, device="cuda")
    d = dcol.view(N, ho, wo, 9, C)
    for t in range(9):
        p[:, t // 3:t // 3 + (ho - 1) * s + 1:s, t % 3:t % 3 + (wo - 1) * s + 1:s] += d[:, :, :, t]
    return p[:, 1:H + 1, 1:W + 1]


@pytest.mark.parametrize("case", CASES)
def test_convolution_tiles(dp, case):
    from paper_2508_13304_amd import proposal as pr
    n, hw, ci, co, s = case
    g = torch.Generator("cuda").manual_seed(sum(case))
    rnd = lambda *sh: torch.randn(sh, device="cuda", generator=g)
    ho = (hw - 1) // s + 1
    x, dz = rnd(n, hw, hw, ci).relu().bfloat16(), rnd(n, ho, ho, co).bfloat16()
    row = (9 * ci + 1 + 7) // 8 * 8
    w, b = (0.1 * rnd(co, row)).bfloat16(), rnd(co)
    X, Z, W = x.double(), dz.double().reshape(-1, co), w[:, :9 * ci].double()
    col = im2col(X, s)
    ref, mag = (col @ W.T + b).relu(), col @ W.abs().T + b.abs()
    y = pr.conv_fwd(x, w, s, b).double().reshape(-1, co)
    assert ((y - ref).abs() <= ref / 256 + 1e-5 * mag).all()
    dw = torch.full((co, row), float("nan"), device="cuda")
    pr.conv_wgrad(x, dz, s, out=dw)
    assert ((dw[:, :9 * ci] - Z.T @ col).abs() <= 1e-5 * (Z.abs().T @ col)).all()
    assert ((dw[:, 9 * ci] - Z.sum(0)).abs() <= 1e-5 * Z.abs().sum(0)).all()
    assert (dw[:, 9 * ci + 1:] == 0).all()
    dx = pr.conv_dgrad_act(dz, w, tuple(x.shape), s, x).double()
    ref, mag = col2im(Z @ W, x.shape, s) * (X > 0), col2im(Z.abs() @ W.abs(), x.shape, s)
    assert ((dx - ref).abs() <= ref.abs() / 256 + 1e-5 * mag).all()


@pytest.mark.parametrize("n,h,w,co,s", [(1, 1, 1, 32, 1), (2, 5, 7, 32, 2), (3, 33, 18, 64, 1), (40, 37, 41, 32, 2),
                                        (300, 61, 61, 32, 2)])
def test_two_channel_layer_equals_the_explicit_products(dp, n, h, w, co, s):
    from paper_2508_13304_amd import proposal as pr
    g = torch.Generator("cuda").manual_seed(n + h)
    rnd = lambda *sh: torch.randn(sh, device="cuda", generator=g)
    x, wt, b = rnd(n, h, w, 2).bfloat16(), rnd(co, 24).bfloat16(), rnd(co)
    col, ho, wo = pr.im2col(x, s, ld=24, ones=True)
    y = pr.conv_c2_fwd(x, wt, s, b)
    assert torch.equal(y.reshape(-1, co), pr.gemm_bias_act(col, wt, 18, b))
    dz = rnd(n, ho, wo, co).bfloat16()
    dw = pr.conv_c2_wgrad(x, dz, s, out=torch.full((co, 24), float("nan"), device="cuda"))
    assert torch.equal(dw, pr.gemm(dz.reshape(-1, co), col, ta=True))


def test_two_channel_input_off_its_alignment(dp):
    """An image pair that does not start on a whole pixel's four bytes is still taken."""
    from paper_2508_13304_amd import proposal as pr
    net = pr.ProposalNet(size=32, channels=(32, 32), seed=3)
    x = torch.randn((2, 32, 32, 2), device="cuda", generator=torch.Generator("cuda").manual_seed(1)).bfloat16()
    flat = torch.zeros(x.numel() + 1, dtype=torch.bfloat16, device="cuda")
    flat[1:] = x.reshape(-1)
    assert torch.equal(net.forward(flat[1:].view(x.shape)), net.forward(x))


@pytest.mark.parametrize("ta", [False, True])
def test_rows_further_apart_than_32_bit_offsets_reach(dp, ta):
    """64 rows (or k) of 2^25 + 8 elements: the last one lies past 2^32 bytes."""
    from paper_2508_13304_amd import proposal as pr
    g = torch.Generator("cuda").manual_seed(11)
    ld = 2 ** 25 + 8
    big = torch.empty((72, ld), dtype=torch.bfloat16, device="cuda")
    a = big[:, :64]
    a.copy_(torch.randn((72, 64), device="cuda", generator=g))
    b = torch.randn((64 if not ta else 72, 40), device="cuda", generator=g).bfloat16()
    A = a.double().T if ta else a.double()
    assert ((pr.gemm(a, b, ta=ta).double() - A @ b.double()).abs() <= 1e-5 * (A.abs() @ b.double().abs())).all()
    if not ta:
        bias = torch.randn(40, device="cuda", generator=g)
        ref, mag = (A @ b.double() + bias).relu(), A.abs() @ b.double().abs() + bias.abs()
        y = pr.gemm_bias_act(a, b.T.contiguous(), 64, bias).double()
        assert ((y - ref).abs() <= ref / 256 + 1e-5 * mag).all()


def test_more_than_2_to_the_24_rows(dp):
    """Rows past 2^24 of an image one pixel wide, with no numbers behind its end: the
    part of the last step beyond K = 72 reads nothing."""
    from paper_2508_13304_amd import proposal as pr
    g = torch.Generator("cuda").manual_seed(12)
    h, n = 2 ** 24 + 40, 300
    buf = torch.full((h + 64, 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    buf[:h] = 0
    buf[h - n:h] = torch.randn((n, 8), device="cuda", generator=g)
    x = buf[:h].view(1, h, 1, 8)
    w, b = (0.1 * torch.randn((8, 80), device="cuda", generator=g)).bfloat16(), torch.zeros(8, device="cuda")
    X, W = x[:, h - n:].double(), w[:, :72].double()
    col = im2col(X, 1)[2:]
    ref, mag = col @ W.T, col.abs() @ W.abs().T
    y = pr.conv_fwd(x, w, 1, b, relu=False)
    assert ((y[0, h - n + 2:, 0].double() - ref).abs() <= ref.abs() / 256 + 1e-5 * mag).all()
    assert (y[0, :h - n - 1] == 0).all()
    ref, mag = col2im(X.reshape(-1, 8) @ W, X.shape, 1), col2im(X.reshape(-1, 8).abs() @ W.abs(), X.shape, 1)
    dx = pr.conv_dgrad_act(x, w, (1, h, 1, 8), 1)
    d = (dx[:, h - n:].double() - ref).abs() - (ref.abs() / 256 + 1e-5 * mag)
    assert (d[:, 2:] <= 0).all() and (dx[0, :h - n - 1] == 0).all()


def test_input_refilled_between_forward_and_backward(dp):
    from paper_2508_13304_amd import proposal as pr
    net = pr.ProposalNet(size=32, channels=(32, 32), seed=4)
    g = torch.Generator("cuda").manual_seed(2)
    x = torch.randn((3, 32, 32, 2), device="cuda", generator=g).bfloat16()
    dout = torch.randn((3, 6), device="cuda", generator=g)
    _, cache = net.forward(x, keep=True)
    net.backward(cache, dout)
    want = net.G.clone()
    _, cache = net.forward(x, keep=True)
    x.zero_()
    net.backward(cache, dout)
    assert torch.equal(net.G, want)
