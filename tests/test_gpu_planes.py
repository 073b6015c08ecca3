"""The kernels on the bf16 matrix instructions (forward 1x1 and 3x3, input and
weight gradients), which take bf16 operands as they are and fp32 ones as three
bf16 planes: integer-exact against the oracle at the edges of their tiles,
fp32 error against 64 bits, and operands that are not finite."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14713_amd as onexn
import workloads
from gpu_helpers import gpu_conv, oracle_conv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    onexn.load_library()


DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
FWD = [  # (n, m, k, stride, pad, B, H, W, N)
    (40, 33, 3, 1, 1, 1, 16, 16, 32),    # one 256-pixel tile exactly, a ragged col-group
    (64, 50, 3, 1, 1, 3, 14, 14, 32),    # tiles spanning images
    (32, 20, 3, 1, 0, 9, 4, 4, 32),      # the narrowest images, many per tile
    (32, 90, 3, 1, 2, 5, 5, 6, 16),      # padding wider than the window's reach
    (48, 17, 3, 1, 1, 1, 7, 200, 16),    # several strips of columns, the last narrower
    (64, 40, 3, 1, 1, 1, 19, 61, 32),
    (33, 70, 3, 1, 1, 2, 31, 8, 16),
    (64, 45, 3, 2, 1, 2, 15, 17, 32),    # parity planes (bf16)
    (48, 24, 3, 2, 0, 1, 9, 70, 16),
    (32, 18, 3, 3, 1, 2, 13, 11, 16),
    (32, 18, 3, 5, 2, 2, 13, 21, 32),    # stride beyond the window
    (70, 130, 1, 1, 0, 2, 9, 7, 16),     # 1x1, pixels not a multiple of four (bf16)
    (70, 130, 1, 1, 0, 2, 8, 34, 16),    # quads, more than one tile per image
    (64, 40, 1, 2, 0, 3, 9, 11, 32),
    (32, 65, 1, 3, 2, 1, 10, 8, 16),
]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("n,m,k,s,pd,B,H,W,N", FWD)
def test_forward_integers(n, m, k, s, pd, B, H, W, N, dt, tune):
    tune("kernel", 2)
    w, x = workloads.gen_integer_layer(n + m + W, n, m, k, B, H, W)
    for p in (0.0, 0.5, 0.9):
        y, _ = gpu_conv(w.to(DTYPES[dt]), x.to(DTYPES[dt]), N, p, True, s, pd, out_dtype=torch.float32)
        ref, _ = oracle_conv(w, x, N, p, True, s, pd)
        np.testing.assert_array_equal(y, ref)


@pytest.mark.parametrize("m,s,B,H,W", [
    (40, 1, 70, 1, 1),       # one-pixel images
    (300, 1, 70, 1, 1),
    (40, 1, 3, 2, 2), (40, 1, 40, 2, 2), (140, 1, 40, 2, 2),     # quads, below and above 32 pixels
    (40, 1, 2, 7, 7), (140, 1, 1, 7, 7), (140, 1, 2, 7, 7),
    (40, 2, 3, 9, 9), (230, 2, 3, 9, 9), (230, 2, 9, 5, 5),
    (40, 1, 1, 211, 211), (70, 2, 8, 211, 211),                  # few channels, many pixels
])
@pytest.mark.parametrize("N", [16, 32])
def test_bf16_1x1_dispatch(m, s, B, H, W, N):
    """1x1 layers on either side of the lines between the general and this kernel."""
    w, x = workloads.gen_integer_layer(m + B, 40, m, 1, B, H, W)
    y, _ = gpu_conv(w.bfloat16(), x.bfloat16(), N, 0.5, True, s, 0, out_dtype=torch.float32)
    ref, _ = oracle_conv(w, x, N, 0.5, True, s, 0)
    np.testing.assert_array_equal(y, ref)


BWD = [  # (n, m, k, stride, pad, B, H, W, N)
    (40, 33, 3, 1, 1, 2, 16, 16, 32),
    (64, 50, 3, 1, 1, 3, 14, 14, 16),
    (72, 20, 3, 1, 0, 7, 6, 6, 8),
    (32, 40, 3, 1, 2, 2, 5, 7, 16),
    (32, 129, 3, 1, 1, 1, 9, 61, 32),
    (80, 45, 1, 1, 0, 3, 7, 9, 32),
    (140, 270, 1, 1, 0, 2, 8, 8, 16),
    (64, 33, 1, 1, 1, 2, 6, 5, 8),
    (48, 40, 3, 2, 1, 2, 11, 17, 16),    # strided: dY spread in the tile, strided octets of X
    (72, 35, 3, 2, 0, 3, 14, 14, 32),
    (40, 33, 3, 3, 2, 1, 17, 90, 8),
    (32, 70, 1, 2, 0, 2, 13, 9, 32),
    (24, 200, 1, 3, 1, 2, 12, 13, 8),
    (136, 64, 1, 1, 0, 3, 12, 12, 8),    # 1x1 in bf16: 64 and 128 input channels per tile
    (300, 130, 1, 1, 0, 1, 10, 26, 32),
    (32, 5, 5, 1, 2, 1, 11, 23, 16),
    (32, 3, 7, 3, 3, 2, 25, 26, 32),
    (32, 600, 1, 1, 0, 40, 5, 5, 32),    # several chunks of 512 pixels
    (8, 33, 3, 1, 1, 2, 11, 17, 8),      # few channels: kernels chosen by them
    (24, 20, 3, 1, 1, 3, 61, 60, 16),
    (64, 8, 3, 1, 1, 2, 9, 9, 32),
    (8, 32, 1, 1, 0, 2, 9, 9, 8),
    (8, 32, 3, 2, 1, 2, 15, 13, 32),
]


def _grads(w, x, dy, N, p, s, pd):
    n, m, k, _ = w.shape
    L = onexn.prepare_layer(w, N, p, True)
    dx = torch.full(x.shape, float("nan"), device="cuda")
    dD = torch.full((L.t, N, k, k), float("nan"), device="cuda")
    onexn.conv2d_bwd_data(L.P, L.I, L.D, n, m, dy.cuda(), x.shape[2:], s, pd, torch.float32, out=dx)
    onexn.conv2d_bwd_weight(L.P, L.I, n, N, (k, k), x.cuda(), dy.cuda(), s, pd, out=dD)
    return L, dx.double().cpu().numpy(), dD.double().cpu().numpy()


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("n,m,k,s,pd,B,H,W,N", BWD)
def test_gradients_integers(n, m, k, s, pd, B, H, W, N, dt, tune):
    w, x = workloads.gen_integer_layer(n + m + W, n, m, k, B, H, W)
    Ho, Wo = onexn.out_hw(H, W, k, k, (s, s), (pd, pd))
    dy = torch.randint(-3, 4, (B, n, Ho, Wo), generator=torch.Generator().manual_seed(W)).float()
    strided = dt == "bf16" and s > 1     # the general kernel may be chosen there, by times
    for kernel, p in [(4, 0.0), (4, 0.5), (4, 0.95)] + [(-1, 0.5)] * strided:
        tune("bwd_kernel", kernel if strided else -1)
        L, dx, dD = _grads(w.to(DTYPES[dt]), x.to(DTYPES[dt]), dy.to(DTYPES[dt]), N, p, s, pd)
        pr = oracle.prune(w.double().numpy(), N, p, True)
        np.testing.assert_array_equal(
            dx, oracle.conv2d_bwd_data(dy.double().numpy(), pr.wbar, (H, W), (s, s), (pd, pd)))
        dw = oracle.conv2d_bwd_weight(x.double().numpy(), dy.double().numpy(), pr.T, N, (k, k), (s, s), (pd, pd))
        np.testing.assert_array_equal(dD, oracle.pack(dw, pr.T, N)[2])


def _one_in(t):
    """t as a contiguous view that starts one element into a larger buffer."""
    v = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape)
    return v.copy_(t)


@pytest.mark.parametrize("n,m,k,s,B,H,W,N", [
    (70, 130, 1, 1, 3, 8, 6, 32),        # (quads that the N = 32 kernels do not take at this alignment)
    (70, 130, 1, 1, 3, 8, 6, 16),
    (40, 130, 1, 1, 2, 9, 7, 32),
    (64, 45, 3, 1, 2, 14, 15, 32),
    (48, 24, 3, 2, 2, 11, 13, 16),
])
def test_bf16_misaligned_operands(n, m, k, s, B, H, W, N, tune):
    """The 8- and 16-byte loads of x and dY at addresses of two bytes' alignment."""
    tune("bwd_kernel", 4)
    w, x = workloads.gen_integer_layer(n + m, n, m, k, B, H, W)
    Ho, Wo = onexn.out_hw(H, W, k, k, (s, s), (k // 2, k // 2))
    dy = torch.randint(-3, 4, (B, n, Ho, Wo), generator=torch.Generator().manual_seed(W)).float()
    L = onexn.prepare_layer(w.bfloat16(), N, 0.5, True)
    pr = oracle.prune(w.double().numpy(), N, 0.5, True)
    xd, dyd = _one_in(x.bfloat16()), _one_in(dy.bfloat16())
    at = ((s, s), (k // 2, k // 2))
    y = L.forward(xd, s, k // 2, out_dtype=torch.float32)
    np.testing.assert_array_equal(y.double().cpu().numpy(), oracle.conv2d(x.double().numpy(), pr.wbar, *at))
    dx = onexn.conv2d_bwd_data(L.P, L.I, L.D, n, m, dyd, (H, W), s, k // 2, torch.float32)
    np.testing.assert_array_equal(dx.double().cpu().numpy(),
                                  oracle.conv2d_bwd_data(dy.double().numpy(), pr.wbar, (H, W), *at))
    dD = onexn.conv2d_bwd_weight(L.P, L.I, n, N, (k, k), xd, dyd, s, k // 2)
    dw = oracle.conv2d_bwd_weight(x.double().numpy(), dy.double().numpy(), pr.T, N, (k, k), *at)
    np.testing.assert_array_equal(dD.double().cpu().numpy(), oracle.pack(dw, pr.T, N)[2])


def test_bf16_weight_gradient_does_not_vary():
    w, x = workloads.gen_integer_layer(3, 64, 48, 3, 4, 20)
    x, dy = torch.randn(4, 48, 20, 20).bfloat16(), torch.randn(4, 64, 20, 20).bfloat16()
    runs = [_grads(w.bfloat16(), x, dy, 32, 0.5, 1, 1)[2] for _ in range(3)]
    assert all(np.array_equal(runs[0], r) for r in runs[1:])


@pytest.mark.parametrize("k,s,pd", [(1, 1, 0), (3, 1, 1), (1, 2, 0), (3, 2, 1)])
@pytest.mark.parametrize("n,m,N", [
    (150, 40, 32),     # few tiles: half the rows of a col-group per workgroup, 22 rows in the last one
    (170, 1400, 32),   # a 1x1 layer of many tiles: all 32 rows; 10 rows in the last col-group
    (170, 30, 16),
])
def test_bf16_weight_gradient_rows(n, m, N, k, s, pd, tune):
    tune("bwd_kernel", 4)
    if k == 3:
        m = max(m // 9, 30)
    w, x = workloads.gen_integer_layer(n + m, n, m, k, 2, 10, 8)
    Ho, Wo = onexn.out_hw(10, 8, k, k, (s, s), (pd, pd))
    dy = torch.randint(-3, 4, (2, n, Ho, Wo), generator=torch.Generator().manual_seed(m)).float()
    for p in (0.0, 0.5):
        L, _, dD = _grads(w.bfloat16(), x.bfloat16(), dy.bfloat16(), N, p, s, pd)
        T = oracle.prune(w.double().numpy(), N, p, True).T
        dw = oracle.conv2d_bwd_weight(x.double().numpy(), dy.double().numpy(), T, N, (k, k), (s, s), (pd, pd))
        np.testing.assert_array_equal(dD, oracle.pack(dw, T, N)[2])


def _norm_err(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("N", [16, 32])
def test_fp32_products(N, tune):
    """One product per output: the planes leave out less than 1.002 * 2^-24 of it,
    the five small products' additions round by 2^-24 of at most 2^-6 each and
    the last one by 2^-24: together under 2.1 * 2^-24, with no preferred sign
    (40000 errors of a spread below 2^-24 average to under 0.05 of it)."""
    tune("kernel", 2)
    gen = torch.Generator().manual_seed(N)
    m, H = 8, 50
    w = torch.zeros(16, m, 3, 3)
    o = torch.arange(16)
    w[o, o % m, 1, 1] = torch.rand(16, generator=gen) + 1
    x = torch.rand(2, m, H, H, generator=gen) + 1
    w[1, 1, 1, 1] = x[:, 1, :, :25] = 1 + 2.0 ** -7 - 2.0 ** -23
    w[2, 2, 1, 1] = x[:, 2, :, :25] = 2 - 2.0 ** -23
    refs = x.double().numpy()[:, o % m] * w[o, o % m, 1, 1].double().numpy()[:, None, None]
    y, _ = gpu_conv(w, x, N, 0.0, False, 1, 1)
    w[m:] = 0                            # (one output channel per input channel)
    dy = torch.cat([x, x], 1)
    L = onexn.prepare_layer(w, N, 0.0, False)
    dx = onexn.conv2d_bwd_data(L.P, L.I, L.D, 16, m, dy.cuda(), (H, H), 1, 1).double().cpu().numpy()
    for got, ref in ((y, refs), (dx, refs[:, :m])):
        err = (got / ref - 1) * 2.0 ** 24
        assert np.abs(err).max() < 2.1
        assert abs(err.mean()) < 0.05


@pytest.mark.parametrize("scale", [1.0, 2.0 ** 60, 2.0 ** -60])
@pytest.mark.parametrize("N", [16, 32])
def test_fp32_error(N, scale, tune):
    """Three planes hold an fp32 value exactly, the six products leave out at most
    1.002 * 2^-24 of a product, and each of at most 9 * 256 / 16 additions per
    accumulator rounds by 2^-24 of a partial sum, at random: together under
    sqrt(144) * 2^-24 = 7e-7 of the result's norm, at any scale."""
    tune("kernel", 2)
    gen = torch.Generator().manual_seed(N)
    w = torch.randn(64, 256, 3, 3, generator=gen) * 0.03
    x = torch.randn(2, 256, 14, 14, generator=gen).clamp_min(0) * scale
    y, _ = gpu_conv(w, x, N, 0.3, False, 1, 1)
    ref, _ = oracle_conv(w, x, N, 0.3, False, 1, 1)
    assert _norm_err(y / scale, ref / scale) < 7e-7
    dy = torch.randn(2, 64, 14, 14, generator=gen) * scale
    _, dx, _ = _grads(w, x, dy, N, 0.3, 1, 1)
    pr = oracle.prune(w.double().numpy(), N, 0.3, True)
    ref = oracle.conv2d_bwd_data(dy.double().numpy(), pr.wbar, (14, 14), (1, 1), (1, 1))
    assert _norm_err(dx / scale, ref / scale) < 7e-7


def _kept_grads(L, x, dy, k, s, pd):
    """Both gradients in fp64 over the kept blocks and in-image taps only."""
    n, N = L.n, L.N
    P, I, D = L.P.cpu().numpy(), L.I.cpu().numpy(), L.D.double().cpu().numpy()
    B, m, H, W = x.shape
    Ho, Wo = dy.shape[2:]
    dx, dD = np.zeros(x.shape), np.zeros(D.shape)
    for g in range(len(P) - 1):
        rows = min(N, n - g * N)
        d = dy[:, g * N:g * N + rows]
        for z in range(P[g], P[g + 1]):
            for q in range(k):
                oh = [o for o in range(Ho) if 0 <= o * s - pd + q < H]
                ih = [o * s - pd + q for o in oh]
                for r in range(k):
                    ow = [o for o in range(Wo) if 0 <= o * s - pd + r < W]
                    iw = [o * s - pd + r for o in ow]
                    part = d[:, :, oh][:, :, :, ow]
                    if not oh or not ow:
                        continue
                    dx[np.ix_(range(B), [I[z]], ih, iw)] += np.einsum("bohw,o->bhw", part, D[z, :rows, q, r])[:, None]
                    xs = x[:, I[z]][:, ih][:, :, iw]
                    dD[z, :rows, q, r] = np.einsum("bohw,bhw->o", part, xs)
    return dx, dD


def _same(got, ref):
    """Non-finite values in the same places and of the same kind, finite ones close."""
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(got)], ref[np.isinf(ref)])
    f = np.isfinite(ref)
    assert np.array_equal(f, np.isfinite(got))
    assert np.abs(got[f] - ref[f]).max() <= 1e-5 * np.abs(ref[f]).max()


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("k,N", [(3, 32), (3, 16), (1, 32), (1, 16)])
def test_not_finite(k, N, dt, tune):
    tune("kernel", 2)
    w, x = workloads.gen_integer_layer(k + N, 2 * N, 24, k, 2, 12, 10)
    dy = torch.randint(1, 4, (2, 2 * N, 12, 10), generator=torch.Generator().manual_seed(N)).float()
    x[0, 3, 4, 5], x[1, 7, 0, 0], x[1, 9, 11, 9] = float("inf"), float("-inf"), float("nan")
    dy[0, 5, 0, 0], dy[1, N + 1, 6, 9], dy[1, 2, 11, 4] = float("inf"), float("nan"), float("-inf")
    w, x, dy = (v.to(DTYPES[dt]) for v in (w, x, dy))
    L = onexn.prepare_layer(w, N, 0.5, True)
    y = L.forward(x.cuda(), 1, k // 2, out_dtype=torch.float32).double().cpu().numpy()
    with np.errstate(invalid="ignore"):
        _same(y, oracle.decode(x.double().numpy(), L.P.cpu().numpy(), L.I.cpu().numpy(),
                               L.D.double().cpu().numpy(), L.n, (1, 1), (k // 2, k // 2)))
        if dt == "f32" and k == 1:
            return      # those gradients run on the fp32 instruction
        L, dx, dD = _grads(w, x, dy, N, 0.5, 1, k // 2)
        rdx, rdD = _kept_grads(L, x.double().numpy(), dy.double().numpy(), k, 1, k // 2)
        _same(dx, rdx)
        if dt == "bf16":
            _same(dD, rdD)


@pytest.mark.parametrize("k,s,N", [(3, 1, 32), (1, 1, 16), (3, 2, 16), (1, 2, 32)])
def test_not_finite_many_pixels(k, s, N, tune):
    """Recomputed sums of several passes of a wave's lanes, whole rows of them, and
    infinities that meet their opposite or a zero late."""
    tune("bwd_kernel", 4)
    w, x = workloads.gen_integer_layer(k + N, N + 9, 48, k, 5, 23, 21)
    Ho, Wo = onexn.out_hw(23, 21, k, k, (s, s), (k // 2, k // 2))
    dy = torch.randint(1, 4, (5, N + 9, Ho, Wo), generator=torch.Generator().manual_seed(N)).float()
    inf = float("inf")
    x[:, 5], x[4, 6, 22, 20], x[0, 7, 0, 0], x[4, 7, 11, 11], x[2, 8] = inf, -inf, inf, -inf, float("nan")
    dy[0, 3], dy[4, 4, Ho - 1, Wo - 1], dy[2, N + 2, 4, 4] = -inf, inf, float("nan")
    w, x, dy = (v.bfloat16() for v in (w, x, dy))
    with np.errstate(invalid="ignore"):
        L, dx, dD = _grads(w, x, dy, N, 0.3, s, k // 2)
        rdx, rdD = _kept_grads(L, x.double().numpy(), dy.double().numpy(), k, s, k // 2)
        _same(dx, rdx)
        _same(dD, rdD)


def _taps(x, w, k, pd):
    """conv2d of one stride-1 image as a sum over taps, in fp32 on the GPU (exact on small integers)."""
    xp = torch.nn.functional.pad(x, (pd, pd, pd, pd))
    Ho, Wo = xp.shape[2] - k + 1, xp.shape[3] - k + 1
    y = 0
    for q in range(k):
        for r in range(k):
            y = y + w[:, :, q, r] @ xp[0, :, q:q + Ho, r:r + Wo].reshape(x.shape[1], -1)
    return y.view(1, -1, Ho, Wo)


@pytest.mark.parametrize("m,k,H,W", [
    (8, 1, 1, 6556022),      # rows and images longer than fp32 reciprocals divide
    (8, 1, 6556022, 1),
    (8, 1, 1, 8388628),      # (quads)
    (8, 1, 2796210, 3),
    (4, 3, 6556022, 4),
])
def test_long_images(m, k, H, W):
    w, x = workloads.gen_integer_layer(m + k, 16, m, k, 1, H, W)
    layer = onexn.prepare_layer(w.bfloat16(), 16, 0.0, False)
    ref = _taps(x.cuda(), w.cuda(), k, k // 2).bfloat16()
    buf = torch.full((ref.numel() + 4096,), float("nan"), dtype=torch.bfloat16, device="cuda")
    y = layer.forward(x.bfloat16().cuda(), 1, k // 2, out=buf[:ref.numel()].view(ref.shape))
    assert torch.equal(y, ref)
    assert buf[ref.numel():].isnan().all()
    if k == 1 and H == 1:
        y = onexn.fc_fwd(layer.P, layer.I, layer.D, 16, x.bfloat16().cuda().view(m, W), "cols")
        assert torch.equal(y, ref.view(16, W))
