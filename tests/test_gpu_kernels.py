"""GPU parity, kernel by kernel: each library kernel, called through the C ABI's kernel-level
entry points on the oracle's own operands, against the oracle's operator."""
import numpy as np
import pytest

from conv_shapes import LAYERS
from oracle import ops
from parity import check_kernel

pytestmark = pytest.mark.gpu
R = np.random.default_rng(20260428)


@pytest.fixture(scope="module")
def S():
    import torch
    import paper_2604_28175_amd as strait
    assert torch.cuda.is_available()
    strait.torch = torch
    return strait


def dev(S, a, dtype=None):
    t = S.torch.from_numpy(np.ascontiguousarray(a))
    if dtype is not None:
        t = t.to(dtype)
    return t.cuda()


def f16(a):
    return np.asarray(a).astype(np.float16)


def act_ref(y, act):
    return {0: y, 1: ops.relu(y), 2: ops.relu6(y), 3: ops.gelu(y)}[act]


CONV_CASES = [
    # N, H, W, C, K, R, stride, pad, act, residual, out_f32     (what it exercises)
    (2, 14, 14, 64, 64, 3, 1, 1, 1, False, False),      # gather path, exact tiles in K
    (3, 15, 13, 32, 96, 3, 2, 1, 1, False, False),      # stride 2, ragged M, ragged N tile
    (2, 9, 9, 16, 40, 3, 1, 1, 0, True, False),         # C = 16: a 32-wide slice straddles taps; residual
    (1, 10, 10, 24, 72, 3, 2, 1, 2, False, False),      # C = 24, ReLU6
    (2, 12, 12, 128, 256, 1, 1, 0, 1, True, False),     # 1x1 GEMM path + residual + ReLU
    (2, 12, 12, 64, 128, 1, 2, 0, 0, False, False),     # strided 1x1 (projection shortcut)
    (2, 20, 20, 3, 16, 7, 2, 3, 1, False, False),       # C = 3: scalar gather path, 7x7
    (1, 8, 8, 5, 10, 3, 1, 1, 0, False, False),         # odd C and K: scalar gather, direct epilogue
    (4, 1, 1, 64, 10, 1, 1, 0, 0, False, True),         # FC as 1x1 conv, fp32 logits
    (1, 40, 40, 64, 64, 3, 1, 1, 1, False, False),      # several 128-pixel tiles and a ragged tail (M = 1600)
    (1, 7, 7, 512, 512, 3, 1, 1, 1, False, False),      # long reduction (K = 4608), small M
    (11, 56, 56, 64, 256, 1, 1, 0, 1, True, False),     # 64 -> 256 pointwise with residual, M = 34496: many tiles, ragged tail, residual requested early
    # wide 3x3 stride-1 layers (which kernel a layer is given: conv_shapes.py and test_every_kernel_..., which assert it)
    (3, 56, 56, 64, 64, 3, 1, 1, 1, False, False),      # 64 channels out, two input slices
    (6, 28, 28, 32, 128, 3, 1, 1, 1, False, False),     # 128 channels out, a single input slice
    (1, 37, 112, 64, 128, 3, 1, 1, 0, False, False),    # wider rows, ragged height, no activation
    (2, 24, 224, 32, 64, 3, 1, 1, 1, False, False),     # widest rows served
    (2, 40, 100, 96, 192, 3, 1, 1, 2, False, False),    # three channel tiles, three input slices, ReLU6
    # more than 768 tiles of 256 x 128
    (64, 56, 56, 32, 256, 3, 1, 1, 1, False, False),    # 1626 tiles, two channel tiles
    (16, 112, 112, 64, 128, 3, 1, 1, 1, False, False),  # patch kernel: rows cut into two strips of 56; two input slices
    (48, 64, 64, 32, 128, 3, 1, 1, 0, False, False),    # 64-pixel rows
    (12, 128, 128, 32, 128, 3, 1, 1, 2, False, False),  # 128-pixel rows
    # 64 channels out, at most 128 in and 1024 or more 256-pixel tiles: workgroups that walk over several tiles each
    (81, 56, 56, 64, 64, 3, 1, 1, 1, False, False),     # 1028 tiles, two input slices
    (24, 112, 112, 32, 64, 3, 1, 1, 2, False, False),   # one slice: every slice is a tile's last; rows in two strips
    (320, 28, 28, 128, 64, 3, 1, 1, 0, False, False),   # four slices
    # few tiles and a reduction worth splitting: groups of wavefronts, or the kernel for small outputs
    (8, 14, 14, 1024, 256, 1, 1, 0, 1, False, False),   # pointwise, 64-wide slices, 16 of them
    (2, 14, 14, 512, 256, 1, 1, 0, 1, True, False),     # pointwise with residual
    (8, 14, 14, 256, 256, 3, 1, 1, 1, False, False),    # 3x3: 72 slices of 32
    (1, 10, 10, 264, 64, 1, 1, 0, 0, False, False),     # nine 32-wide slices, the last one ragged
    (3, 9, 9, 160, 96, 3, 2, 1, 2, False, False),       # stride 2, ragged tiles in both directions, 45 slices
]


@pytest.mark.parametrize("case", CONV_CASES, ids=lambda c: "x".join(map(str, c[:8])))
def test_conv2d(S, case):
    N, H, W, C, K, Rk, stride, pad, act, use_res, out_f32 = case
    x = f16(R.standard_normal((N, H, W, C)))
    w = f16(R.standard_normal((K, C, Rk, Rk)) * (2.0 / (C * Rk * Rk)) ** 0.5)
    b = R.standard_normal(K).astype(np.float32)
    ref = ops.conv2d(x, w, b, stride, pad)
    res = f16(R.standard_normal(ref.shape)) if use_res else None
    if use_res:
        ref = ref + res.astype(np.float64)
    ref = act_ref(ref, act)
    w_krsc = np.ascontiguousarray(np.transpose(w, (0, 2, 3, 1)))
    y = S.k_conv2d(dev(S, x), dev(S, w_krsc), dev(S, b), stride, pad, act, None if res is None else dev(S, res), out_f32)
    S.torch.cuda.synchronize()
    check_kernel(y.float().cpu().numpy(), ref, f"conv {case}")


def test_conv2d_split_in_the_workgroup_integer_data_is_bit_exact(S):
    """Few tiles and 9 to 32 slices, pointwise and 3x3: exact on integer data, partial sums included.  (The kernels that split the
    reduction over groups of wavefronts have their own shapes in test_every_kernel_integer_data_is_bit_exact.)"""
    for (N, H, W, C, K, Rk, stride, pad) in ((4, 14, 14, 512, 128, 1, 1, 0), (1, 10, 10, 264, 64, 1, 1, 0), (2, 14, 14, 96, 64, 3, 1, 1)):
        x = R.integers(-2, 3, (N, H, W, C)).astype(np.float16)
        w = (R.integers(-1, 2, (K, C, Rk, Rk)) * (R.random((K, C, Rk, Rk)) < 0.2)).astype(np.float16)
        b = R.integers(-5, 6, K).astype(np.float32)
        ref = ops.conv2d(x, w, b, stride, pad)
        assert np.abs(ref).max() < 2048
        y = S.k_conv2d(dev(S, x), dev(S, np.ascontiguousarray(np.transpose(w, (0, 2, 3, 1)))), dev(S, b), stride, pad)
        assert np.array_equal(y.float().cpu().numpy().astype(np.float64), ref), (N, H, W, C, K, Rk)


def test_conv2d_integer_data_is_bit_exact(S):
    """Small integers are exact in fp16 and fp32, so the GPU must reproduce the oracle exactly."""
    x = R.integers(-3, 4, (2, 11, 9, 16)).astype(np.float16)
    w = R.integers(-2, 3, (24, 16, 3, 3)).astype(np.float16)
    b = R.integers(-5, 6, 24).astype(np.float32)
    for stride in (1, 2):
        ref = ops.conv2d(x, w, b, stride, 1)
        assert np.abs(ref).max() < 2048
        y = S.k_conv2d(dev(S, x), dev(S, np.ascontiguousarray(np.transpose(w, (0, 2, 3, 1)))), dev(S, b), stride, 1)
        assert np.array_equal(y.float().cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("N,H,W,C,K", [(4, 40, 60, 32, 64), (2, 36, 128, 32, 128), (1, 29, 224, 64, 64), (40, 15, 14, 32, 64), (30, 19, 17, 32, 128),
                                       (2, 70, 65, 32, 64), (2, 40, 130, 32, 64), (3, 21, 200, 32, 64),
                                       # 768 tiles of 256 x 128 or more, the last one in the patch kernel: two strips of 64
                                       (64, 56, 56, 32, 256), (16, 112, 112, 32, 128), (48, 64, 64, 32, 128), (12, 128, 128, 64, 128),
                                       # 64 channels out, 1024 tiles of 256 or more; in the patch kernel (81, 300 and 6 images): workgroups that
                                       # walk over tiles with two and three slices (the patch buffers swap roles from tile to tile)
                                       (81, 56, 56, 64, 64), (72, 60, 60, 32, 64), (300, 30, 30, 96, 64), (50, 40, 130, 32, 64),
                                       (6, 224, 224, 64, 64)])   # and four strips of 56
def test_conv2d_wide_3x3_integer_data_is_bit_exact(S, N, H, W, C, K):
    """Wide 3x3 stride-1 layers, from an input patch in LDS addressed through the bordered image or gathered: with
    integer data every border, strip seam and tile seam must come out exactly."""
    x = R.integers(-3, 4, (N, H, W, C)).astype(np.float16)
    w = R.integers(-2, 3, (K, C, 3, 3)).astype(np.float16)
    b = R.integers(-5, 6, K).astype(np.float32)
    ref = ops.conv2d(x, w, b, 1, 1)
    assert np.abs(ref).max() < 2048
    y = S.k_conv2d(dev(S, x), dev(S, np.ascontiguousarray(np.transpose(w, (0, 2, 3, 1)))), dev(S, b), 1, 1)
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), ref)


def test_conv2d_tap_count_pattern(S):
    y = S.k_conv2d(dev(S, np.ones((1, 6, 6, 8), np.float16)), dev(S, np.ones((8, 3, 3, 8), np.float16)), None, 2, 1)
    got = y.float().cpu().numpy()[0, :, :, 0] / 8
    cnt = lambda i: sum(0 <= 2 * i + r - 1 < 6 for r in range(3))
    assert np.array_equal(got, [[cnt(i) * cnt(j) for j in range(3)] for i in range(3)])


@pytest.mark.parametrize("M,N,K,act,use_res,out_f32", [(256, 768, 768, 0, True, False), (130, 3072, 768, 3, False, False),
                                                        (64, 768, 3072, 0, True, False), (5, 1000, 2048, 0, False, True),
                                                        (300, 2304, 768, 0, False, False)])
def test_gemm(S, M, N, K, act, use_res, out_f32):
    x = f16(R.standard_normal((M, K)))
    w = f16(R.standard_normal((N, K)) * K ** -0.5)
    b = (R.standard_normal(N) * 0.1).astype(np.float32)
    ref = ops.linear(x, w, b)
    res = f16(R.standard_normal(ref.shape)) if use_res else None
    if use_res:
        ref = ref + res.astype(np.float64)
    ref = act_ref(ref, act)
    y = S.k_gemm(dev(S, x), dev(S, w), dev(S, b), act, None if res is None else dev(S, res), out_f32)
    check_kernel(y.float().cpu().numpy(), ref, f"gemm {M}x{N}x{K}")


@pytest.mark.parametrize("M,K1,N1,N2,use_res", [(9001, 64, 256, 64, True),       # many 32-pixel tiles and a ragged tail
                                                 (5000, 64, 256, 128, True),      # the seam into the next stage: twice as wide
                                                 (70, 64, 256, 64, True),         # fewer tiles than one workgroup has wavefronts
                                                 (97001, 64, 256, 64, True),      # every wavefront of the full grid walks over several tiles
                                                 (70003, 64, 256, 128, True)])
def test_pointwise_pair(S, M, K1, N1, N2, use_res):
    """y = relu(x W3^T + b3 + res), z = relu(fp16(y) W1^T + b1) in one launch: against the oracle's operators, and bit
    for bit against the same two layers as two launches."""
    x = f16(R.standard_normal((M, K1)))
    w3 = f16(R.standard_normal((N1, K1)) * (0.5 / K1) ** 0.5)
    b3 = (R.standard_normal(N1) * 0.1).astype(np.float32)
    res = f16(R.standard_normal((M, N1))) if use_res else None
    w1 = f16(R.standard_normal((N2, N1)) * (2.0 / N1) ** 0.5)
    b1 = (R.standard_normal(N2) * 0.1).astype(np.float32)
    y_ref = ops.linear(x, w3, b3)
    if use_res:
        y_ref = y_ref + res.astype(np.float64)
    y_ref = ops.relu(y_ref)
    z_ref = ops.relu(ops.linear(y_ref.astype(np.float16), w1, b1))      # the second layer reads the fp16 tensor
    dx, dw3, db3, dw1, db1 = dev(S, x), dev(S, w3), dev(S, b3), dev(S, w1), dev(S, b1)
    dres = None if res is None else dev(S, res)
    y, z = S.k_pointwise_pair(dx, dw3, db3, dres, dw1, db1)
    S.torch.cuda.synchronize()
    check_kernel(y.float().cpu().numpy(), y_ref, f"pair y {M}x{K1}x{N1}")
    check_kernel(z.float().cpu().numpy(), z_ref, f"pair z {M}x{N1}x{N2}", rel=2.0 ** -9)
    y2 = S.k_gemm(dx, dw3, db3, S.ACT_RELU, dres)
    assert S.torch.equal(y, y2)
    if -(-M // 64) * -(-N2 // 64) > 256:   # (with fewer tiles the stand-alone kernel splits its reduction and adds in another order)
        assert S.torch.equal(z, S.k_gemm(y2, dw1, db1, S.ACT_RELU))


def test_pointwise_pair_integer_data_is_bit_exact(S):
    M, K1, N1, N2 = 777, 64, 256, 64
    x = R.integers(-2, 3, (M, K1)).astype(np.float16)
    w3 = R.integers(-1, 2, (N1, K1)).astype(np.float16)
    b3 = R.integers(-3, 4, N1).astype(np.float32)
    res = R.integers(-4, 5, (M, N1)).astype(np.float16)
    w1 = (R.integers(-1, 2, (N2, N1)) * (R.random((N2, N1)) < 0.1)).astype(np.float16)     # sparse: sums stay exact in fp16
    b1 = R.integers(-3, 4, N2).astype(np.float32)
    y_ref = ops.relu(ops.linear(x, w3, b3) + res.astype(np.float64))
    z_ref = ops.relu(ops.linear(y_ref, w1, b1))
    assert np.abs(y_ref).max() < 2048 and np.abs(z_ref).max() < 2048
    y, z = S.k_pointwise_pair(dev(S, x), dev(S, w3), dev(S, b3), dev(S, res), dev(S, w1), dev(S, b1))
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), y_ref)
    assert np.array_equal(z.float().cpu().numpy().astype(np.float64), z_ref)


def test_pointwise_pair_rejects_other_shapes(S):
    t = S.torch.zeros((256, 96), dtype=S.torch.float16, device="cuda")
    w3 = S.torch.zeros((256, 96), dtype=S.torch.float16, device="cuda")
    w1 = S.torch.zeros((64, 256), dtype=S.torch.float16, device="cuda")
    res = S.torch.zeros((256, 256), dtype=S.torch.float16, device="cuda")
    with pytest.raises(S.StraitError) as e:
        S.k_pointwise_pair(t, w3, None, res, w1, None)             # 96 input channels
    assert e.value.status == S.E_SHAPE
    with pytest.raises(S.StraitError) as e:
        S.k_pointwise_pair(S.torch.zeros((256, 128), dtype=S.torch.float16, device="cuda"),
                           S.torch.zeros((512, 128), dtype=S.torch.float16, device="cuda"), None,
                           S.torch.zeros((256, 512), dtype=S.torch.float16, device="cuda"),
                           S.torch.zeros((128, 512), dtype=S.torch.float16, device="cuda"), None)   # weights that do not fit in LDS
    assert e.value.status == S.E_SHAPE
    with pytest.raises(S.StraitError) as e:
        S.k_pointwise_pair(t[:, :64].contiguous(), w3[:, :64].contiguous(), None, None, w1, None)   # no residual tensor
    assert e.value.status == S.E_INVALID


@pytest.mark.parametrize("N,P,Q,C,H2,W2,K2,s2,Cout", [(2, 14, 14, 128, 28, 28, 256, 2, 512),      # few tiles: the reduction is split
                                                        (16, 28, 28, 128, 56, 56, 256, 2, 512),    # 128-wide tiles
                                                        (3, 7, 7, 512, 14, 14, 1024, 2, 2048),     # ragged rows, long second part
                                                        (5, 8, 9, 64, 15, 17, 64, 2, 256),         # odd second tensor
                                                        (4, 20, 20, 64, 20, 20, 64, 1, 256),       # stride 1
                                                        (44, 28, 28, 128, 56, 56, 256, 2, 512)])   # enough tiles for the 256 x 128 shape
def test_conv1x1_proj(S, N, P, Q, C, H2, W2, K2, s2, Cout):
    """A pointwise convolution with a subsampling pointwise projection of a second tensor inside its reduction, against
    the oracle's two convolutions added in fp64."""
    x = f16(R.standard_normal((N, P, Q, C)))
    x2 = f16(R.standard_normal((N, H2, W2, K2)))
    w3 = f16(R.standard_normal((Cout, C)) * (0.5 / C) ** 0.5)
    wd = f16(R.standard_normal((Cout, K2)) * (0.5 / K2) ** 0.5)
    bias = (R.standard_normal(Cout) * 0.1).astype(np.float32)
    sub = x2[:, ::s2, ::s2][:, :P, :Q]
    ref = ops.relu(ops.linear(x, w3, None) + ops.linear(sub, wd, None) + bias.astype(np.float64))
    wcat = np.ascontiguousarray(np.concatenate([w3, wd], axis=1))
    y = S.k_conv1x1_proj(dev(S, x), dev(S, x2), s2, dev(S, wcat), dev(S, bias), S.ACT_RELU)
    check_kernel(y.float().cpu().numpy(), ref, f"conv1x1+proj {N}x{P}x{Q}x{C}+{K2}->{Cout}")


def test_conv1x1_proj_integer_data_and_errors(S):
    N, P, Q, C, K2, Cout = 3, 9, 10, 64, 128, 72
    x = R.integers(-2, 3, (N, P, Q, C)).astype(np.float16)
    x2 = R.integers(-2, 3, (N, 2 * P, 2 * Q, K2)).astype(np.float16)
    wcat = (R.integers(-1, 2, (Cout, C + K2)) * (R.random((Cout, C + K2)) < 0.5)).astype(np.float16)
    bias = R.integers(-3, 4, Cout).astype(np.float32)
    ref = ops.linear(np.concatenate([x, x2[:, ::2, ::2]], axis=-1), wcat, bias)
    assert np.abs(ref).max() < 2048
    y = S.k_conv1x1_proj(dev(S, x), dev(S, x2), 2, dev(S, wcat), dev(S, bias))
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), ref)
    with pytest.raises(S.StraitError) as e:                      # a first part that is not whole 64-wide slices
        S.k_conv1x1_proj(dev(S, x[..., :32].copy()), dev(S, x2), 2, dev(S, wcat[:, 32:].copy()), dev(S, bias))
    assert e.value.status == S.E_SHAPE
    with pytest.raises(S.StraitError) as e:                      # second tensor too small for the last output pixel
        S.k_conv1x1_proj(dev(S, x), dev(S, x2[:, :2 * P - 2].copy()), 2, dev(S, wcat), dev(S, bias))
    assert e.value.status == S.E_SHAPE


@pytest.mark.parametrize("M", [9001, 70, 97001])
def test_pointwise_pair_proj(S, M):
    """The pair whose shortcut is a 1x1 projection of a second tensor: y = relu(x W3^T + x2 Wd^T + b3 + bd) with the two
    products in one reduction, z = relu(fp16(y) W1^T + b1): against the oracle's operators, and bit for bit against one
    product over the concatenated inputs."""
    K1 = K2 = 64; N1, N2 = 256, 64
    x, x2 = f16(R.standard_normal((M, K1))), f16(R.standard_normal((M, K2)))
    w3 = f16(R.standard_normal((N1, K1)) * (0.5 / K1) ** 0.5)
    wd = f16(R.standard_normal((N1, K2)) * (0.5 / K2) ** 0.5)
    b3 = (R.standard_normal(N1) * 0.1).astype(np.float32)
    bd = (R.standard_normal(N1) * 0.1).astype(np.float32)
    w1 = f16(R.standard_normal((N2, N1)) * (2.0 / N1) ** 0.5)
    b1 = (R.standard_normal(N2) * 0.1).astype(np.float32)
    bsum = b3 + bd
    y_ref = ops.relu(ops.linear(x, w3, None) + ops.linear(x2, wd, None) + bsum.astype(np.float64))
    z_ref = ops.relu(ops.linear(y_ref.astype(np.float16), w1, b1))
    wcat = np.ascontiguousarray(np.concatenate([w3, wd], axis=1))
    dx, dx2, dw, db, dw1, db1 = dev(S, x), dev(S, x2), dev(S, wcat), dev(S, bsum), dev(S, w1), dev(S, b1)
    y, z = S.k_pointwise_pair_proj(dx, dx2, dw, db, dw1, db1)
    S.torch.cuda.synchronize()
    check_kernel(y.float().cpu().numpy(), y_ref, f"pair-proj y {M}")
    check_kernel(z.float().cpu().numpy(), z_ref, f"pair-proj z {M}", rel=2.0 ** -9)
    if M * N1 > 128 * 4096:           # (below that the stand-alone kernel splits its reduction and adds in another order)
        xcat = S.torch.cat([dx, dx2], dim=1).contiguous()
        assert S.torch.equal(y, S.k_gemm(xcat, dw, db, S.ACT_RELU))


def test_pointwise_pair_proj_integer_data_and_errors(S):
    M, N1, N2 = 777, 256, 64
    x = R.integers(-2, 3, (M, 64)).astype(np.float16)
    x2 = R.integers(-2, 3, (M, 64)).astype(np.float16)
    wcat = R.integers(-1, 2, (N1, 128)).astype(np.float16)
    b = R.integers(-3, 4, N1).astype(np.float32)
    w1 = (R.integers(-1, 2, (N2, N1)) * (R.random((N2, N1)) < 0.1)).astype(np.float16)     # sparse: sums stay exact in fp16
    b1 = R.integers(-3, 4, N2).astype(np.float32)
    y_ref = ops.relu(ops.linear(np.concatenate([x, x2], axis=1), wcat, b))
    z_ref = ops.relu(ops.linear(y_ref, w1, b1))
    assert np.abs(y_ref).max() < 2048 and np.abs(z_ref).max() < 2048
    y, z = S.k_pointwise_pair_proj(dev(S, x), dev(S, x2), dev(S, wcat), dev(S, b), dev(S, w1), dev(S, b1))
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), y_ref)
    assert np.array_equal(z.float().cpu().numpy().astype(np.float64), z_ref)
    with pytest.raises(S.StraitError) as e:                      # the next stage's 128 channels do not fit beside the wider weights
        S.k_pointwise_pair_proj(dev(S, x), dev(S, x2), dev(S, wcat), dev(S, b), S.torch.zeros((128, 256), dtype=S.torch.float16, device="cuda"), None)
    assert e.value.status == S.E_SHAPE
    with pytest.raises(S.StraitError) as e:
        S.k_pointwise_pair_proj(dev(S, x), None, dev(S, wcat), dev(S, b), dev(S, w1), dev(S, b1))
    assert e.value.status == S.E_INVALID


@pytest.mark.parametrize("N,H,W,C,stride", [(2, 14, 14, 96, 1), (2, 15, 13, 144, 2), (1, 7, 7, 960, 1), (3, 28, 28, 32, 2), (1, 9, 10, 8, 1),
                                            # stride 1 with enough work for the column kernel: few channels, ragged height, many channels
                                            (6, 56, 56, 32, 1), (5, 30, 27, 144, 1), (16, 7, 7, 960, 1)])
def test_dwconv3x3(S, N, H, W, C, stride):
    x = f16(R.standard_normal((N, H, W, C)) * 2)
    w = f16(R.standard_normal((C, 1, 3, 3)) * 0.47)
    b = R.standard_normal(C).astype(np.float32)
    ref = ops.relu6(ops.dwconv2d(x, w, b, stride, 1))
    w_rsc = np.ascontiguousarray(np.transpose(w[:, 0], (1, 2, 0)))
    y = S.k_dwconv3x3(dev(S, x), dev(S, w_rsc), dev(S, b), stride, S.ACT_RELU6)
    check_kernel(y.float().cpu().numpy(), ref, "dwconv")
    assert (ref == 6).any() and (ref == 0).any()


def test_pools_bit_exact_and_avg(S):
    x = f16(R.standard_normal((2, 13, 12, 64)) - 3.0)      # mostly negative: padding must never win
    y = S.k_maxpool3x3s2(dev(S, x))
    assert np.array_equal(y.cpu().numpy().astype(np.float64), ops.maxpool2d(x, 3, 2, 1))
    g = S.k_global_avgpool(dev(S, x))
    check_kernel(g.float().cpu().numpy(), ops.global_avg_pool(x.astype(np.float64)), "gap")
    c = S.k_global_avgpool(dev(S, np.full((1, 7, 7, 8), 3.25, np.float16)))
    assert np.array_equal(c.cpu().numpy(), np.full((1, 8), 3.25, np.float16))


@pytest.mark.parametrize("rows,n", [(4, 10), (33, 1000), (1, 7), (5, 64)])
def test_softmax_top1(S, rows, n):
    x = (R.standard_normal((rows, n)) * 4).astype(np.float32)
    x[0, min(3, n - 1)] = x[0].max() + 1.0
    x[-1, 0] = x[-1, n - 1] = x[-1].max() + 2.0             # exact tie: lowest index wins
    p, t = S.k_softmax_top1(dev(S, x))
    ref = ops.softmax(x)
    assert np.abs(p.cpu().numpy() - ref).max() < 1e-5
    assert np.abs(p.cpu().numpy().sum(-1) - 1).max() < 1e-5
    assert np.array_equal(t.cpu().numpy(), ops.argmax_first(x))
    assert t.cpu().numpy()[-1] == 0


@pytest.mark.parametrize("rows,n", [(7, 768), (130, 768), (3, 64), (2, 3072), (5, 256), (13, 512), (9, 1024)])
def test_layernorm(S, rows, n):
    x = f16(R.standard_normal((rows, n)) * 3 + 1)
    g = R.uniform(0.8, 1.2, n).astype(np.float32)
    b = (R.standard_normal(n) * 0.02).astype(np.float32)
    y = S.k_layernorm(dev(S, x), dev(S, g), dev(S, b), 1e-12)
    check_kernel(y.float().cpu().numpy(), ops.layernorm(x, g, b, 1e-12), "layernorm")


@pytest.mark.parametrize("B,Sq,heads,lens", [(3, 128, 12, (128, 32, 77)), (2, 64, 2, (64, 5)), (4, 32, 1, (1, 16, 31, 32)),
                                             (2, 128, 4, (33, 100)),
                                             # lengths that are no multiple of the 32-row blocks, and more than 128 keys
                                             (3, 197, 12, (197, 197, 150)), (2, 37, 2, (37, 20)), (3, 17, 1, (17, 1, 16)),
                                             (2, 256, 2, (256, 129)), (2, 129, 3, (129, 128)), (2, 255, 1, (255, 97))])
def test_attention(S, B, Sq, heads, lens):
    hid = heads * 64
    qkv = f16(R.standard_normal((B, Sq, 3 * hid)))
    vl = np.array(lens, np.int32)
    ref = ops.attention(qkv[..., :hid], qkv[..., hid:2 * hid], qkv[..., 2 * hid:], vl, heads)
    out = S.k_attention(dev(S, qkv), dev(S, vl), heads).float().cpu().numpy()
    for b in range(B):
        L = int(vl[b])
        check_kernel(out[b, :L], ref[b, :L], f"attention seq {b}", rel=2.0 ** -9, abs_rel=2e-3)
        assert np.isfinite(out[b]).all()
    # padded keys never matter: scribble over them (including non-finite values) and compare bit for bit
    qkv2 = qkv.copy()
    for b in range(B):
        qkv2[b, vl[b]:, hid:] = np.float16(np.inf)
    out2 = S.k_attention(dev(S, qkv2), dev(S, vl), heads).float().cpu().numpy()
    for b in range(B):
        assert np.array_equal(out2[b, :vl[b]], out[b, :vl[b]])


@pytest.mark.parametrize("B,Sq,heads", [(64, 160, 6), (65, 160, 6), (1, 129, 1)])
def test_attention_query_blocks_per_workgroup(S, B, Sq, heads):
    """Sequences of more than 4 query blocks, on both sides of the line between one workgroup per head and two; lengths around
    the 16-key steps, the 32-key blocks and the 64-key passes, one of them empty (all output rows zero)."""
    hid = heads * 64
    qkv = f16(R.standard_normal((B, Sq, 3 * hid)))
    vl = np.resize(np.array([Sq, 1, 64, 65, 16, 0, 79, 127, 128, 97, Sq - 1], np.int32), B)
    out = S.k_attention(dev(S, qkv), dev(S, vl), heads).float().cpu().numpy()
    for b in range(min(B, 11)):
        L = int(vl[b])
        if L:
            ref = ops.attention(qkv[b:b + 1, :, :hid], qkv[b:b + 1, :, hid:2 * hid], qkv[b:b + 1, :, 2 * hid:], vl[b:b + 1], heads)[0]
            check_kernel(out[b, :L], ref[:L], f"attention length {L}", rel=2.0 ** -9, abs_rel=2e-3)
        assert not out[b, -(-L // 32) * 32:].any()
    assert np.isfinite(out).all()


@pytest.mark.parametrize("dead", [1, 64, 70, 128])
def test_attention_leading_scores_of_minus_infinity(S, dead):
    """Keys whose scores are -inf have probability 0, also where they fill the first 64-key passes of the running maximum."""
    qkv = f16(R.standard_normal((1, 150, 192)))
    qkv[..., 0] = 1
    ref = ops.attention(qkv[:, :, :64], qkv[:, dead:, 64:128], qkv[:, dead:, 128:], np.array([150 - dead], np.int32), 1)[0]
    qkv[0, :dead, 64] = -np.inf
    out = S.k_attention(dev(S, qkv), dev(S, np.array([150], np.int32)), 1).float().cpu().numpy()[0]
    check_kernel(out, ref, f"{dead} keys at -inf", rel=2.0 ** -9, abs_rel=2e-3)


def test_attention_rows_of_more_than_31_bits(S):
    """One sequence whose rows span more than 2 GB: 23040 heads, every 64th group the same values."""
    qkv = f16(R.standard_normal((1, 256, 3, 64 * 64)))
    out = S.k_attention(dev(S, np.tile(qkv, 360).reshape(1, 256, -1)), dev(S, np.array([250], np.int32)), 360 * 64)[0]
    one = S.k_attention(dev(S, qkv.reshape(1, 256, -1)), dev(S, np.array([250], np.int32)), 64)[0]
    assert (out.reshape(256, 360, -1) == one[:, None, :]).all()


def stem_pool_weights(w_oihw):
    """[64,3,7,7] -> the fused stem kernel's [64][176] layout (strait.h, strait_k_stem_pool)."""
    wf = np.zeros((64, 22 * 8), np.float16)
    for r in range(7):
        for s in range(7):
            for c in range(3):
                wf[:, r * 24 + 1 + s * 3 + c] = w_oihw[:, c, r, s]
    return wf


@pytest.mark.parametrize("n,h,w", [(2, 64, 64), (1, 224, 224), (3, 50, 38), (2, 7, 8), (1, 33, 66), (2, 1, 2), (1, 130, 226)])
def test_stem_pool(S, n, h, w):
    x = f16(R.standard_normal((n, h, w, 3)))
    wt = f16(R.standard_normal((64, 3, 7, 7)) * (2.0 / 147) ** 0.5)
    b = (R.standard_normal(64) * 0.5).astype(np.float32)
    ref = ops.maxpool2d(ops.relu(ops.conv2d(x, wt, b, 2, 3)), 3, 2, 1)
    y = S.k_stem_pool(dev(S, x), dev(S, stem_pool_weights(wt)), dev(S, b)).float().cpu().numpy()
    assert y.shape == ref.shape
    check_kernel(y, ref, f"stem+pool {n}x{h}x{w}")


def stem3_weights(w_oihw):
    """[K,3,3,3] -> the direct 3x3/2 stem's [32][48] layout (strait.h, strait_k_stem3x3s2)."""
    wf = np.zeros((32, 48), np.float16)
    k = w_oihw.shape[0]
    for r in range(3):
        for s in range(3):
            for c in range(3):
                wf[:k, r * 16 + 1 + s * 3 + c] = w_oihw[:, c, r, s]
    return wf


@pytest.mark.parametrize("n,h,w,k,act", [(2, 64, 64, 32, 2), (1, 224, 224, 32, 2), (3, 51, 38, 32, 1), (2, 7, 8, 16, 0), (1, 33, 66, 24, 2),
                                         (2, 1, 2, 8, 0), (1, 130, 226, 32, 2), (5, 18, 130, 32, 2), (40, 96, 96, 32, 2)])
def test_stem3x3s2(S, n, h, w, k, act):
    x = f16(R.standard_normal((n, h, w, 3)))
    wt = f16(R.standard_normal((k, 3, 3, 3)) * (2.0 / 27) ** 0.5)
    b = (R.standard_normal(k) * 0.5).astype(np.float32)
    ref = act_ref(ops.conv2d(x, wt, b, 2, 1), act)
    y = S.k_stem3x3s2(dev(S, x), dev(S, stem3_weights(wt)), dev(S, b), k, act=act).float().cpu().numpy()
    assert y.shape == ref.shape
    check_kernel(y, ref, f"stem 3x3/2 {n}x{h}x{w}->{k}")


def test_stem3x3s2_integer_data_and_errors(S):
    # small integers: every product and partial sum is exact in fp16 and fp32, so any order of summation gives the same bits
    x = R.integers(-3, 4, (3, 45, 70, 3)).astype(np.float16)
    wt = R.integers(-2, 3, (32, 3, 3, 3)).astype(np.float16)
    b = R.integers(-4, 5, 32).astype(np.float32)
    y = S.k_stem3x3s2(dev(S, x), dev(S, stem3_weights(wt)), dev(S, b), 32, act=2).float().cpu().numpy()
    assert np.array_equal(y, ops.relu6(ops.conv2d(x, wt, b, 2, 1)))
    with pytest.raises(S.StraitError):       # odd width
        S.k_stem3x3s2(dev(S, x[:, :, :69]), dev(S, stem3_weights(wt)), dev(S, b), 32)
    with pytest.raises(S.StraitError):       # a channel count the kernel does not take
        S.k_stem3x3s2(dev(S, x), dev(S, stem3_weights(wt)), dev(S, b), 12)


@pytest.mark.parametrize("n,h,w,k,act", [(2, 32, 32, 16, 1), (1, 224, 224, 64, 1), (3, 51, 38, 32, 0), (2, 1, 2, 64, 0), (1, 5, 64, 16, 2), (2, 4, 66, 64, 1),
                                         (1, 9, 130, 32, 1), (7, 3, 126, 64, 2), (30, 96, 96, 64, 1)])
def test_stem3x3s1(S, n, h, w, k, act):
    """One launch from the image: random data against the oracle, integers exactly, and non-finite pixels reach the outputs they are taps of alone."""
    def layout(wt):
        wf = np.zeros((max(k, 32), 2, 3, 16), np.float16)
        rows = np.transpose(wt, (0, 2, 3, 1)).reshape(k, 3, 9)
        wf[:k, 0, :, 1:10] = rows
        wf[:k, 1, :, 0:9] = rows
        return wf.reshape(-1)
    wt = f16(R.standard_normal((k, 3, 3, 3)) * (2.0 / 27) ** 0.5)
    b = (R.standard_normal(k) * 0.5).astype(np.float32)
    x = f16(R.standard_normal((n, h, w, 3)))
    y = S.k_stem3x3s1(dev(S, x), dev(S, layout(wt)), dev(S, b), k, act=act).float().cpu().numpy()
    check_kernel(y, act_ref(ops.conv2d(x, wt, b, 1, 1), act), f"stem 3x3/1 {n}x{h}x{w}->{k}")
    xi, wi, bi = R.integers(-3, 4, x.shape).astype(np.float16), R.integers(-2, 3, wt.shape).astype(np.float16), R.integers(-4, 5, k).astype(np.float32)
    yi = S.k_stem3x3s1(dev(S, xi), dev(S, layout(wi)), dev(S, bi), k, act=0).float().cpu().numpy()
    assert np.array_equal(yi, ops.conv2d(xi, wi, bi, 1, 1))
    py, px = h // 2, w // 2
    xi[0, py, px, 1] = np.nan
    yn = S.k_stem3x3s1(dev(S, xi), dev(S, layout(wi)), dev(S, bi), k, act=0).float().cpu().numpy()
    touched = np.zeros(yn.shape[:3], bool)
    touched[0, max(py - 1, 0):py + 2, max(px - 1, 0):px + 2] = True
    assert not np.isfinite(yn[touched]).any() and np.array_equal(yn[~touched], yi[~touched])
    with pytest.raises(S.StraitError):       # odd width
        S.k_stem3x3s1(dev(S, x[:, :, :w - 1]), dev(S, layout(wt)), dev(S, b), k)
    with pytest.raises(S.StraitError):       # a channel count the kernel does not take
        S.k_stem3x3s1(dev(S, x), dev(S, layout(wt)), dev(S, b), 48)


@pytest.mark.parametrize("n,h,w", [(2, 64, 64), (1, 224, 224), (3, 51, 38), (2, 7, 8), (2, 1, 2), (1, 130, 226), (5, 18, 122), (40, 96, 96)])
def test_stem3x3s2_dw(S, n, h, w):
    """Stem 3x3/2 (3 -> 32) + depthwise 3x3 as one launch: against the oracle's two operators, and bit for bit against the
    two stand-alone kernels."""
    x = f16(R.standard_normal((n, h, w, 3)))
    wt = f16(R.standard_normal((32, 3, 3, 3)) * (2.0 / 27) ** 0.5)
    b = (R.standard_normal(32) * 0.5).astype(np.float32)
    wd = f16(R.standard_normal((32, 1, 3, 3)) * 0.47)
    bd = R.standard_normal(32).astype(np.float32)
    ref = ops.relu6(ops.dwconv2d(ops.relu6(ops.conv2d(x, wt, b, 2, 1)), wd, bd, 1, 1))
    wf_d, wd_d = dev(S, stem3_weights(wt)), dev(S, np.ascontiguousarray(np.transpose(wd[:, 0], (1, 2, 0))))
    y = S.k_stem3x3s2_dw(dev(S, x), wf_d, dev(S, b), wd_d, dev(S, bd))
    y2 = S.k_dwconv3x3(S.k_stem3x3s2(dev(S, x), wf_d, dev(S, b), 32, act=2), wd_d, dev(S, bd), 1, 2)
    S.torch.cuda.synchronize()
    assert tuple(y.shape) == ref.shape
    assert S.torch.equal(y, y2), f"fused differs from the two launches {n}x{h}x{w}"
    check_kernel(y.float().cpu().numpy(), ref, f"stem + dw {n}x{h}x{w}")
    with pytest.raises(S.StraitError):       # odd width
        S.k_stem3x3s2_dw(dev(S, x[:, :, :w - 1]), wf_d, dev(S, b), wd_d, dev(S, bd))


EXPAND_DW_CASES = [
    # N, H, W, Cin, Chid, stride      (MobileNetV2's blocks at their real shapes, then ragged ones)
    (2, 112, 112, 16, 96, 2), (2, 56, 56, 24, 144, 1), (2, 56, 56, 24, 144, 2), (3, 28, 28, 32, 192, 1), (3, 28, 28, 32, 192, 2),
    (4, 14, 14, 64, 384, 1), (4, 14, 14, 96, 576, 1), (4, 14, 14, 96, 576, 2), (5, 7, 7, 160, 960, 1),
    (2, 15, 13, 40, 88, 1),       # 40 input channels in a 64-wide reduction, 88 = 2 groups of 32 and 24 channels, odd image
    (1, 9, 10, 8, 8, 2),          # one group with 8 channels, the smallest of everything
    (2, 37, 45, 48, 200, 2),      # stride 2 with ragged tiles in both directions, a ragged last group
    (70, 14, 14, 64, 384, 1),     # enough tiles that a workgroup takes all twelve groups
    (1, 20, 70, 160, 64, 2),      # 160 input channels at stride 2: only the smallest tile fits LDS
]


@pytest.mark.parametrize("case", EXPAND_DW_CASES, ids=lambda c: "x".join(map(str, c)))
def test_expand_dw(S, case):
    """1x1 expansion + depthwise 3x3 as one launch: against the oracle's two operators, and bit for bit against the two
    stand-alone kernels."""
    N, H, W, Cin, Chid, stride = case
    x = f16(R.standard_normal((N, H, W, Cin)))
    w1 = f16(R.standard_normal((Chid, Cin, 1, 1)) * (2.0 / Cin) ** 0.5)
    b1 = R.standard_normal(Chid).astype(np.float32)
    wd = f16(R.standard_normal((Chid, 1, 3, 3)) * 0.47)
    bd = R.standard_normal(Chid).astype(np.float32)
    hid = ops.relu6(ops.conv2d(x, w1, b1, 1, 0))
    ref = ops.relu6(ops.dwconv2d(hid, wd, bd, stride, 1))
    w1_d = dev(S, np.ascontiguousarray(w1[:, :, 0, 0]))
    wd_d = dev(S, np.ascontiguousarray(np.transpose(wd[:, 0], (1, 2, 0))))
    y = S.k_expand_dw(dev(S, x), w1_d, dev(S, b1), wd_d, dev(S, bd), stride)
    t = S.k_conv2d(dev(S, x), w1_d.reshape(Chid, 1, 1, Cin), dev(S, b1), 1, 0, 2)
    y2 = S.k_dwconv3x3(t, wd_d, dev(S, bd), stride, 2)
    S.torch.cuda.synchronize()
    assert tuple(y.shape) == ref.shape
    assert S.torch.equal(y, y2), f"fused differs from the two launches {case}"
    check_kernel(y.float().cpu().numpy(), ref, f"expand+dw {case}")


@pytest.mark.parametrize("case", [(1, 28, 30, 32, 200, 1), (16, 56, 56, 24, 144, 1), (128, 55, 57, 24, 144, 1), (64, 28, 28, 32, 192, 1), (32, 13, 14, 96, 576, 1),
                                  (96, 14, 14, 64, 384, 1), (48, 7, 6, 160, 968, 1), (17, 14, 14, 96, 576, 2), (64, 28, 27, 32, 192, 2), (32, 80, 82, 16, 96, 2)],
                         ids=lambda c: "x".join(map(str, c)))
def test_expand_dw_every_cut(S, case):
    """Batches for which each way to cut a layer is chosen (smallest tiles, large tiles with one group of channels per workgroup, with
    several, workgroups that walk over tiles): bit for bit what the two stand-alone kernels give."""
    N, H, W, Cin, Chid, stride = case
    x = dev(S, f16(R.standard_normal((N, H, W, Cin))))
    w1 = dev(S, f16(R.standard_normal((Chid, Cin)) * (2.0 / Cin) ** 0.5))
    b1 = dev(S, R.standard_normal(Chid).astype(np.float32))
    wd = dev(S, f16(R.standard_normal((3, 3, Chid)) * 0.47))
    bd = dev(S, R.standard_normal(Chid).astype(np.float32))
    y = S.k_expand_dw(x, w1, b1, wd, bd, stride)
    y2 = S.k_dwconv3x3(S.k_conv2d(x, w1.reshape(Chid, 1, 1, Cin), b1, 1, 0, 2), wd, bd, stride, 2)
    S.torch.cuda.synchronize()
    assert S.torch.equal(y, y2)


@pytest.mark.parametrize("w", [466000, 470001])          # 18 rows of 128 channels: one side and the other of 2^31 bytes
def test_expand_dw_long_rows(S, w):
    """Rows that a tile's 32-bit offsets do not span are read through addresses: bit for bit what the two stand-alone kernels give."""
    t = S.torch
    x = t.randn((1, 2, w, 128), device="cuda", dtype=t.float16)
    w1, b1 = dev(S, f16(R.standard_normal((8, 128)) * 0.125)), dev(S, R.standard_normal(8).astype(np.float32))
    wd, bd = dev(S, f16(R.standard_normal((3, 3, 8)) * 0.47)), dev(S, R.standard_normal(8).astype(np.float32))
    y = S.k_expand_dw(x, w1, b1, wd, bd, 1)
    y2 = S.k_dwconv3x3(S.k_conv2d(x, w1.reshape(8, 1, 1, 128), b1, 1, 0, 2), wd, bd, 1, 2)
    t.cuda.synchronize()
    assert t.equal(y, y2)


def test_expand_dw_errors(S):
    x = dev(S, np.zeros((1, 8, 8, 12), np.float16))
    with pytest.raises(S.StraitError):       # Cin % 8 != 0
        S.k_expand_dw(x, dev(S, np.zeros((16, 12), np.float16)), None, dev(S, np.zeros((3, 3, 16), np.float16)), None, 1)
    x = dev(S, np.zeros((1, 8, 8, 16), np.float16))
    with pytest.raises(S.StraitError):       # stride 3
        S.k_expand_dw(x, dev(S, np.zeros((16, 16), np.float16)), None, dev(S, np.zeros((3, 3, 16), np.float16)), None, 3)


@pytest.mark.parametrize("n,h,w,c", [(2, 8, 6, 16), (3, 14, 14, 512), (1, 224, 224, 64)])
def test_maxpool2x2(S, n, h, w, c):
    x = f16(R.standard_normal((n, h, w, c)))
    y = S.k_maxpool2x2s2(dev(S, x)).float().cpu().numpy()
    assert np.array_equal(y, ops.maxpool2d(x, 2, 2, 0))          # selection only: bit-exact


@pytest.mark.parametrize("n,t,d", [(2, 9, 64), (3, 196, 768)])
def test_vit_tokens(S, n, t, d):
    patch = f16(R.standard_normal((n, t, d)))
    cls = f16(R.standard_normal(d) * 0.02).astype(np.float32)
    pos = f16(R.standard_normal((t + 1, d)) * 0.02).astype(np.float32)
    z = S.k_vit_tokens(dev(S, patch), dev(S, cls), dev(S, pos)).float().cpu().numpy()
    ref = np.concatenate([np.broadcast_to(cls.astype(np.float64), (n, 1, d)), patch.astype(np.float64)], axis=1) + pos.astype(np.float64)
    check_kernel(z, ref, "vit tokens", rel=2.0 ** -10, abs_rel=1e-3)


def test_argmax_f16(S):
    x = f16(R.standard_normal((6, 16, 768)))
    x[2, 0, 5] = x[2, 0, 700] = 50.0
    t = S.k_argmax_f16(dev(S, x), 768, 16 * 768, 6)
    assert np.array_equal(t.cpu().numpy(), ops.argmax_first(x[:, 0, :].astype(np.float64)))


def test_launchers_reject_bad_shapes(S):
    x = dev(S, np.zeros((1, 8, 8, 12), np.float16))
    with pytest.raises(S.StraitError):
        S.k_dwconv3x3(x, dev(S, np.zeros((3, 3, 12), np.float16)), None, 1)       # C % 8 != 0
    with pytest.raises(S.StraitError):
        S.k_attention(dev(S, np.zeros((1, 300, 192), np.float16)), dev(S, np.array([300], np.int32)), 1)   # more than 256 keys
    with pytest.raises(S.StraitError):
        S.k_layernorm(dev(S, np.zeros((2, 12), np.float16)), dev(S, np.ones(12, np.float32)), dev(S, np.zeros(12, np.float32)), 1e-5)


SPLITK_CASES = [
    # N, H, W, C, K, R, stride, pad, act, residual, out_f32   (few output tiles + long reduction, shared out inside a workgroup;
    # split over several: test_split_reductions_integer_data_is_bit_exact)
    (1, 7, 7, 512, 512, 3, 1, 1, 1, True, False),       # 49 pixels, K = 4608, residual + ReLU
    (2, 14, 14, 256, 256, 3, 2, 1, 1, False, False),    # strided 3x3, slices start in the middle of the tap sequence
    (1, 7, 7, 1024, 512, 1, 1, 0, 2, False, False),     # 1x1, ReLU6
    (8, 1, 1, 2048, 1000, 1, 1, 0, 0, False, True),     # classifier head: fp32 logits
    (3, 9, 11, 64, 72, 3, 1, 1, 0, False, False),       # ragged M and N tiles, uneven split of the 18 slices
]


@pytest.mark.parametrize("case", SPLITK_CASES, ids=lambda c: "x".join(map(str, c[:8])))
def test_conv2d_split_k(S, case):
    N, H, W, C, K, Rk, stride, pad, act, use_res, out_f32 = case
    x = f16(R.standard_normal((N, H, W, C)))
    w = f16(R.standard_normal((K, C, Rk, Rk)) * (2.0 / (C * Rk * Rk)) ** 0.5)
    b = R.standard_normal(K).astype(np.float32)
    ref = ops.conv2d(x, w, b, stride, pad)
    res = f16(R.standard_normal(ref.shape)) if use_res else None
    if use_res:
        ref = ref + res.astype(np.float64)
    ref = act_ref(ref, act)
    w_krsc = np.ascontiguousarray(np.transpose(w, (0, 2, 3, 1)))
    args = (dev(S, x), dev(S, w_krsc), dev(S, b), stride, pad, act, None if res is None else dev(S, res), out_f32)
    y1 = S.k_conv2d(*args).float().cpu().numpy()
    check_kernel(y1, ref, f"split-K conv {case}")
    # partial sums are added in a fixed order: a second launch gives the same bits
    y2 = S.k_conv2d(*args).float().cpu().numpy()
    assert np.array_equal(y1, y2)


def test_gemm_gelu_and_ragged_k(S):
    """GELU epilogue of the pipelined kernel and a reduction that is not a multiple of the slice."""
    for (M, N, K, act) in [(512, 768, 776, 3), (1000, 256, 40, 0), (4096, 3072, 768, 3)]:
        x = f16(R.standard_normal((M, K)))
        w = f16(R.standard_normal((N, K)) * K ** -0.5)
        b = (R.standard_normal(N) * 0.1).astype(np.float32)
        ref = act_ref(ops.linear(x, w, b), act)
        y = S.k_gemm(dev(S, x), dev(S, w), dev(S, b), act)
        check_kernel(y.float().cpu().numpy(), ref, f"gemm {M}x{N}x{K} act {act}")


def test_gelu_over_its_range(S):
    """Every fp16 value from -9 to 9 and the specials through the activation alone (identity weights).  Per element: half a unit of
    fp16's last place (6e-8 apart below 6.1e-5), and the 2.5e-7 that the polynomial may be off."""
    v = np.arange(65536, dtype=np.uint16).view(np.float16)
    v = np.concatenate([v[np.isfinite(v) & (np.abs(v.astype(np.float64)) <= 9)], np.zeros(7, np.float16)])
    v = v[:v.size // 8 * 8].reshape(-1, 8)
    y = S.k_gemm(dev(S, v), dev(S, np.eye(8, dtype=np.float16)), None, 3).float().cpu().numpy().astype(np.float64)
    ref = ops.gelu(v.astype(np.float64))
    ulp = np.maximum(2.0 ** (np.floor(np.log2(np.maximum(np.abs(ref), 1e-30))) - 10), 2.0 ** -24)
    assert np.all(np.abs(y - ref) <= 0.5 * ulp * 1.001 + 2.5e-7)
    bias = np.array([np.inf, -np.inf, np.nan, 6.5, -6.5, -30000, 30000, 0], np.float32)
    y = S.k_gemm(dev(S, np.zeros((1, 8), np.float16)), dev(S, np.eye(8, dtype=np.float16)), dev(S, bias), 3).float().cpu().numpy()[0]
    assert y[0] == np.inf and not np.isfinite(y[2]) and np.array_equal(y[[1, 3, 4, 5, 6, 7]], [0, 6.5, 0, 0, 30000, 0])


@pytest.mark.parametrize("M,H,N,act,spread", [
    # one row; a ragged last tile of each size; one to sixteen groups of 64 channels; GELU
    (1, 64, 64, 0, 1.0), (37, 192, 576, 0, 1.0), (129, 768, 2304, 0, 1.0), (300, 768, 3072, 3, 1.0), (1025, 1024, 256, 0, 1.0), (1379, 768, 2304, 0, 1.0),
    (2600, 768, 768, 3, 1.0), (5000, 512, 2304, 0, 1.0), (8200, 768, 768, 0, 1.0), (12608, 768, 3072, 3, 1.0),
    # a row mean of 200 times the deviation
    (260, 768, 768, 0, 0.005)])
def test_gemm_with_folded_layernorm(S, M, H, N, act, spread):
    """y1 = x0 w0^T + b0 + res with its statistics, then act(LN(y1) w1^T + b1), then LN(y1) as the residual of a third product."""
    eps, rows = 1e-6, min(M, 400)
    x0, w0, b0 = f16(R.standard_normal((M, 128)) * spread), f16(R.standard_normal((H, 128)) * 128 ** -0.5), np.zeros(H, np.float32)
    res = f16(R.standard_normal((M, H)) * spread + 1.0)
    g, be = R.uniform(0.8, 1.2, H).astype(np.float32), (R.standard_normal(H) * 0.1).astype(np.float32)
    w1, b1 = f16(R.standard_normal((N, H)) * H ** -0.5), (R.standard_normal(N) * 0.1).astype(np.float32)
    y1, st = S.k_gemm_ln(dev(S, x0), dev(S, w0), dev(S, b0), res=dev(S, res), stats=True)
    plain = S.k_gemm(dev(S, x0), dev(S, w0), dev(S, b0), res=dev(S, res))
    v = y1.cpu().numpy().astype(np.float64)
    check_kernel(v, plain.cpu().numpy().astype(np.float64), "folded: first product")
    q = v.reshape(M, H // 64, 64)
    ref = np.stack([q.sum(-1), ((q - q.mean(-1, keepdims=True)) ** 2).sum(-1)], -1)
    # 64 additions and 64 squares in 32 bits
    assert np.all(np.abs(st.cpu().numpy() - ref) <= 1e-5 * np.stack([np.abs(q).sum(-1), ref[..., 1] + 1e-6 * (q ** 2).sum(-1)], -1))
    wl, cs, bl = S.k_fold_layernorm(dev(S, w1), dev(S, b1), dev(S, g), dev(S, be))
    wg = w1.astype(np.float64) * g                     # rounded to fp16 once, or to fp32 and then to fp16
    assert np.all(np.abs(wl.cpu().numpy() - wg) <= np.abs(wg) * 2.0 ** -11 * 1.001 + 2.0 ** -25)
    y2, _ = S.k_gemm_ln(y1, wl, bl, act, ln_stats=st, ln_csum=cs, ln_eps=eps)
    at = np.linspace(0, M - 1, rows).astype(int)
    norm = ops.layernorm(v[at], g, be, eps)
    check_kernel(y2.float().cpu().numpy()[at], act_ref(ops.linear(norm, w1, b1), act), f"folded: {M}x{N}x{H} act {act}")
    # the third product's residual is LN(y1); K of 1088 and few tiles: the residual goes through LDS, else it is fetched early
    for K in (64, 1088):
        x3, w3 = f16(R.standard_normal((M, K))), f16(R.standard_normal((H, K)) * K ** -0.5)
        y3, s3 = S.k_gemm_ln(dev(S, x3), dev(S, w3), dev(S, b0), res=y1, ln_stats=st, ln_g=dev(S, g), ln_b=dev(S, be), ln_eps=eps, stats=True)
        o = y3.cpu().numpy().astype(np.float64)
        check_kernel(o[at], norm + ops.linear(x3[at], w3, b0), f"folded residual: {M}x{H}x{K}")
        assert np.all(np.abs(s3.cpu().numpy()[..., 0] - o.reshape(M, H // 64, 64).sum(-1)) <= 1e-5 * np.abs(o).reshape(M, H // 64, 64).sum(-1))


def test_gemm_with_folded_layernorm_of_equal_numbers_and_errors(S):
    """A row of equal numbers normalises to beta alone; infinities stay in their row; what the kernel has no form for is refused."""
    x = np.full((70, 128), 3.0, np.float16)
    x[1], x[2, 5], x[3] = 0, np.inf, R.standard_normal(128)
    w, b = f16(R.standard_normal((64, 128))), np.ones(64, np.float32)
    g, be = np.full(128, 2, np.float32), R.standard_normal(128).astype(np.float32)
    wl, cs, bl = S.k_fold_layernorm(dev(S, w), dev(S, b), dev(S, g), dev(S, be))
    q = x.astype(np.float32).reshape(70, 2, 64)
    with np.errstate(invalid="ignore"):
        st = np.stack([q.sum(-1), ((q - q.mean(-1, keepdims=True)) ** 2).sum(-1)], -1)
    y = S.k_gemm_ln(dev(S, x), wl, bl, ln_stats=dev(S, st), ln_csum=cs, ln_eps=1e-12)[0].float().cpu().numpy()
    beta = ops.linear(be[None], w, b)[0]
    ok = np.r_[0, 1, 4:70]
    check_kernel(y[ok], np.broadcast_to(beta, (68, 64)), "equal rows")
    check_kernel(y[3:4], ops.linear(ops.layernorm(x[3:4].astype(np.float64), g, be, 1e-12), w, b), "ordinary row")
    x, st, r = dev(S, x), dev(S, st), dev(S, np.zeros((70, 64), np.float16))
    for bad in (dict(w=wl), dict(w=wl, ln_stats=st), dict(w=wl, ln_stats=st, ln_csum=cs, res=r), dict(w=wl, stats=True), dict(w=wl, ln_stats=st, ln_csum=cs, act=1),
                dict(w=wl, ln_stats=st, ln_csum=cs, stats=True, res=r), dict(w=wl, res=r, stats=True, ln_stats=st), dict(w=wl[:40], ln_stats=st, ln_csum=cs)):
        with pytest.raises(S.StraitError):
            S.k_gemm_ln(x, bias=bl, **bad)


@pytest.mark.parametrize("H", [448, 832, 896, 960, 768, 1024])      # of the first four, 1 / H is no fp32 number whose product with a sum gives the mean
@pytest.mark.parametrize("M", [70, 2600])
def test_folded_layernorm_of_equal_numbers_at_every_kind_of_width(S, H, M):
    """A row of equal numbers, any finite one, is beta alone: as a residual to the last bit, as an input to the product's rounding."""
    rng = np.random.default_rng(H + M)
    v = rng.integers(0, 65536, 4 * M, dtype=np.uint16).view(np.float16)
    v = v[np.isfinite(v)][:M]
    v[:2] = 1.75, 100
    g, be = rng.uniform(0.8, 1.2, H).astype(np.float32), (rng.standard_normal(H) * 0.1).astype(np.float32)
    zero, wz, bz = np.zeros((M, 64), np.float16), np.ones((H, 64), np.float16), np.zeros(H, np.float32)
    y1, st = S.k_gemm_ln(dev(S, zero), dev(S, wz), dev(S, bz), res=dev(S, np.repeat(v[:, None], H, 1)), stats=True)
    assert np.array_equal(y1.cpu().numpy(), np.repeat(v[:, None], H, 1))
    y, _ = S.k_gemm_ln(dev(S, zero), dev(S, wz), dev(S, bz), res=y1, ln_stats=st, ln_g=dev(S, g), ln_b=dev(S, be), ln_eps=1e-12, stats=True)
    assert np.array_equal(y.cpu().numpy(), np.broadcast_to(be.astype(np.float16), (M, H)))
    w, b = f16(rng.standard_normal((192, H)) * H ** -0.5), (rng.standard_normal(192) * 0.1).astype(np.float32)
    wl, cs, bl = S.k_fold_layernorm(dev(S, w), dev(S, b), dev(S, g), dev(S, be))
    y, _ = S.k_gemm_ln(y1, wl, bl, ln_stats=st, ln_csum=cs, ln_eps=1e-12)
    check_kernel(y.float().cpu().numpy(), np.broadcast_to(ops.linear(be[None], w, b), (M, 192)), f"equal rows of {H}")


@pytest.mark.parametrize("M,N,K,use_res", [
    # many sizes of output, ragged in pixels and (where the layer allows it) in channels and slices
    (6311, 2304, 512, False), (8617, 1160, 64, False), (8347, 456, 64, True), (6455, 1184, 136, False), (8298, 280, 192, True),
    (4881, 1584, 136, False), (8491, 208, 136, True), (8466, 72, 520, False), (8894, 648, 64, True), (8514, 200, 64, False),
    (8387, 72, 64, True), (8250, 16, 192, False), (77, 40, 64, False), (45, 72, 520, True),
    # longer reductions
    (2891, 136, 768, True), (661, 208, 512, False),
    # one slice, fewer slices than the ring holds, exactly as many, one more
    (300, 64, 32, False), (300, 64, 96, False), (300, 64, 128, True), (9000, 256, 192, False), (9000, 256, 256, False)])
def test_gemm_tiles_integer_data_is_bit_exact(S, M, N, K, use_res):
    """Small integers are exact in fp16 and fp32: every tile, its ring of slices and its edges must reproduce the product."""
    x = R.integers(-2, 3, (M, K)).astype(np.float16)
    w = (R.integers(-1, 2, (N, K)) * (R.random((N, K)) < 0.3)).astype(np.float16)
    b = R.integers(-5, 6, N).astype(np.float32)
    res = R.integers(-9, 10, (M, N)).astype(np.float16) if use_res else None
    ref = x.astype(np.float64) @ w.astype(np.float64).T + b + (0 if res is None else res.astype(np.float64))
    assert np.abs(ref).max() < 2048
    y = S.k_gemm(dev(S, x), dev(S, w), dev(S, b), 0, None if res is None else dev(S, res))
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("M,N,K", [(300, 64, 96), (9000, 256, 96), (9000, 256, 160), (6455, 1184, 136), (1000, 264, 40), (77, 40, 72)])
def test_gemm_infinite_weights_stay_in_their_channel(S, M, N, K):
    """Reductions that end inside a slice: what lies behind a weight row's end is the next row, whose infinities must not
    meet the zeros that fill up the slice of the input."""
    x = R.integers(1, 3, (M, K)).astype(np.float16)
    w = R.integers(-1, 2, (N, K)).astype(np.float16)
    want = x.astype(np.float64) @ w.astype(np.float64).T
    w[3::7] = np.inf
    want[:, 3::7] = np.inf
    y = S.k_gemm(dev(S, x), dev(S, w), None)
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), want)


@pytest.mark.parametrize("N,H,C,K,Rk", [
    (97, 1, 3072, 768, 1), (128, 1, 3072, 768, 1), (192, 1, 3072, 768, 1),    # a transformer block's second product, one or two short sequences
    (33, 1, 3072, 768, 1), (640, 1, 4096, 768, 1), (500, 1, 3104, 520, 1),    # fewer rows, the largest output (120 tiles), ragged everywhere
    (1, 7, 512, 512, 3), (8, 14, 128, 256, 3), (3, 9, 160, 72, 3)])           # gathered: three sizes of output
def test_residual_is_added_before_the_only_rounding(S, N, H, C, K, Rk):
    """Long reductions for few outputs: products between 2048 and 4096, of which fp16 holds the even ones, and a residual that
    leaves 0 or 1 of them.  Exact only if the sum is formed in fp32 and rounded once."""
    kg = C * Rk * Rk
    x = R.integers(0, 3, (N, H, H, C)).astype(np.float16)
    w = (np.floor(2900 / kg) + (R.random((K, C, Rk, Rk)) < 2900 / kg % 1)).astype(np.float16)      # 2900 on average away from the border
    b = R.integers(0, 6, K).astype(np.float32)
    full = ops.conv2d(x, w, b, 1, Rk // 2)
    inside = (full > 2048) & (full < 4096)
    assert inside.mean() > 0.4
    res = np.where(inside, -2 * np.floor(full / 2), 0)
    want = np.where(inside, full + res, 0)
    y = S.k_conv2d(dev(S, x), dev(S, np.ascontiguousarray(np.transpose(w, (0, 2, 3, 1)))), dev(S, b), 1, Rk // 2, 0, dev(S, res.astype(np.float16)))
    assert np.array_equal(np.where(inside, y.float().cpu().numpy().astype(np.float64), 0), want)


@pytest.mark.parametrize("N,H,C,K,Rk,stride,pad,use_res,out_f32", [
    (1, 7, 512, 512, 3, 1, 1, False, False),     # 49 pixels: a ragged fourth tile; 72 super-slices over four wavefronts
    (1, 14, 192, 40, 3, 2, 1, True, False),      # stride 2, channels ragged in the tile; 27 super-slices: unequal parts
    (3, 1, 192, 10, 1, 1, 0, False, True),       # three super-slices: one wavefront has none; ten fp32 outputs
    (5, 1, 2048, 1000, 1, 1, 0, False, True),    # a classifier
    (1, 1, 64, 7, 1, 1, 0, False, True),         # the smallest: one row, one super-slice, odd outputs
    (1, 9, 256, 96, 1, 2, 0, False, False)])     # a strided projection
def test_small_outputs_integer_data_is_bit_exact(S, N, H, C, K, Rk, stride, pad, use_res, out_f32):
    """Few outputs, the reduction shared out over the wavefronts of a workgroup: partial sums and their meeting in LDS are
    exact on integer data."""
    x = R.integers(-2, 3, (N, H, H, C)).astype(np.float16)
    w = (R.integers(-1, 2, (K, C, Rk, Rk)) * (R.random((K, C, Rk, Rk)) < 0.2)).astype(np.float16)
    b = R.integers(-5, 6, K).astype(np.float32)
    ref = ops.conv2d(x, w, b, stride, pad)
    res = R.integers(-9, 10, ref.shape).astype(np.float16) if use_res else None
    if use_res:
        ref = ref + res.astype(np.float64)
    assert np.abs(ref).max() < 2048
    y = S.k_conv2d(dev(S, x), dev(S, np.ascontiguousarray(np.transpose(w, (0, 2, 3, 1)))), dev(S, b), stride, pad, 0,
                   None if res is None else dev(S, res), out_f32)
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), ref)


def test_small_outputs_gelu_and_second_source(S):
    """The same kernel with GELU on a short token sequence, and with a second source of its reduction."""
    x, w, b = f16(R.standard_normal((19, 768))), f16(R.standard_normal((136, 768)) * 768 ** -0.5), R.standard_normal(136).astype(np.float32)
    y = S.k_gemm(dev(S, x), dev(S, w), dev(S, b), 3)
    check_kernel(y.float().cpu().numpy(), ops.gelu(ops.linear(x, w, b)), "gemm 19x136x768 gelu")
    x1, x2 = R.integers(-2, 3, (1, 7, 7, 128)).astype(np.float16), R.integers(-2, 3, (1, 14, 14, 192)).astype(np.float16)
    wp = (R.integers(-1, 2, (72, 320)) * (R.random((72, 320)) < 0.3)).astype(np.float16)
    bp = R.integers(-5, 6, 72).astype(np.float32)
    ref = np.concatenate([x1, x2[:, ::2, ::2]], -1).astype(np.float64) @ wp.astype(np.float64).T + bp
    y = S.k_conv1x1_proj(dev(S, x1), dev(S, x2), 2, dev(S, wp), dev(S, bp))
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("N,H,C,K,Rk,act,use_res,out_f32,kernel", [
    (13, 1, 25088, 1000, 1, 0, False, False, "slabs 64x64x64"),      # ragged rows and channels, 392 slices over many parts
    (9, 1, 16352, 72, 1, 1, True, False, "slabs 64x64x32"),          # a reduction of no whole 64-wide slices, residual and ReLU in the second launch
    (385, 1, 8192, 1024, 1, 0, True, True, "slabs 64x64x64"),        # 112 tiles in a few parts, fp32 residual sums out
    (270, 1, 4096, 512, 1, 2, False, True, "slabs 64x64x64"),        # ReLU6
    (8, 7, 1024, 512, 3, 0, True, True, "slabs 64x64x64"),           # gathered: parts start in the middle of a filter
    (2, 9, 544, 64, 3, 0, False, False, "slabs 64x64x32")])          # ... with channels in halves of a slice
def test_split_reductions_integer_data_is_bit_exact(S, N, H, C, K, Rk, act, use_res, out_f32, kernel):
    """Few outputs behind a long reduction: fp32 slabs of several workgroups per tile, added and finished by a second launch.
    Small integers: exact in any order."""
    assert S.k_conv2d_kernel(N, H, H, C, K, Rk, 1, Rk // 2, act, use_res, out_f32) == kernel
    x = R.integers(-2, 3, (N, H, H, C)).astype(np.float16)
    w = (R.integers(-1, 2, (K, C, Rk, Rk)) * (R.random((K, C, Rk, Rk)) < 0.1)).astype(np.float16)
    b = R.integers(-5, 6, K).astype(np.float32)
    ref = ops.conv2d(x, w, b, 1, Rk // 2)
    res = R.integers(-9, 10, ref.shape).astype(np.float16) if use_res else None
    ref = act_ref(ref + (0 if res is None else res.astype(np.float64)), act)
    assert np.abs(ref).max() < 2048
    y = S.k_conv2d(dev(S, x), dev(S, np.ascontiguousarray(np.transpose(w, (0, 2, 3, 1)))), dev(S, b), 1, Rk // 2, act,
                   None if res is None else dev(S, res), out_f32)
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("kernel,shape,use_res", LAYERS, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v).replace(" ", "_"))
def test_every_kernel_integer_data_is_bit_exact(S, kernel, shape, use_res):
    """Small integers are exact in fp16 and fp32, in any order of addition: every kernel, its ring of slices, its edges and its way
    to add a residual against the taps' products in fp32."""
    N, H, W, C, K, Rk, stride, pad = shape
    assert S.k_conv2d_kernel(N, H, W, C, K, Rk, stride, pad, res=use_res) == kernel
    g = S.torch.Generator(device="cuda").manual_seed(N * H + C * K)
    ints = lambda lo, hi, size: S.torch.randint(lo, hi, size, generator=g, device="cuda").float()
    x = ints(-2, 3, (N, H, W, C))
    w = ints(-1, 2, (K, Rk, Rk, C)) * (ints(0, 10, (K, Rk, Rk, C)) < 3)
    b = ints(-5, 6, (K,))
    P, Q = (H + 2 * pad - Rk) // stride + 1, (W + 2 * pad - Rk) // stride + 1
    xp = S.torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    ref = b.expand(N * P * Q, K).clone()
    for r in range(Rk):
        for s in range(Rk):
            ref += xp[:, r:r + (P - 1) * stride + 1:stride, s:s + (Q - 1) * stride + 1:stride].reshape(-1, C) @ w[:, r, s].T.contiguous()
    res = ints(-9, 10, (N, P, Q, K)) if use_res else None
    if use_res:
        ref += res.reshape(ref.shape)
    assert ref.abs().max() < 2048
    y = S.k_conv2d(x.half(), w.half(), b, stride, pad, 0, None if res is None else res.half())
    assert S.torch.equal(y.float().reshape(ref.shape), ref)


@pytest.mark.parametrize("tile,shapes", [
    # one slice, a few, more than the ring holds; short patches and, in the second half, the longest ones
    ("32x16", [(9, 42, 4, 64, 16), (17, 52, 8, 128, 16), (40, 10, 6, 512, 16), (2, 59, 27, 64, 16), (3, 14, 24, 192, 96), (2, 4, 22, 320, 160)]),
    ("64x16", [(17, 43, 4, 64, 64), (3, 52, 5, 192, 256), (9, 29, 6, 320, 80), (1, 25, 55, 64, 160), (2, 34, 17, 192, 160), (9, 3, 62, 320, 96)]),
    ("64x32", [(40, 56, 6, 64, 32), (5, 34, 8, 128, 256), (17, 40, 8, 320, 64), (1, 33, 50, 64, 160), (9, 17, 45, 192, 64), (9, 56, 28, 512, 32)]),
    ("128x32", [(9, 32, 19, 64, 160), (3, 43, 30, 192, 160), (9, 40, 30, 512, 64), (3, 46, 62, 64, 96), (3, 46, 62, 192, 96), (5, 43, 50, 704, 64)])])
def test_small_3x3_integer_data_is_bit_exact(S, tile, shapes):
    """The 3x3 kernel of small images, each tile: ragged last tiles, images of any height, rounds of workgroups."""
    for N, H, W, C, K in shapes:
        test_every_kernel_integer_data_is_bit_exact(S, "small 3x3 " + tile, (N, H, W, C, K, 3, 1, 1), False)
        x, w = f16(R.standard_normal((N, H, W, C))), f16(R.standard_normal((K, 3, 3, C)) * (9 * C) ** -0.5)
        y = S.k_conv2d(dev(S, x), dev(S, w), None, 1, 1, 2)                 # no bias, ReLU6
        ref = S.torch.nn.functional.conv2d(dev(S, x).float().permute(0, 3, 1, 2), dev(S, w).float().permute(0, 3, 1, 2), padding=1).permute(0, 2, 3, 1)
        check_kernel(y.float().cpu().numpy(), ref.clamp(0, 6).cpu().numpy(), f"small 3x3 {tile} {N}x{H}x{W}x{C}->{K}")


@pytest.mark.parametrize("kernel,shape,use_res", [
    ("128x64x64", (1659, 1, 1, 2768, 904, 1, 1, 0), False), ("128x64x64", (5191, 1, 1, 1312, 368, 1, 1, 0), False), ("128x64x64", (1379, 1, 1, 768, 768, 1, 1, 0), True),
    ("128x64x64", (8827, 1, 1, 1960, 144, 1, 1, 0), True), ("128x64x64", (35, 9, 33, 384, 344, 3, 2, 1), False), ("128x64x64", (25, 27, 41, 256, 144, 3, 2, 1), True),
    # either side of the length from which the 128 x 128 tile of 8 wavefronts reads its operands three steps ahead
    ("128x128x64, 8 wavefronts", (12877, 1, 1, 448, 144, 1, 1, 0), True), ("128x128x64, 8 wavefronts", (2740, 1, 1, 920, 1160, 1, 1, 0), True),
    ("128x128x64, 8 wavefronts", (4975, 1, 1, 2376, 680, 1, 1, 0), True)])
def test_operands_read_ahead_integer_data_is_bit_exact(S, kernel, shape, use_res):
    """Tiles whose operands are read three steps ahead: ragged rows, channels and slices, few slices and many."""
    test_every_kernel_integer_data_is_bit_exact(S, kernel, shape, use_res)


@pytest.mark.parametrize("tile,shapes", [
    # each length of the patch, odd and even numbers of slices, the narrowest and the widest images
    ("96x128", [(17, 7, 46, 128, 384), (32, 44, 4, 192, 384), (10, 13, 42, 192, 384), (2, 58, 47, 128, 384), (33, 3, 55, 192, 384), (3, 29, 63, 192, 384), (2, 41, 62, 512, 256)]),
    ("192x128", [(24, 64, 30, 128, 128), (40, 64, 5, 192, 384), (4, 58, 47, 192, 384), (25, 59, 31, 128, 128), (22, 33, 63, 128, 128), (27, 19, 64, 192, 128)])])
def test_mid_3x3_integer_data_is_bit_exact(S, tile, shapes):
    """The 3x3 kernel of mid-size layers, each tile: ragged last tiles, images of any height, two rounds of workgroups."""
    for N, H, W, C, K in shapes:
        test_every_kernel_integer_data_is_bit_exact(S, "mid 3x3 " + tile, (N, H, W, C, K, 3, 1, 1), False)
        x, w = f16(R.standard_normal((N, H, W, C))), f16(R.standard_normal((K, 3, 3, C)) * (9 * C) ** -0.5)
        y = S.k_conv2d(dev(S, x), dev(S, w), None, 1, 1, 2)                 # no bias, ReLU6
        ref = S.torch.nn.functional.conv2d(dev(S, x).float().permute(0, 3, 1, 2), dev(S, w).float().permute(0, 3, 1, 2), padding=1).permute(0, 2, 3, 1)
        check_kernel(y.float().cpu().numpy(), ref.clamp(0, 6).cpu().numpy(), f"mid 3x3 {tile} {N}x{H}x{W}x{C}->{K}")


def test_split_reduction_under_capture(S):
    """A product whose reduction is split allocates a workspace; on a stream that records a graph it takes a kernel that needs none."""
    M, N, K = 270, 512, 4096
    assert S.k_conv2d_kernel(M, 1, 1, K, N, 1, 1, 0, out_f32=True).startswith("slabs")
    x = R.integers(-2, 3, (M, K)).astype(np.float16)
    w = R.integers(-1, 2, (N, K)).astype(np.float16)
    want = x.astype(np.float64) @ w.astype(np.float64).T
    dx, dw = dev(S, x), dev(S, w)
    eager = S.k_gemm(dx, dw, None, 0, None, True)
    S.torch.cuda.synchronize()
    graph = S.torch.cuda.CUDAGraph()
    with S.torch.cuda.graph(graph):
        y = S.k_gemm(dx, dw, None, 0, None, True)
    for _ in range(3):
        y.fill_(float("nan"))
        graph.replay()
        S.torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().astype(np.float64), want)
        assert S.torch.equal(S.k_gemm(dx, dw, None, 0, None, True), eager)
    assert np.array_equal(eager.cpu().numpy().astype(np.float64), want)


@pytest.mark.parametrize("n,k,act,res", [(576, 96, 2, False), (384, 128, 0, False), (768, 768, 1, True), (3072, 768, 3, False), (1280, 320, 2, False), (768, 3072, 0, False)])
def test_products_of_fewer_rows_on_other_tiles_have_the_same_bits(S, n, k, act, res):
    """What batches that are computed part by part rely on: on all tiles on which one group of wavefronts reduces, a row's result is the same bit for bit, wherever in a tile it lies."""
    t = S.torch
    full = 25600
    x, w = t.randn((full, k), device="cuda").half(), (t.randn((n, k), device="cuda") * (2.0 / k) ** 0.5).half()
    b, r = t.randn(n, device="cuda") * 0.02, t.randn((full, n), device="cuda").half() if res else None
    y, tiles = S.k_gemm(x, w, b, act=act, res=r), set()
    for at, m in ((0, 60), (100, 200), (7, 900), (0, 1500), (4000, 3300), (33, 5000), (1000, 12600), (95, 20000)):
        tile = S.k_conv2d_kernel(m, 1, 1, k, n, 1, 1, 0, act=act, res=res)
        if not tile[0].isdigit() or "groups" in tile:
            continue
        tiles.add(tile)
        part = S.k_gemm(x[at:at + m].contiguous(), w, b, act=act, res=r[at:at + m].contiguous() if res else None)
        assert t.equal(part, y[at:at + m]), (tile, m, int((part != y[at:at + m]).sum()))
    assert len(tiles) >= 3, tiles
