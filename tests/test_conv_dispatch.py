"""Which kernel and tile a layer is given: host code, checked without a GPU."""
import paper_2604_28175_amd as S
from conv_shapes import LAYERS


def test_a_refused_layer_has_no_kernel():
    assert S.k_conv2d_kernel(1, 2, 2, 8, 8, 5, 1, 1) is None            # window larger than the padded image
    assert "invalid shape" in S.last_error()
    assert S.k_conv2d_kernel(1, 8, 8, 3, 16, 3, 1, 1) == "through registers 64x64"     # odd channels: element by element


def test_wide_3x3_layers_between_the_measured_networks():
    """Layers that had been given kernels up to 1.7 times slower than the best one that takes them."""
    for n, h, c, k, stride, want in ((16, 112, 64, 128, 1, "patch 256x128"), (33, 56, 128, 256, 1, "patch 256x128"), (261, 28, 128, 128, 1, "patch 256x128"),
                                     (588, 14, 512, 64, 1, "patch 256x64"), (64, 56, 256, 256, 1, "patch 256x128"),
                                     (118, 40, 160, 512, 2, "256x128x32"), (60, 10, 160, 2048, 1, "256x128x32")):
        assert S.k_conv2d_kernel(n, h, h, c, k, 3, stride, 1) == want, (n, h, c, k, stride)


def test_outputs_that_are_no_whole_fp16_chunks():
    """fp32 outputs and odd numbers of channels: large products go through registers, few outputs to the kernels that share the
    reduction out (they had all been given the small-output kernel, up to six times slower)."""
    def gemm(m, n, k, out_f32=True):
        return S.k_conv2d_kernel(m, 1, 1, k, n, 1, 1, 0, out_f32=out_f32)
    assert gemm(16384, 768, 4096) == gemm(8192, 1001, 1024, False) == "through registers 128x128"
    assert gemm(4096, 1000, 2048) == gemm(4096, 1001, 2048, False) == "through registers 128x64"
    assert gemm(600, 1001, 256) == gemm(2221, 1000, 768) == "through registers 64x64"
    assert gemm(9, 1000, 2048) == gemm(3, 10, 64) == gemm(12, 1001, 2048, False) == "small outputs 16x16"
    assert gemm(385, 1024, 8192) == gemm(270, 512, 4096) == "slabs 64x64x64"


def test_long_reductions_are_split_again():
    def gemm(m, n, k):
        return S.k_conv2d_kernel(m, 1, 1, k, n, 1, 1, 0)
    assert gemm(13, 1000, 25088) == gemm(20, 64, 16384) == gemm(533, 64, 16320) == "slabs 64x64x64"
    assert gemm(9, 72, 16352) == "slabs 64x64x32"                       # no whole slices of 64
    assert gemm(6, 4096, 25088) == "small outputs 16x16"                # bound by its weights: nothing to gain
    assert gemm(64, 768, 4096).startswith(("32x64x64", "64x64x64", "small"))


def test_every_kernel_has_a_layer():
    """What the bit-exactness test on the GPU relies on: its layers reach every kernel and tile, and the one they say."""
    for kernel, (n, h, w, c, k, r, stride, pad), res in LAYERS:
        assert S.k_conv2d_kernel(n, h, w, c, k, r, stride, pad, res=res) == kernel, (kernel, n, h, w, c, k, r, stride, res)
    assert len({kernel for kernel, _, _ in LAYERS}) == 19
