"""Which kernel and tile a layer is given: host code, checked without a GPU."""
import paper_2604_28175_amd as S


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
