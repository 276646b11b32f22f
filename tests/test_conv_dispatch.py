"""Which kernel and tile a layer is given: host code, checked without a GPU."""
import paper_2604_28175_amd as S


def test_a_refused_layer_has_no_kernel():
    assert S.k_conv2d_kernel(1, 2, 2, 8, 8, 5, 1, 1) is None            # window larger than the padded image
    assert "invalid shape" in S.last_error()
    assert S.k_conv2d_kernel(1, 8, 8, 3, 16, 3, 1, 1) == "through registers 64x64"     # odd channels: element by element
