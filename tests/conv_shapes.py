"""For every kernel and tile of the convolution dispatch, pointwise and gathered, with and without a residual, a small layer that
it is chosen for: ragged in pixels, and in channels and slices where the kernel allows it."""

# kernel, (N, H, W, C, K, R, stride, pad), residual
LAYERS = [
    ("128x128x64", (9305, 1, 1, 264, 840, 1, 1, 0), False),
    ("128x128x64", (4978, 1, 1, 192, 1584, 1, 1, 0), True),
    ("128x128x64", (178, 14, 22, 64, 72, 3, 1, 1), False),
    ("128x128x64, 8 wavefronts", (12955, 1, 1, 104, 152, 1, 1, 0), False),
    ("128x128x64, 8 wavefronts", (12877, 1, 1, 128, 144, 1, 1, 0), True),
    ("128x128x64, 8 wavefronts", (16, 44, 18, 64, 136, 3, 1, 1), False),
    ("128x256x64", (10824, 1, 1, 120, 648, 1, 1, 0), False),
    ("128x256x64", (28285, 1, 1, 256, 152, 1, 1, 0), True),
    ("128x256x64", (9, 58, 50, 64, 144, 3, 1, 1), False),
    ("128x64x32, 2 slices", (33071, 1, 1, 8, 8, 1, 1, 0), False),
    ("128x64x32, 2 slices", (33603, 1, 1, 8, 8, 1, 1, 0), True),
    ("128x64x32, 2 slices", (115, 53, 35, 32, 8, 3, 1, 1), False),
    ("128x64x32, 3 slices", (16898, 1, 1, 8, 8, 1, 1, 0), False),
    ("128x64x32, 3 slices", (16557, 1, 1, 8, 8, 1, 1, 0), True),
    ("128x64x32, 3 slices", (18, 21, 50, 32, 8, 3, 1, 1), False),
    ("128x64x32, 3 slices", (5, 47, 70, 64, 8, 3, 1, 1), True),
    ("192x128x64", (4366, 1, 1, 8, 1360, 1, 1, 0), False),
    ("192x128x64", (34146, 1, 1, 40, 72, 1, 1, 0), True),
    ("192x128x64", (91, 40, 40, 64, 72, 3, 2, 1), False),
    ("256x128x32", (49817, 1, 1, 8, 72, 1, 1, 0), False),
    ("256x128x32", (53363, 1, 1, 72, 72, 1, 1, 0), True),
    ("256x128x32", (37, 60, 64, 32, 72, 3, 2, 1), False),
    ("256x192x64", (59493, 1, 1, 40, 136, 1, 1, 0), False),
    ("256x192x64", (54591, 1, 1, 128, 144, 1, 1, 0), True),
    ("256x192x64", (10, 60, 60, 64, 136, 3, 1, 1), False),
    ("256x192x64", (16, 66, 130, 64, 160, 3, 2, 1), True),
    ("256x256x64", (16485, 1, 1, 512, 672, 1, 1, 0), False),
    ("256x256x64", (50923, 1, 1, 512, 216, 1, 1, 0), True),
    ("256x256x64", (160, 27, 29, 64, 216, 3, 2, 1), False),
    ("32x64x64", (24, 1, 1, 104, 8, 1, 1, 0), False),
    ("32x64x64", (20, 1, 1, 120, 8, 1, 1, 0), True),
    ("32x64x64", (5571, 1, 1, 1032, 8, 1, 1, 0), True),        # the residual added in fp32
    ("32x64x64", (7, 47, 21, 64, 8, 3, 1, 1), False),
    ("32x64x64", (10, 55, 55, 128, 48, 3, 2, 1), True),        # the residual added in fp32
    ("32x64x64, 4 groups", (20, 1, 1, 608, 8, 1, 1, 0), False),
    ("32x64x64, 4 groups", (21, 1, 1, 600, 8, 1, 1, 0), True),
    ("32x64x64, 4 groups", (20, 1, 1, 1072, 8, 1, 1, 0), True),        # the residual added in fp32
    ("32x64x64, 4 groups", (5, 9, 130, 128, 8, 3, 1, 1), False),
    ("32x64x64, 4 groups", (13, 17, 27, 128, 8, 3, 1, 1), True),        # the residual added in fp32
    ("64x128x64", (8337, 1, 1, 320, 72, 1, 1, 0), False),
    ("64x128x64", (10930, 1, 1, 256, 72, 1, 1, 0), True),
    ("64x128x64", (7, 29, 43, 64, 72, 3, 1, 1), False),
    ("64x64x32", (20, 1, 1, 8, 8, 1, 1, 0), False),
    ("64x64x32", (21, 1, 1, 8, 8, 1, 1, 0), True),
    ("64x64x32", (1, 27, 27, 32, 8, 3, 2, 1), False),
    ("64x64x32", (7, 6, 6, 160, 16, 3, 2, 1), True),        # the residual added in fp32
    ("64x64x64", (8670, 1, 1, 168, 8, 1, 1, 0), False),
    ("64x64x64", (9896, 1, 1, 168, 8, 1, 1, 0), True),
    ("64x64x64", (3, 29, 100, 64, 8, 3, 1, 1), False),
    ("64x64x64, 2 groups", (8348, 1, 1, 1896, 8, 1, 1, 0), False),
    ("64x64x64, 2 groups", (8718, 1, 1, 1752, 8, 1, 1, 0), True),
    ("64x64x64, 2 groups", (5, 42, 42, 192, 8, 3, 1, 1), False),
    ("64x64x64, 2 groups", (9, 19, 53, 192, 8, 3, 1, 1), True),
    ("96x128x64", (17600, 1, 1, 120, 72, 1, 1, 0), False),
    ("96x128x64", (16463, 1, 1, 120, 72, 1, 1, 0), True),
    ("96x128x64", (5, 60, 60, 64, 72, 3, 1, 1), False),
    ("patch 128x128", (4, 41, 100, 32, 128, 3, 1, 1), False),        # four patch transfers per wavefront
    ("patch 128x128", (17, 14, 69, 32, 128, 3, 1, 1), False),        # six patch transfers per wavefront
    ("patch 256x128", (41, 20, 20, 32, 256, 3, 1, 1), False),        # three patch transfers per wavefront
    ("patch 256x128", (15, 34, 65, 32, 128, 3, 1, 1), False),        # four patch transfers per wavefront
    ("patch 256x64", (5, 66, 100, 32, 64, 3, 1, 1), False),        # six patch transfers per wavefront
    ("patch 256x64", (8, 65, 65, 32, 64, 3, 1, 1), False),        # eight patch transfers per wavefront
    ("patch 256x64", (26, 47, 224, 32, 64, 3, 1, 1), False),        # workgroups that walk over tiles, six patch transfers
    ("patch 256x64", (61, 35, 128, 32, 64, 3, 1, 1), False),        # ... eight
]
