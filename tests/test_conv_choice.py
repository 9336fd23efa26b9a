"""The built-in choice of a convolution configuration (host code, no GPU)."""
import ctypes

import pytest

from paper_1511_07376_amd import cnn

FIRST_SPLIT, FIRST_DIRECT = 16, 22  # configurations below take the fp32 tiles


def choice(n, c, h, w, k, r, s, stride, pad, groups, in_net=False):
    """conv2d_heuristic_config of the shape."""
    p, q = cnn.cnn_conv2d_out_shape(h, w, r, s, stride, pad)
    shape = (ctypes.c_int * 14)(n, c, h, w, k, r, s, stride, stride, pad, pad, groups, p, q)
    return cnn.lib._ZN3cnn23conv2d_heuristic_configERKNS_9ConvShapeEb(ctypes.byref(shape), in_net)


# N, C, H, W, K, R, S, stride, pad, groups; us on the fp32 choice, and on the
# split or direct kernel that an earlier fit of the estimates took instead
@pytest.mark.parametrize("shape", [
    (75, 206, 11, 11, 322, 3, 3, 1, 0, 1),   # 106.5, 150.5
    (163, 298, 18, 16, 127, 3, 3, 1, 0, 1),  # 235.9, 329.8
    (40, 4, 78, 93, 89, 7, 1, 2, 0, 1),      # 23.2, 32.3
    (5, 54, 32, 29, 22, 5, 5, 1, 0, 1),      # 13.6, 18.6
    (58, 8, 83, 82, 76, 1, 3, 2, 0, 1),      # 23.5, 31.7
    (26, 115, 22, 19, 194, 3, 3, 1, 0, 1),   # 62.2, 82.1
], ids=lambda s: "x".join(map(str, s)))
def test_fp32_tiles_where_they_are_faster(shape):
    assert 0 <= choice(*shape) < FIRST_SPLIT


@pytest.mark.parametrize("shape,first,last", [
    ((64, 256, 28, 28, 256, 3, 3, 1, 1, 1), FIRST_SPLIT, FIRST_DIRECT),  # 502.6 us on fp32 tiles, 390.6
    ((64, 3, 227, 227, 96, 11, 11, 4, 0, 1), FIRST_SPLIT, FIRST_DIRECT),  # 137.8, 131.9
    ((64, 512, 14, 14, 512, 3, 3, 1, 1, 1), FIRST_SPLIT, FIRST_DIRECT),  # 551.8, 378.8
    ((16, 20, 12, 12, 50, 5, 5, 1, 0, 1), FIRST_DIRECT, 25),             # 17.5, 8.4
    ((1, 64, 56, 56, 64, 3, 3, 1, 1, 1), FIRST_DIRECT, 25),              # 19.4, 8.6
], ids=str)
def test_split_and_direct_kernels_where_they_are_faster(shape, first, last):
    assert first <= choice(*shape) < last


def test_launch_bound_calls_keep_the_fp32_tiles():
    for shape in ((2, 24, 18, 15, 118, 3, 3, 1, 0, 2), (1, 3, 9, 9, 16, 3, 3, 1, 0, 1), (2, 8, 79, 61, 20, 3, 3, 1, 1, 2)):
        assert choice(*shape) < FIRST_SPLIT


@pytest.mark.parametrize("n", [1, 8, 64, 256])
def test_sums_of_one_tap_stay_in_fp32(n):
    """The split kernels are less accurate there; the direct ones are fp32."""
    for c, groups in ((1, 1), (64, 64), (512, 512)):
        for k in (512, 1024):
            for h in (7, 56, 112):
                if n * max(c, k) * h * h < 1 << 31:
                    assert not FIRST_SPLIT <= choice(n, c, h, h, k, 1, 1, 1, 0, groups) < FIRST_DIRECT
    takes = cnn.lib._ZN3cnn19conv2d_config_takesERKNS_9ConvShapeEi
    takes.restype = ctypes.c_bool
    one, two = ((ctypes.c_int * 14)(n, c, 14, 14, 64, 1, 1, 1, 1, 0, 0, 1, 14, 14) for c in (1, 2))
    for cfg in range(cnn.cnn_conv2d_num_configs()):
        assert takes(ctypes.byref(two), cfg)
        assert takes(ctypes.byref(one), cfg) == (not FIRST_SPLIT <= cfg < FIRST_DIRECT)
    # a reduction beyond the direct kernels' tap tables is not tuned under their names
    long = (ctypes.c_int * 14)(16, 1024, 15, 15, 60, 3, 3, 1, 1, 1, 1, 1, 15, 15)
    assert [takes(ctypes.byref(long), cfg) for cfg in range(FIRST_DIRECT, cnn.cnn_conv2d_num_configs())] == [False] * 3


@pytest.mark.parametrize("shape", [
    (16, 256, 15, 15, 384, 3, 3, 1, 0, 1),  # AlexNet's conv3 at batch 16
    (1, 256, 15, 15, 384, 3, 3, 1, 0, 1),   # ... on one image
], ids=["b16", "b1"])
def test_split_reductions_are_cheaper_inside_a_network(shape):
    """Their fill and ReLU cost a standalone call two launches, a network none."""
    assert choice(*shape) >= FIRST_DIRECT
    assert choice(*shape, in_net=True) < FIRST_SPLIT
