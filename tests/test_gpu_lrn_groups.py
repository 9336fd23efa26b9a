"""LRN at the edges of its pixel groups (4) and channel chunks (8), on planes
below one group, and on outputs stored past L2."""
import numpy as np
import pytest
import torch

import oracle
from conftest import to_dev, to_host
from paper_1511_07376_amd import workloads as wl
from parity import assert_elementwise_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1, 3, 5, 7, 9])
@pytest.mark.parametrize("shape", [
    (3, 1, 1, 1), (2, 9, 1, 3), (65, 8, 1, 2), (2, 7, 2, 2), (5, 17, 1, 5), (1, 16, 7, 9), (67, 33, 3, 5),
    (1, 8, 16, 16), (3, 40, 15, 17),
], ids=lambda s: "x".join(map(str, s)))
def test_lrn_group_and_chunk_edges(gpu, shape, size):
    x = wl.normal(shape, 20.0, 50, 0)
    print(shape, size, flush=True)
    y = to_host(gpu.cnn_lrn_fwd(to_dev(x), size, 1e-2, 0.75, 1.0))
    assert_elementwise_close(y, oracle.lrn_fwd(x, size, 1e-2, 0.75, 1.0), np.abs(x).max(), f"lrn {shape} {size}")


def test_lrn_output_larger_than_l2(gpu):
    """37 MB: the same values per image as the image by itself (plain stores)."""
    x = to_dev(wl.normal((31, 96, 55, 57), 20.0, 51, 0))
    y = gpu.cnn_lrn_fwd(x, 5)
    for n in (0, 15, 30):
        np.testing.assert_array_equal(to_host(y[n:n + 1]), to_host(gpu.cnn_lrn_fwd(x[n:n + 1].contiguous(), 5)))


@pytest.mark.parametrize("batch", [2, 31, 116])
def test_lrn_in_a_network_gives_the_same_values(gpu, batch):
    """1, 37 and 140 MB: a network's line between the kinds of stores (input and
    output together 256 MiB) lies elsewhere than a standalone call's."""
    net = wl.Net(name="lrn", input_chw=(96, 55, 57), layers=(wl.lrn(5),), weight_std=0.0, bias_std=0.0,
                 default_batch=batch, batches=(batch,))
    x = torch.rand((batch, 96, 55, 57), device="cuda") * 20
    y = gpu.Network(net, [None])(x)
    assert torch.equal(y, gpu.cnn_lrn_fwd(x, 5))
