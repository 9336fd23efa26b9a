"""Fully connected layers on bf16 parts where they can go wrong: ragged blocks
of images and features, waves with no, one or a partial 32-tap chunk, rows of
any alignment, values that do not survive the split, and accuracy."""
import numpy as np
import pytest
import torch

import oracle
from conftest import to_dev, to_host
from paper_1511_07376_amd import workloads as wl
from parity import assert_gemm_close

pytestmark = pytest.mark.gpu


def _configs(gpu):
    return [i for i in range(gpu.cnn_fc_num_configs()) if gpu.cnn_fc_config_name(i).startswith("bf16 parts")]


@pytest.mark.parametrize("N", [3, 32, 33, 65, 129])
@pytest.mark.parametrize("I", [1, 31, 32, 33, 255, 257, 515, 1000, 1023, 1025, 2049])
def test_fc_parts_edges(gpu, N, I):
    O = 31 if N == 65 else 70
    x, w, b = wl.normal((N, I), 1.0, 60, 0), wl.normal((O, I), 1.0, 60, 1), wl.normal((O,), 1.0, 60, 2)
    for relu in (False, True):
        ref = oracle.fc_fwd(x, w, b, relu)
        for cfg in [-1] + _configs(gpu):
            print(f"N{N} I{I} relu{int(relu)} config {cfg}", flush=True)
            y = gpu.cnn_fc_fwd(to_dev(x), to_dev(w), to_dev(b), relu, config=cfg)
            assert_gemm_close(to_host(y), ref, I, f"N{N} I{I} relu{int(relu)} config {cfg}")


@pytest.mark.parametrize("I", [40, 1100])
def test_fc_parts_values_that_do_not_split(gpu, I):
    """Infinities, NaN and a value whose leading part rounds to infinity: the
    same non-finite outputs as the fp32 tiles give."""
    x, w = wl.normal((5, I), 1.0, 61, 0), wl.normal((37, I), 1.0, 61, 1)
    x[0, 2], x[1, I - 1], x[2, 7], x[3, 11] = np.inf, -np.inf, np.nan, np.float32(3.4e38)
    w[4, 3], w[36, 0] = -np.inf, np.float32(-3.395e38)
    args = to_dev(x), to_dev(w), None, False
    want = to_host(gpu.cnn_fc_fwd(*args, config=0))
    fin = np.isfinite(want) & (np.abs(want) < 1e30)
    assert np.isnan(want).any() and np.isinf(want).any() and fin.any()
    for cfg in _configs(gpu):
        got = to_host(gpu.cnn_fc_fwd(*args, config=cfg))
        np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
        np.testing.assert_array_equal(np.isinf(got) * np.sign(got), np.isinf(want) * np.sign(want))
        # each a sum of I products in fp32, within I * 2^-24 of the sum of magnitudes (below 8 I here)
        assert np.abs(got[fin] - want[fin]).max() <= 2 * I * 2.0 ** -24 * 8 * I


@pytest.mark.parametrize("I", [2, 6, 333, 4000])
def test_fc_parts_no_less_accurate_than_fp32(gpu, I):
    x, w = wl.normal((24, I), 1.0, 62, 0), wl.normal((96, I), 1.0, 62, 1)
    ref = (torch.from_numpy(x).double() @ torch.from_numpy(w).double().t()).numpy()

    def err(cfg):
        y = to_host(gpu.cnn_fc_fwd(to_dev(x), to_dev(w), None, False, config=cfg)).astype(np.float64)
        return np.linalg.norm(y - ref) / np.linalg.norm(ref)

    for cfg in _configs(gpu):
        print(f"I {I} config {cfg}: {err(cfg) / err(0):.3f}", flush=True)
        assert err(cfg) <= err(0)


@pytest.mark.parametrize("xs,ws", [(-115, 0), (0, -120), (-140, 60), (-60, -70)])
@pytest.mark.parametrize("I", [27, 333])
def test_fc_parts_of_small_values(gpu, I, xs, ws):
    """As test_parts_of_small_values of the convolutions, against the fp32 tiles."""
    x = wl.normal((24, I), 1.0, 63, 0) * np.float32(2.0 ** xs)
    w = (wl.normal((96, I), 1.0, 63, 1).astype(np.float64) * 2.0 ** ws).astype(np.float32)
    ref = (torch.from_numpy(x).double() @ torch.from_numpy(w).double().t()).numpy()

    def err(cfg):
        y = to_host(gpu.cnn_fc_fwd(to_dev(x), to_dev(w), None, False, config=cfg)).astype(np.float64)
        return np.sqrt(np.mean((y - ref) ** 2))

    for cfg in _configs(gpu):
        assert err(cfg) <= 1.02 * err(0) + 2.0 ** -150, f"config {cfg}"


@pytest.mark.parametrize("sign", [1, -1])
def test_fc_parts_just_inside_the_range(gpu, sign):
    """Products and sums within 0.1% of the largest float, of inputs whose leading parts round up."""
    for I, live in ((1, 1), (40, 16), (1100, 16)):
        x = np.zeros((5, I), np.float32)
        x[:, :live] = np.float32(1.998 * 2.0 ** 63 / live)
        w = np.full((37, I), sign * 2.0 ** 64, np.float32)
        ref = x.astype(np.float64) @ w.astype(np.float64).T
        for cfg in [0] + _configs(gpu):
            got = to_host(gpu.cnn_fc_fwd(to_dev(x), to_dev(w), None, False, config=cfg))
            assert (np.abs(got - ref) <= live * 2.0 ** -23 * np.abs(ref)).all(), f"I {I} config {cfg}"


def test_fc_of_one_input_stays_in_fp32(gpu):
    """One product a sum: the fp32 value itself, which the parts miss by up to 3% more than its rounding."""
    x, w = wl.normal((24, 1), 1.0, 64, 0), wl.normal((96, 1), 1.0, 64, 1)
    np.testing.assert_array_equal(to_host(gpu.cnn_fc_fwd(to_dev(x), to_dev(w), None, False)), x * w.T)
