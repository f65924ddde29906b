"""Plaintext correlations on both sides of the lines at which they change kernel
or split: 2^26 multiply-adds, few columns over a little more than one grid of
workgroups, short parts of a contraction, and the digit bounds of the f64 kernel
with the shapes that reach it (two digits: 2^15 windowed indices, eight columns;
three digits: a 47-bit t, 2^21 indices), on operands of the largest centred
magnitude there."""
import numpy as np
import pytest
import torch

from oracle import linear as LN
from workloads import T_PLAIN as T
from workloads import conv, conv1d, fc

from gpu_common import dev, host_i64

pytestmark = pytest.mark.gpu

KW = dict(log2_n=10, num_limbs=2, prime_bits=50)
T47 = 140737488355213
_ctx = {}


def context(t):
    from paper_2403_11166_amd import Context
    if t not in _ctx:
        _ctx[t] = Context(10, 2, 50, 5, t=t)
    return _ctx[t]


CASES = {
    "below_line": (fc(64, 1024, 1023, **KW), "fwd"),
    "at_line": (fc(64, 1024, 1024, **KW), "fwd"),
    "few_columns_f64": (conv(30, 169, 6, 29, k=5, pad=0, **KW), "fwd"),
    "few_columns_f64_flipped": (conv(44, 14, 134, 21, k=5, pad=0, **KW), "dx"),
    "few_columns_int8": (conv(84, 12, 84, 14, k=3, pad=1, **KW), "dx"),
    "few_columns_one_round": (conv(84, 87, 8, 16, k=5, pad=0, **KW), "fwd"),
    "scattered_parts": (conv1d(16, 128, 256, 30, k=5, pad=2, **KW), "dx"),
    "scattered_unsplit": (fc(128, 784, 800, **KW), "dw"),
    "second_round_refused": (conv(109, 49, 53, 11, k=3, pad=0, **KW), "fwd"),
    "contiguous_parts": (fc(203, 1076, 314, **KW), "dx"),
}


@pytest.mark.parametrize("case", CASES)
def test_lines(case):
    layer, op = CASES[case]
    rng = np.random.default_rng(len(case))
    x, w, dy = (rng.integers(0, T, s, dtype=np.int64) for s in (layer.x_shape(), layer.w_shape(), layer.y_shape()))
    a, b = {"fwd": (x, w), "dx": (dy, w), "dw": (x, dy)}[op]
    got = host_i64(context(T).zt_linear(layer, op, dev(a), dev(b)))
    pts = [tuple(0 for _ in got.shape), tuple(n - 1 for n in got.shape)]
    pts += [tuple(int(rng.integers(n)) for n in got.shape) for _ in range(60)]
    assert [int(got[p]) for p in pts] == LN.layer_op_at(layer, op, a, b, T, pts)
    assert got.min() >= 0 and got.max() < T


@pytest.mark.parametrize("c_in", [32768, 32769])
def test_two_digit_bound(c_in):
    """2^15 indices: 512 steps of each of 16 waves, as many as two digits hold in
    53 bits; one more takes the int8 kernel."""
    layer = conv(2, c_in, 8, 91, k=1, pad=0, **KW)  # 16562 rows: 259 tiles of 64 x 64
    h = (T - 1) // 2
    x = torch.full(layer.x_shape(), h, dtype=torch.int64, device="cuda")
    w = torch.full(layer.w_shape(), h, dtype=torch.int64, device="cuda")
    got = context(T).zt_linear(layer, "fwd", x, w)
    assert got.numel() == 16562 * 8
    assert bool((got == c_in * h * h % T).all())


def test_three_digit_bound():
    """A 47-bit t: three digits, 2^15 steps of each of 16 waves."""
    batch = 1 << 21
    layer = fc(batch, 128, 64, **KW)
    h = (T47 - 1) // 2
    x = torch.full(layer.x_shape(), h, dtype=torch.int64, device="cuda")
    dy = torch.full(layer.y_shape(), h, dtype=torch.int64, device="cuda")
    got = context(T47).zt_linear(layer, "dw", x, dy)
    assert got.numel() == 128 * 64
    assert bool((got == batch * h * h % T47).all())
