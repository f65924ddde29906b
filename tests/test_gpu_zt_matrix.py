"""Large plaintext correlations (from 2^26 multiply-adds) on the int8 matrix cores,
bit for bit against the plain layer operators: outputs around multiples of 64,
contractions with remainders of 16 and shorter than a window row's step, windows
with padding and a flipped kernel, operands strided along the contraction, one
and several parts of the contraction, t next to the digits' bound, and operands
of the largest value."""
import numpy as np
import pytest

from oracle import linear as LN
from workloads import T_PLAIN, conv, conv1d, fc

from gpu_common import dev, host_i64

pytestmark = pytest.mark.gpu

KW = dict(log2_n=10, num_limbs=2, prime_bits=50)
T46 = (1 << 46) - 21  # the digits' bound is t < 2^46
_ctx = {}


def context(t):
    from paper_2403_11166_amd import Context
    if t not in _ctx:
        _ctx[t] = Context(10, 2, 50, 5, t=t)
    return _ctx[t]


def work(layer):
    per = layer.c_out * layer.c_in * layer.batch
    return per if layer.kind == "fc" else per * layer.h_out * layer.w_out * layer.kh * layer.kw


CASES = {
    "fc_fwd_split": (fc(65, 8191, 129, **KW), "fwd"),
    "fc_dx_unsplit": (fc(2049, 2047, 17, **KW), "dx"),
    "fc_dw_remainder": (fc(1033, 257, 255, **KW), "dw"),
    "fc_five_columns": (fc(1700, 8001, 5, **KW), "fwd"),
    "conv_fwd": (conv(21, 66, 71, 9, k=3, pad=1, **KW), "fwd"),
    "conv_dx_flipped": (conv(21, 66, 71, 9, k=3, pad=1, **KW), "dx"),
    "conv_dw": (conv(21, 66, 71, 9, k=3, pad=1, **KW), "dw"),
    "conv_valid_k5": (conv(25, 40, 33, 14, k=5, pad=0, **KW), "fwd"),
    "conv_k1": (conv(30, 130, 90, 16, k=1, pad=0, **KW), "dw"),
    "conv1d_fwd": (conv1d(33, 100, 127, 37, k=5, pad=2, **KW), "fwd"),
    "conv1d_dw": (conv1d(33, 100, 127, 37, k=5, pad=0, **KW), "dw"),
}


@pytest.mark.parametrize("t", [T_PLAIN, T46])
@pytest.mark.parametrize("case", CASES)
def test_large_correlations(case, t):
    layer, op = CASES[case]
    assert work(layer) >= 1 << 26
    rng = np.random.default_rng(len(case) + t % 97)
    x, w, dy = (rng.integers(0, t, s, dtype=np.int64) for s in (layer.x_shape(), layer.w_shape(), layer.y_shape()))
    a, b = {"fwd": (x, w), "dx": (dy, w), "dw": (x, dy)}[op]
    got = host_i64(context(t).zt_linear(layer, op, dev(a), dev(b)))
    if t == T_PLAIN:
        assert np.array_equal(got, LN.layer_op(layer, op, a, b, t))
    else:
        pts = [tuple(0 for _ in got.shape), tuple(n - 1 for n in got.shape)]
        pts += [tuple(int(rng.integers(n)) for n in got.shape) for _ in range(30)]
        assert [int(got[p]) for p in pts] == LN.layer_op_at(layer, op, a, b, t, pts)


@pytest.mark.parametrize("batch", [8192, 8193, 70000])
def test_accumulators_at_their_bound(batch):
    """One part holds up to 8192 indices in 32 bits: operands whose digits are
    -128 (but the highest), and t - 1."""
    layer = fc(batch, 1030, 1030, **KW)  # 17 x 17 tiles: more than a part per CU
    for v in (0x3f7f_7f7f_7f80, T46 - 1):
        x = dev(np.full(layer.x_shape(), v % T46, dtype=np.int64))
        dy = dev(np.full(layer.y_shape(), v % T46, dtype=np.int64))
        got = host_i64(context(T46).zt_linear(layer, "dw", x, dy))
        assert got.size == 1030 * 1030
        assert (got == batch * (v % T46) ** 2 % T46).all()
