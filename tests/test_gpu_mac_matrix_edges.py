"""The matrix-core multiply-accumulate where its index arithmetic has more than
one case, with every product checked to run there: output windows and kernel
windows in several tiles, ragged Conv1d tiles, contractions of one block, and
its bound of 8192 contraction indices on operands whose digits are -128."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import linear as LN
from workloads import T_PLAIN as T
from workloads import conv, conv1d, fc, layer_tensors

from gpu_common import dev, host_i64, host_u64

pytestmark = pytest.mark.gpu

OP = {"fwd": 0, "dx": 1, "dw": 2}
_ctx = {}


def context(log2_n, limbs, bits):
    from paper_2403_11166_amd import Context
    key = (log2_n, limbs, bits)
    if key not in _ctx:
        _ctx[key] = Context(log2_n, limbs, bits, 47)
    return _ctx[key]


def on_matrix_cores(layer, op, plan):
    from paper_2403_11166_amd import _abi as A
    from paper_2403_11166_amd.api import layer_struct, plan_struct
    p, out = A.Params(), ctypes.c_int(-1)
    p.log2_n, p.num_limbs, p.prime_bits = layer.log2_n, layer.num_limbs, layer.prime_bits
    A.check(A.load().pencil_product_kernel(ctypes.byref(p), ctypes.byref(layer_struct(layer)),
                                           ctypes.byref(plan_struct(plan)), OP[op], ctypes.byref(out)))
    return out.value == 1


def product(layer, op, tile, seed):
    ctx = context(layer.log2_n, layer.num_limbs, layer.prime_bits)
    plan = {op: tile, "sched": (3, 3, 3)}
    assert on_matrix_cores(layer, op, plan)
    ts = layer_tensors(layer, seed)
    d = {k: dev(v) for k, v in ts.items()}
    if op == "fwd":
        ct = ctx.encrypt(layer, plan, "x_fwd", d["x1"], 7)
        out, s = ctx.linear_fwd(layer, plan, ct, d["x0"], d["W"], 8)
        want = LN.layer_op(layer, op, ts["X"], ts["W"], T)
    elif op == "dx":
        ct = ctx.encrypt(layer, plan, "dy_dx", d["dy1"], 7)
        out, s, _, _ = ctx.linear_bwd(layer, plan, ct, None, None, d["dy0"], d["x0"], d["W"], 8, do_dw=False)
        want = LN.layer_op(layer, op, ts["dY"], ts["W"], T)
    else:
        cx = ctx.encrypt(layer, plan, "x_dw", d["x1"], 7)
        cy = ctx.encrypt(layer, plan, "dy_dw", d["dy1"], 7)
        _, _, out, s = ctx.linear_bwd(layer, plan, None, cx, cy, d["dy0"], d["x0"], d["W"], 8, do_dx=False)
        want = (LN.layer_op(layer, op, ts["x0"], ts["dy1"], T) + LN.layer_op(layer, op, ts["x1"], ts["dy0"], T)) % T
    got = (host_i64(ctx.decrypt(layer, plan, op, out)) + host_i64(s)) % T
    assert np.array_equal(got, want)


KW = dict(log2_n=11, num_limbs=3)
SHAPES = {
    "split_rows": (lambda kw: conv(20, 28, 34, 6, k=3, pad=1, **kw), "fwd", (1, 1, 1, 3, 6, 3, 3)),
    "split_rows_cols": (lambda kw: conv(13, 30, 33, 6, k=3, pad=1, **kw), "fwd", (1, 1, 1, 3, 3, 3, 3)),
    "dx_split_rows": (lambda kw: conv(20, 34, 28, 6, k=3, pad=1, **kw), "dx", (1, 1, 1, 3, 6, 3, 3)),
    "dw_split_rows": (lambda kw: conv(24, 16, 34, 6, k=3, pad=1, **kw), "dw", (1, 1, 1, 1, 3, 6, 6)),
    "split_kernel": (lambda kw: conv(24, 11, 34, 6, k=3, pad=1, **kw), "fwd", (1, 1, 1, 6, 6, 1, 3)),
    "dw_split_window": (lambda kw: conv(9, 30, 34, 6, k=3, pad=1, **kw), "dw", (1, 1, 1, 3, 3, 2, 6)),
    "conv1d_ragged": (lambda kw: conv1d(23, 61, 33, 12, k=5, **kw), "fwd", (1, 1, 2, 1, 5, 1, 5)),
    "conv1d_dx_ragged": (lambda kw: conv1d(24, 33, 61, 12, k=5, **kw), "dx", (1, 1, 2, 1, 12, 1, 5)),
    "one_block": (lambda kw: fc(64, 16, 64, **kw), "fwd", (1,) * 7),
    "one_ragged_block": (lambda kw: fc(64, 15, 64, **kw), "fwd", (1,) * 7),
    "dw_one_block": (lambda kw: fc(15, 64, 64, **kw), "dw", (1,) * 7),
}


@pytest.mark.parametrize("bits", [50, 60])
@pytest.mark.parametrize("shape", SHAPES)
def test_partitions_and_blocks(shape, bits):
    make, op, tile = SHAPES[shape]
    product(make(dict(KW, prime_bits=bits)), op, tile, 91)


def extreme(bits, q):
    """The largest residue below q whose digits are all -128 but the highest."""
    n = (bits - 1) // 8
    low = 128 * (256 ** n - 1) // 255
    return (q + low) // 256 ** n * 256 ** n - low


def split30(v):
    return (v & 0x3FFFFFFF) | (v >> 30) << 32


@pytest.mark.parametrize("bits", [50, 60])
@pytest.mark.parametrize("op", ["fwd", "dw"])
def test_contraction_at_its_bound(op, bits):
    """8192 indices, the most the int32 diagonals hold.  Every tile is one entry, a
    constant polynomial, and every ciphertext component one residue in all slots, so
    the product adds one constant to coefficient 0 of each output; the mask and the
    flood, the same for zero operands, cancel in the difference.  One index more
    goes to the vector kernel."""
    ctx = context(10, 2, bits)
    kw = dict(log2_n=10, num_limbs=2, prime_bits=bits)
    make = lambda k: fc(32, k, 16, **kw) if op == "fwd" else fc(k, 32, 16, **kw)  # noqa: E731
    k = 8192 if op == "fwd" else 4096  # the weight gradient has two terms
    layer, plan = make(k), {op: (1,) * 7, "sched": (3, 3, 3)}
    assert on_matrix_cores(layer, op, plan) and not on_matrix_cores(make(k + 1), op, plan)
    w_small = (1 << 40) - 128 * (256 ** 5 - 1) // 255  # five digits of -128, at most t / 2: lifts to itself
    w_large = T - 1 - (1 << 20)                       # lifts to q - 1 - 2^20
    sz = ctx.layout(layer, plan)

    def cts(count, swap):
        ct = ctx.empty_cts(count)
        for l, q in enumerate(ctx.primes):
            v = [extreme(bits, q), q - 1]
            for c in range(2):
                ct[:, c, l] = split30(v[c ^ swap])
        return ct

    def full(shape, v):
        return torch.full(shape, v, dtype=torch.int64, device="cuda")

    def run(zero):
        if op == "fwd":
            ct = cts(sz.n_ct[0], 0)
            if zero:
                ct.zero_()
            return host_u64(ctx.linear_fwd(layer, plan, ct, full(layer.x_shape(), 0),
                                           full(layer.w_shape(), 0 if zero else w_small), 3)[0])
        cx, cy = cts(sz.n_ct[2], 0), cts(sz.n_ct[3], 1)
        if zero:
            cx.zero_(), cy.zero_()
        return host_u64(ctx.linear_bwd(layer, plan, None, cx, cy, full(layer.y_shape(), 0 if zero else w_small),
                                       full(layer.x_shape(), 0 if zero else w_large), full(layer.w_shape(), 0), 3,
                                       do_dx=False)[2])

    a, b = run(False), run(True)
    assert a.shape[0] == 32 * 16
    for l, q in enumerate(ctx.primes):
        v = [extreme(bits, q), q - 1]
        for c in range(2):
            want = k * v[c] * w_small if op == "fwd" else k * (v[c] * w_small + (q - 1 - (1 << 20)) * v[c ^ 1])
            x, y = a[:, c, l].astype(object), b[:, c, l].astype(object)
            diff = (x - y) % q
            assert (diff[:, 0] == want % q).all()
            assert not diff[:, 1:].any()
