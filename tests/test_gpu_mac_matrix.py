"""The matrix-core multiply-accumulate at the edges of its tiles: output grids
and contractions around multiples of 16, both forms of products (one term; the
weight gradient's two), moduli below and just below 2^60, and partitions of
images.  Every operand tile holds one channel, so the grid of output tiles is the
layer's channel grid; reconstructed products are compared bit for bit with the
plain layer operators."""
import numpy as np
import pytest

from oracle import linear as LN
from workloads import T_PLAIN, conv, conv1d, fc, layer_tensors

from gpu_common import dev, host_i64

pytestmark = pytest.mark.gpu

T = T_PLAIN
_ctx = {}


def context(log2_n, limbs, bits):
    from paper_2403_11166_amd import Context
    key = (log2_n, limbs, bits)
    if key not in _ctx:
        _ctx[key] = Context(log2_n, limbs, bits, 43)
    return _ctx[key]


def product(ctx, layer, op, tile, seed):
    plan = {op: tile, "sched": (3, 3, 3)}
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
        want = LN.layer_op(layer, op, ts["X"], ts["dY"], T)
        want = (want - LN.layer_op(layer, op, ts["x0"], ts["dy0"], T) - LN.layer_op(layer, op, ts["x1"], ts["dy1"], T)) % T
    got = (host_i64(ctx.decrypt(layer, plan, op, out)) + host_i64(s)) % T
    assert np.array_equal(got, want)


# rows x columns x contraction of output tiles; N = 1024, L = 2 (50-bit) or 3 (60-bit)
GRIDS = [(24, 32, 16), (16, 33, 33), (33, 17, 47), (8, 64, 130), (48, 16, 7), (25, 31, 15), (64, 64, 1)]


@pytest.mark.parametrize("limbs,bits", [(2, 50), (3, 60)])
@pytest.mark.parametrize("rows,cols,k", GRIDS)
def test_tile_edges(rows, cols, k, limbs, bits):
    ctx = context(10, limbs, bits)
    product(ctx, fc(rows, k, cols, log2_n=10, num_limbs=limbs, prime_bits=bits), "fwd", (1,) * 7, 51)
    product(ctx, fc(k, rows, cols, log2_n=10, num_limbs=limbs, prime_bits=bits), "dw", (1,) * 7, 52)


@pytest.mark.parametrize("op,tile", [("fwd", (1, 1, 1, 3, 6, 3, 3)), ("dx", (1, 1, 1, 3, 6, 3, 3)),
                                     ("fwd", (1, 1, 1, 6, 6, 1, 3)), ("dw", (1, 1, 1, 3, 3, 6, 6))],
                         ids=["split_rows", "dx_split_rows", "split_kernel", "dw"])
def test_image_partitions(op, tile):
    """Output windows split (several A tiles per row and contraction index) or the
    kernel window split (several contraction indices per channel)."""
    layer = conv(9, 14, 18, 6, k=3, pad=1, log2_n=11, num_limbs=3, prime_bits=60)
    product(context(11, 3, 60), layer, op, tile, 53)


def test_conv1d_ragged():
    layer = conv1d(17, 20, 33, 12, k=5, log2_n=11, num_limbs=3, prime_bits=60)
    ctx = context(11, 3, 60)
    product(ctx, layer, "fwd", (1, 2, 1, 1, 8, 1, 5), 54)
    product(ctx, layer, "dx", (1, 1, 2, 1, 12, 1, 5), 55)
