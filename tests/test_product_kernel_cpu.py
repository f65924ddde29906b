"""Which kernel multiplies a product (host only).  The grids are those of output
tiles and contraction indices at which both kernels were timed."""
import ctypes

import pytest

from workloads.configs import fc

OP = {"fwd": 0, "dx": 1, "dw": 2}


def matrix(layer, op, plan, ret=False):
    from paper_2403_11166_amd import _abi as A
    from paper_2403_11166_amd.api import layer_struct, plan_struct
    lib = A.load()
    p, out = A.Params(), ctypes.c_int(-1)
    p.log2_n, p.num_limbs, p.prime_bits = layer.log2_n, layer.num_limbs, layer.prime_bits
    st = lib.pencil_product_kernel(ctypes.byref(p), ctypes.byref(layer_struct(layer)),
                                   ctypes.byref(plan_struct(plan)), OP[op], ctypes.byref(out))
    return st if ret else out.value


def grid(params, rows, cols, k, op):
    log2_n, limbs, bits = params
    kw = dict(log2_n=log2_n, num_limbs=limbs, prime_bits=bits)
    layer = fc(rows, k, cols, **kw) if op == "fwd" else fc(k, rows, cols, **kw)
    return matrix(layer, op, {op: (1,) * 7})


# (parameters, rows, columns, indices, product): vector and matrix kernel's us, batched
VECTOR = [((13, 3, 50), 16, 16, 7, "fwd"),   # 74, 103
          ((12, 2, 50), 40, 24, 12, "fwd"),  # 133, 184
          ((12, 2, 50), 16, 32, 6, "dw"),    # 67, 86
          ((13, 3, 50), 64, 64, 7, "fwd"),   # 1478, 1830
          ((12, 2, 60), 32, 32, 7, "fwd"),   # 103, 123
          ((13, 3, 60), 8, 16, 7, "fwd"),    # 40, 47
          ((13, 3, 60), 8, 8, 2, "fwd")]
MATRIX = [((12, 2, 50), 32, 32, 25, "fwd"), ((13, 3, 50), 64, 64, 48, "fwd"), ((13, 3, 60), 16, 16, 25, "fwd"),
          ((14, 4, 60), 40, 24, 16, "fwd"), ((14, 4, 60), 64, 64, 24, "dw"), ((13, 3, 60), 24, 128, 96, "fwd")]


@pytest.mark.parametrize("point", VECTOR)
def test_vector_kernel_where_it_is_faster(point):
    assert grid(*point) == 0


@pytest.mark.parametrize("point", MATRIX)
def test_matrix_kernel_where_it_is_faster(point):
    assert grid(*point) == 1


def test_launch_limit():
    """A launch holds fewer than 2^32 threads, 1024 per 16 slots and output tile: at N
    = 16384, L = 4 below 1024 tiles of 16 x 16.  Larger products keep the vector kernel."""
    assert grid((14, 4, 60), 248, 512, 32, "fwd") == 1  # 31 x 32 tiles
    assert grid((14, 4, 60), 256, 512, 32, "fwd") == 0  # 32 x 32
    assert grid((14, 4, 60), 256, 1000, 16, "dw") == 0
    assert grid((10, 1, 60), 4096, 4096, 16, "dw") == 0


def test_requests_are_checked():
    from paper_2403_11166_amd import _abi as A
    layer = fc(4, 5, 6, log2_n=10, num_limbs=2, prime_bits=60)
    assert matrix(layer, "fwd", {"fwd": (1, 1, 2048, 1, 1, 1, 1)}, ret=True) == A.PENCIL_EINVAL
    assert A.load().pencil_product_kernel(None, None, None, 0, None) == A.PENCIL_EINVAL
