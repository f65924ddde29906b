"""The autotuner measures schedules only where they matter: a product that runs on
the matrix cores under its chosen tile gets no schedule line in the cache and keeps
the plan's schedule; the vector kernel's products get one."""
import ctypes
import re

import pytest

from workloads import fc

pytestmark = pytest.mark.gpu

OPS = ("fwd", "dx", "dw")


def test_no_schedule_is_recorded_for_matrix_products(tmp_path):
    from paper_2403_11166_amd import Context
    from paper_2403_11166_amd import _abi as A
    from paper_2403_11166_amd.api import layer_struct
    ctx = Context(10, 2, 60, 39)
    p = A.Params()
    p.log2_n, p.num_limbs, p.prime_bits = 10, 2, 60
    kinds = set()
    for layer in (fc(64, 2048, 128, log2_n=10, num_limbs=2, prime_bits=60),
                  fc(4, 10, 6, log2_n=10, num_limbs=2, prime_bits=60)):
        path = tmp_path / f"tune{layer.c_in}.txt"
        plan = ctx.plan_auto(layer)
        tuned = ctx.autotune(layer, plan, str(path))
        lines = path.read_text()
        for i, op in enumerate(OPS):
            matrix = ctypes.c_int()
            A.check(A.load().pencil_product_kernel(ctypes.byref(p), ctypes.byref(layer_struct(layer)),
                                                   ctypes.byref(tuned), i, ctypes.byref(matrix)))
            kinds.add(matrix.value)
            assert bool(re.search(rf"op={i} sched", lines)) == (matrix.value == 0)
            assert 0 <= tuned.sched[i] < 9
    assert kinds == {0, 1}
