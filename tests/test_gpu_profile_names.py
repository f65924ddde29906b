"""Kernel timing by name: the entries a reader of the statistics looks up are
there, in their order, and the launches of the calls are counted under them."""
import ctypes

import pytest

from workloads import fc, layer_tensors

from gpu_common import dev

pytestmark = pytest.mark.gpu

NAMES = ["ntt_ct", "ntt_pt", "ntt_ternary", "mac", "intt_out", "flood_mask", "encrypt", "phase", "decode", "ntt_plain",
         "step_ntt", "step_mac", "step_intt", "step_flood"]


def stats(ctx):
    from paper_2403_11166_amd import _abi as A
    arr, cnt = (A.KernelStat * 32)(), ctypes.c_int()
    ctx._check(ctx.lib.pencil_profile_read(ctx.h, arr, 32, ctypes.byref(cnt)))
    return [(arr[i].name.decode(), arr[i].launches) for i in range(cnt.value)]


def test_names_and_launches():
    from paper_2403_11166_amd import Context
    ctx = Context(10, 2, 50, 37)
    layer = fc(4, 10, 6, log2_n=10, num_limbs=2, prime_bits=50)
    plan, d = ctx.plan_auto(layer), {k: dev(v) for k, v in layer_tensors(layer, 81).items()}
    ctx._check(ctx.lib.pencil_profile_enable(ctx.h, 1))
    cx, cdx = ctx.encrypt(layer, plan, "x_fwd", d["x1"], 1), ctx.encrypt(layer, plan, "dy_dx", d["dy1"], 2)
    cxw, cdyw = ctx.encrypt(layer, plan, "x_dw", d["x1"], 3), ctx.encrypt(layer, plan, "dy_dw", d["dy1"], 4)
    out, _ = ctx.linear_fwd(layer, plan, cx, d["x0"], d["W"], 5)
    ctx.linear_bwd(layer, plan, cdx, cxw, cdyw, d["dy0"], d["x0"], d["W"], 6)
    ctx.decrypt(layer, plan, "fwd", out)
    got = stats(ctx)
    assert [n for n, _ in got][:len(NAMES)] == NAMES
    want = dict.fromkeys(NAMES, 0) | {"ntt_ct": 2, "ntt_pt": 1, "ntt_ternary": 4, "encrypt": 4, "mac": 3, "intt_out": 3,
                                      "flood_mask": 3, "phase": 1, "decode": 1}
    assert {n: c for n, c in got if n in want} == want
