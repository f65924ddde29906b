"""Decryption takes ciphertext residues as a caller's own additions leave them: the
word-wise sums of two and three returned ciphertexts, not reduced mod q_l,
decrypt to the sums of their messages for both kinds of moduli (just below 2^60
and 50-bit).  The default flood of three products, 3/8 of q / t, stays below the
rounding's 1/2."""
import numpy as np
import pytest

from workloads import conv, fc

from gpu_common import dev, host_i64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2_n,limbs,bits", [(10, 2, 60), (11, 2, 50), (12, 2, 60), (13, 3, 60), (14, 4, 60)])
def test_unreduced_sums_decrypt(log2_n, limbs, bits):
    from paper_2403_11166_amd import Context
    ctx = Context(log2_n, limbs, bits, 31)
    kw = dict(log2_n=log2_n, num_limbs=limbs, prime_bits=bits)
    for layer in (fc(5, 70, 11, **kw), conv(3, 2, 5, 9, k=3, pad=1, **kw)):
        plan = ctx.plan_auto(layer)
        rng = np.random.default_rng(log2_n)
        w = dev(rng.integers(0, ctx.t, layer.w_shape(), dtype=np.int64))
        cts, want = [], 0
        for i in range(3):
            x0, x1 = (dev(rng.integers(0, ctx.t, layer.x_shape(), dtype=np.int64)) for _ in range(2))
            ct = ctx.encrypt(layer, plan, "x_fwd", x1, 10 * i)
            out, _ = ctx.linear_fwd(layer, plan, ct, x0, w, 10 * i + 1)
            cts.append(out)
            want = want + host_i64(ctx.decrypt(layer, plan, "fwd", out))
            total = cts[0]
            for c in cts[1:]:
                total = total + c
            assert np.array_equal(host_i64(ctx.decrypt(layer, plan, "fwd", total)), want % ctx.t)
