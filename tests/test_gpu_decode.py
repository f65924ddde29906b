"""Decryption with one to four limbs (each its own width of multiword arithmetic):
ragged output tiles of FC and convolution products, a small and the default-sized
plaintext modulus, with and without the noise measurement, bit for bit against the
plain layer operator."""
import numpy as np
import pytest

from oracle import linear as LN
from workloads import conv, fc

from gpu_common import dev, host_i64

pytestmark = pytest.mark.gpu

LAYERS = [lambda **kw: fc(5, 70, 11, **kw), lambda **kw: conv(3, 2, 5, 9, k=3, pad=1, **kw)]


@pytest.mark.parametrize("limbs,t", [(1, 257), (1, 65537), (2, 65537), (2, 2199023255531), (3, 2199023255531),
                                     (4, 2199023255531)])
def test_decrypt_per_limb_count(limbs, t):
    from paper_2403_11166_amd import Context
    ctx = Context(10, limbs, 60, 9, t=t)
    for make in LAYERS:
        layer = make(log2_n=10, num_limbs=limbs, prime_bits=60)
        rng = np.random.default_rng(limbs)
        x0, x1 = (rng.integers(0, t, layer.x_shape(), dtype=np.int64) for _ in range(2))
        w = rng.integers(0, t, layer.w_shape(), dtype=np.int64)
        plan = ctx.plan_auto(layer)
        ct = ctx.encrypt(layer, plan, "x_fwd", dev(x1), 3)
        out, s = ctx.linear_fwd(layer, plan, ct, dev(x0), dev(w), 4)
        want = LN.layer_op(layer, "fwd", (x0 + x1) % t, w, t)
        y = host_i64(ctx.decrypt(layer, plan, "fwd", out))
        assert np.array_equal((y + host_i64(s)) % t, want)
        again, _ = ctx.decrypt_checked(layer, plan, "fwd", out)
        assert np.array_equal(host_i64(again), y)
