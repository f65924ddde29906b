"""The NTT width (residues per thread) is a schedule: changed by the autotuner
between a step's creation and its bind, after a bind, or before a second one, it
leaves every output as it was.  The width comes from a cache file, so that no
measurement decides it."""
import numpy as np
import pytest
import torch

from workloads import conv, fc, layer_tensors

from gpu_common import dev

pytestmark = pytest.mark.gpu

OUTS = ("ct_y", "y0", "ct_dx", "dx0", "ct_dw", "dw_mask")


def set_width(ctx, layer, plan, loge, path):
    path.write_text('{"key": "gfx950 N=%d L=%d ntt_loge", "choice": %d}\n' % (ctx.n, ctx.L, loge))
    ctx.autotune(layer, plan, str(path))
    assert ctx.ntt_loge() == loge


@pytest.mark.parametrize("log2_n,limbs,bits", [(12, 2, 60), (13, 2, 50), (13, 3, 60), (14, 2, 60)])
def test_width_changed_around_bind(log2_n, limbs, bits, tmp_path):
    from paper_2403_11166_amd import Context, Step
    ctx = Context(log2_n, limbs, bits, 35)
    kw = dict(log2_n=log2_n, num_limbs=limbs, prime_bits=bits)
    layers = [fc(6, 40, 24, **kw), conv(3, 4, 5, 9, k=3, pad=1, **kw)]
    ents, ios = [], []
    for i, layer in enumerate(layers):
        plan, d = ctx.plan_auto(layer), {k: dev(v) for k, v in layer_tensors(layer, 71 + i).items()}
        sz = ctx.layout(layer, plan)
        ents.append((ctx, layer, plan))
        ios.append(dict(ct_x1=ctx.encrypt(layer, plan, "x_fwd", d["x1"], 500 + i),
                        ct_dy_dx=ctx.encrypt(layer, plan, "dy_dx", d["dy1"], 600 + i),
                        ct_x_dw=ctx.encrypt(layer, plan, "x_dw", d["x1"], 700 + i),
                        ct_dy_dw=ctx.encrypt(layer, plan, "dy_dw", d["dy1"], 800 + i),
                        x0=d["x0"], dy0=d["dy0"], w=d["W"], ct_y=ctx.empty_cts(sz.n_out[0]),
                        ct_dx=ctx.empty_cts(sz.n_out[1]), ct_dw=ctx.empty_cts(sz.n_out[2]),
                        y0=torch.empty_like(d["dy0"]), dx0=torch.empty_like(d["x0"]),
                        dw_mask=torch.empty_like(d["W"])))

    def outputs():
        torch.cuda.synchronize()
        return [io[k].cpu().numpy().copy() for io in ios for k in OUTS]

    for i, ((_, layer, plan), io) in enumerate(zip(ents, ios)):
        ctx.linear_fwd(layer, plan, io["ct_x1"], io["x0"], io["w"], 90 + 2 * i, out=(io["ct_y"], io["y0"]))
        ctx.linear_bwd(layer, plan, io["ct_dy_dx"], io["ct_x_dw"], io["ct_dy_dw"], io["dy0"], io["x0"], io["w"],
                       91 + 2 * i, out=(io["ct_dx"], io["dx0"], io["ct_dw"], io["dw_mask"]))
    want = outputs()

    def check(step):
        for io in ios:
            for k in OUTS:
                io[k].zero_()
        step.run(90)
        assert all(np.array_equal(a, b) for a, b in zip(outputs(), want))

    tune = tmp_path / "tune.txt"
    step = Step(ents)
    ws = torch.empty(step.workspace_bytes(), dtype=torch.uint8, device="cuda")
    assert ctx.ntt_loge() == 4
    set_width(ctx, layers[0], ents[0][2], 5, tune)  # created at one width, bound at the other
    step.bind(ios, ws)
    check(step)
    set_width(ctx, layers[0], ents[0][2], 4, tune)  # bound at one width, run at the other
    check(step)
    step.bind(ios, ws)  # and bound a second time
    check(step)
