"""Performance cases of the encrypted linear-layer product.

Each case is one call or short sequence of calls a training program makes:
the model owner's products of one layer or of a whole step, the data owner's
encryption and decryption, the plaintext terms both parties compute over Z_t,
the online phase of the preprocessed products, and a layer differentiated by
autograd.  Shapes are those of the workloads of this repository (MNIST MLP and
CNN, AGNews TextCNN, CIFAR-shaped convolutions, the largest fully connected
layer), parameters N = 4096 .. 16384 with 2 .. 4 limbs.

A layer is written "kind batch c_in c_out h w k pad stride"; several layers
are separated by ";".
"""
import numpy as np
import torch

from paper_2403_11166_amd import api, autograd, pencil_plus
from workloads.configs import LayerSpec

T_PLAIN = 2199023255531  # the library's default plaintext modulus
FRAC = 4096.0            # fixed-point scale 2^12
MASKS = 8                # masks per operand of the preprocessed products


def _case(name, kind, layers, log2_n, limbs, bits=60, option=""):
    return dict(name=name, kind=kind, layers=layers, log2_n=log2_n, limbs=limbs, bits=bits, option=option)


def listed():
    return [
        # inference on a small classifier head: one forward product, launch latency
        _case("fwd_fc64x10_b8", "fwd", "fc 8 64 10 1 1 1 0 1", 12, 2, 50),
        # the MNIST MLP's first layer, every product of a training step
        _case("step_fc784x128_b64", "step", "fc 64 784 128 1 1 1 0 1", 13, 3),
        # a network's first convolution (three input channels)
        _case("step_conv3x64_b64", "step", "conv 64 3 64 32 32 3 1 1", 13, 3),
        # a text layer through the per-product calls; odd length, ragged tiles
        _case("layer_conv1d_128x128_l30_b64", "layer", "conv1d 64 128 128 1 30 5 0 1", 13, 3),
        # the widest fully connected layer, ragged output count
        _case("step_fc2048x1001_b64", "step", "fc 64 2048 1001 1 1 1 0 1", 13, 3),
        # one layer of each width of the eight-layer CIFAR stack, batched
        _case("step_conv64_128_256_b64", "step",
              "conv 64 64 64 32 32 3 1 1;conv 64 128 128 16 16 3 1 1;conv 64 256 256 8 8 3 1 1", 14, 4),
        # the data owner's side of the stack's first layer: its input's encryption
        _case("encrypt_conv64_b64", "encrypt", "conv 64 64 64 32 32 3 1 1", 14, 4, option="x_fwd"),
        # ... and the decryption of what the model owner returns
        _case("decrypt_conv64_b64", "decrypt", "conv 64 64 64 32 32 3 1 1", 14, 4, option="fwd"),
        # a party's local term of the weight gradient of a convolution
        _case("local_dw_conv64_b64", "local", "conv 64 64 64 16 16 3 1 1", 13, 3, option="dw"),
        # a plaintext forward product of the MNIST CNN's first FC layer
        _case("local_fwd_fc980x100_b64", "local", "fc 64 980 100 1 1 1 0 1", 13, 3, option="fwd"),
        # online phase of the preprocessed products on the MNIST MLP's layer
        _case("online_fwd_fc784x128_b64", "online", "fc 64 784 128 1 1 1 0 1", 13, 3, option="fwd"),
        # the MNIST CNN's strided convolution as a differentiable layer, forward and backward
        _case("train_conv1x5_s2_b64", "train", "conv 64 1 5 28 28 5 2 2", 13, 3),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _draw_layer(rng, kind, stride):
    what = rng.choice(("fc", "conv", "conv1d"))
    batch = _log(rng, 4, 128)
    if what == "fc":
        return "fc %d %d %d 1 1 1 0 1" % (batch, _log(rng, 10, 2048), _log(rng, 4, 1001))
    s = rng.choice((1, 2)) if stride else 1
    k = rng.choice((1, 3, 5)) if what == "conv" else rng.choice((3, 5))
    pad = rng.choice((0, k // 2))
    ci, co = _log(rng, 1, 256), _log(rng, 4, 256)
    if what == "conv1d":
        return "conv1d %d %d %d 1 %d %d %d %d" % (batch, ci, co, _log(rng, 12, 64), k, pad, s)
    hw = _log(rng, 7, 32)
    return "conv %d %d %d %d %d %d %d %d" % (batch, ci, co, hw, hw, k, pad, s)


def draw(rng):
    most = work(listed()[5])
    while True:
        kind = rng.choice(("fwd", "step", "step", "layer", "layer", "encrypt", "decrypt", "local", "online", "train"))
        log2_n, limbs, bits = rng.choice(((12, 2, 50), (13, 3, 60), (13, 3, 60), (14, 4, 60)))
        count = rng.choice((1, 2)) if kind == "step" else 1
        layers = ";".join(_draw_layer(rng, kind, kind == "train") for _ in range(count))
        option = {"encrypt": rng.choice(("x_fwd", "dy_dx", "x_dw", "dy_dw")), "decrypt": rng.choice(("fwd", "dx", "dw")),
                  "local": rng.choice(("fwd", "dx", "dw")), "online": rng.choice(pencil_plus.KINDS)}.get(kind, "")
        c = dict(kind=kind, layers=layers, log2_n=log2_n, limbs=limbs, bits=bits, option=option)
        w = work(c)
        # no costlier than the largest listed case; the whole protocol of a
        # layer and the preprocessed shares (64 tensors per party) much smaller
        share = {"train": 8, "online": 4, "local": 4}.get(kind, 2)
        if w["bytes"] * share <= most["bytes"] and w["flops"] * share <= most["flops"]:
            return c


# ------------------------------------------------------------------- inputs

def _layers(case):
    out = []
    for text in case["layers"].split(";"):
        kind, *v = text.split()
        b, ci, co, h, w, k, pad, s = (int(x) for x in v)
        out.append(LayerSpec(kind, b, ci, co, h, w, k, pad, s, log2_n=case["log2_n"], num_limbs=case["limbs"],
                             prime_bits=case["bits"]))
    return out


def _context(case, seed):
    return api.Context(case["log2_n"], case["limbs"], case["bits"], seed=1 + seed)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _uniform(g, shape):
    """A share: uniform over Z_t."""
    return torch.randint(0, T_PLAIN, tuple(shape), generator=g, device="cuda", dtype=torch.int64)


def _fixed(g, shape, std):
    """Fixed-point normal values, the integers floor(x 2^12)."""
    return torch.floor(torch.randn(tuple(shape), generator=g, device="cuda", dtype=torch.float64) * (std * FRAC))


def _weights(g, layer):
    w = _fixed(g, layer.w_shape(), (2.0 / (layer.c_in * layer.kh * layer.kw)) ** 0.5)
    return torch.remainder(w.to(torch.int64), T_PLAIN)


def _buffers(ctx, layer, plan, seed, ops):
    """Device buffers of one layer's products, ciphertexts encrypted by the data owner."""
    g = _generator(seed)
    s = ctx.layout(layer, plan)
    w, x0, x1 = _weights(g, layer), _uniform(g, layer.x_shape()), _uniform(g, layer.x_shape())
    d = dict(w=w, x0=x0)
    if "fwd" in ops:
        d["ct_x1"] = ctx.encrypt(layer, plan, "x_fwd", x1, 101)
        d["bias"] = _uniform(g, (layer.c_out,))
        d["ct_y"], d["y0"] = ctx.empty_cts(s.n_out[0]), torch.empty_like(_uniform(g, layer.y_shape()))
    if "dx" in ops or "dw" in ops:
        d["dy0"], dy1 = _uniform(g, layer.y_shape()), _uniform(g, layer.y_shape())
    if "dx" in ops:
        d["ct_dy_dx"] = ctx.encrypt(layer, plan, "dy_dx", dy1, 102)
        d["ct_dx"], d["dx0"] = ctx.empty_cts(s.n_out[1]), torch.empty_like(x0)
    if "dw" in ops:
        d["ct_x_dw"] = ctx.encrypt(layer, plan, "x_dw", x1, 103)
        d["ct_dy_dw"] = ctx.encrypt(layer, plan, "dy_dw", dy1, 104)
        d["ct_dw"], d["dw_mask"] = ctx.empty_cts(s.n_out[2]), torch.empty_like(w)
    return d


def prepare(case, seed):
    kind, layers = case["kind"], _layers(case)
    layer, ctx, g = layers[0], _context(case, seed), _generator(seed)
    st = dict(kind=kind, ctx=ctx, layer=layer, option=case["option"])
    if kind == "step":
        plans = [ctx.plan_auto(l) for l in layers]
        ios = [_buffers(ctx, l, p, seed + 7 * i, ("fwd", "dx", "dw")) for i, (l, p) in enumerate(zip(layers, plans))]
        step = api.Step([(ctx, l, p) for l, p in zip(layers, plans)])
        step.bind(ios, torch.empty(step.workspace_bytes(), dtype=torch.uint8, device="cuda"))
        st.update(step=step, ios=ios)
    elif kind in ("fwd", "layer"):
        plan = st["plan"] = ctx.plan_auto(layer)
        st["io"] = _buffers(ctx, layer, plan, seed, ("fwd",) if kind == "fwd" else ("fwd", "dx", "dw"))
        s = ctx.layout(layer, plan)
        need = s.ws_fwd_bytes if kind == "fwd" else max(s.ws_fwd_bytes, s.ws_bwd_bytes)
        st["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    elif kind in ("encrypt", "decrypt"):
        plan = st["plan"] = ctx.plan_auto(layer)
        s = ctx.layout(layer, plan)
        if kind == "encrypt":
            op = api.OPERANDS[case["option"]]
            st["share"] = _uniform(g, layer.y_shape() if case["option"].startswith("dy") else layer.x_shape())
            st["out"] = ctx.empty_cts(s.n_ct[op])
            st["ws"] = torch.empty(s.ws_enc_bytes, dtype=torch.uint8, device="cuda")
        else:
            d = _buffers(ctx, layer, plan, seed, (case["option"],))
            if case["option"] == "fwd":
                st["ct"] = ctx.linear_fwd(layer, plan, d["ct_x1"], d["x0"], d["w"], 7, bias=d["bias"])[0]
            else:
                dx = case["option"] == "dx"
                r = ctx.linear_bwd(layer, plan, d.get("ct_dy_dx"), d.get("ct_x_dw"), d.get("ct_dy_dw"), d["dy0"],
                                   d["x0"], d["w"], 7, do_dx=dx, do_dw=not dx)
                st["ct"] = r[0] if dx else r[2]
            st["ws"] = torch.empty(s.ws_dec_bytes, dtype=torch.uint8, device="cuda")
    elif kind == "local":
        st["a"], st["b"] = _local_inputs(layer, case["option"], seed)
    elif kind == "online":
        st.update(_online_inputs(layer, case["option"], seed))
    elif kind == "train":
        st["engine"] = autograd.EncryptedLinearEngine(layer, ctx)
        st.update(_train_inputs(layer, seed))
    return st


def _local_inputs(layer, op, seed):
    """Shares on both sides: x or dY, and W or dY."""
    g = _generator(seed)
    a = _uniform(g, layer.y_shape() if op == "dx" else layer.x_shape())
    return a, _uniform(g, layer.y_shape() if op == "dw" else layer.w_shape())


def _online_inputs(layer, kind, seed):
    g = _generator(seed)
    x, y, w = layer.x_shape(), layer.y_shape(), layer.w_shape()
    ush, vsh, osh = {"fwd": (w, x, y), "dx": (w, y, x), "dw01": (y, x, w), "dw10": (x, y, w)}[kind]
    rng = np.random.default_rng(seed)
    return dict(u=_uniform(g, ush), v=_uniform(g, vsh), u_masks=[_uniform(g, ush) for _ in range(MASKS)],
                v_masks=[_uniform(g, vsh) for _ in range(MASKS)],
                share0=[[_uniform(g, osh) for _ in range(MASKS)] for _ in range(MASKS)],
                share1=[[_uniform(g, osh) for _ in range(MASKS)] for _ in range(MASKS)],
                k=[int(c) for c in rng.integers(-1024, 1025, MASKS)],
                l=[int(c) for c in rng.integers(-1024, 1025, MASKS)])


def _train_inputs(layer, seed):
    g = _generator(seed)
    fan = layer.c_in * layer.kh * layer.kw
    return dict(x=_fixed(g, layer.x_shape(), 1.0).requires_grad_(),
                w=_fixed(g, layer.w_shape(), (2.0 / fan) ** 0.5).requires_grad_(),
                b=(_fixed(g, (layer.c_out,), 0.1) * FRAC).requires_grad_(), dy=_fixed(g, layer.y_shape(), 0.05))


# --------------------------------------------------------------------- a pass

def run(st):
    kind, ctx, layer = st["kind"], st["ctx"], st["layer"]
    if kind == "step":
        st["step"].run(1000)
        return [{k: d[k] for k in ("ct_y", "y0", "ct_dx", "dx0", "ct_dw", "dw_mask")} for d in st["ios"]]
    if kind in ("fwd", "layer"):
        d, plan = st["io"], st["plan"]
        ct_y, y0 = ctx.linear_fwd(layer, plan, d["ct_x1"], d["x0"], d["w"], 1000, bias=d["bias"], ws=st["ws"],
                                  out=(d["ct_y"], d["y0"]))
        if kind == "fwd":
            return ct_y, y0
        return (ct_y, y0) + tuple(ctx.linear_bwd(
            layer, plan, d["ct_dy_dx"], d["ct_x_dw"], d["ct_dy_dw"], d["dy0"], d["x0"], d["w"], 1001, ws=st["ws"],
            out=(d["ct_dx"], d["dx0"], d["ct_dw"], d["dw_mask"])))
    if kind == "encrypt":
        return ctx.encrypt(layer, st["plan"], st["option"], st["share"], 1000, out=st["out"], ws=st["ws"])
    if kind == "decrypt":
        return ctx.decrypt(layer, st["plan"], st["option"], st["ct"], ws=st["ws"])
    if kind == "local":
        return ctx.zt_linear(layer, st["option"], st["a"], st["b"])
    if kind == "online":
        return pencil_plus.online(ctx, layer, st["option"], st["u"], st["v"], st["u_masks"], st["v_masks"],
                                  st["share0"], st["share1"], st["k"], st["l"])
    y = autograd.encrypted_linear(st["x"], st["w"], st["engine"], st["b"])
    grads = torch.autograd.grad(y, (st["x"], st["w"], st["b"]), st["dy"])
    return (y.detach(),) + grads


# ----------------------------------------------------------------- its work

def _counts(layer, plan):
    """Per product (A tiles, K tiles, outputs, products) of the plan's partition."""
    l = layer
    out = []
    for t, (M, R, K, OH, OW, KH, KW) in (
            (plan.fwd, (l.batch, l.c_out, l.c_in, l.h_out, l.w_out, l.kh, l.kw)),
            (plan.dx, (l.batch, l.c_in, l.c_out, l.h, l.w, l.kh, l.kw)),
            (plan.dw, (l.c_in, l.c_out, l.batch, l.kh, l.kw, l.h_out, l.w_out))):
        nM, nR, nK, nY, nX, nky, nkx = (-(-a // b) for a, b in zip((M, R, K, OH, OW, KH, KW), t.astuple()))
        k = nK * nky * nkx
        out.append((nM * nY * nX * k, nR * k, nM * nR * nY * nX, nM * nR * nY * nX * k))
    return out


def _plan(layer):
    import ctypes
    p = api.A.Plan()
    api.A.check(api.A.load().pencil_plan_auto_n(layer.log2_n, ctypes.byref(api.layer_struct(layer)), ctypes.byref(p)))
    return p


def work(case):
    """Bytes each ciphertext and tensor moved once; operations: a residue
    multiply-accumulate counts 2, a butterfly 3 (multiply, add, subtract), a Z_t
    multiply-add 2."""
    kind, bytes_, flops = case["kind"], 0, 0
    poly = (1 << case["log2_n"]) * case["limbs"]
    ntt = 3 * poly * case["log2_n"] / 2
    for layer in _layers(case):
        X, Y, W = (int(np.prod(s)) for s in (layer.x_shape(), layer.y_shape(), layer.w_shape()))
        macs = Y * (W // layer.c_out)
        if kind in ("local", "online"):
            a, b, o = {"fwd": (X, W, Y), "dx": (Y, W, X), "dw": (X, Y, W), "dw01": (Y, X, W), "dw10": (X, Y, W)}[case["option"]]
            if kind == "online" and case["option"] in ("fwd", "dx"):
                a, b = b, a
            if kind == "local":
                bytes_, flops = bytes_ + 8 * (a + b + o), flops + 2 * macs
            else:
                n = MASKS
                bytes_ += 8 * ((n + 2) * (a + b) + (2 * n * n + 2) * o)
                flops += 4 * macs + 2 * (n * (a + 2 * b) + 2 * n * n * o)
            continue
        eq = layer
        if layer.stride > 1:
            e = api.stride_map(layer)
            eq = LayerSpec(e["kind"], e["batch"], e["c_in"], e["c_out"], e["h"], e["w"], e["k"], e["pad"],
                           log2_n=case["log2_n"], num_limbs=case["limbs"])
        n = _counts(eq, _plan(eq))
        if kind in ("encrypt", "decrypt"):
            if kind == "encrypt":
                which = {"x_fwd": (0, 0), "dy_dx": (1, 0), "x_dw": (2, 0), "dy_dw": (2, 1)}[case["option"]]
                cts = n[which[0]][which[1]]
                bytes_ += 16 * poly * cts + 8 * (Y if case["option"].startswith("dy") else X)
                flops += cts * (3 * ntt + 6 * poly)
            else:
                i = ("fwd", "dx", "dw").index(case["option"])
                bytes_ += 16 * poly * n[i][2] + 8 * (Y, X, W)[i]
                flops += n[i][2] * (2 * ntt + 4 * poly)
            continue
        for i in range(1 if kind == "fwd" else 3):
            na, nk, no, np_ = n[i]
            cts, pts, terms = (na, nk, 1) if i < 2 else (na + nk, na + nk, 2)
            bytes_ += 16 * poly * (cts + no) + 8 * (X + Y + W)
            flops += 4 * poly * (np_ * terms + no) + ntt * (pts + 3 * no + (na if i < 2 else 0))
            if kind == "train":  # the parties' ends around each product
                bytes_ += 16 * poly * (cts + no)
                flops += ntt * (3 * cts + 2 * no)
        if kind == "train":
            flops += 4 * macs
    return {"bytes": float(bytes_), "flops": float(flops)}


# ------------------------------------------------------------- exact results

def _mulmod_pow2(v, bits):
    for _ in range(bits // 14):
        v = (v << 14) % T_PLAIN
    return v


def _correlate(layer, op, a, b):
    """The layer's operator mod t of int64 arrays, from float64 products of
    14-bit digits (every sum is an integer below 2^53)."""
    F = torch.nn.functional
    a, b = a.cpu(), b.cpu()
    four = lambda v: v if v.dim() == 4 else v[:, :, None, :] if v.dim() == 3 else v[:, :, None, None]  # noqa: E731
    ph, pw, kh, kw = layer.pad_h, layer.pad_w, layer.kh, layer.kw
    s = layer.stride

    def plain(x, y):
        if layer.kind == "fc":
            return x @ y.T if op == "fwd" else x @ y if op == "dx" else y.T @ x
        x, y = four(x), four(y)
        if op == "fwd":
            return F.conv2d(x, y, stride=(1 if layer.kind == "conv1d" else s, s), padding=(ph, pw))
        if op == "dx":
            return F.conv2d(x, y.flip(2, 3).transpose(0, 1), padding=(kh - 1 - ph, kw - 1 - pw))
        return F.conv2d(x.transpose(0, 1), y.transpose(0, 1), padding=(ph, pw)).transpose(0, 1)

    total = None
    digits = lambda v: [((v >> (14 * i)) & 16383).double() for i in range(3)]  # noqa: E731
    for i, x in enumerate(digits(a)):
        for j, y in enumerate(digits(b)):
            p = _mulmod_pow2(plain(x, y).to(torch.int64) % T_PLAIN, 14 * (i + j))
            total = p if total is None else (total + p) % T_PLAIN
    shape = {"fwd": layer.y_shape(), "dx": layer.x_shape(), "dw": layer.w_shape()}[op]
    return total.reshape(shape)


def _combine(base, terms, coeffs):
    """base + sum c x mod t, products split at bit 21."""
    out = base.cpu()
    for x, c in zip(terms, coeffs):
        c, x = c % T_PLAIN, x.cpu()
        hi = (x * (c >> 21)) % T_PLAIN
        for _ in range(3):
            hi = (hi << 7) % T_PLAIN
        out = (out + hi + (x * (c & ((1 << 21) - 1))) % T_PLAIN) % T_PLAIN
    return out


def exact(case, seed):
    kind, layer = case["kind"], _layers(case)[0]
    macs = int(np.prod(layer.y_shape())) * layer.c_in * layer.kh * layer.kw
    if macs > 2e9:  # about 20 s of digit products
        return None
    if kind == "local":
        return _correlate(layer, case["option"], *_local_inputs(layer, case["option"], seed))
    if kind == "online":
        s = _online_inputs(layer, case["option"], seed)
        u, v, um, vm, k, l = s["u"], s["v"], s["u_masks"], s["v_masks"], s["k"], s["l"]
        op = case["option"][:2] if case["option"].startswith("dw") else case["option"]
        apply = lambda a, b: _correlate(layer, op, *((a, b) if case["option"] == "dw10" else (b, a)))  # noqa: E731
        u_t, v_t = _combine(u, um, [-c for c in k]), _combine(v, vm, [-c for c in l])
        kl = [a * b for a in k for b in l]
        out1 = _combine(apply(u_t, _combine(torch.zeros_like(v), vm, l)), sum(s["share1"], []), kl)
        out0 = _combine(apply(u, v_t), sum(s["share0"], []), kl)
        return out0, out1, u_t, v_t
    if kind == "train":
        d = {n: t.detach().cpu() for n, t in _train_inputs(layer, seed).items()}
        x, w, b = (d[n].requires_grad_() for n in ("x", "w", "b"))
        F = torch.nn.functional
        if layer.kind == "fc":
            y = F.linear(x, w, b)
        elif layer.kind == "conv":
            y = F.conv2d(x, w, b, stride=layer.stride, padding=layer.pad)
        else:
            y = F.conv1d(x, w, b, stride=layer.stride, padding=layer.pad)
        return (y.detach(),) + torch.autograd.grad(y, (x, w, b), d["dy"])
    return None
