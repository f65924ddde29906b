#!/usr/bin/env python3
"""Throughput of the model owner's encrypted linear-layer products (fwd + bwd).

One step = every product of the workload's layers: the forward product
(Alg. 1), the input-gradient product and the weight-gradient cross terms
(Alg. 2), each through the whole hot path (share add + encode, NTT,
multiply-accumulate, re-randomise, inverse NTT, flood and mask), with the data
owner's ciphertexts and both parties' shares already resident in HBM.
Encryption and decryption (the data owner's ends) are outside the timed region.

Default workload: the eight-layer stack of 3x3 convolutions (3 x 64->64 on
32x32, 3 x 128->128 on 16x16, 2 x 256->256 on 8x8), batch 64, forward and
backward, N = 16384 with four 60-bit RNS primes.  `--config 2` is the FC layer
784 -> 128 (the first layer of the paper's MNIST MLP).  After the timed region
the outputs are decrypted and checked bit for bit against exact modular linear
algebra (float64 digit products, exact below 2^53).

Prints one JSON line.  `--gpus N` with N > 1 exits: the benchmark runs on one GPU.
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# 32-bit integer multiply peak: 256 CUs x 64 lanes x 2.4 GHz, the full VALU
# issue rate.  On gfx950 the multiply forms the kernels use (v_mad_u64_u32,
# v_mul_lo_u32, v_mul_hi_u32) issue at close to that rate: the library's probe
# (pencil_probe_mul32, `--mul-probe`) measures 30-34 T/s.
MUL32_PEAK_TOPS = 256 * 64 * 2.4e9 / 1e12
# int8 matrix-core peak: 256 CUs x 8192 operations per clock x 2.4 GHz, dense.
INT8_PEAK_TOPS = 256 * 8192 * 2.4e9 / 1e12
# 32-bit multiplies of a butterfly: 5 with moduli within 2^26 below 2^60 (four for
# the product by the split twiddle, one to fold it), else 9 (3 for Shoup's
# quotient estimate y1 ws1 + hi(y0 ws1) + hi(y1 ws0), 3 + 3 for the low halves of
# y w and est q).
MUL32_PER_BUTTERFLY = {True: 5, False: 9}
# A multiply-accumulate of two residues: 4 32-bit multiplies of split 30-bit
# operands on the vector units, 64 products of 8-bit digits on the matrix cores
# (a multiplication and an addition each; the windows' zero padding is not counted).
MUL32_PER_MAC = 4
INT8_PER_MAC = 128


def mul32_per_butterfly(ctx):
    return MUL32_PER_BUTTERFLY[all((1 << 60) - q <= 1 << 26 for q in ctx.primes)]


# Schedule choices measured on MI355X, reused so that the benchmark and its
# rocprofv3 summaries run the same kernels.
DEFAULT_TUNE_CACHE = os.path.join(ROOT, "paper_2403_11166_amd", "autotune_gfx950.txt")


def parse():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", type=int, default=5, help="workload index (1..5); default: the largest, the "
                    "eight-layer convolution stack at N = 16384")
    ap.add_argument("--workload", default="", help="one of the extra layer-shape workloads by name "
                    "(MNIST CNN with its stride-2 layer, TextCNN's Conv1d layers, FC 2048->1001); overrides --config")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=15.0, help="CPU oracle sample budget")
    ap.add_argument("--no-verify", action="store_true")
    ap.add_argument("--mode", choices=("step", "graph", "layer"), default="step",
                    help="timed launch path: batched step (phase launches with live kernel events), "
                         "its captured HIP graph, or one launch sequence per product and layer")
    ap.add_argument("--compare-steps", type=int, default=3, help="steps timed for the other launch paths")
    ap.add_argument("--pencil-plus", type=int, default=-1, metavar="M",
                    help="also measure Pencil+ (preprocessed products, M masks per party) on the first "
                         "layer; default 8 on the default workload, 0 (off) on the others")
    ap.add_argument("--no-do-side", action="store_true",
                    help="skip timing the data owner's encryption and decryption after the measured region")
    ap.add_argument("--no-autotune", action="store_true",
                    help="use the planner's default schedules instead of timing the candidates first")
    ap.add_argument("--tune-cache", default=DEFAULT_TUNE_CACHE,
                    help="autotuner cache file (earlier choices are reused, new ones appended); '' = none")
    ap.add_argument("--mul-probe", action="store_true",
                    help="only measure the issue rate of the 32-bit multiply forms (the integer peak) and print it")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="MIB",
                    help="only run a plain device copy of MIB MiB (the reference kernel that scales "
                         "HBM counters into bytes) and print its size and time")
    return ap.parse_args()


# ------------------------------------------------------------- hbm traffic

def kernel_source_hash():
    """sha256 over the device sources (the .hip and .h files) and the committed
    autotuning cache, which fixes the plans and schedules the benchmark runs; a
    traffic record holds for this hash only."""
    import hashlib
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2403_11166_amd", "csrc")
    files = [os.path.join(csrc, n) for n in sorted(os.listdir(csrc)) if n.endswith((".hip", ".h"))]
    for path in files + [DEFAULT_TUNE_CACHE]:
        if os.path.exists(path):
            with open(path, "rb") as f:
                h.update(f.read())
    return h.hexdigest()


def recorded_traffic(kernel, workload):
    """HBM bytes per launch of `kernel` on `workload` from the rocprofv3 counter
    summaries under profiles/ (FETCH_SIZE + WRITE_SIZE, scaled by a plain copy of
    known size), or None when none was taken from the current kernel sources."""
    pdir = os.path.join(ROOT, "profiles")
    if not os.path.isdir(pdir):
        return None
    want = kernel_source_hash()
    for name in sorted(os.listdir(pdir)):
        with open(os.path.join(pdir, name)) as f:
            for line in f:
                if not line.startswith("traffic:"):
                    continue
                kv = dict(tok.split("=", 1) for tok in line.split()[1:] if "=" in tok)
                if kv.get("kernel") == kernel and kv.get("workload") == workload and kv.get("source_sha256") == want:
                    return int(kv["fetch_bytes_per_launch"]) + int(kv["write_bytes_per_launch"])
    return None


def copy_probe(mib):
    import torch
    n = mib << 20
    src = torch.ones(n, dtype=torch.uint8, device="cuda")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    reps = 5
    ev0.record()
    for _ in range(reps):
        dst.copy_(src)
    ev1.record()
    torch.cuda.synchronize()
    ms = ev0.elapsed_time(ev1) / reps
    print(json.dumps({"copy_probe_bytes_read": n, "copy_probe_bytes_written": n, "launches": reps + 1,
                      "avg_ms": round(ms, 4), "GBps_read_plus_write": round(2 * n / (ms / 1e3) / 1e9, 1)}),
          flush=True)


# ------------------------------------------------------------- exact check

def _digits(v, t):
    import torch
    v = torch.where(v > (t - 1) // 2, v - t, v)
    out = []
    for _ in range(2):
        d = torch.remainder(v, 1 << 14)
        out.append(d.double())
        v = torch.div(v - d, 1 << 14, rounding_mode="floor")
    out.append(v.double())
    return out


def _lin_f64(layer, op, a, b):
    """The layer's product over float64 tensors holding integers (no rounding below 2^53)."""
    import torch
    import torch.nn.functional as F
    if layer.kind == "fc":
        return {"fwd": lambda: a @ b.t(), "dx": lambda: a @ b, "dw": lambda: b.t() @ a}[op]()
    k, p = (layer.kh, layer.kw), (layer.pad_h, layer.pad_w)
    st = (1, layer.stride) if layer.kind == "conv1d" else (layer.stride, layer.stride)
    ho, wo = layer.h_out, layer.w_out
    as4 = (lambda v: v.reshape(v.shape[0], v.shape[1], 1, v.shape[-1])) if layer.kind == "conv1d" else (lambda v: v)
    a, b = as4(a), as4(b)
    if op == "fwd":
        cols = F.unfold(a, k, padding=p, stride=st)                # (B, ci*kh*kw, ho*wo)
        out = (b.reshape(b.shape[0], -1) @ cols).reshape(a.shape[0], b.shape[0], ho, wo)
    elif op == "dx":                                             # a = dY, b = W
        cols = b.reshape(b.shape[0], -1).t() @ a.reshape(a.shape[0], a.shape[1], -1)  # (B, ci*kh*kw, ho*wo)
        out = F.fold(cols, (layer.h, layer.w), k, padding=p, stride=st)
    else:
        cols = F.unfold(a, k, padding=p, stride=st)                # a = X, b = dY
        g = torch.einsum("bop,bcp->oc", b.reshape(b.shape[0], b.shape[1], -1), cols)
        out = g.reshape(b.shape[1], a.shape[1], k[0], k[1])
    return out.reshape(out.shape[0], out.shape[1], out.shape[-1]) if layer.kind == "conv1d" else out


def exact_mod_t(layer, op, a, b, t):
    """Exact Z_t result of the layer's product on int64 tensors in [0, t)."""
    import torch
    da, db = _digits(a, t), _digits(b, t)
    T = [None] * 5
    for i in range(3):
        for j in range(3):
            s = torch.remainder(torch.round(_lin_f64(layer, op, da[i], db[j])).long(), t)
            T[i + j] = s if T[i + j] is None else torch.remainder(T[i + j] + s, t)
    acc = T[4]
    for d in range(3, -1, -1):
        acc = torch.remainder(acc * (1 << 14) + T[d], t)
    return acc


# ------------------------------------------------------------- work model

def kernel_work(entries):
    """Algorithmic HBM bytes and operations per kernel kind over one step, for
    (context, layer, plan, sizes, products) entries.

    bytes: every polynomial the kernel must read and write once (8-byte
    residues); operations: 32-bit multiplies, mul32_per_butterfly per butterfly
    ((N/2) log2 N per limb-polynomial) and MUL32_PER_MAC per multiply-accumulate
    (one per product, component, limb and slot), or INT8_PER_MAC int8 operations
    for one on the matrix cores.  The flood's Philox and reductions are not
    counted (0).
    """
    work = {}
    for ctx_, layer_, plan_, sz, ops in entries:
        n, L = ctx_.n, ctx_.L
        lg = n.bit_length() - 1
        poly = L * n * 8
        bfly = L * (n // 2) * lg
        for opi, op in enumerate(("fwd", "dx", "dw")):
            if op not in ops:
                continue
            n_out = sz.n_out[opi]
            if op == "fwd":
                n_ct_in, n_pt = sz.n_ct[0], sz.n_pt[0]
            elif op == "dx":
                n_ct_in, n_pt = sz.n_ct[1], sz.n_pt[1]
            else:
                n_ct_in, n_pt = sz.n_ct[2] + sz.n_ct[3], sz.n_pt[2]
            add = lambda k, b, o: work.__setitem__(k, (work.get(k, (0, 0))[0] + b, work.get(k, (0, 0))[1] + o))  # noqa
            b10 = mul32_per_butterfly(ctx_) * bfly
            # one launch holds a product's forward transforms: plaintexts, masks and,
            # for the forward and input-gradient products, the model owner's share,
            # added to component 0 of the input ciphertexts, which is read and
            # written once (staged copy; they arrive in the NTT domain, and the
            # multiply-accumulate reads the rest in place)
            n_share = n_ct_in if op != "dw" else 0
            add("ntt_ct" if n_share else "ntt_pt", (2 * n_share + n_pt + n_out) * poly, (n_share + n_pt + n_out) * b10)
            matrix = ctx_.on_matrix_cores(layer_, plan_, op)
            add("mac_matrix" if matrix else "mac", (2 * n_ct_in + n_pt + n_out + 2 * n_out) * poly,
                (INT8_PER_MAC if matrix else MUL32_PER_MAC) * sz.n_products[opi] * 2 * L * n)
            add("intt_out", 2 * n_out * 2 * poly, 2 * n_out * b10)
            add("flood_mask", 2 * n_out * 2 * poly, 0)
    # the batched step's phase launches cover the same work
    get = lambda k: work.get(k, (0, 0))  # noqa: E731
    work["step_ntt"] = tuple(get("ntt_ct")[i] + get("ntt_pt")[i] for i in range(2))
    work["step_mac"] = get("mac")
    work["step_mac_matrix"] = get("mac_matrix")
    work["step_intt"] = get("intt_out")
    work["step_flood"] = get("flood_mask")
    return work


# ------------------------------------------------------------- Pencil+

def pencil_plus_bench(e, m, he_step_ms, torch):
    """Pencil+ on one layer (Alg. 3, Alg. 4): the homomorphic preprocessing of the
    four operators (m^2 products each) and the online phase of one training
    step (the four operators' online phases), timed after the main region.
    The online results are reconstructed and checked against exact modular
    linear algebra."""
    from paper_2403_11166_amd import pencil_plus as GP
    ctx, L_, plan, d = e["ctx"], e["layer"], e["plan"], e["d"]
    t = ctx.t
    gen = torch.Generator(device="cpu").manual_seed(1234)

    def rnd(shape):
        return torch.randint(0, t, shape, generator=gen, dtype=torch.int64).cuda()

    ops = {"fwd": (d["W"], d["x1"]), "dx": (d["W"], d["dy1"]), "dw01": (d["dy0"], d["x1"]), "dw10": (d["x0"], d["dy1"])}
    masks, shares, prep_ms, prep_products = {}, {}, 0.0, 0
    sz = e["sz"]
    per_op = {"fwd": sz.n_products[0], "dx": sz.n_products[1], "dw01": sz.n_products[2] // 2,
              "dw10": sz.n_products[2] // 2}
    for i, (kind, (u, v)) in enumerate(ops.items()):
        um = [rnd(tuple(u.shape)) for _ in range(m)]
        vm = [rnd(tuple(v.shape)) for _ in range(m)]
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        sh = GP.prep(ctx, L_, plan, kind, um, vm, 50000 + 1000 * i)
        torch.cuda.synchronize()
        prep_ms += (time.perf_counter() - t0) * 1e3
        prep_products += m * m * per_op[kind]
        masks[kind], shares[kind] = (um, vm), sh
    k = [int(x) for x in torch.randint(1, t, (m,), generator=gen)]
    l = [int(x) for x in torch.randint(1, t, (m,), generator=gen)]

    def online_step():
        return {kind: GP.online(ctx, L_, kind, u, v, masks[kind][0], masks[kind][1], shares[kind][0],
                                shares[kind][1], k, l) for kind, (u, v) in ops.items()}

    res = online_step()
    torch.cuda.synchronize()
    reps = 5

    def timed_reps(fn):
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ev0.record()
        for _ in range(reps):
            fn()
        ev1.record()
        torch.cuda.synchronize()
        return ev0.elapsed_time(ev1) / reps

    eager_ms = timed_reps(online_step)
    # the online phase is ~100 short launches: replay it as one captured graph
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        online_step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        gres = online_step()
    g.replay()
    torch.cuda.synchronize()
    replay_same = all(torch.equal(gres[kd][q], res[kd][q]) for kd in ops for q in range(4))
    online_ms = timed_reps(g.replay)
    torch.cuda.synchronize()
    replay_same &= all(torch.equal(gres[kd][q], res[kd][q]) for kd in ops for q in range(4))
    want = {"fwd": exact_mod_t(L_, "fwd", d["x1"], d["W"], t), "dx": exact_mod_t(L_, "dx", d["dy1"], d["W"], t),
            "dw01": exact_mod_t(L_, "dw", d["x1"], d["dy0"], t), "dw10": exact_mod_t(L_, "dw", d["x0"], d["dy1"], t)}
    exact = all(torch.equal(torch.remainder(res[kd][0] + res[kd][1], t), want[kd]) for kd in ops)
    # the online phase's dense part, one Z_t correlation per operator timed alone:
    # output entries x contraction length multiply-adds
    macs = L_.batch * L_.c_out * L_.h_out * L_.w_out * L_.c_in * L_.kh * L_.kw
    corr = {}
    for kind, (u, v) in ops.items():
        ms = timed_reps(lambda: GP.apply(ctx, L_, kind, u, v))
        corr[kind] = {"ms": round(ms, 4), "macs_Tps": round(macs / (ms / 1e3) / 1e12, 3)}
    return {"m": m, "layer": f"{L_.kind} {L_.c_in}->{L_.c_out} {L_.h}x{L_.w} b{L_.batch}",
            "prep": {"products": int(prep_products), "wall_ms": round(prep_ms, 2),
                     "products_per_s": round(prep_products / (prep_ms / 1e3), 1),
                     "note": "per-call launches from Python, wall clock, includes the data owner's "
                             "encryptions and decryptions"},
            "online": {"ms_per_step": round(online_ms, 4), "launch": "HIP graph replay",
                       "eager_ms_per_step": round(eager_ms, 4), "operators": list(ops),
                       "he_step_ms": round(he_step_ms, 4), "speedup_vs_he_step": round(he_step_ms / online_ms, 2),
                       "bit_exact": bool(exact), "graph_replays_match_eager": bool(replay_same)},
            "zt_correlation": {"macs_per_call": int(macs), "calls_per_step": 8, "per_operator": corr}}


# ------------------------------------------------------------- cpu baseline

def _host_threads():
    """Host cores this process may use (its CPU affinity), capped at 16 (one GPU's share of the host)."""
    try:
        avail = len(os.sched_getaffinity(0))
    except AttributeError:
        avail = os.cpu_count() or 1
    return max(1, min(avail, 16))


def cpu_baseline(layer, seconds):
    """The oracle timed on host cores, in two legs.

    (ii) its plaintext x ciphertext product (schoolbook negacyclic
    multiplication per limb and component, in the oracle's plain-C helper,
    which releases the GIL) on one thread and then on every usable host core;
    products/s is the all-core rate.  (i) its plaintext Z_t layer operators
    (forward, input gradient, weight gradient) on the layer's full shape.
    About `seconds` of wall time per product leg."""
    from concurrent.futures import ThreadPoolExecutor
    from oracle import bfv
    from oracle import linear as LN
    from oracle import params as PR
    P = PR.params_for(layer)
    rng = np.random.default_rng(0)
    ct = np.stack([np.stack([rng.integers(0, q, P.n, dtype=np.uint64) for q in P.moduli]) for _ in range(2)])
    w = rng.integers(0, P.t, P.n)

    def one_product(_=None):
        acc = [[[0] * P.n for _ in range(P.num_limbs)] for _ in range(2)]
        bfv.mul_plain_acc(P, acc, ct, w, P.t)
        return 1

    def rate(threads):
        done, t0 = 0, time.perf_counter()
        with ThreadPoolExecutor(threads) as ex:
            while True:
                done += sum(ex.map(one_product, range(threads)))
                el = time.perf_counter() - t0
                if el >= seconds:
                    return done, el

    n1, el1 = rate(1)
    threads = _host_threads()
    nall, elall = rate(threads) if threads > 1 else (n1, el1)
    # (i) the plaintext layer operators at full size, once each
    xs = rng.integers(0, P.t, layer.x_shape(), dtype=np.int64)
    ws = rng.integers(0, P.t, layer.w_shape(), dtype=np.int64)
    dys = rng.integers(0, P.t, layer.y_shape(), dtype=np.int64)
    t0 = time.perf_counter()
    LN.layer_op(layer, "fwd", xs, ws, P.t)
    LN.layer_op(layer, "dx", dys, ws, P.t)
    LN.layer_op(layer, "dw", xs, dys, P.t)
    plain_s = time.perf_counter() - t0
    return {"value": round(nall / elall, 3), "unit": "products/s", "cores": threads, "kind": "oracle",
            "nproc": os.cpu_count(), "single_core_products_per_s": round(n1 / el1, 3),
            "plaintext_layer_ops_s": round(plain_s, 3),
            "sample": f"{nall} plaintext x ciphertext products at N={P.n}, L={P.num_limbs} (schoolbook "
                      f"negacyclic, both components, all limbs) in {elall:.1f} s on {threads} threads, and "
                      f"{n1} in {el1:.1f} s on one; plaintext leg: the forward, input-gradient and "
                      f"weight-gradient Z_t operators of {layer.kind} {layer.c_in}->{layer.c_out} "
                      f"{layer.h}x{layer.w} b{layer.batch} once each (numpy, its own BLAS threads)"}


# ------------------------------------------------------------- main

def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py: measures one GPU; --gpus {args.gpus} is not supported "
              "(sharding across GPUs is designed, not built)", file=sys.stderr)
        sys.exit(2)
    if args.copy_probe:
        copy_probe(args.copy_probe)
        return
    if args.mul_probe:
        import ctypes
        import torch
        from paper_2403_11166_amd import _abi as A
        torch.cuda.init()
        lib = A.load()
        rates = {}
        for kind, name in enumerate(("v_mad_u64_u32", "v_mul_lo_u32", "v_mul_hi_u32")):
            r = ctypes.c_double()
            A.check(lib.pencil_probe_mul32(kind, ctypes.byref(r)))
            rates[name] = round(r.value / 1e12, 3)
        print(json.dumps({"mul32_probe_T_per_s": rates, "assumed_peak_T_per_s": round(MUL32_PEAK_TOPS, 3),
                          "cus": torch.cuda.get_device_properties(0).multi_processor_count}), flush=True)
        return
    import torch
    from paper_2403_11166_amd import Context
    from paper_2403_11166_amd import _abi as A
    from paper_2403_11166_amd.api import stride_map
    from workloads import CONFIGS, EXTRA_WORKLOADS, LayerSpec
    from workloads.gen import config_tensors
    import ctypes
    import dataclasses

    cfg = EXTRA_WORKLOADS[args.workload] if args.workload else CONFIGS[args.config]
    tensors = config_tensors(cfg)
    torch.cuda.init()
    dev = torch.device("cuda", 0)
    ctxs = {}
    tuned = {}
    layers = []
    relayout_ms = 0.0
    for li, (layer, ts) in enumerate(zip(cfg.layers, tensors)):
        key = (layer.log2_n, layer.num_limbs, layer.prime_bits)
        if key not in ctxs:
            ctxs[key] = Context(layer.log2_n, layer.num_limbs, layer.prime_bits, seed=cfg.seed)
        ctx = ctxs[key]
        strided = None
        if layer.stride > 1:
            # both parties move their shares (and the MO its weights) to the
            # stride-1 space-to-depth equivalent; the products run on that layer
            eqd = stride_map(layer)
            eq = dataclasses.replace(layer, **{k: eqd[k] for k in ("kind", "c_in", "h", "w", "k", "pad", "stride")})
            d0 = {k: torch.from_numpy(v).to(dev) for k, v in ts.items()}
            ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            ev0.record()
            moved = {"x0": ctx.stride_relayout(layer, "x", d0["x0"]), "x1": ctx.stride_relayout(layer, "x", d0["x1"]),
                     "W": ctx.stride_relayout(layer, "w", d0["W"])}
            ev1.record()
            torch.cuda.synchronize()
            relayout_ms += ev0.elapsed_time(ev1)
            ts = dict(ts, **{k: v.cpu().numpy() for k, v in moved.items()})
            strided, layer = (layer, d0), eq
        plan = ctx.plan_auto(layer)
        if not args.no_autotune:
            # schedule-only choices (bit-identical results), timed outside the measured region
            tkey = (key, layer.kind, layer.batch, layer.c_in, layer.c_out, layer.h, layer.w, layer.k, layer.pad)
            if tkey not in tuned:
                tuned[tkey] = ctx.autotune(layer, plan, args.tune_cache or None)
            plan = tuned[tkey]
        sz = ctx.layout(layer, plan)
        d = {k: torch.from_numpy(v).to(dev) for k, v in ts.items()}
        ent = dict(layer=layer, ctx=ctx, plan=plan, sz=sz, d=d, strided=strided)
        ent["ct_x"] = ctx.encrypt(layer, plan, "x_fwd", d["x1"], 1000 + li)
        if "dx" in cfg.ops:
            ent["ct_dy_dx"] = ctx.encrypt(layer, plan, "dy_dx", d["dy1"], 2000 + li)
        if "dw" in cfg.ops:
            ent["ct_x_dw"] = ctx.encrypt(layer, plan, "x_dw", d["x1"], 3000 + li)
            ent["ct_dy_dw"] = ctx.encrypt(layer, plan, "dy_dw", d["dy1"], 4000 + li)
        ent["ws_f"] = ctx._ws(sz.ws_fwd_bytes)
        ent["ws_b"] = ctx._ws(sz.ws_bwd_bytes)
        ent["out_f"] = (ctx.empty_cts(sz.n_out[0]), torch.empty(layer.y_shape(), dtype=torch.int64, device=dev))
        ent["out_b"] = (ctx.empty_cts(sz.n_out[1]), torch.empty(layer.x_shape(), dtype=torch.int64, device=dev),
                        ctx.empty_cts(sz.n_out[2]), torch.empty(layer.w_shape(), dtype=torch.int64, device=dev))
        layers.append(ent)
    torch.cuda.synchronize()

    def layer_step(nonce):
        for li, e in enumerate(layers):
            L_, c, d = e["layer"], e["ctx"], e["d"]
            c.linear_fwd(L_, e["plan"], e["ct_x"], d["x0"], d["W"], nonce + 2 * li, ws=e["ws_f"], out=e["out_f"])
            if "dx" in cfg.ops or "dw" in cfg.ops:
                c.linear_bwd(L_, e["plan"], e.get("ct_dy_dx"), e.get("ct_x_dw"), e.get("ct_dy_dw"), d["dy0"],
                             d["x0"], d["W"], nonce + 2 * li + 1, ws=e["ws_b"], out=e["out_b"],
                             do_dx="dx" in cfg.ops, do_dw="dw" in cfg.ops)

    from paper_2403_11166_amd import Step
    step_obj = Step([(e["ctx"], e["layer"], e["plan"]) for e in layers], ops=cfg.ops)
    step_ws = torch.empty(step_obj.workspace_bytes(), dtype=torch.uint8, device=dev)
    step_obj.bind([dict(ct_x1=e["ct_x"], ct_dy_dx=e.get("ct_dy_dx"), ct_x_dw=e.get("ct_x_dw"),
                        ct_dy_dw=e.get("ct_dy_dw"), x0=e["d"]["x0"], dy0=e["d"]["dy0"], w=e["d"]["W"],
                        ct_y=e["out_f"][0], y0=e["out_f"][1], ct_dx=e["out_b"][0], dx0=e["out_b"][1],
                        ct_dw=e["out_b"][2], dw_mask=e["out_b"][3]) for e in layers], step_ws)
    n_layers = len(layers)
    stream = torch.cuda.current_stream()

    def timed(fn, steps, profile):
        for c in ctxs.values():
            c._check(c.lib.pencil_profile_enable(c.h, 1 if profile else 0))
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ev0.record(stream)
        for i in range(steps):
            fn(i)
        ev1.record(stream)
        torch.cuda.synchronize()
        return ev0.elapsed_time(ev1) / steps, time.perf_counter() - t0

    def read_stats():
        stats = {}
        for c in ctxs.values():
            arr = (A.KernelStat * 16)()
            cnt = ctypes.c_int()
            c._check(c.lib.pencil_profile_read(c.h, arr, 16, ctypes.byref(cnt)))
            for i in range(cnt.value):
                nm = arr[i].name.decode()
                l0, m0 = stats.get(nm, (0, 0.0))
                stats[nm] = (l0 + arr[i].launches, m0 + arr[i].total_ms)
            c._check(c.lib.pencil_profile_enable(c.h, 0))
        return stats

    runners = {
        "layer": lambda i: layer_step(1000 + 2 * n_layers * i),
        "step": lambda i: step_obj.run(1000 + 2 * n_layers * i),
    }
    for i in range(args.warmup):
        runners["layer"](i)
        runners["step"](i)
    step_obj.capture()
    step_obj.set_nonce(1000)
    runners["graph"] = lambda i: step_obj.replay()
    for i in range(args.warmup):
        runners["graph"](i)
    torch.cuda.synchronize()

    compare = {}
    for mode in ("layer", "step", "graph"):
        if mode != args.mode:
            compare[mode] = round(timed(runners[mode], args.compare_steps, False)[0], 4)
    # the timed region: kernel events on (graph replays carry no events; their
    # kernels are timed from an eager run of the same step just after)
    ms_step, wall = timed(runners[args.mode], args.steps, args.mode != "graph")
    if args.mode == "graph":
        timed(runners["step"], args.steps, True)
    stats = read_stats()
    compare[args.mode] = round(ms_step, 4)

    products = sum(sum(e["sz"].n_products[i] for i, op in enumerate(("fwd", "dx", "dw")) if op in cfg.ops)
                   for e in layers)
    value = products / (ms_step / 1e3)

    # ------------------------------------------------------ bit-exact check
    bit_exact = None
    if not args.no_verify:
        bit_exact = True
        for e in layers:
            L_, c, d, t = e["layer"], e["ctx"], e["d"], e["ctx"].t
            # a strided layer is checked against its own definition: outputs of
            # the stride-1 equivalent, gradients mapped back by each party
            S, o = e["strided"] if e["strided"] else (L_, d)
            back = (lambda which, v: c.stride_relayout(S, which, v)) if e["strided"] else (lambda which, v: v)
            y1 = c.decrypt(L_, e["plan"], "fwd", e["out_f"][0])
            ok = torch.equal(torch.remainder(e["out_f"][1] + y1, t), exact_mod_t(S, "fwd", d["X"], o["W"], t))
            if "dx" in cfg.ops:
                dx1 = c.decrypt(L_, e["plan"], "dx", e["out_b"][0])
                ok &= torch.equal(torch.remainder(back("dx", e["out_b"][1]) + back("dx", dx1), t),
                                  exact_mod_t(S, "dx", d["dY"], o["W"], t))
            if "dw" in cfg.ops:
                dw1 = c.decrypt(L_, e["plan"], "dw", e["out_b"][2])
                cross = torch.remainder(exact_mod_t(S, "dw", o["x1"], d["dy0"], t)
                                        + exact_mod_t(S, "dw", o["x0"], d["dy1"], t), t)
                ok &= torch.equal(torch.remainder(back("dw", e["out_b"][3]) + back("dw", dw1), t), cross)
            bit_exact &= bool(ok)

    # ------------------------------------------------------ roofline
    work = kernel_work([(e["ctx"], e["layer"], e["plan"], e["sz"], cfg.ops) for e in layers])
    per_step = {k: (stats[k][0] / args.steps, stats[k][1] / args.steps) for k in stats if stats[k][0]}
    dom = max(per_step, key=lambda k: per_step[k][1])
    launches, ms = per_step[dom]
    bytes_step, ops_step = work.get(dom, (0, 0))
    # per launch: algorithmic work of one launch over its average duration
    avg_ms = ms / launches
    gbs = bytes_step / launches / (avg_ms / 1e3) / 1e9
    tops = ops_step / launches / (avg_ms / 1e3) / 1e12
    on_matrix = dom.endswith("mac_matrix")
    peak = INT8_PEAK_TOPS if on_matrix else MUL32_PEAK_TOPS
    roof = {"kernel": dom, "launches_per_step": launches, "avg_launch_ms": round(avg_ms, 5),
            "bound": "mfma" if on_matrix else "alu", "achieved": round(tops, 3), "peak": round(peak, 3),
            "unit": "T int8-op/s" if on_matrix else "T int32-multiply/s", "frac": round(tops / peak, 4),
            "traffic": recorded_traffic(dom, cfg.name),
            "work_per_launch": {"int8_ops" if on_matrix else "mul32": int(ops_step / launches),
                                "algo_bytes": int(bytes_step / launches)},
            "hbm": {"achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                    "frac": round(gbs / HBM_PEAK_GBS, 4)}}
    breakdown = {k: {"launches": v[0], "ms": round(v[1], 4),
                     "algo_GBps": round(work.get(k, (0, 0))[0] / (v[1] / 1e3) / 1e9, 1) if v[1] else None,
                     ("int8_Tops" if k.endswith("mac_matrix") else "mul32_Tps"):
                         round(work.get(k, (0, 0))[1] / (v[1] / 1e3) / 1e12, 3) if v[1] else None}
                 for k, v in sorted(per_step.items(), key=lambda kv: -kv[1][1])}

    # ------------------------------------------------------ NTT throughput
    # The metric's second figure: forward and inverse negacyclic NTTs over a
    # batch of the first layer's input ciphertexts (both components, every
    # limb), 16 N bytes per limb-polynomial (read and write once).
    e0 = layers[0]
    c0 = e0["ctx"]
    polys = e0["ct_x"].clone()
    npoly = polys.numel() // c0.n
    lg = c0.n.bit_length() - 1

    def ntt_ms(inverse):
        c0.ntt(polys, inverse)
        torch.cuda.synchronize()
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ev0.record(stream)
        for _ in range(5):
            c0.ntt(polys, inverse)
        ev1.record(stream)
        torch.cuda.synchronize()
        return ev0.elapsed_time(ev1) / 5

    ntt_rec = {"limb_polys": int(npoly), "N": c0.n, "L": c0.L, "bytes": int(16 * c0.n * npoly)}
    for name, inv in (("forward", False), ("inverse", True)):
        ms = ntt_ms(inv)
        gbs = 16 * c0.n * npoly / (ms / 1e3) / 1e9
        mul = mul32_per_butterfly(c0) * npoly * (c0.n // 2) * lg / (ms / 1e3) / 1e12
        ntt_rec[name] = {"ms": round(ms, 4), "GBps": round(gbs, 1), "hbm_frac": round(gbs / HBM_PEAK_GBS, 4),
                         "mul32_Tps": round(mul, 3), "mul32_frac": round(mul / MUL32_PEAK_TOPS, 4)}
    del polys

    # ------------------------------------------------------ data owner's ends
    # Encryption of the first layer's input ciphertexts and decryption of its
    # forward outputs, timed after the measured region (they are not part of
    # the model owner's step).
    do_side = None
    if not args.no_do_side:
        e = layers[0]
        c, L_, plan, sz = e["ctx"], e["layer"], e["plan"], e["sz"]
        enc_ws = c._ws(sz.ws_enc_bytes)
        dec_ws = c._ws(sz.ws_dec_bytes)
        out_ct = c.empty_cts(sz.n_ct[0])
        reps = 5

        def timed_calls(fn):
            fn(0)
            torch.cuda.synchronize()
            ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            ev0.record(stream)
            for r in range(reps):
                fn(r + 1)
            ev1.record(stream)
            torch.cuda.synchronize()
            return ev0.elapsed_time(ev1) / reps

        enc_ms = timed_calls(lambda r: c.encrypt(L_, plan, "x_fwd", e["d"]["x1"], 9000 + r, out=out_ct, ws=enc_ws))
        dec_ms = timed_calls(lambda r: c.decrypt(L_, plan, "fwd", e["out_f"][0], ws=dec_ws))
        # rooflines of the two ends: encryption transforms u, e0 + round(q m / t)
        # and e1 (3 L limb-transforms per ciphertext) and writes both components;
        # decryption transforms c1 forward and the phase back (2 L) and reads both
        # components.  Both are bound by the transforms' 32-bit multiplies.
        n_, lg_ = c.n, c.n.bit_length() - 1
        bfly_ = mul32_per_butterfly(c) * (n_ // 2) * lg_
        ct_bytes = 2 * c.L * n_ * 8

        def ends_roof(count, ms, transforms):
            mul = count * transforms * c.L * bfly_
            return {"bound": "alu", "mul32_Tps": round(mul / (ms / 1e3) / 1e12, 3),
                    "frac": round(mul / (ms / 1e3) / 1e12 / MUL32_PEAK_TOPS, 4),
                    "GBps": round(count * ct_bytes / (ms / 1e3) / 1e9, 1),
                    "hbm_frac": round(count * ct_bytes / (ms / 1e3) / 1e9 / HBM_PEAK_GBS, 4)}

        do_side = {"encrypt": {"ciphertexts": int(sz.n_ct[0]), "ms": round(enc_ms, 4),
                               "ciphertexts_per_s": round(sz.n_ct[0] / (enc_ms / 1e3), 1),
                               "roofline": ends_roof(int(sz.n_ct[0]), enc_ms, 3)},
                   "decrypt": {"ciphertexts": int(sz.n_out[0]), "ms": round(dec_ms, 4),
                               "ciphertexts_per_s": round(sz.n_out[0] / (dec_ms / 1e3), 1),
                               "roofline": ends_roof(int(sz.n_out[0]), dec_ms, 2)},
                   "layer": f"{L_.kind} {L_.c_in}->{L_.c_out} {L_.h}x{L_.w} b{L_.batch}"}

    # ------------------------------------------- bias gradient and DP noise
    # The weight-update terms that finish Alg. 2 (Sec. III.B.2) on every layer
    # of the workload: the bias-gradient share of dY and the DO's perturbation
    # of its dW and db shares.  Both are HBM-bound streams; the bias gradient
    # is checked against an int64 sum in torch.
    wupd = None
    if not args.no_do_side:
        reps = 10
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

        def time_reps(fn):
            fn(0)
            torch.cuda.synchronize()
            ev0.record(stream)
            for r in range(reps):
                fn(r + 1)
            ev1.record(stream)
            torch.cuda.synchronize()
            return ev0.elapsed_time(ev1) / reps

        bg_ms = dp_ms = 0.0
        bg_bytes = dp_bytes = 0
        bg_ok = True
        for e in layers:
            c, L_, d = e["ctx"], e["layer"], e["d"]
            dy = d["dy1"]
            db = c.bias_grad(L_, dy)
            dims = [i for i in range(dy.dim()) if i != 1]
            bg_ok = bg_ok and bool(torch.equal(db, dy.sum(dim=dims) % c.t))
            bg_ms += time_reps(lambda r: c.bias_grad(L_, dy))
            bg_bytes += 8 * (dy.numel() + db.numel())
            dwt = d["W"].clone()
            dp_ms += time_reps(lambda r: c.dp_noise_(dwt, 2.0 ** 24 * 0.05, 7000 + r, 0))
            dp_bytes += 16 * dwt.numel()
        wupd = {"bias_grad": {"ms": round(bg_ms, 4), "GBps": round(bg_bytes / (bg_ms / 1e3) / 1e9, 1),
                              "hbm_frac": round(bg_bytes / (bg_ms / 1e3) / 1e9 / HBM_PEAK_GBS, 4),
                              "algo_bytes": bg_bytes, "matches_torch_sum": bg_ok},
                "dp_noise_dW": {"ms": round(dp_ms, 4), "GBps": round(dp_bytes / (dp_ms / 1e3) / 1e9, 1),
                                "hbm_frac": round(dp_bytes / (dp_ms / 1e3) / 1e9 / HBM_PEAK_GBS, 4),
                                "algo_bytes": dp_bytes,
                                "normals_per_s": round(dp_bytes / 16 / (dp_ms / 1e3), 1)},
                "layers": len(layers)}

    # ------------------------------------------------------ Pencil+
    plus = None
    m_plus = args.pencil_plus if args.pencil_plus >= 0 else (8 if args.config == 2 and not args.workload else 0)
    if m_plus > 0:
        plus = pencil_plus_bench(layers[0], m_plus, compare["step"] if "step" in compare else ms_step, torch)

    # the integer peak's evidence: issue rates of the multiply forms on this GPU
    probe = {}
    for kind, name in enumerate(("v_mad_u64_u32", "v_mul_lo_u32", "v_mul_hi_u32")):
        r = ctypes.c_double()
        A.check(A.load().pencil_probe_mul32(kind, ctypes.byref(r)))
        probe[name] = round(r.value / 1e12, 3)

    cpu = None
    if not args.no_cpu_baseline:
        cpu = cpu_baseline(layers[0]["layer"], args.cpu_seconds)

    first = layers[0]
    rec = {
        "metric": "encrypted linear-layer fwd+bwd products/sec at bit-exact; NTT GB/s vs HBM roofline",
        "value": round(value, 1),
        "unit": "products/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "steps_per_s": round(1e3 / ms_step, 1),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u64",
        "data": "synthetic",
        "config": {"workload": cfg.name, "N": first["ctx"].n, "L": first["ctx"].L,
                   "layers": [f"{S.kind} {S.c_in}->{S.c_out} {S.h}x{S.w} k{S.k} s{S.stride} b{S.batch}"
                              + (" (as its stride-1 equivalent)" if e["strided"] else "")
                              for e in layers for S in [e["strided"][0] if e["strided"] else e["layer"]]],
                   "ops": list(cfg.ops), "products_per_step": int(products),
                   "plans": [{"fwd": e["plan"].fwd.astuple(), "dx": e["plan"].dx.astuple(),
                              "dw": e["plan"].dw.astuple(), "sched": list(e["plan"].sched)} for e in layers],
                   "autotuned": not args.no_autotune,
                   "autotune_cache": os.path.relpath(args.tune_cache, ROOT) if args.tune_cache else None,
                   "ntt_loge": {f"N={c.n},L={c.L}": c.ntt_loge() for c in ctxs.values()},
                   "launch": {"step": "batched phase launches (all layers and products)",
                              "graph": "the batched step replayed as one HIP graph",
                              "layer": "one launch sequence per product and layer"}[args.mode]},
        "bit_exact": bit_exact,
        "wall_s_timed": round(wall, 3),
        "launch_paths_ms_per_step": compare,
        "batched_speedup_vs_unbatched": round(compare["layer"] / min(compare["step"], compare["graph"]), 3),
        "roofline": roof,
        "mul32_probe_T_per_s": probe,
        "kernels": breakdown,
        "cpu_baseline": cpu,
        "ntt": ntt_rec,
        "data_owner_ends": do_side,
        "weight_update_terms": wupd,
        "stride_relayout_ms": round(relayout_ms, 4) if any(e["strided"] for e in layers) else None,
        "pencil_plus": plus,
    }
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()
