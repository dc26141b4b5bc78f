#!/usr/bin/env python3
"""Throughput of the K-replica LSAM hot path on one MI355X.

One "step" is one pass of the whole path over one batch of synthetic input: `lsam_step`
(forward/backward, gradient norm, ascent perturbation, second forward/backward, descent +
coupling for all K replicas) followed by `lsam_sync` (schedule test and, when replicas are
due, the center update).  Inputs are resident in HBM before the timed region starts.

Prints ONE JSON line: replica-samples/s plus a `roofline` object for the dominant kernel
class (HIP-event durations measured inside the library on its own stream over a second run
of the same steps) and a `cpu_baseline` object (the CPU oracle timed on a bounded sample).
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

import workloads  # noqa: E402

PEAK_HBM_GBS = 8000.0
PEAK_TFLOPS = {0: 157.3, 1: 2500.0}   # dense MFMA: fp32, bf16
SPLIT_PRODUCTS = 6                    # bf16 products an fp32 product of exact pieces is formed from (plane tensors)


# HBM bytes per launch of each kernel class, from two `rocprofv3 --pmc` runs of this script
# (FETCH_SIZE, then WRITE_SIZE; KiB per dispatch scaled by what the same counter reads for a plain
# 1 GiB device copy: x2.0 and x1.0), summed over the dispatches of a class and divided by its
# launches (a split-K GEMM and its reduce count as one launch; kernels that serve several classes
# are told apart by empty marker kernels launched between the classes in a copy of the library).
# The figures belong to the kernel sources that serve the workload (traffic_family), as long as their digest is the one
# in TRAFFIC_SOURCES; with any other sources `traffic` is null.
TRAFFIC_SOURCES = {"raw": "7ecdbed4756e4dd1", "dense_bf16": "5226c8879f5d946e", "all": "532e42178a1df6bb"}
TRAFFIC = {
    "cfg2": {"center": 84162976, "descent": 538478884, "gemm_dw": 96747181, "gemm_dx": 42137399,
             "gemm_fwd": 91313573, "perturb": 201939879},
    "cfg3": {"bias_grad": 69965355, "center": 1393527072, "gemm_dw_ascend": 732938428,
             "gemm_dw_norm": 74834581, "gemm_dw_step": 2904271437, "gemm_dx": 250151232,
             "gemm_fwd": 233113689, "softmax_ce": 1428949},
    "cfg4": {"center": 2400048928, "descent": 32005545216, "sumsq_partials": 3417931339},
    "cfg5": {"bias_grad": 836635733, "gemm_dw_ascend": 6220483834, "gemm_dw_norm": 1683837749,
             "gemm_dw_step": 27280532194, "gemm_dx": 2584784242, "gemm_fwd": 2034203236,
             "softmax_ce": 96475915},
    "cnn5": {"bias_grad": 7143764, "conv_first": 80178413, "descent": 79475846,
             "gemm_dw": 51929342, "gemm_dx": 107749902, "gemm_fwd": 42564241, "perturb": 29814018,
             "pool": 56534275},
    "cnn5bn": {"batchnorm": 86030533, "conv_first": 80335276, "descent": 79541381,
             "gemm_dw": 51969009, "gemm_dx": 113816528, "gemm_fwd": 42744123, "perturb": 29838593},
    "resnet18": {"batchnorm": 201102826, "conv_first": 221362047, "descent": 1430937488,
             "gemm_dw": 252846617, "gemm_dx": 366479652, "gemm_fwd": 293660952,
             "perturb": 536610566, "pool": 26264216},
    "resnet18bf": {"batchnorm": 149142329, "conv_first": 223411678, "descent": 1430936934,
             "gemm_dw": 102601357, "gemm_dx": 187866395, "gemm_fwd": 110345231,
             "perturb": 536610225, "pool": 26264207, "softmax_ce": 124241},
    "resnet20": {"batchnorm": 72500733, "conv_first": 60550145, "descent": 34871469,
             "gemm_dw": 72397848, "gemm_dx": 93903104, "gemm_fwd": 65008708, "perturb": 13087403,
             "pool": 9487317},
    "resnet34": {"batchnorm": 194503825, "conv_first": 221389946, "descent": 2731132935,
             "gemm_dw": 245768897, "gemm_dx": 335356277, "gemm_fwd": 261628590,
             "perturb": 1024183307, "pool": 26264217, "softmax_ce": 485024},
    "vgg16": {"batchnorm": 101264297, "conv_first": 221832774, "descent": 1952501434,
             "gemm_dw": 174100766, "gemm_dx": 198164842, "gemm_fwd": 160359164,
             "perturb": 732196776},
    "vgg16bf": {"batchnorm": 76753255, "conv_first": 223642959, "descent": 1952501374,
             "gemm_dw": 77534825, "gemm_dx": 101127042, "gemm_fwd": 76220015, "perturb": 732196675,
             "softmax_ce": 123900},
    "wrn16x10": {"batchnorm": 595628892, "conv_first": 60565709, "descent": 2191727505,
             "gemm_dw": 1164417129, "gemm_dx": 1485016044, "gemm_fwd": 1660644325,
             "perturb": 821906336},
    "wrn16x10bf": {"batchnorm": 416333942, "conv_first": 60510081, "descent": 2191726234,
             "gemm_dw": 330248064, "gemm_dx": 582511328, "gemm_fwd": 447066536,
             "perturb": 821906007, "softmax_ce": 123900},
    "wrn28x10": {"batchnorm": 643008090, "conv_first": 60615942, "descent": 4678080460,
             "gemm_dw": 1349570907, "gemm_dx": 1599117019, "gemm_fwd": 1818108096,
             "perturb": 1754287219, "softmax_ce": 484683},
    "wrn40x10": {"batchnorm": 659650300, "conv_first": 60544820, "descent": 7157051358,
             "gemm_dw": 1430426883, "gemm_dx": 1643661000, "gemm_fwd": 1911413329,
             "perturb": 2683899873, "softmax_ce": 484683},
}


def traffic_family(w):
    """Which sources hold the kernels a workload launches."""
    return "raw" if not w.dims else "dense_bf16" if w.gemm_dtype == 1 and not w.n_conv else "all"


def kernel_sources_digest(family):
    import glob
    import hashlib
    h = hashlib.sha256()
    # the files that hold device code (the host engine, lsam_api.hip and engine.h, launches
    # these kernels but does not change what one launch of them moves)
    csrc = os.path.join(ROOT, "paper_2509_03110_amd", "csrc")
    files = {"raw": ["kernels_stream.hip", "langevin.h"],
             "dense_bf16": ["kernels_ce.hip", "kernels_gemm_bf16.hip", "kernels_stream.hip", "b32s.h", "dense_gradients.h",
                            "langevin.h"],
             "all": sorted(os.path.basename(f) for f in glob.glob(os.path.join(csrc, "kernels_*.hip"))) +
                    ["b32s.h", "dense_gradients.h", "langevin.h", "planes.h"]}[family]
    for f in files:
        with open(os.path.join(csrc, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def layer_table(eng, w):
    """What the library reports about each layer (`lsam_layer_info`): which kernels serve it, the
    rows of its matrix products, whether its gradients are stored."""
    return [eng.lsam_layer_info(l) for l in range(len(w.dims) - 1)]


def plane_table(eng, w):
    """bfloat16 values per number in the operands of each layer's products (0: stored fp32 numbers)."""
    return [eng.lsam_layer_planes(l) for l in range(len(w.dims) - 1)]


def matrix_units(w, layers, planes):
    """Per product class: the share of its flops that each kind of product forms ("fp32", "bf16", or
    "split": fp32 from exact bf16 pieces)."""
    from paper_2509_03110_amd import lsam

    def shares(lo):
        out = {}
        for (kind, _, _, rows, fi, fo, pc, _), np_ in list(zip(layers, planes))[lo:]:
            if kind in (lsam.LAYER_HEAD, lsam.LAYER_CONV_FIRST):
                continue
            unit = "split" if np_ == 3 else "bf16" if np_ == 1 or w.gemm_dtype == 1 else "fp32"
            out[unit] = out.get(unit, 0.0) + float(rows) * (fi + pc) * fo
        total = sum(out.values())
        return {k: v / total for k, v in out.items()}
    return {name: s for name, s in (("gemm_fwd", shares(0)), ("gemm_dx", shares(1)), ("gemm_dw", shares(0))) if s}


def mixed_rate(shares, fp32, bf16):
    """The rate of a class whose flops are shared out like that among units of these rates."""
    rate = {"fp32": fp32, "bf16": bf16, "split": bf16 / SPLIT_PRODUCTS}
    return 1.0 / sum(v / rate[k] for k, v in shares.items())


def gemm_flops(w, layers):
    """Per all-replica step (both passes): flops of the forward, dX and dW GEMM classes and of
    the first convolution layer's own kernels.  On the fused path (bf16 dense model) the
    weight-gradient product is formed for the perturbed operand copy and, at the perturbed
    point, for the sampler step; the norm of the first-pass gradient comes from the Gram
    matrices of the product's factors, 2 B^2 (out + in) flops, or from a product whose result
    is only summed."""
    from paper_2509_03110_amd import lsam
    K = w.K
    per = [float(rows) * fi * fo if kind not in (lsam.LAYER_HEAD, lsam.LAYER_CONV_FIRST) else 0.0
           for kind, _, _, rows, fi, fo, _, _ in layers]
    first = sum(float(rows) * fi * fo for kind, _, _, rows, fi, fo, _, _ in layers if kind == lsam.LAYER_CONV_FIRST)
    proj = sum(float(rows) * pc * fo for _, _, _, rows, _, fo, pc, _ in layers)    # 1x1 projections
    sw, sw_dx = sum(per) + proj, sum(per[1:]) + proj
    out = {"gemm_fwd": 2 * 2.0 * sw * K, "gemm_dx": 2 * 2.0 * sw_dx * K}
    if first:
        out["conv_first"] = 2 * 2 * 2.0 * first * K      # forward and weight gradient
    if any(r[2] for r in layers):
        out["gemm_dw_ascend"] = out["gemm_dw_step"] = 2.0 * sw * K
        out["gemm_dw_norm"] = K * sum(1.0 * rows * rows * (fi + fo) if route == 2 else 2.0 * rows * fi * fo
                                      for _, _, route, rows, fi, fo, _, _ in layers)
    else:
        out["gemm_dw"] = 2 * 2.0 * sw * K
    return out


def conv_routes(w, layers, planes):
    """What the library keeps of each convolution's output and where a normalisation's sums are taken, as its layout
    decides it."""
    from paper_2509_03110_amd import lsam
    n = w.n_conv
    bit = lambda mask, l: l < n and bool((mask >> l) & 1)
    proj = lambda l: l < n and bool(layers[l][6])
    opens = lambda l: bit(w.skip_mask, l + 1) and (proj(l + 1) or not w.preact)
    direct_dx = lambda l: 0 < l < n and not layers[l][1]
    # the shortcut's gradient joins the product that writes the block input's
    joins = lambda l: (l > 0 and opens(l) and planes[l] and direct_dx(l) and not bit(w.pool_mask, l - 1) and
                       not bit(w.stride_mask, l + 1))
    reads_planes = lambda l: planes[l] > 0 and layers[l][0] == lsam.LAYER_CONV_DIRECT
    out = []
    for l in range(n):
        bn, pool, last = bit(w.bn_mask, l), bit(w.pool_mask, l), l + 1 == n
        post_sum = bit(w.skip_mask, l) and not w.preact
        # what writes this layer's gradient is a plane product that completes it
        complete = not last and planes[l + 1] and direct_dx(l + 1) and (not opens(l + 1) or joins(l + 1))
        r = dict(bn=bn, pool=pool, post_sum=post_sum, bn_pool=bn and pool and not post_sum,
                 bn_gap=bn and not pool and last and bool(w.global_avg_pool) and joined_average(w, layers[l][3], w.dims[l + 1], post_sum))
        r["bits"] = pool or (bn and bool(complete if not last else w.global_avg_pool))
        r["pooled_floats"] = pool and (last or not reads_planes(l + 1))
        closing = l + 2 if bit(w.skip_mask, l + 2) else None
        if pool or last:
            r["floats"] = not r["bn_pool"] and not r["bn_gap"]
        else:
            r["floats"] = (not r["bits"] or not reads_planes(l + 1) or
                           (closing is not None and (not planes[closing] if proj(closing) else not w.preact)))
        # (a product cut over workgroups leaves no sums: its bytes then count less than it moves)
        r["sums_forward"] = layers[l][0] == lsam.LAYER_CONV_FIRST or planes[l] > 0
        r["sums_backward"] = bool(complete and bn and (not pool or r["bn_pool"]))
        r["joins"] = bool(joins(l))
        # the gradient of a last image's average is formed where it is used
        r["from_average"] = r["bn_gap"] and not (post_sum and not proj(l))
        out.append(r)
    return out


def joined_average(w, rows, channels, shortcut):
    hw = rows // w.batch
    if hw <= (16 if shortcut else 64):
        return True
    work = w.K * w.batch * channels
    return (hw <= 256 and work >= 20480) if shortcut else work >= 6144


def conv_bytes(w, layers, planes):
    """Algorithmic bytes per all-replica step (both passes) of the kernels around the
    convolution products: what they read and write once each, as the library's layout has it (conv_routes).
    Where an unfolded image is stored it is written once (plus the image
    read), where its gradient is stored that is read once (plus the image gradient written).
    Where plane tensors serve a layer (`planes` values of 2 bytes
    per number) its image's and its output gradient's planes are written by the kernels that form
    them, or from the stored floats by one of their own.  Outputs are written as floats only where
    something reads them, their signs as a bit a value."""
    from paper_2509_03110_amd import lsam
    unfold = pool = bn = 0.0
    routes = conv_routes(w, layers, planes)
    for l in range(w.n_conv):
        kind, dx_stored, _, rows, _, _, proj_c, proj_step = layers[l]
        np_, r = planes[l], routes[l]
        skip, proj = (w.skip_mask >> l) & 1, bool(proj_c)
        cin, cout = w.dims[l], w.dims[l + 1]
        v = rows * cout                               # values of the output
        last, first = l + 1 == w.n_conv, kind == lsam.LAYER_CONV_FIRST
        st2 = 4 if (w.stride_mask >> l) & 1 else 1    # pixels of the image read per output pixel
        if kind == lsam.LAYER_CONV_STORED:
            unfold += rows * (st2 * cin * 4.0 + 9 * cin * (2.0 * np_ if np_ else 4.0))
        # planes of the image it reads, also for the projection of the block it opens
        image = np_ if kind == lsam.LAYER_CONV_DIRECT else 0
        if l + 1 < w.n_conv and layers[l + 1][6]:
            image = max(image, planes[l + 1])
        if image and l > 0 and (routes[l - 1]["pool"] and not routes[l - 1]["bn_pool"]):
            pool += rows * st2 * cin * 2.0 * image
        elif image and l > 0 and routes[l - 1]["bn"]:
            bn += rows * st2 * cin * 2.0 * image
        elif image:
            unfold += rows * st2 * cin * (4.0 + 2.0 * image)
        if np_ and not r["bn"] and not r["pool"]:
            unfold += v * (4.0 + 2.0 * np_)
        if dx_stored:
            unfold += rows * (9 * cin + st2 * cin) * 4.0
        # what is written of the output gradient behind its normalisation, bytes a value
        dz = 2.0 * np_ + (4.0 if w.preact and skip and not proj else 0.0) if np_ else 4.0
        bits = 0.25
        if r["bn"]:
            # statistics read Z unless the product has left them; the normalisation reads Z again
            bn += v * 4.0 * ((0 if r["sums_forward"] else 1) + 1)
            if r["bn_pool"]:
                bn += v / 4 * (4.0 + 2 * bits + (4.0 if r["pooled_floats"] else 0.0))
            else:
                bn += v * ((4.0 if r["floats"] else 0.0) + (bits if r["bits"] and not r["pool"] else 0.0))
            # backward: sums of dY and Z unless the product has left them, then dZ from both (which a first
            # layer's weight gradient forms itself)
            if not r["sums_backward"]:
                bn += v / 4 * (8.0 + bits) if r["bn_pool"] else v * (4.0 + bits) if r["from_average"] else v * 8.0
            handed = w.preact and l + 2 < w.n_conv and (w.skip_mask >> (l + 2)) & 1 and not layers[l + 2][6]
            if r["bn_pool"]:
                bn += v * (4.0 + dz) + v / 4 * (4.0 + 2 * bits)
            elif r["from_average"]:
                bn += v * (4.0 + bits + dz)
            elif not first or handed:
                bn += v * (8.0 + dz + (4.0 if handed and np_ else 0.0))
        if r["pool"] and not r["bn_pool"]:
            # forward reads the image; what the backward pass writes goes to a normalisation or, without one, to the products
            pool += v * 4.0 + v / 4 * (2 * bits + (4.0 if r["pooled_floats"] else 0.0))
            pool += v / 4 * (4.0 + 2 * bits) + v * (2.0 * np_ if np_ and not r["bn"] else 4.0)
        if last and w.global_avg_pool:
            if not r["bn_gap"]:
                pool += (v / 4 if r["pool"] else v) * 4.0
            if not r["from_average"]:
                pool += v / 4 * 4.0 if r["pool"] else v * (4.0 + (bits if r["bits"] else 4.0))
        if proj:
            # projection: its normalisation is the layer's own once more, from stored sums backward, and its
            # output is read where the two branches meet; the pixels a strided one
            # keeps are read in place on plane tensors, gathered (read and written) otherwise;
            # backward, the gradient of those pixels joins the product that writes the block input's gradient, or
            # is added to it under that input's mask (3 reads, 1 write).  A pre-activation block's bare
            # projection joins the convolution's product, or is added to its output (two reads and a write)
            if not w.preact:
                dy = 4.0 if not r["from_average"] else bits
                bn += v * ((0.0 if np_ else 4.0) + 4.0 + 2 * (4.0 + dy) + (2.0 * np_ if np_ else 4.0))
            elif not np_:
                pool += v * 4.0 * 3
            if proj_step == 2 and not np_:
                unfold += rows * proj_c * 4.0 * 2
            if not routes[l - 1]["joins"]:
                pool += rows * proj_c * 4.0 * 4
        elif skip and w.preact:
            # identity shortcut of a pre-activation block: the sum two convolutions below joins this one's
            # product, or is added to it; backward, where no plane tensor is formed, likewise
            if not np_:
                pool += v * 4.0 * 3
            if not planes[l - 2]:
                pool += v * 4.0 * 3
        elif skip:
            # shortcut: read with the normalisation (forward); backward joins the product that writes the block
            # input's gradient, or reads dY, the mask and that gradient and writes the latter
            bn += rows * min(cout, w.dims[l - 1]) * 4.0
            if not routes[l - 1]["joins"]:
                pool += rows * min(cout, w.dims[l - 1]) * 4.0 * 4
    out = {}
    if bn:
        out["batchnorm"] = 2 * bn * w.K
    if unfold:
        out["unfold_fold"] = 2 * unfold * w.K
    if pool:
        out["pool"] = 2 * pool * w.K
    return out


def stream_bytes(w, fused_step=False, restarts=0.0):
    """Algorithmic bytes per all-replica step of the update-path kernels (reads + writes
    the method itself requires; y is shared by the K replicas): descent reads x, g2, v, S
    (16 B per parameter) and writes x, v, S (12 B), plus the bf16 operand copy (2 B) in bf16
    mode, plus y once for all replicas.  `restarts`: replicas per step, on average, whose sum
    of iterates starts again from zero (served by the center update one tick before): their S
    is written but not read."""
    n = float(w.K) * w.d
    bf = w.gemm_dtype == 1 and not w.n_conv
    out = {"sumsq_partials": 4 * n,
           "perturb": (10 if bf else 12) * n,
           "descent": (30 if bf else 28) * n + 4.0 * w.d - 4.0 * restarts * w.d}
    if not w.dims and w.rho and w.algorithm == 0:
        # both gradients are at hand: the descent's pass reads g1 and writes the perturbed point too
        out["descent"] += 8 * n
        del out["perturb"]
    if fused_step:
        # the weight matrices take their step where the second-pass gradient is produced: that
        # kernel reads x, v, S (12 B per parameter) and y once, writes x, v, S (12 B) and the
        # bf16 operand copy (2 B), and neither writes nor reads g2; the separate kernel is left
        # with the bias vectors
        nw = sum(a * b for a, b in w.layer_shapes)
        nb = w.d - nw
        out["gemm_dw_step"] = 26.0 * w.K * nw + 4.0 * nw - 4.0 * restarts * nw
        out["descent"] = 28.0 * w.K * nb + 4.0 * nb - 4.0 * restarts * nb
        # the ascent GEMMs read x and write the bf16 copy of x~; no perturbation kernel runs
        out["gemm_dw_ascend"] = 6.0 * w.K * nw
        del out["perturb"]
    return out


def make_inputs(w, torch, dev, n_sets):
    sets = []
    if w.dims:
        for s in range(n_sets):
            X, lab = workloads.batch(w, s)
            Xd = torch.from_numpy(X).to(dev)
            if w.gemm_dtype == 1 and not w.n_conv:
                Xd = Xd.to(torch.bfloat16)
            sets.append((Xd.contiguous(), torch.from_numpy(lab).to(dev)))
    else:
        # raw-vector mode: fixed gradient buffers ~ N(0, grad_std^2), generated on the device
        gen = torch.Generator(device=dev)
        gen.manual_seed(w.data_seed)
        g1 = torch.randn(w.K, w.d_raw, device=dev, generator=gen) * w.grad_std
        g2 = torch.randn(w.K, w.d_raw, device=dev, generator=gen) * w.grad_std
        sets.append((g1, g2))
    return sets


def cpu_baseline(w, budget_s=20.0):
    """Times the oracle, single-threaded, on a bounded sample of the workload."""
    from threadpoolctl import threadpool_limits
    sys.path.insert(0, os.path.join(ROOT, "tests"))
    from util import oracle_from
    with threadpool_limits(limits=1):
        if w.dims:
            # one replica; shrink the batch for the two largest workloads
            frac = {"cfg5": 8, "cfg3": 2, "vgg16": 16, "vgg16bf": 16, "resnet20": 4}.get(w.name, 1)
            ws = w.scaled(K=1, batch=max(w.batch // frac, 1), tau=(10 ** 6,))
            o = oracle_from(ws, workloads.init_params(ws))
            X, lab = workloads.batch(ws, 0)
            n, t0 = 0, time.perf_counter()
            while True:
                o.step(X, lab)
                n += 1
                if time.perf_counter() - t0 > budget_s / 2 or n >= 20:
                    break
            dt = time.perf_counter() - t0
            value = n * ws.batch / dt
            sample = ("%d step(s) of 1 replica at batch %d (of K=%d, B=%d); samples/s of that bounded "
                      "sample, taken as the rate of the whole workload (work per sample is the same: "
                      "extrapolated)" % (n, ws.batch, w.K, w.batch))
            unit = "replica-samples/s"
        else:
            d = min(w.d_raw, 10_000_000)
            ws = w.scaled(K=1, d_raw=d, tau=(4,))
            o = oracle_from(ws, workloads.init_params(ws))
            g1, g2 = workloads.raw_grads(ws, 0)
            n, t0 = 0, time.perf_counter()
            while True:
                o.step_grads(g1, g2)
                o.sync()
                n += 1
                if time.perf_counter() - t0 > budget_s / 2 or n >= 20:
                    break
            dt = time.perf_counter() - t0
            value = n * d / dt
            sample = ("%d iteration(s) of 1 replica at d=%d (of K=%d, d=%d); extrapolated as above"
                      % (n, d, w.K, w.d_raw))
            unit = "replica-params/s"
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"value": value, "unit": unit, "cores": 1, "kind": "oracle", "sample": sample,
            "host_cpu": model, "host_cores": os.cpu_count()}


def default_steps(w):
    return {"cfg1": 200, "cfg2": 200, "cnn5": 100, "cnn5bn": 100}.get(w.name, 20)


def run_workload(w, steps, warmup, kernel_timing=True):
    """Times `steps` steps of workload `w` after `warmup` untimed ones; returns the fields of
    the JSON line that belong to this workload."""
    import torch
    from paper_2509_03110_amd import lsam
    dev = torch.device("cuda:0")
    cfg, keep = lsam.config_from_workload(w)
    eng = lsam.Lsam(cfg, workloads.init_params(w), device=dev, keep=keep)
    sets = make_inputs(w, torch, dev, w.batch_pool or 8)
    loss = torch.zeros(w.K, device=dev)

    def one(i):
        a, b = sets[i % len(sets)]
        if w.dims:
            eng.lsam_step(a, b, loss)
        else:
            eng.lsam_step_grads(a, b)
        eng.lsam_sync()

    for i in range(warmup):
        one(i)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(steps):
        one(i)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    ms = dt / steps * 1e3

    if w.dims:
        value, unit, metric = w.K * w.batch / (dt / steps), "replica-samples/s", \
            "replica-samples/sec per LSAM step"
    else:
        value, unit, metric = w.K * w.d_raw / (dt / steps), "replica-params/s", \
            "replica-params/sec per LSAM update iteration"

    roof, kernels = None, {}
    if kernel_timing:
        eng.lsam_timing_enable(True)
        for i in range(steps):
            one(i)
        stats = eng.lsam_timing_read()
        eng.lsam_timing_enable(False)
        layers, planes = (layer_table(eng, w), plane_table(eng, w)) if w.dims else ([], [])
        units = matrix_units(w, layers, planes) if w.dims else {}
        fused_step = any(r[2] for r in layers)
        flops = gemm_flops(w, layers) if w.dims else {}
        # center update: 4 B/param per due replica (S read; starting it again from zero costs
        # no write, the next step simply does not read it) + 16 B/param (y and g'_prev read and
        # written), summed over the ticks of this run that had a sync
        first = warmup + steps
        due, _ = lsam.lsam_schedule_replay(cfg, first + steps)
        nd = due[first:].sum(axis=1)
        restarts = float(due[first - 1:-1].sum()) / steps     # served one tick earlier
        nbytes = stream_bytes(w, fused_step, restarts)
        nbytes.update(conv_bytes(w, layers, planes))
        nbytes["center"] = float(np.sum((4.0 * nd + 16.0) * (nd > 0))) * w.d / steps
        family = traffic_family(w)
        traffic = TRAFFIC.get(w.name, {}) if kernel_sources_digest(family) == TRAFFIC_SOURCES[family] else {}
        for name, (cnt, tot) in stats.items():
            if cnt == 0:
                continue
            k = {"launches_per_step": cnt / steps, "ms_per_step": tot / steps,
                 "avg_launch_ms": tot / cnt}
            if name in ("gemm_dw_step", "gemm_dw_ascend") and name in nbytes and tot > 0:
                # a contraction whose epilogue streams the sampler state: priced against the
                # roof that binds it (HBM), with its matrix-unit rate beside it
                k.update(bound="hbm", achieved=nbytes[name] * steps / (tot * 1e-3) / 1e9,
                         peak=PEAK_HBM_GBS, unit="GB/s",
                         algorithmic_bytes_per_launch=nbytes[name] * steps / cnt,
                         mfma_tflops=flops[name] * steps / (tot * 1e-3) / 1e12)
            elif name in flops and tot > 0:
                k.update(bound="mfma", achieved=flops[name] * steps / (tot * 1e-3) / 1e12,
                         peak=mixed_rate(units[name], PEAK_TFLOPS[0], PEAK_TFLOPS[1]) if name in units
                         else PEAK_TFLOPS[w.gemm_dtype], unit="TFLOP/s",
                         algorithmic_flops_per_launch=flops[name] * steps / cnt)
            elif name in nbytes and tot > 0:
                k.update(bound="hbm", achieved=nbytes[name] * steps / (tot * 1e-3) / 1e9,
                         peak=PEAK_HBM_GBS, unit="GB/s",
                         algorithmic_bytes_per_launch=nbytes[name] * steps / cnt)
            if "achieved" in k:
                k["frac"] = k["achieved"] / k["peak"]
            if name in units and k.get("bound") == "mfma" and "split" in units[name]:
                k["units"] = units[name]
            k["traffic"] = traffic.get(name)
            kernels[name] = k
        ranked = [n for n in sorted(kernels, key=lambda n: -kernels[n]["ms_per_step"])
                  if "achieved" in kernels[n]]
        if ranked:
            top = kernels[ranked[0]]
            roof = {"kernel": ranked[0], "bound": top["bound"], "achieved": top["achieved"],
                    "peak": top["peak"], "unit": top["unit"], "frac": top["frac"],
                    "traffic": top["traffic"], "avg_launch_ms": top["avg_launch_ms"]}
            if "units" in top:
                roof["units"] = top["units"]

    out = {
        "metric": metric, "value": value, "unit": unit, "n_gpus": 1, "steps": steps,
        "warmup": warmup, "ms_per_step": ms, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32" if (w.gemm_dtype == 0) else "bf16 operands, f32 accumulate and master weights",
        "data": "synthetic",
        "config": {"workload": w.name, "K": w.K, "dims": list(w.dims), "n_conv": w.n_conv,
                   "image": [w.img_h, w.img_w], "pool_mask": w.pool_mask, "bn_mask": w.bn_mask,
                   "d": w.d, "batch": w.batch,
                   "rho": w.rho, "lr": w.lr, "momentum": w.momentum, "algorithm": w.algorithm,
                   "noise_scale": w.noise_scale,
                   "periods": eng.lsam_get_schedule()[0]},
        "roofline": roof, "kernels": kernels,
    }
    eng.close()
    del eng, sets
    torch.cuda.empty_cache()
    return out


def add_measured_fractions(out, w, peaks):
    """The same fractions against what the simplest kernels reach on this very device."""
    copy_gbs, bf16_tf, f32_tf = peaks
    mfma_meas = bf16_tf if w.gemm_dtype == 1 else f32_tf
    for k in list(out["kernels"].values()) + ([out["roofline"]] if out["roofline"] else []):
        if k.get("bound") == "mfma":
            k["frac_of_measured"] = k["achieved"] / (mixed_rate(k["units"], f32_tf, bf16_tf) if "units" in k else mfma_meas)
        elif k.get("bound") == "hbm":
            k["frac_of_measured"] = k["achieved"] / copy_gbs


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=None)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="cfg5", choices=sorted(workloads.WORKLOADS),
                    help="the timed workload (default: the largest configuration that fits one GPU)")
    ap.add_argument("--also", default=None,
                    help="comma-separated workloads reported in short form under `other_workloads` "
                         "(default: cfg2,cfg3,cfg4 when the workload is cfg5; 'none' for none)")
    ap.add_argument("--algorithm", type=int, default=0, choices=[0, 1],
                    help="0 = LSAM (default), 1 = synchronous data-parallel baseline")
    ap.add_argument("--noise-scale", type=float, default=0.0,
                    help="sigma of the Langevin sampler (0 = noise-free, the default)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-kernel-timing", action="store_true")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU: the path holds all K replicas on a single MI355X and "
              "uses no collectives, so --gpus %d is not supported." % args.gpus, file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2509_03110_amd import lsam
    if not torch.cuda.is_available():
        print("no GPU visible", file=sys.stderr)
        sys.exit(1)
    dev = torch.device("cuda:0")
    w = workloads.WORKLOADS[args.workload]
    if args.algorithm or args.noise_scale:
        w = w.scaled(algorithm=args.algorithm, noise_scale=args.noise_scale, noise_seed=1)
    steps = args.steps if args.steps is not None else default_steps(w)
    timing = not args.no_kernel_timing

    out = run_workload(w, steps, args.warmup, timing)
    also = args.also if args.also is not None else ("cfg2,cfg3,cfg4" if w.name == "cfg5" else "none")
    others = {}
    for name in [n for n in also.split(",") if n and n != "none" and n != w.name]:
        wo = workloads.WORKLOADS[name]
        others[name] = (wo, run_workload(wo, min(default_steps(wo), 50), args.warmup, timing))
    if timing:
        scratch = torch.empty(1 << 28, dtype=torch.float32, device=dev)          # 1 GiB
        peaks = lsam.lsam_probe_peaks(scratch)
        del scratch
        out["measured_peaks"] = {"copy_GBps": peaks[0], "mfma_bf16_TFLOPs": peaks[1],
                                 "mfma_f32_TFLOPs": peaks[2]}
        add_measured_fractions(out, w, peaks)
        for wo, r in others.values():
            add_measured_fractions(r, wo, peaks)
    if others:
        keep = ("bound", "achieved", "peak", "unit", "frac", "frac_of_measured", "ms_per_step",
                "avg_launch_ms", "launches_per_step")
        out["other_workloads"] = {
            name: {"value": r["value"], "unit": r["unit"], "ms_per_step": r["ms_per_step"],
                   "steps": r["steps"], "dtype": r["dtype"],
                   "kernels": {k: {f: v[f] for f in keep if f in v} for k, v in r["kernels"].items()
                               if "achieved" in v}}
            for name, (wo, r) in others.items()}
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(w)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
