"""The work that users of this framework have it do, as cases that can be timed.

A case is a dict of plain values.  `listed()` gives the fixed ones, `draw(rng)` one more from the
same ranges, `prepare(case, seed)` what a program holds before the call (inputs made from the seed,
the layer handle or the network), `run(state)` one pass through the public entry points, `work(case)`
the bytes and operations the pass cannot do without and `tolerance(case)` how far another correct
implementation at the same precision may be off.

Two kinds of case: one gated layer (`GatedConv.forward`: 3x3, 1x1 or fully connected) and a whole
channel-gated ResNet-18 forward pass (`GatedResNet18.forward`).  Activations are ReLU outputs times a
smooth per-image magnitude field, weights are normal with the usual variance; gate thresholds are set so
that a given fraction of the activations fires, and each threshold is put into the widest gap between
neighbouring sums close to that quantile, so that a decision does not hang on the order of a sum.
"""
import functools
import math

import numpy as np
import torch

from paper_1805_12549_amd import binding as B
from paper_1805_12549_amd import resnet18

_DTYPES = {"f32": (B.CG_F32, torch.float32, 4), "bf16": (B.CG_BF16, torch.bfloat16, 2),
           "int8": (B.CG_I8, torch.int8, 1), "int32": (B.CG_I32, torch.int32, 4)}


def _layer(name, n, h, w, cin, cout, **kw):
    case = dict(kind="layer", name=name, n=n, h=h, w=w, cin=cin, cout=cout, k=3, stride=1, g=4, dtype="bf16",
                out="bf16", maps="coherent", rho=0.3, affine=False, residual=False, grouped=False, shuffle=False,
                tau=0.0, two_sided=False, counts=False, alloc=False)
    case.update(kw)
    return case


def _network(name, n, size, g, rho):
    return dict(kind="network", name=name, n=n, size=size, g=g, rho=rho)


def listed():
    return [
        # the smallest layer of the repository's configurations, called the way a first user calls it:
        # fp32, every output asked for and allocated by the call
        _layer("fp32 16@32 n1", 1, 32, 32, 16, 16, dtype="f32", out="f32", maps="iid", counts=True, alloc=True),
        # one image through a deep int8 layer: latency
        _layer("int8 256@14 n1", 1, 14, 14, 256, 256, dtype="int8", out="int8", affine=True),
        # one image through the whole network: latency, and the host work of some twenty calls
        _network("network 224 n1", 1, 224, 4, 0.3),
        # a CIFAR-shaped layer at training-size batch, unstructured inputs
        _layer("256@8 n128", 128, 8, 8, 256, 256, maps="iid", rho=0.25),
        # a channel-width-scaled layer on an odd feature map and batch: sizes that are multiples of nothing large
        _layer("96>80@45x33 n5", 5, 45, 33, 96, 80),
        # int8 serving batch, requantised output
        _layer("int8 128@28 n32", 32, 28, 28, 128, 128, dtype="int8", out="int8", affine=True),
        # the benchmark's first layer: few channels, many pixels, clustered gate maps
        _layer("64@56 n64", 64, 56, 56, 64, 64),
        # a stride-2 layer whose gate maps do not cluster across channels
        _layer("128>256@28s2 n64", 64, 28, 28, 128, 256, stride=2, maps="literal"),
        # channel grouping with the shuffled store and the fired counts
        _layer("grouped 128@28 n64", 64, 28, 28, 128, 128, grouped=True, shuffle=True, counts=True),
        # a residual block's second layer at large batch: scale/shift by decision, residual, ReLU
        _layer("fused 256@14 n256", 256, 14, 14, 256, 256, affine=True, residual=True),
        # a point-wise layer of a MobileNet-style network
        _layer("1x1 1024@14 n64", 64, 14, 14, 1024, 1024, k=1),
        # the whole network at throughput batch
        _network("network 224 n256", 256, 224, 4, 0.3),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    what = rng.random()
    if what < 0.12:
        size = rng.randint(64, 224)
        return _no_name(_network("", _log_int(rng, 1, 140), size, rng.choice((2, 4, 8)), round(rng.uniform(0.1, 0.6), 2)))
    maps = rng.choice(("coherent", "coherent", "literal", "iid"))
    rho = round(rng.uniform(0.1, 0.7), 2)
    dtype = rng.choice(("bf16", "bf16", "bf16", "int8", "int8", "f32"))
    ragged = rng.random() < 0.25                 # channel counts that are multiples of 16 only
    g = rng.choice((2, 4, 4, 8))
    if what < 0.22:                              # a fully connected layer
        unit = 64
        cin, cout = unit * _log_int(rng, 4, 64), unit * _log_int(rng, 4, 64)
        n, h, w, k, stride = _log_int(rng, 1, 2048), 1, 1, 1, 1
        maps = rng.choice(("coherent", "iid"))
        cap = 17e9
    elif what < 0.40:                            # a point-wise layer
        unit = 16 if ragged else 64
        cin, cout = unit * _log_int(rng, 1, 1024 // unit), unit * _log_int(rng, 1, 1024 // unit)
        n, h, k = _log_int(rng, 1, 256), _log_int(rng, 4, 56), 1
        w, stride = h if rng.random() < 0.5 else _log_int(rng, 4, 56), rng.choice((1, 1, 1, 2))
        cap = 13e9
    else:                                        # a 3x3 layer
        unit = 16 if ragged else 64
        cin = unit * _log_int(rng, 1, 512 // unit)
        stride = rng.choice((1, 1, 1, 2))
        cout = cin if rng.random() < 0.6 else min(512, 2 * cin) if rng.random() < 0.6 else unit * _log_int(rng, 1, 512 // unit)
        n, h, k = _log_int(rng, 1, 256), _log_int(rng, 4, 112), 3
        w = h if rng.random() < 0.6 else _log_int(rng, 4, 112)
        cap = 30e9
    grouped = k == 3 and cout % g == 0 and rng.random() < 0.15
    narrow = cin // g * _DTYPES[dtype][2] % 32 != 0 or (grouped and cout // g % 64 and 64 % (cout // g))
    if dtype == "f32" or ragged or narrow:       # small models: at most a few hundred million products
        cap = 0.4e9
    ho, wo = -(-h // stride), -(-w // stride)
    macs = ho * wo * cout * cin * k * k
    n = max(1, min(n, int(cap // macs), int(1.5e8 // (h * w * max(cin, cout)))))
    while macs * n > cap and h > 4:              # one image alone is too much: a smaller one
        h, w = max(4, h // 2), max(4, w // 2)
        ho, wo = -(-h // stride), -(-w // stride)
        macs = ho * wo * cout * cin * k * k
    if macs * n > cap:
        cin = cout = unit
    out = {"bf16": rng.choice(("bf16", "bf16", "bf16", "f32")), "int8": rng.choice(("int8", "int8", "int8", "int32")),
           "f32": "f32"}[dtype]
    return _no_name(_layer("", n, h, w, cin, cout, k=k, stride=stride, g=g, dtype=dtype, out=out, maps=maps, rho=rho,
                           affine=out == "int8" or (out != "int32" and rng.random() < 0.5), residual=rng.random() < 0.3, grouped=grouped,
                           shuffle=grouped and rng.random() < 0.5, tau=0.3 if rng.random() < 0.08 else 0.0,
                           two_sided=dtype != "int8" and rng.random() < 0.06, counts=rng.random() < 0.25,
                           alloc=rng.random() < 0.2))


def _no_name(case):
    return {k: v for k, v in case.items() if k != "name"}


# ---------------------------------------------------------------------------------------------------
# inputs of one layer
# ---------------------------------------------------------------------------------------------------

def _blur(size, sigma=4.0):
    i = np.arange(size)
    m = np.exp(-0.5 * ((i[:, None] - i[None, :]) / sigma) ** 2)
    return torch.from_numpy((m / m.sum(1, keepdims=True)).astype(np.float32)).cuda()


def _magnitude(case, gen):
    """[n, h, w] field the activations are multiplied by."""
    u = torch.rand((case["n"], case["h"], case["w"]), generator=gen, device="cuda")
    f = torch.matmul(torch.matmul(_blur(case["h"]), u).contiguous(), _blur(case["w"]).t().contiguous())
    if case["maps"] == "literal":
        lo, hi = f.amin((1, 2), keepdim=True), f.amax((1, 2), keepdim=True)
        return (f - lo) / (hi - lo).clamp_min(1e-9)
    on = min(1.0, case["rho"] + 0.10)            # on/off regions that cover a little more than what shall fire
    flat = f.flatten().sort().values
    q = flat[min(flat.numel() - 1, int((1.0 - on) * flat.numel()))]
    return ((f - q) / 0.05 + 0.5).clamp(0.0, 1.0)


def _base_channels(case, group):
    cb = case["cin"] // case["g"]
    return slice(group * cb, (group + 1) * cb)


def _base_sums(case, x, w_base):
    """The base-path sums [pixels, cout] of the layer, from plain matrix products (fp32; fp64 for int8)."""
    dt = torch.float64 if case["dtype"] == "int8" else torch.float32
    n, h, w, k, s = case["n"], case["h"], case["w"], case["k"], case["stride"]
    pad = 1 if k == 3 else 0
    ho, wo = (h + 2 * pad - k) // s + 1, (w + 2 * pad - k) // s + 1
    groups = case["g"] if case["grouped"] else 1
    cpg = case["cout"] // groups
    parts = []
    for grp in range(groups):
        xp = torch.nn.functional.pad(x[..., _base_channels(case, grp)].to(dt), (0, 0, pad, pad, pad, pad))
        acc = torch.zeros((n * ho * wo, cpg), dtype=dt, device="cuda")
        for r in range(k):
            for c in range(k):
                tap = xp[:, r:r + (ho - 1) * s + 1:s, c:c + (wo - 1) * s + 1:s, :].reshape(n * ho * wo, -1)
                acc += tap @ w_base[grp * cpg:(grp + 1) * cpg, r, c, :].to(dt).t().contiguous()
        parts.append(acc)
    return torch.cat(parts, 1)


def _threshold(sums, mean, sd, z):
    """Per channel: the middle of the widest gap between neighbouring sums near mean + z * sd."""
    cols = sums.t().contiguous().sort(dim=1).values
    cols = torch.cat([cols[:, :1] - sd[:, None], cols, cols[:, -1:] + sd[:, None]], 1).contiguous()
    m = cols.shape[1]
    at = torch.searchsorted(cols, (mean + z * sd)[:, None].contiguous()).clamp(1, m - 1)
    half = min(512, max(1, m // 200))
    idx = (at + torch.arange(-half, half + 1, device="cuda")[None, :]).clamp(1, m - 1)
    hi, lo = cols.gather(1, idx), cols.gather(1, idx - 1)
    best = (hi - lo).argmax(1, keepdim=True)
    return ((hi + lo) * 0.5).gather(1, best)[:, 0]


def _gate(case, sums):
    mean, var = sums.mean(0), sums.var(0, unbiased=False)
    var = torch.where(var > 1e-9, var, torch.ones_like(var))
    sd = var.sqrt()

    def quantile(fraction_above):
        z = ((sums - mean) / sd).flatten().sort().values
        return z[min(z.numel() - 1, max(0, int((1.0 - fraction_above) * z.numel())))]

    z = quantile(case["rho"])
    if case["dtype"] == "int8":
        return dict(gate_thr_i32=torch.ceil(mean + z * sd).clamp(-2 ** 31, 2 ** 31 - 1).cpu().numpy().astype(np.int32))
    mean64, sd64 = mean.double().cpu().numpy(), sd.double().cpu().numpy()

    def delta(zz):
        return (_threshold(sums, mean, sd, zz).double().cpu().numpy() - mean64) / sd64

    gate = dict(gate_mean=mean64, gate_var=sd64 ** 2, delta=delta(z))
    if case["two_sided"]:
        gate["delta_hi"] = delta(quantile(case["rho"] * 0.1))
    return gate


def _prepare_layer(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, h, w, cin, cout, k, g = (case[f] for f in ("n", "h", "w", "cin", "cout", "k", "g"))
    cb = cin // g
    x = torch.relu(torch.randn((n, h, w, cin), generator=gen, device="cuda"))
    if case["maps"] != "iid":
        x *= _magnitude(case, gen)[..., None]
    std = math.sqrt(2.0 / (k * k * cin))
    wfull = torch.randn((cout, k, k, cin), generator=gen, device="cuda") * std
    groups = g if case["grouped"] else 1
    cpg = cout // groups
    if case["maps"] == "coherent":               # sums of all channels follow the local magnitude
        for grp in range(groups):
            wfull[grp * cpg:(grp + 1) * cpg, ..., _base_channels(case, grp)] += 2.0 * std
    in_dtype, tdt, _ = _DTYPES[case["dtype"]]
    out_dtype, odt, _ = _DTYPES[case["out"]]
    options = {}
    if case["dtype"] == "int8":
        s_x = (x.max() / 127.0).clamp_min(1e-9)
        s_w = (wfull.abs().amax((1, 2, 3)) / 127.0).clamp_min(1e-9)
        x = (x / s_x).round().clamp(0, 127).to(tdt)
        wfull = (wfull / s_w[:, None, None, None]).round().clamp(-127, 127).to(tdt)
        if case["affine"]:                       # fixed-point requantisation to the int8 range
            s_y = s_x * s_w.mean() * math.sqrt(k * k * cin) * 64.0 / 127.0
            mult = (s_x * s_w / s_y * 65536.0).round().clamp(1, 2 ** 30)
            options.update(rq_mult1=mult.cpu().numpy().astype(np.int32), rq_shift=16,
                           rq_mult0=(mult * (0.9 + 0.6 * torch.rand(cout, generator=gen, device="cuda"))).round().clamp(
                               1, 2 ** 30).cpu().numpy().astype(np.int32),
                           rq_bias=torch.randint(-8, 9, (cout,), generator=gen, device="cuda").cpu().numpy().astype(np.int32))
    else:
        x, wfull = x.to(tdt), wfull.to(tdt)
        if case["affine"]:
            table = torch.rand((4, cout), generator=gen, device="cuda").cpu().numpy()
            options.update(scale0=0.5 + table[0], shift0=0.2 * table[1] - 0.1, scale1=0.5 + table[2], shift1=0.2 * table[3] - 0.1)
    w_base = torch.cat([wfull[grp * cpg:(grp + 1) * cpg, ..., _base_channels(case, grp)] for grp in range(groups)]).contiguous()
    w_cond = torch.cat([torch.cat([wfull[grp * cpg:(grp + 1) * cpg, ..., :grp * cb],
                                   wfull[grp * cpg:(grp + 1) * cpg, ..., (grp + 1) * cb:]], -1)
                        for grp in range(groups)]).contiguous()
    options.update(_gate(case, _base_sums(case, x, w_base)))
    epilogue = B.CG_EPI_RELU
    if case["affine"] and case["dtype"] != "int8":
        epilogue |= B.CG_EPI_AFFINE
    residual = None
    pad = 1 if k == 3 else 0
    ho, wo = (h + 2 * pad - k) // case["stride"] + 1, (w + 2 * pad - k) // case["stride"] + 1
    if case["residual"]:
        epilogue |= B.CG_EPI_RESIDUAL
        shape = (n, ho, wo, cout)
        if case["dtype"] == "int8":
            residual = torch.randint(0, 128, shape, generator=gen, device="cuda", dtype=torch.int8)
            options["rq_res_mult"] = 30000
        else:
            residual = torch.relu(torch.randn(shape, generator=gen, device="cuda")).to(odt)
    layer = B.GatedConv(n_max=n, h=h, w=w, c_in=cin, c_out=cout, c_base=cb, w_base=w_base, w_cond=w_cond,
                        in_dtype=in_dtype, out_dtype=out_dtype, kh=k, kw=k, stride=case["stride"], pad=pad,
                        epilogue=epilogue, groups=g if case["grouped"] else 0, shuffle=case["shuffle"], tau_c=case["tau"],
                        **options)
    state = dict(kind="layer", layer=layer, x=x, residual=residual, alloc=case["alloc"], counts=case["counts"])
    if not case["alloc"]:                        # a serving loop keeps its output buffers
        state["y"] = torch.empty((n, ho, wo, cout), dtype=odt, device="cuda")
        state["bitmap"] = torch.empty((n * ho * wo, (cout + 31) // 32), dtype=torch.int32, device="cuda")
        state["count_buf"] = torch.empty(2 + n * cout, dtype=torch.int32, device="cuda") if case["counts"] else False
    return state


@functools.lru_cache(maxsize=2)
def _net(n, size, g, rho):
    return resnet18.GatedResNet18(max(n, 4), size=size, groups=g, rho=rho)      # (it calibrates on four pictures)


def prepare(case, seed):
    if case["kind"] == "layer":
        return _prepare_layer(case, seed)
    net = _net(case["n"], case["size"], case["g"], case["rho"])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    size, n = case["size"], case["n"]
    # synthetic pictures: noise times a large-scale magnitude, as the network was calibrated on
    u = torch.rand((n, size, size), generator=gen, device="cuda")
    blur = _blur(size, size / 14.0)
    f = torch.matmul(torch.matmul(blur, u).contiguous(), blur.t().contiguous())
    lo, hi = f.amin((1, 2), keepdim=True), f.amax((1, 2), keepdim=True)
    x = torch.relu(torch.randn((n, size, size, 3), generator=gen, device="cuda")) * ((f - lo) / (hi - lo))[..., None]
    return dict(kind="network", net=net, x=x.to(torch.bfloat16).contiguous())


def run(state):
    if state["kind"] == "network":
        return state["net"].forward(state["x"])
    layer = state["layer"]
    if state["alloc"]:
        return layer.forward(state["x"], residual=state["residual"], counts=state["counts"])
    return layer.forward(state["x"], residual=state["residual"], y=state["y"], bitmap=state["bitmap"],
                         counts=state["count_buf"])


# ---------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------

def _layer_work(n, h, w, cin, cout, k, stride, g, rho, eb, ob, residual, bitmap, counts):
    pad = 1 if k == 3 else 0
    m = n * ((h + 2 * pad - k) // stride + 1) * ((w + 2 * pad - k) // stride + 1)
    cb = cin // g
    pixels = n * h * w if k == 3 or stride == 1 else m
    nbytes = pixels * cin * eb + cout * k * k * cin * eb + m * cout * ob * (2 if residual else 1)
    nbytes += m * ((cout + 31) // 32) * 4 * bitmap + (8 + 4 * n * cout) * counts
    return nbytes, 2.0 * m * cout * k * k * (cb + rho * (cin - cb))


def work(case):
    if case["kind"] == "layer":
        rb = 1 if case["dtype"] == "int8" else _DTYPES[case["out"]][2]
        nbytes, flops = _layer_work(*(case[f] for f in ("n", "h", "w", "cin", "cout", "k", "stride", "g", "rho")),
                                    _DTYPES[case["dtype"]][2], _DTYPES[case["out"]][2], False, 1, int(case["counts"]))
        ho, wo = -(-case["h"] // case["stride"]), -(-case["w"] // case["stride"])
        nbytes += case["n"] * ho * wo * case["cout"] * rb * case["residual"]
        return {"bytes": nbytes, "flops": flops}
    n, size = case["n"], case["size"]
    # the layers' activations are counted once each: written by one layer, read by the next
    conv = (size - 1) // 2 + 1
    nbytes = n * size * size * 3 * 2 + 64 * 147 * 2 + n * ((conv - 1) // 2 + 1) ** 2 * 64 * 2
    flops = 2.0 * n * conv * conv * 64 * 147
    for spec in resnet18.conv_specs(size):
        b, f = _layer_work(n, spec.hw, spec.hw, spec.c_in, spec.c_out, 3, spec.stride, case["g"], case["rho"], 2, 2,
                           spec.residual, 0, 0)
        nbytes, flops = nbytes + b, flops + f
        if spec.stride == 2:                     # the block's 1x1 shortcut
            b, f = _layer_work(n, spec.hw, spec.hw, spec.c_in, spec.c_out, 1, 2, 1, 1.0, 2, 2, False, 0, 0)
            nbytes, flops = nbytes + b, flops + f
    last = resnet18.conv_specs(size)[-1].hw
    return {"bytes": nbytes + n * last * last * 512 * 2 + 512 * 1000 * 2 + n * 4000, "flops": flops + 2.0 * n * 512 * 1000}


def tolerance(case):
    if case["kind"] == "network":
        return {"rel": 1e-2}          # bf16 activations through twenty layers
    if case["dtype"] == "int8":
        return "exact"
    if case["out"] == "bf16":
        return {"rel": 3e-3, "differ": 1e-4}      # a few sums fall to the other side of a bf16 rounding
    return {"rel": 1e-5, "differ": 1e-4}          # fp32 sums of at most some thousand products
