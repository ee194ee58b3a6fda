"""The work that a user of this framework has it do, as cases that can be timed and compared.

A case is one pass through the public entry points on inputs made from a seed: a reassembled low-bit linear layer
(norm, channel disassembly and assembly, per-token quantization, integer GEMM, dequantising epilogue) as a serving
program calls it in decode, in small batches and in prefill; the same layer behind the gated activation of an MLP;
and the device side of calibrating one layer.  Shapes are those of `paper_2310_08041_amd/workloads.py` (the layers of
its five configurations and their transposes), of the tests, or generic.

  listed(), draw(rng)      the cases
  prepare(case, seed)      inputs, map, packed weights, workspace and output buffer on the GPU
  run(state)               one pass
  exact(case, seed)        the same outputs from plain torch in 64 bits
  work(case), tolerance(case)
"""
import math

import numpy as np
import torch

from paper_2310_08041_amd import binding as b

NORMS = {"none": b.NORM_NONE, "layer": b.NORM_LAYER, "rms": b.NORM_RMS}
CALIB_TOKENS = 256
EPS = 1e-5


def _linear(name, n, c, o, a_bits, w_bits, norm="rms", x="bf16", y="bf16", bulk="normal", outliers=None, theta="expand 0.01",
            swiglu=False):
    return dict(name=name, kind="linear", n=n, c=c, o=o, a_bits=a_bits, w_bits=w_bits, norm=norm, x=x, y=y, bulk=bulk,
                outliers=max(1, c // 200) if outliers is None else outliers, theta=theta, swiglu=swiglu)


def listed():
    return [
        # one token through a q/k/v projection: a single interactive request, the smallest call there is
        _linear("decode_1_qkv_w4a4", 1, 4096, 12288, 4, 4),
        # sixteen requests decoded together, 6-bit codes (the decode configuration)
        _linear("decode_16_q_w6a6", 16, 8192, 8192, 6, 6),
        # the tiny configuration: float32 activations, LayerNorm, float32 result
        _linear("tiny_layernorm_f32", 64, 512, 512, 4, 4, norm="layer", x="f32", y="f32", outliers=8, theta="fixed 4"),
        # a hundred requests decoded together (continuous batching), an up/gate projection; not a multiple of a tile
        _linear("batch_100_upgate_w4a4", 100, 5120, 27648, 4, 4, bulk="laplace"),
        # a short prompt or a larger decode batch through a down projection, 6-bit codes, nothing to normalise
        _linear("batch_200_down_w6a6", 200, 13824, 5120, 6, 6, norm="none"),
        # prefill of one 2048-token segment through q/k/v (the 7B configuration)
        _linear("prefill_2048_qkv_w4a4", 2048, 4096, 12288, 4, 4),
        # prefill of two segments through up/gate (the 13B configuration)
        _linear("prefill_4096_upgate_w4a4", 4096, 5120, 27648, 4, 4, bulk="laplace"),
        # prefill through the widest layer (the 70B configuration): the headline shape
        _linear("prefill_2048_down_w4a4", 2048, 28672, 8192, 4, 4, bulk="student_t3", theta="tmax 8"),
        # the same layer as a model has it, fed by silu(gate) * up, with 6-bit codes
        _linear("prefill_2048_swiglu_down_w6a6", 2048, 28672, 8192, 6, 6, norm="none", theta="expand 0.01", swiglu=True),
        # a ragged prompt with ragged widths: LayerNorm, float32 in and out, 8-bit activations on 4-bit weights
        _linear("ragged_777_layernorm_w4a8", 777, 5000, 4999, 8, 4, norm="layer", x="f32", y="f32"),
        # an expansion ratio of 5 % instead of 1 % (the ablation over the ratio): many computed channels
        _linear("prefill_2048_qkv_expand5", 2048, 4096, 12288, 4, 4, theta="expand 0.05"),
        # calibrating one layer: channel statistic, nearest pairs under the weighted distance, full-precision output, its error
        dict(name="calibrate_1024_proj", kind="calibrate", n=1024, c=4096, o=4096, norm="rms", x="bf16", bulk="normal", outliers=20),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    if rng.random() < 0.1:
        return dict(kind="calibrate", n=log(64, 1024), c=8 * log(32, 512), o=log(256, 4096), norm=rng.choice(["rms", "layer"]),
                    x=rng.choice(["bf16", "f32"]), bulk=rng.choice(["normal", "laplace"]), outliers=rng.randint(1, 20))
    while True:
        n, c, o = log(1, 4096), log(256, 28672), log(256, 27648)
        if rng.random() < 0.75:  # widths of real layers are multiples of 128, the others are ragged
            c, o = max(256, c // 128 * 128), max(256, o // 128 * 128)
        if n * c * o <= 4096 * 5120 * 27648 and n * c <= 2048 * 28672 and c * o <= 28672 * 8192:
            break
    a_bits, w_bits = rng.choice([(4, 4), (4, 4), (4, 4), (6, 6), (8, 8), (8, 4)])
    x = rng.choice(["bf16", "bf16", "bf16", "f32"])
    swiglu = x == "bf16" and rng.random() < 0.15
    case = _linear("", n, c, o, a_bits, w_bits, norm="none" if swiglu else rng.choice(["rms", "rms", "layer", "none"]), x=x,
                   y=rng.choice(["bf16", "bf16", "f32"]), bulk=rng.choice(["normal", "laplace", "student_t3"]),
                   theta=rng.choice(["expand 0.01", "expand 0.01", "tmax 8", "expand 0.05"]), swiglu=swiglu)
    del case["name"]
    return case


# ---------------------------------------------------------------- inputs, from the seed alone (plain torch)

def _bulk(kind, shape, g):
    z = torch.randn(shape, generator=g, device="cuda")
    if kind == "laplace":
        u = torch.rand(shape, generator=g, device="cuda").clamp_(1e-7, 1 - 1e-7).sub_(0.5)
        return -u.sign() * torch.log1p(-2 * u.abs())
    if kind == "student_t3":
        s = sum(torch.randn(shape, generator=g, device="cuda").square_() for _ in range(3))
        return z / (s / 3).sqrt_().clamp_(min=1e-3)
    return z


def _inputs(case, seed):
    """Everything the layer is made from: activations of this call and of a calibration batch with the same outlier
    channels, norm parameters, the map in the paper's terms, and the quantized weights."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n, c, o = case["n"], case["c"], case["o"]
    kind = torch.bfloat16 if case["x"] == "bf16" else torch.float32
    chans = torch.randperm(c, generator=g, device="cuda")[:min(case["outliers"], c)]
    factor = torch.ones(c, device="cuda")
    factor[chans] = torch.empty(chans.numel(), device="cuda").uniform_(30.0, 100.0, generator=g)
    s = {"gamma": torch.empty(c, device="cuda").uniform_(0.5, 1.5, generator=g),
         "beta": torch.randn(c, generator=g, device="cuda") * 0.1 if case["norm"] == "layer" else None}
    if case.get("swiglu"):
        s["gate"] = (_bulk(case["bulk"], (n, c), g)).to(kind)
        s["up"] = (_bulk(case["bulk"], (n, c), g) * factor).to(kind)
        gate, up = _bulk(case["bulk"], (CALIB_TOKENS, c), g), _bulk(case["bulk"], (CALIB_TOKENS, c), g) * factor
        calib = torch.nn.functional.silu(gate) * up
    else:
        s["x"] = (_bulk(case["bulk"], (n, c), g) * factor).to(kind)
        calib = _bulk(case["bulk"], (CALIB_TOKENS, c), g) * factor
    if case["kind"] == "calibrate":
        s["W"] = torch.randn((c, o), generator=g, device="cuda") * 0.02
        s["pick"] = torch.randperm(c, generator=g, device="cuda").to(torch.int32)
        s["got"] = torch.randn((n, o), generator=g, device="cuda")
        return s
    y = _norm(case, calib.to(kind).float(), s["gamma"], s["beta"])
    s["map"] = _paper_map(y, case["theta"])
    w = torch.randn((o, c), generator=g, device="cuda") * 0.02
    s["w"] = _quantize(_reassemble(s["map"], w, weights=True), case["w_bits"])
    return s


def _norm(case, x, gamma, beta):
    if case["norm"] == "layer":
        y = (x - x.mean(1, keepdim=True)) * torch.rsqrt(x.var(1, unbiased=False, keepdim=True) + EPS) * gamma
        return y if beta is None else y + beta
    if case["norm"] == "rms":
        return x * torch.rsqrt(x.square().mean(1, keepdim=True) + EPS) * gamma
    return x


def _paper_map(y, rule):
    """Disassembly counts from the calibration maxima and the threshold, then as many merged pairs as there are new
    sub-channels: the nearest member of set B for every member of set A, the shortest edges first."""
    m = y.abs().amax(0).cpu().numpy().astype(np.float32)
    kind, val = rule.split()
    if kind == "fixed":
        theta = float(val)
    elif kind == "tmax":
        theta = float(m.max()) / float(val)
    else:
        want, lo, hi = max(1, round(float(val) * m.size)), float(m.max()) / 4096, float(m.max())
        for _ in range(40):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if (np.ceil(m / mid) - 1).clip(0).sum() >= want else (lo, mid)
        theta = lo
    theta = float(np.float32(theta))
    split = np.maximum(1, np.ceil(m.astype(np.float64) / theta)).astype(np.int64)
    first = np.concatenate([[0], np.cumsum(split)])[:-1]
    single = split == 1
    a, bb = np.nonzero(single & (first % 2 == 0))[0], np.nonzero(single & (first % 2 == 1))[0]
    r = min(int((split - 1).sum()), a.size) if bb.size else 0
    ta, tb = torch.from_numpy(a).cuda(), torch.from_numpy(bb).cuda()
    if r:
        ya, yb = y[:, ta].t().contiguous(), y[:, tb].t().contiguous()
        best = [torch.cdist(p, yb).min(1) for p in ya.split(4096)]
        d, j = torch.cat([v.values for v in best]), torch.cat([v.indices for v in best])
        pick = torch.sort(torch.sort(d, stable=True).indices[:r]).values
        src, dst = (first[a[pick.cpu().numpy()]] // 2), (first[bb[j[pick].cpu().numpy()]] // 2)
    else:
        src = dst = np.zeros(0, np.int64)
    return dict(absmax=m, theta=theta, split=split, src=src.astype(np.int32), dst=dst.astype(np.int32))


def _reassemble(m, y, weights=False):
    """[rows, C] -> [rows, C^]: activations are divided by the split and averaged over a merged group, weights are
    repeated and summed."""
    chan = torch.from_numpy(np.repeat(np.arange(m["split"].size), m["split"])).cuda()
    z = y[:, chan]
    src, dst = torch.from_numpy(m["src"]).long().cuda() * 2, torch.from_numpy(m["dst"]).long().cuda() * 2 + 1
    if not weights:
        z = z / torch.from_numpy(m["split"]).cuda()[chan].to(y.dtype)
    if src.numel():
        # the k-th source of every destination at a time: one order of additions, the same on every run
        order, seen = np.zeros(m["dst"].size, np.int64), {}
        for i, v in enumerate(m["dst"].tolist()):
            order[i] = seen[v] = seen.get(v, -1) + 1
        group = torch.ones(z.shape[1], dtype=y.dtype, device=y.device)
        for k in range(int(order.max()) + 1):
            now = torch.from_numpy(np.nonzero(order == k)[0]).cuda()
            z[:, dst[now]] += z[:, src[now]]
            group[dst[now]] += 1
        if not weights:
            z = z / group
    keep = torch.ones(z.shape[1], dtype=torch.bool, device=y.device)
    keep[src] = False
    return z[:, keep]


def _quantize(v, bits):
    """Asymmetric codes per row."""
    top = (1 << bits) - 1
    lo, hi = v.amin(1, keepdim=True), v.amax(1, keepdim=True)
    scale = torch.where(hi > lo, (hi - lo) / top, torch.ones_like(hi))
    zero = -torch.round(lo / scale)
    codes = (torch.round(v / scale) + zero).clamp_(0, top)
    return dict(codes=codes.to(torch.uint8), scale=scale[:, 0], zero=zero[:, 0].to(torch.int32))


def _pack(codes, bits):
    rows, k = codes.shape
    c = torch.zeros((rows, (k + 255) // 256 * 256), dtype=torch.uint8, device=codes.device)
    c[:, :k] = codes
    if bits == 4:
        c = c[:, 0::2] | (c[:, 1::2] << 4)
    elif bits == 6:
        q = [c[:, i::4] for i in range(4)]
        c = torch.stack([q[0] | (q[1] << 6), (q[1] >> 2) | (q[2] << 4), (q[2] >> 4) | (q[3] << 2)], 2).reshape(rows, -1)
    return c.contiguous()


# ---------------------------------------------------------------- what the program has in hand, and the pass

def prepare(case, seed):
    s = _inputs(case, seed)
    n, c, o = case["n"], case["c"], case["o"]
    st = {"case": case, "norm": NORMS[case["norm"]], "gamma": s["gamma"], "beta": s["beta"]}
    if case["kind"] == "calibrate":
        half = c // 2
        st.update(x=s["x"], W=s["W"], got=s["got"], a=s["pick"][:half].sort().values.contiguous(),
                  b=s["pick"][half:].sort().values.contiguous(), n_match=min(n, CALIB_TOKENS),
                  y=torch.empty((n, c), device="cuda"), ref=torch.empty((n, o), dtype=torch.float64, device="cuda"),
                  loss=torch.empty(1, dtype=torch.float64, device="cuda"),
                  j=torch.empty(half, dtype=torch.int32, device="cuda"), d=torch.empty(half, dtype=torch.float64, device="cuda"),
                  ws=torch.empty(b.qllm_match_workspace_bytes(half, c - half), dtype=torch.uint8, device="cuda"),
                  err_ws=torch.empty(b.qllm_sq_error_workspace_bytes(n), dtype=torch.uint8, device="cuda"))
        return st
    m, w = s["map"], s["w"]
    built = b.qllm_build_map_host(m["absmax"], m["theta"], m["src"], m["dst"])
    st["map"] = b.DeviceMap(built["row_ptr"], built["src"], built["scale"], c, built["plan"])
    k, a_bits, w_bits = st["map"].C_out, case["a_bits"], case["w_bits"]
    st["w"] = b.DeviceWeight(_pack(w["codes"], w_bits).cpu().numpy(), w["scale"].cpu().numpy(), w["zero"].cpu().numpy(),
                             w["codes"].sum(1, dtype=torch.int32).cpu().numpy(), k, w_bits, tiles8=True if a_bits > 4 else None)
    st["ws"] = torch.empty(b.qllm_workspace_bytes(n, k, o, a_bits), dtype=torch.uint8, device="cuda")
    st["y"] = torch.empty((n, o), dtype=torch.bfloat16 if case["y"] == "bf16" else torch.float32, device="cuda")
    if case["swiglu"]:
        st.update(gate=s["gate"], up=s["up"], x=torch.empty_like(s["gate"]))
    else:
        st["x"] = s["x"]
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "calibrate":
        absmax = torch.zeros(case["c"], device="cuda")
        b.qllm_norm_channel_absmax(st["x"], st["norm"], st["gamma"], st["beta"], EPS, absmax, st["y"])
        b.qllm_match_nearest(st["y"][:st["n_match"]], st["W"], st["a"], st["b"], st["j"], st["d"], st["ws"])
        b.qllm_linear_f64(st["y"], st["W"], st["ref"])
        b.qllm_sq_error(st["got"], st["ref"], st["loss"], st["err_ws"])
        return {"absmax": absmax, "y": st["y"], "best_j": st["j"], "best_d": st["d"], "ref": st["ref"], "loss": st["loss"]}
    if case["swiglu"]:
        b.qllm_swiglu(st["gate"], st["up"], st["x"])
    b.qllm_reassembled_linear(st["x"], st["norm"], st["gamma"], st["beta"], EPS, st["map"], case["a_bits"], st["w"], st["y"], st["ws"])
    return {"x": st["x"], "y": st["y"]} if case["swiglu"] else st["y"]


def exact(case, seed):
    s = _inputs(case, seed)
    f64 = {k: (v.double() if isinstance(v, torch.Tensor) and v.is_floating_point() else v) for k, v in s.items()}
    if case["kind"] == "calibrate":
        y, W = _norm(case, f64["x"], f64["gamma"], f64["beta"]), f64["W"]
        half = case["c"] // 2
        a, bb = s["pick"][:half].sort().values.long(), s["pick"][half:].sort().values.long()
        ym = y[:min(case["n"], CALIB_TOKENS)]
        d = (torch.cdist(ym[:, a].t().contiguous(), ym[:, bb].t().contiguous()) * torch.cdist(W[a], W[bb]) / 2).square().min(1)
        ref = y @ W
        return {"absmax": y.abs().amax(0), "y": y, "best_j": d.indices.to(torch.int32), "best_d": d.values, "ref": ref,
                "loss": (f64["got"] - ref).square().sum().reshape(1)}
    if case["swiglu"]:
        x = torch.nn.functional.silu(f64["gate"]) * f64["up"]
        xin = x.to(s["gate"].dtype).double()  # the layer's input is what the activation stored
    else:
        xin = f64["x"]
    q = _quantize(_reassemble(s["map"], _norm(case, xin, f64["gamma"], f64["beta"]).contiguous()), case["a_bits"])
    xq = (q["codes"].double() - q["zero"].double()[:, None]) * q["scale"][:, None]
    w = f64["w"]
    wq = (w["codes"].double() - w["zero"].double()[:, None]) * w["scale"].double()[:, None]
    y = xq @ wq.t().contiguous()
    return {"x": x, "y": y} if case["swiglu"] else y


def work(case):
    """Inputs once, results once; the products of the contraction.  Nothing for codes, tiles or partial sums."""
    n, c, o = case["n"], case["c"], case["o"]
    size = {"bf16": 2, "f32": 4}
    if case["kind"] == "calibrate":
        half = c // 2
        return {"bytes": n * c * (size[case["x"]] + 4) + 4 * c * o + 12 * n * o + 12 * half,
                "flops": 2 * n * c * o + 2 * half * (c - half) * (min(n, CALIB_TOKENS) + o)}
    swiglu = 3 * n * c * 2 if case["swiglu"] else 0
    return {"bytes": swiglu + n * c * size[case["x"]] + o * c * case["w_bits"] / 8 + 12 * o + n * o * size[case["y"]],
            "flops": 2 * n * c * o}


def tolerance(case):
    """About four times what the path shows against exact(): 1.7e-3 for a bfloat16 result (its rounding; 3.7e-3 where
    bfloat16 activations are quantized as they are, with ties); 3e-5 for a float32 one (codes that a row statistic
    rounded otherwise moves by one); 4e-8 for the calibration's float32 and float64 values."""
    if case["kind"] == "calibrate":
        return {"rel": 1e-6, "max": 1e-5, "differ": 2e-3}
    if case["y"] == "f32" and not case["swiglu"]:
        return {"rel": 2e-4, "max": 2e-2}
    return {"rel": 7e-3, "max": 5e-2}
