"""Performance cases of the activation-compression path, through the package's public entry points.

A case is one call sequence a pipeline stage makes for one activation tensor (or one group of
microbatches): the sender path (statistics, directed search, quantize + pack), the receiver
(unpack + dequantize), several sender paths in flight with their receivers, or the step-by-step
calls that bring their results to the host.  Sizes are those of the repository's configurations
(ViT-Base, ViT-Large and ViT-Huge stage boundaries, and the 151 M-element bf16 tensor) plus smaller
and ragged ones.  Tensors are drawn on the GPU with the same recipes as synth_inputs.py.
"""
import ctypes
import math

import torch

import paper_2211_04515_amd as qp

DEVICE = "cuda"
BITS = (2, 3, 4, 6, 8, 16)

# the most elements of one drawn case: what its path is used for, and no more work than the listed cases
MIN_N = 4_000
MAX_SEND_F32 = 32_000_000
MAX_BF16 = 151_257_088
MAX_STREAM = 64_000_000
MAX_STEPS_F32 = 16_000_000


def _case(path, n, dtype, bits, values, flags=0, dist=0, count=1, name=None):
    c = {"path": path, "n": n, "dtype": dtype, "bits": bits, "values": values, "flags": flags, "dist": dist, "count": count}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a few dozen tokens of one request at the lowest bitwidth: launches and latency are all there is
        _case("send", 38_411, "bf16", 2, "laplace", name="send_tokens_bf16_2bit"),
        # one image's activations, 1x197x768
        _case("send", 151_296, "f32", 4, "laplace", name="send_image_f32_4bit"),
        # a partly filled microbatch of odd size, between one image and a full batch
        _case("send", 1_234_567, "f32", 6, "mixture", name="send_ragged_f32_6bit"),
        # the ViT-Base stage boundary, 64x197x768, at the bitwidth of a narrow link and at the usual one
        _case("send", 9_682_944, "f32", 2, "mixture", name="send_base_f32_2bit"),
        _case("send", 9_682_944, "f32", 8, "mixture", name="send_base_f32_8bit"),
        # the same boundary under the deployment policy: no search above 4 bit
        _case("send", 9_682_944, "f32", 16, "mixture", flags=qp.QP_SEARCH_LOW_BITS_ONLY, name="send_base_f32_16bit_policy"),
        # the ViT-Large boundary after a GELU, 64x197x1024: skewed, one-sided values
        _case("send", 12_910_592, "f32", 4, "gelu", name="send_gelu_f32_4bit"),
        # ViT-L/16 at 384 px, 256x577x1024 in bf16: heavy-tailed values, the largest tensor
        _case("send", 151_257_088, "bf16", 3, "student", name="send_large_bf16_3bit"),
        # the receiving stage of the ViT-Base boundary, and of the largest tensor
        _case("receive", 9_682_944, "f32", 4, "mixture", name="receive_base_4bit"),
        _case("receive", 151_257_088, "f32", 3, "student", name="receive_large_3bit"),
        # six ViT-Huge microbatches (32x257x1280) in flight on three lanes, each expanded again by its receiver
        _case("stream", 10_526_720, "f32", 2, "laplace", count=6, name="stream_huge_f32_2bit"),
        # the four steps called one by one with their results on the host (a controller that logs them), with the
        # coarse-to-fine sweep
        _case("steps", 9_682_944, "f32", 3, "mixture", flags=qp.QP_SEARCH_COARSE_TO_FINE, name="steps_base_f32_3bit_c2f"),
    ]


def _log_uniform(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    n = min(max(n, lo), hi)
    # odd and ragged sizes as often as round ones
    return n if rng.random() < 0.5 else max(lo, n - n % 768)


def draw(rng):
    path = rng.choice(("send", "send", "send", "send", "receive", "receive", "stream", "steps"))
    bits = rng.choice(BITS)
    dtype = rng.choice(("f32", "f32", "bf16"))
    values = rng.choice(("laplace", "mixture", "gelu", "student", "gauss"))
    flags, dist, count = 0, qp.QP_LAPLACE, 1
    if path == "receive":
        return _case(path, _log_uniform(rng, MIN_N, MAX_BF16), "f32", bits, values)
    if path == "send":
        n = _log_uniform(rng, MIN_N, MAX_SEND_F32 if dtype == "f32" else MAX_BF16)
    elif path == "stream":
        count = rng.randrange(2, 9)
        n = _log_uniform(rng, MIN_N, MAX_STREAM // count)
    else:
        n = _log_uniform(rng, MIN_N, MAX_STEPS_F32)
    # most calls are the paper's method; the variants are used now and then
    if rng.random() < 0.4:
        flags = rng.choice((qp.QP_SEARCH_CLIP_TO_DATA, qp.QP_SEARCH_LOW_BITS_ONLY, qp.QP_SEARCH_COARSE_TO_FINE))
        if flags == qp.QP_SEARCH_COARSE_TO_FINE and dtype == "bf16" and n >= 1 << 20:
            flags = 0   # not offered there
    if rng.random() < 0.2:
        dist = rng.choice((qp.QP_GAUSS, qp.QP_DIST_AUTO)) if path != "steps" else qp.QP_GAUSS
    return _case(path, n, dtype, bits, values, flags, dist, count)


# ---- inputs -----------------------------------------------------------------------------------

def _laplace(n, g):
    x = torch.empty(n, device=DEVICE).exponential_(generator=g)
    return x * (torch.randint(0, 2, (n,), device=DEVICE, generator=g, dtype=torch.int8) * 2 - 1)


def _outliers(x, g, share, factor):
    k = int(round(share * x.numel()))
    if k:
        at = torch.randint(0, x.numel(), (k,), device=DEVICE, generator=g).unique()
        x[at] *= factor


def _values(kind, n, dtype, g):
    if kind == "laplace":
        x = _laplace(n, g) * 0.5
        _outliers(x, g, 0.001, 20.0)
    elif kind == "mixture":
        x = torch.where(torch.rand(n, device=DEVICE, generator=g) < 0.7, _laplace(n, g) * 0.4,
                        torch.randn(n, device=DEVICE, generator=g) + 0.1)
        _outliers(x, g, 0.0005, 30.0)
    elif kind == "gelu":
        x = torch.nn.functional.gelu(torch.randn(n, device=DEVICE, generator=g) * 1.5)
    elif kind == "student":   # three degrees of freedom
        chi2 = torch.randn(n, device=DEVICE, generator=g).square_()
        for _ in range(2):
            chi2 += torch.randn(n, device=DEVICE, generator=g).square_()
        x = torch.randn(n, device=DEVICE, generator=g) / (chi2 / 3.0).sqrt_() * 0.5
    else:
        x = torch.randn(n, device=DEVICE, generator=g) * 0.8 + 0.05
    return x.to(torch.bfloat16) if dtype == "bf16" else x


def _config(case):
    cfg = qp.qp_default_search_cfg()
    cfg.flags, cfg.dist = case["flags"], case["dist"]
    return cfg


def _records(ws):
    """What a call leaves in its workspace, as views: statistics, search result, winner's index, all scores."""
    at = qp.qp_ws_offset(qp.QP_WS_STATS)
    res = qp.qp_ws_offset(qp.QP_WS_RESULT)
    sc = qp.qp_ws_offset(qp.QP_WS_SCORES)
    return {"moments": ws[at + 16:at + 64].view(torch.float64), "density": ws[at + 72:at + 88].view(torch.float64),
            "result": ws[res:res + 48].view(torch.float64), "winner": ws[res + 48:res + 56].view(torch.int32),
            "scores": ws[sc:sc + 101 * 8].view(torch.float64)}


def prepare(case, seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    n, bits, dtype = case["n"], case["bits"], case["dtype"]
    s = {"path": case["path"], "bits": bits}
    if case["path"] == "receive":
        # a payload as it comes off the link, and the record that travels beside it
        nbytes = qp.qp_packed_bytes(n, bits)
        s["packed"] = torch.randint(-2**31, 2**31 - 1, (nbytes // 4,), device=DEVICE, generator=g, dtype=torch.int32).view(torch.uint8)
        alpha = float(0.5 + torch.rand(1, device=DEVICE, generator=g).item())
        s["q"] = qp.qp_make_qparams(0.01, qp.qp_aciq_constant(bits) * alpha, bits, n)
        s["y"] = torch.empty(n, device=DEVICE)
        return s
    s["cfg"] = _config(case)
    if case["path"] == "send":
        s["x"] = _values(case["values"], n, dtype, g)
        s["ws"] = qp.alloc_workspace(n, s["cfg"])
        s["packed"] = qp.alloc_packed(n, bits)
        s["grid"] = torch.empty(ctypes.sizeof(qp.qp_qparams_t), dtype=torch.uint8, device=DEVICE)
        s["out"] = {"packed": s["packed"], "grid": s["grid"][16:].view(torch.float32), **_records(s["ws"])}
    elif case["path"] == "stream":
        count = case["count"]
        s["x"] = [_values(case["values"], n, dtype, g) for _ in range(count)]
        s["packed"] = [qp.alloc_packed(n, bits) for _ in range(count)]
        s["grid"] = [torch.empty(ctypes.sizeof(qp.qp_qparams_t), dtype=torch.uint8, device=DEVICE) for _ in range(count)]
        s["y"] = [torch.empty(n, device=DEVICE) for _ in range(count)]
        s["lanes"] = [(qp.alloc_workspace(n, s["cfg"]), torch.cuda.Stream()) for _ in range(min(3, count))]
        s["jobs"] = [(x, bits, p, q.data_ptr()) for x, p, q in zip(s["x"], s["packed"], s["grid"])]
        s["out"] = {"packed": s["packed"], "grid": [q[16:].view(torch.float32) for q in s["grid"]], "y": s["y"]}
    else:
        s["x"] = _values(case["values"], n, dtype, g)
        s["ws"] = qp.alloc_workspace(n, s["cfg"])
        s["packed"] = qp.alloc_packed(n, bits)
        s["y"] = torch.empty(n, device=DEVICE)
    return s


# ---- one pass -----------------------------------------------------------------------------------

def run(s):
    bits = s["bits"]
    if s["path"] == "send":
        qp.qp_compress_async(s["x"], bits, s["ws"], s["packed"], s["grid"].data_ptr(), s["cfg"])
        return s["out"]
    if s["path"] == "receive":
        qp.qp_unpack_dequant(s["packed"], s["q"], s["y"])
        return s["y"]
    if s["path"] == "stream":
        here = torch.cuda.current_stream()
        for _, stream in s["lanes"]:
            stream.wait_stream(here)
        qp.qp_compress_many_async(s["jobs"], s["lanes"], s["cfg"])
        for i, (packed, grid, y) in enumerate(zip(s["packed"], s["grid"], s["y"])):
            qp.qp_unpack_dequant_dev(packed, bits, grid.data_ptr(), y, s["lanes"][i % len(s["lanes"])][1])
        for _, stream in s["lanes"]:
            here.wait_stream(stream)
        return s["out"]
    st = qp.qp_stats(s["x"], s["ws"])
    res, q = qp.qp_dsaciq_search(s["x"], st, bits, s["ws"], s["cfg"])
    qp.qp_quant_pack(s["x"], q, s["packed"])
    qp.qp_unpack_dequant(s["packed"], q, s["y"])
    return {"mean": st.mean, "mad": st.mad, "var": st.var, "b_r": st.b_r, "peak": st.peak_count, "alpha": res.alpha_star,
            "winner": res.j_star, "mse": res.mse_star, "mse_aciq": res.mse_aciq, "packed": s["packed"], "y": s["y"]}


def work(case):
    """Each tensor read once, each payload and expanded tensor written once; about 30 operations per element of a
    sender path (moments, a bin, a code), whatever the search costs."""
    n, bits = case["n"], case["bits"]
    elem = 2 if case["dtype"] == "bf16" else 4
    packed = qp.qp_packed_bytes(n, bits)
    if case["path"] == "send":
        return {"bytes": n * elem + packed, "flops": 30 * n}
    if case["path"] == "receive":
        return {"bytes": packed + 4 * n, "flops": 2 * n}
    if case["path"] == "stream":
        return {"bytes": case["count"] * (n * elem + 2 * packed + 4 * n), "flops": case["count"] * 32 * n}
    return {"bytes": n * elem + 2 * packed + 4 * n, "flops": 32 * n}


def tolerance(case):
    """The receiver has one correct result.  The sender's sums are 64-bit (another order of them changes a record
    by about 1e-13); its grid is rounded to 32 bits once, so a grid that falls on the other side of a rounding
    differs by 1.2e-7 and moves the few codes whose values lie that close to a threshold."""
    if case["path"] == "receive":
        return "exact"
    return {"rel": 2e-7, "max": 1e-6, "differ": 4e-6}


# ---- the same results in 64 bits ------------------------------------------------------------------

def _constant(bits, dist):
    """The minimiser a of ACIQ's expected error at this bitwidth: Laplace a e^a = 3 4^q, Gaussian phi(a) - a Q(a) = a / (6 4^q)."""
    def excess(a):
        if dist == qp.QP_GAUSS:
            return math.exp(-0.5 * a * a) / math.sqrt(2 * math.pi) - a * 0.5 * math.erfc(a / math.sqrt(2)) - a / (6.0 * 4.0 ** bits)
        return math.log(3.0 * 4.0 ** bits) - math.log(a) - a
    lo, hi = 1e-3, 100.0
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if excess(mid) > 0 else (lo, mid)
    return 0.5 * (lo + hi)


def _grid(center, alpha, bits, clip):
    """[lo, hi, scale, 1/scale] as the record holds them, in 32 bits."""
    def f32(v):
        return torch.tensor(v, dtype=torch.float64).to(torch.float32).item()
    lo, hi = f32(f32(center) - f32(alpha)), f32(f32(center) + f32(alpha))
    if clip:
        lo, hi = max(lo, clip[0]), min(hi, clip[1])
    if not hi > lo:
        return [lo, hi, 0.0, 0.0]
    levels = 2.0 ** bits - 1
    return [lo, hi, f32((hi - lo) / levels), f32(levels / (hi - lo))]


def _expanded(x, grid, bits):
    """What the receiver holds: codes by the 32-bit rule, lo + code scale in 64 bits rounded once."""
    lo, hi, scale, inv = grid
    code = ((x.clamp(lo, hi) - torch.tensor(lo, device=DEVICE)) * torch.tensor(inv, device=DEVICE)).round_().clamp_(0, 2 ** bits - 1)
    return code.double().mul_(scale).add_(lo).float()


def _sender(x, bits, flags, dist):
    x = x.float()
    n, d = x.numel(), x.double()
    mean, mn, mx = d.mean().item(), x.min(), x.max()
    nbins = 2048
    bins = ((x - mn) * (nbins / (mx - mn).double()).float()).clamp_(0, nbins - 1).to(torch.int64)
    hist = torch.bincount(bins, minlength=nbins).double()
    width = (mx.double() - mn.double()).item() / nbins
    peak = int(hist.max().item())
    stats = {"mean": mean, "mad": (d - mean).abs_().mean().item(), "abs_mean": d.abs().mean().item(),
             "var": (d - mean).square_().mean().item(), "min": mn.item(), "max": mx.item(), "peak": peak,
             "peak_density": peak / (n * width)}
    stats["b_r"] = 1.0 / (2.0 * stats["peak_density"])
    if dist == qp.QP_DIST_AUTO:
        z = mn.double() + (torch.arange(nbins, device=DEVICE, dtype=torch.float64) + 0.5) * width - mean
        dens, b, var = hist / (n * width), stats["mad"], stats["var"]
        fit_l = (dens - (-z.abs() / b).exp() / (2 * b)).square().sum().item()
        fit_g = (dens - (-z * z / (2 * var)).exp() / math.sqrt(2 * math.pi * var)).square().sum().item()
        dist = qp.QP_GAUSS if fit_g < fit_l else qp.QP_LAPLACE
    if dist == qp.QP_GAUSS:
        s_e, s_r = math.sqrt(stats["var"]), 1.0 / (math.sqrt(2 * math.pi) * stats["peak_density"])
    else:
        s_e, s_r = stats["mad"], stats["b_r"]
    t, c = 100, _constant(bits, dist)
    step = (s_r - s_e) / t
    clip = (stats["min"], stats["max"]) if flags & qp.QP_SEARCH_CLIP_TO_DATA else None
    scores = [math.nan] * (t + 1)

    def score(js):
        for j in js:
            if scores[j] != scores[j]:
                scores[j] = (d - _expanded(x, _grid(mean, c * (s_e + j * step), bits, clip), bits).double()).square_().sum().item()
        return min(js, key=lambda j: (scores[j], j))

    if flags & qp.QP_SEARCH_LOW_BITS_ONLY and bits > 4:
        win = 0
    elif flags & qp.QP_SEARCH_COARSE_TO_FINE:
        first = score(list(range(0, t + 1, 10)))
        win = score(list(range(max(0, first - 9), min(t, first + 9) + 1)))
    else:
        win = score(list(range(t + 1)))
    alpha = c * (s_e + win * step)
    result = [s_e, s_r, s_e + win * step, alpha, scores[0] / n, scores[win] / n]
    return stats, scores, result, _grid(mean, alpha, bits, clip), x


def exact(case, seed):
    s = prepare(case, seed)
    bits = case["bits"]

    def f64(v):
        return torch.tensor(v, dtype=torch.float64)
    if case["path"] == "receive":
        n = case["n"]
        words = torch.cat([s["packed"].view(torch.int32), torch.zeros(1, dtype=torch.int32, device=DEVICE)])
        y = torch.empty(n, dtype=torch.float64, device=DEVICE)
        for at in range(0, n, 1 << 24):
            bit = torch.arange(at, min(n, at + (1 << 24)), device=DEVICE, dtype=torch.int64) * bits
            word = bit >> 5
            both = (words[word].long() & 0xffffffff) | ((words[word + 1].long() & 0x7fffffff) << 32)
            y[at:at + bit.numel()] = ((both >> (bit & 31)) & (2 ** bits - 1)).double() * s["q"].scale + s["q"].lo
        return y
    if case["path"] == "stream":
        grids, ys = [], []
        for x in s["x"]:
            *_, grid, x32 = _sender(x, bits, case["flags"], case["dist"])
            grids.append(f64(grid))
            ys.append(_expanded(x32, grid, bits).double())
        return {"packed": [None] * len(grids), "grid": grids, "y": ys}
    stats, scores, result, grid, x32 = _sender(s["x"], bits, case["flags"], case["dist"])
    if case["path"] == "send":
        return {"packed": None, "grid": f64(grid), "moments": f64([stats[k] for k in ("mean", "mad", "abs_mean", "var", "min", "max")]),
                "density": f64([stats["peak_density"], stats["b_r"]]), "result": f64(result), "winner": None, "scores": f64(scores)}
    return {"mean": stats["mean"], "mad": stats["mad"], "var": stats["var"], "b_r": stats["b_r"], "peak": None, "alpha": result[3],
            "winner": None, "mse": result[5], "mse_aciq": result[4], "packed": None, "y": _expanded(x32, grid, bits).double()}
