"""Timed cases of the framework: what a program that quantizes a network with it does.

A search case finds the breakpoints of a layer's or a model's weights (exhaustively, or
with the prefix-sum search) and quantizes the weights with them; a selector case chooses
the breakpoints from an assumed law instead and asks for their error; an inner-product
case multiplies 8-bit activations with packed weights.  Inputs are drawn on the GPU, in
the shapes of the networks the paper evaluates and with the values of its weights:
bell-shaped or long-tailed, with a scale of its own per channel.
"""
from __future__ import annotations

import math

import torch

from paper_2002_00104_amd import pwlq, synth

PER_CHANNEL, PER_TENSOR = pwlq.PER_CHANNEL, pwlq.PER_TENSOR


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _text(shapes):
    return ";".join("%dx%d" % synth.as_ck(s) for s in shapes)


def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split(";")]


def _search(name, shapes, dist, bits=4, n_cand=1000, mode=PER_CHANNEL, fast=False, out="bytes"):
    return dict(name=name, kind="search", shapes=shapes, dist=dist, bits=bits, n_cand=n_cand,
                mode=mode, fast=fast, out=out)


def _linear(name, M, K, N, bits, sums=False):
    return dict(name=name, kind="linear", M=M, K=K, N=N, bits=bits, sums=sums)


def listed():
    resnet = _text(synth.resnet50_shapes())
    transformer = _text(synth.transformer_shapes())
    return [
        # the smallest call: one 3x3 convolution, a coarse grid, as in a loop over layers
        _search("conv_layer", "64x576", "laplace", n_cand=100),
        # one layer of no round size, at five bits, kept packed and dequantized for a check of accuracy
        _search("ragged_layer", "515x1155", "gauss", bits=5, n_cand=300, out="packed_hat"),
        # a whole network in one call, the grid and width of the paper's main tables
        _search("resnet50", resnet, "gauss"),
        # a network of many short channels (depthwise filters: nine weights each), kept packed
        _search("mobilenetv2", _text(synth.mobilenetv2_shapes()), "laplace", out="packed"),
        # one breakpoint per layer, three bits, a fine grid
        _search("inceptionv3_per_tensor", _text(synth.inceptionv3_shapes()), "student_t",
                bits=3, n_cand=2000, mode=PER_TENSOR),
        # the linear layers of a transformer block; the largest call
        _search("transformer", transformer, "laplace_outliers"),
        # the search that a program in a hurry takes, with the storage format
        _search("resnet50_fast", resnet, "gauss", fast=True, out="packed"),
        _search("transformer_fast", transformer, "laplace_outliers", fast=True),
        # the paper's own selector (Gaussian, solved), its error, and the packed weights
        dict(name="resnet50_selector", kind="select", shapes=resnet, dist="gauss", bits=4,
             mode=PER_CHANNEL, selector=pwlq.GAUSS_SOLVE),
        # inference on packed weights: a long prompt, a few tokens of decoding, and a
        # classifier head whose integer sums are wanted apart
        _linear("linear_prefill", 4096, 4096, 4096, 4),
        _linear("linear_decode", 8, 4096, 11008, 4),
        _linear("linear_head_sums", 250, 2048, 1000, 6, sums=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shapes(rng, most):
    """One to forty tensors of 16..4096 channels of 9..11008 weights, at most `most` weights."""
    left, got = most, []
    for _ in range(_log(rng, 1, 40)):
        C, K = _log(rng, 16, 4096), _log(rng, 9, 11008)
        C = min(C, left // K)
        if C < 1:
            break
        got.append("%dx%d" % (C, K))
        left -= C * K
    return ";".join(got)


def draw(rng):
    kind = rng.choice(("search", "fast", "select", "linear", "linear"))
    bits = rng.choice((4, 4, 4, 2, 3, 5, 6, 7, 8))
    if kind == "linear":
        M, K, N = _log(rng, 1, 4096), 16 * _log(rng, 8, 688), _log(rng, 32, 11008)
        M = max(1, min(M, 4096 ** 3 // (K * N)))
        return dict(kind="linear", M=M, K=K, N=N, bits=bits, sums=rng.random() < 0.25)
    dist = rng.choice(("gauss", "laplace", "student_t", "laplace_outliers"))
    mode = PER_TENSOR if rng.random() < 0.3 else PER_CHANNEL
    if kind == "select":
        return dict(kind="select", shapes=_draw_shapes(rng, 60_000_000), dist=dist, bits=bits,
                    mode=mode, selector=rng.choice((pwlq.GAUSS_FIT, pwlq.GAUSS_SOLVE, pwlq.LAPLACE_SOLVE)))
    n_cand = _log(rng, 50, 2000)
    most = min(60_000_000, 25_000_000_000 // n_cand)
    return dict(kind="search", shapes=_draw_shapes(rng, most), dist=dist, bits=bits, n_cand=n_cand,
                mode=mode, fast=kind == "fast", out=rng.choice(("bytes", "packed", "packed_hat")))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _weights(C, K, dist, gen):
    def normal():
        return torch.randn((C, K), generator=gen, device="cuda")

    def laplace():
        e = torch.empty((C, K), device="cuda").exponential_(generator=gen)
        return e.mul_(torch.randint(0, 2, (C, K), generator=gen, device="cuda").mul_(2).sub_(1))

    if dist == "student_t":
        chi2 = normal().square_().add_(normal().square_()).add_(normal().square_())
        return normal().div_(chi2.div_(3.0).sqrt_().clamp_min_(1e-6)).mul_(0.02)
    if dist == "laplace_outliers":
        w = laplace().mul_(0.02)
        w[torch.rand((C, K), generator=gen, device="cuda") < 0.001] *= 10.0
        return w
    scale = torch.randn((C, 1), generator=gen, device="cuda").mul_(0.5).sub_(3.0).exp_()
    return (normal() if dist == "gauss" else laplace()).mul_(scale)


def _tensors(case, seed):
    gen = _generator(seed)
    return [_weights(C, K, case["dist"], gen) for C, K in _shapes(case)]


def _linear_inputs(case, seed):
    """Activations, and weights as a quantized network stores them: codes and region flags
    (per channel, breakpoint near where the search puts it), the parameters p and m."""
    gen = _generator(seed)
    M, K, N, bits = case["M"], case["K"], case["N"], case["bits"]
    L = float(2 ** (bits - 1) - 1)
    w = _weights(N, K, "laplace", gen)
    a = w.abs()
    m = a.amax(1)
    p = m * (0.2 + 0.2 * torch.rand(N, generator=gen, device="cuda"))
    tail = a > p[:, None]
    x = torch.where(tail, (a - p[:, None]) * (L / (m - p))[:, None], a * (L / p)[:, None])
    code = x.round().clamp_(max=L).to(torch.uint8)
    code |= (w < 0).to(torch.uint8) << (bits - 1)
    xq = torch.randint(-128, 128, (M, K), generator=gen, device="cuda").to(torch.int8)
    return xq, code, tail, p, m


S_X, Z_X = 0.0123, -0.57          # step and offset of the activations


def _bit_stream(values, bits):
    """uint8 values as one little-endian stream of `bits` bits each (size a multiple of 8)."""
    by = values.reshape(-1, 8).to(torch.int64)
    word = torch.zeros(by.shape[0], dtype=torch.int64, device=by.device)
    for i in range(8):
        word |= by[:, i] << (i * bits)
    return torch.stack([(word >> (8 * i)) & 255 for i in range(bits)], 1).to(torch.uint8).reshape(-1)


def prepare(case, seed):
    if case["kind"] == "linear":
        xq, code, tail, p, m = _linear_inputs(case, seed)
        M, N = case["M"], case["N"]
        ws = torch.empty(max(256, pwlq.lib.pwlq_linear_workspace_bytes(N)), dtype=torch.uint8, device="cuda")
        y = torch.empty((M, N), dtype=torch.float32, device="cuda")
        acc = torch.empty((3, M, N), dtype=torch.int32, device="cuda") if case["sums"] else None
        return dict(case=case, xq=xq, codes=_bit_stream(code, case["bits"]),
                    flags=_bit_stream(tail.to(torch.uint8), 1), p=p, m=m, workspace=ws, out=(y, acc))
    tensors = _tensors(case, seed)
    if len(tensors) == 1:
        return dict(case=case, w=tensors[0])
    # a model-level program keeps the tensor list, its workspace and its output arrays
    tl = pwlq.TensorList(tensors, case["mode"])
    st = dict(case=case, tl=tl)
    bits = case["bits"]
    if case["kind"] == "select":
        nbytes = max(pwlq.select_list_workspace_bytes(tl), pwlq.mse_list_workspace_bytes(tl),
                     pwlq.quantize_list_workspace_bytes(tl, bits))
        packed, hat = True, False
        st["sel"] = (torch.empty(tl.n_groups, dtype=torch.float32, device="cuda"),
                     torch.empty(tl.n_groups, dtype=torch.float32, device="cuda"))
        st["mse"] = torch.empty(tl.n_groups, dtype=torch.float64, device="cuda")
    else:
        nbytes = max(pwlq.search_list_workspace_bytes(tl, bits, case["n_cand"]),
                     pwlq.quantize_list_workspace_bytes(tl, bits))
        packed, hat = case["out"] != "bytes", case["out"] == "packed_hat"
        st["found"] = pwlq.alloc_search_outputs(tl.n_groups, "cuda")
    st["workspace"] = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
    if packed:
        st["layout"] = pwlq.PackedLayout(tl, bits)
        # cleared once: the bytes between two streams belong to nobody
        st["out"] = (torch.zeros(st["layout"].code_bytes, dtype=torch.uint8, device="cuda"),
                     torch.zeros(st["layout"].flag_bytes, dtype=torch.uint8, device="cuda"),
                     torch.empty(tl.n_elements, dtype=torch.float32, device="cuda") if hat else None)
    else:
        st["out"] = pwlq.alloc_quantize_outputs(tl.n_elements, "cuda")
    return st


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def _run_layer(case, w):
    """One tensor, through the calls that allocate their outputs."""
    bits, mode = case["bits"], case["mode"]
    if case["kind"] == "select":
        p, m = pwlq.select_analytic(w, case["selector"], mode)
        found = dict(p_star=p, m=m, mse=pwlq.mse(w, bits, p, m, mode))
        out = "packed"
    else:
        found = pwlq.search(w, bits, case["n_cand"], mode, fast=case["fast"])
        out = case["out"]
    if out == "bytes":
        q = pwlq.quantize(w, bits, found["p_star"], found["m"], mode)
    else:
        q = pwlq.quantize_packed(w, bits, found["p_star"], found["m"], mode, want_w_hat=out == "packed_hat")
    return dict(found, codes=q[0], flags=q[1], w_hat=q[2])


def run(state):
    case = state["case"]
    if case["kind"] == "linear":
        y, acc = pwlq.linear_i8(state["xq"], S_X, Z_X, state["codes"], state["flags"], case["N"], case["bits"],
                                state["p"], state["m"], want_acc=case["sums"], workspace=state["workspace"],
                                out=state["out"])
        return dict(y=y, acc=acc)
    if "w" in state:
        return _run_layer(case, state["w"])
    tl, bits, ws = state["tl"], case["bits"], state["workspace"]
    if case["kind"] == "select":
        p, m = pwlq.select_analytic_list(tl, case["selector"], ws, state["sel"])
        found = dict(p_star=p, m=m, mse=pwlq.mse_list(tl, bits, p, m, ws, state["mse"]))
    else:
        found = pwlq.search_list(tl, bits, case["n_cand"], ws, state["found"], case["fast"])
    if "layout" in state:
        c, f, h, _ = pwlq.quantize_packed_list(tl, bits, found["p_star"], found["m"], state["layout"],
                                               state["out"][2] is not None, ws, state["out"])
    else:
        c, f, h = pwlq.quantize_list(tl, bits, found["p_star"], found["m"], ws, state["out"])
    return dict(found, codes=c, flags=f, w_hat=h)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    bits = case["bits"]
    if case["kind"] == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        # activations, codes and region bits, parameters, outputs; the integer products of
        # the two regions that keep their own step (three sums where they are wanted apart)
        sums = 3 if case["sums"] else 2
        return dict(bytes=M * K + N * K * (bits + 1) / 8 + 8 * N + M * N * (16 if case["sums"] else 4),
                    flops=2.0 * M * N * K * sums)
    shapes = _shapes(case)
    elements = sum(C * K for C, K in shapes)
    groups = sum(C for C, _ in shapes) if case["mode"] == PER_CHANNEL else len(shapes)
    # the weights once for the breakpoints, once more to quantize them with the result; the outputs
    out = case.get("out", "packed")
    written = 6.0 if out == "bytes" else (bits + 1) / 8 + (4.0 if out == "packed_hat" else 0.0)
    moved = elements * (8.0 + written) + 20.0 * groups
    if case["kind"] == "select":
        return dict(bytes=moved + 4.0 * elements, flops=10.0 * elements)     # read a third time for the error
    if case["fast"]:
        # a cumulative count and sum per level and candidate, and the sums themselves
        return dict(bytes=moved, flops=groups * case["n_cand"] * (2 ** bits - 1) * 4.0 + 5.0 * elements)
    # every weight at every candidate: position in steps, round, error, square and sum
    return dict(bytes=moved, flops=5.0 * elements * case["n_cand"])


def tolerance(case):
    if case["kind"] == "linear":
        # whole sums are exact; y is a few 32-bit roundings of terms of its own size:
        # measured 5e-8 against 64 bits over the range of sizes
        return dict(rel=2e-7, max=4e-6, differ=0.0)
    if case["kind"] == "select":
        # the breakpoint is a 64-bit root rounded to 32 bits: one unit in the last place
        # (1.2e-7 of a value), and a code in ten million that sits on the moved boundary
        return dict(rel=1.2e-7, max=1e-6, differ=1e-6)
    # codes are decided in the same 32-bit steps by every implementation and the error is
    # summed in 64 bits (up to two million terms): the order of the sum is all that is free
    return dict(rel=1e-12, max=1e-11, differ=0.0)


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------
def _groups(w, mode):
    a = w.double().abs()
    return a if mode == PER_CHANNEL else a.reshape(1, -1)


def _errors(a, p, m, L):
    """Squared error summed over each row of magnitudes a[G, K] for breakpoints p[G, k]."""
    best = torch.empty_like(p)
    for g in range(0, a.shape[0], max(1, 50_000_000 // (a.shape[1] * p.shape[1]))):
        h = min(a.shape[0], g + max(1, 50_000_000 // (a.shape[1] * p.shape[1])))
        pp, aa = p[g:h, :, None], a[g:h, None, :]
        tail = aa > pp
        z = torch.where(tail, pp, 0.0)
        s = torch.where(tail, (m[g:h, None, None] - pp) / L, pp / L)
        x = aa - z
        del z, tail
        e = x.div(s).round_().clamp_(max=L).mul_(s).sub_(x)
        e = torch.nan_to_num_(e, nan=0.0, posinf=0.0, neginf=0.0)       # a group of zeros has no step
        best[g:h] = e.square_().sum(-1)
    return best


def _curve(a, m, n, L):
    """Squared error of every candidate, [G, n]."""
    G, K = a.shape
    k = torch.arange(1, n + 1, device=a.device, dtype=torch.float64)
    p = m[:, None] * (k / n)
    if K <= 16384:
        step = max(1, 50_000_000 // K)
        return torch.cat([_errors(a, p[:, i:i + step].contiguous(), m, L) for i in range(0, n, step)], 1)
    total = torch.zeros((G, n), dtype=torch.float64, device=a.device)
    for at in range(0, K, 16384):
        total += _curve_part(a[:, at:at + 16384].contiguous(), p, m, L)
    return total


def _curve_part(a, p, m, L):
    step = max(1, 50_000_000 // a.shape[1])
    return torch.cat([_errors(a, p[:, i:i + step].contiguous(), m, L) for i in range(0, p.shape[1], step)], 1)


def _select(a, m, selector):
    """Section 5.1's fit, or the root of Eq.8 in (0, m/2) by bisection."""
    sigma, beta = a.square().mean(1).sqrt(), a.mean(1)
    if selector == pwlq.GAUSS_FIT:
        return torch.minimum((sigma * torch.log(0.8614 * m / sigma + 0.6079)).clamp_min(0.0), m)

    def slope(p):
        if selector == pwlq.LAPLACE_SOLVE:
            z = -torch.expm1(-m / beta)
            F = 0.5 - 0.5 * torch.expm1(-p / beta) / z
            f = torch.exp(-p / beta) / (2.0 * beta) / z
        else:
            r = math.sqrt(0.5)
            z = torch.erf(m / sigma * r)
            F = 0.5 + 0.5 * torch.erf(p / sigma * r) / z
            f = torch.exp(-0.5 * (p / sigma) ** 2) / (sigma * math.sqrt(2 * math.pi)) / z
        return p - 2 * m + 2 * m * F + m * (2 * p - m) * f

    lo, hi = torch.zeros_like(m), 0.5 * m
    end = slope(hi) <= 0
    for _ in range(100):
        mid = 0.5 * (lo + hi)
        up = slope(mid) > 0
        hi, lo = torch.where(up, mid, hi), torch.where(up, lo, mid)
    return torch.where(end, 0.5 * m, 0.5 * (lo + hi))


def exact(case, seed):
    bits = case["bits"]
    L = float(2 ** (bits - 1) - 1)
    if case["kind"] == "linear":
        xq, code, tail, p, m = _linear_inputs(case, seed)
        p, m = p.double()[:, None], m.double()[:, None]
        mag = (code & int(L)).double()
        w = torch.where(tail, p + mag * ((m - p) / L), mag * (p / L))
        # a tail weight carries its sign on the offset too, whatever its code
        w = torch.where((code >> (bits - 1)) > 0, -w, w)
        # the activations' step and offset are 32-bit numbers
        s_x, z_x = (float(torch.tensor(v, dtype=torch.float32)) for v in (S_X, Z_X))
        return dict(y=(xq.double() * s_x + z_x) @ w.t().contiguous(), acc=None)
    found = dict(p_star=[], m=[], mse=[])
    hats = []
    want_hat = case.get("out", "packed") != "packed"
    for w in _tensors(case, seed):
        a = _groups(w, case["mode"])
        m = a.amax(1)
        if case["kind"] == "select":
            p = _select(a, m, case["selector"])
            sse = sum(_errors(a[:, i:i + 16384].contiguous(), p[:, None], m, L) for i in range(0, a.shape[1], 16384))[:, 0]
        else:
            sse, k = _curve(a, m, case["n_cand"], L).min(1)
            p = m * ((k + 1).double() / case["n_cand"])
        found["p_star"].append(p)
        found["m"].append(m)
        found["mse"].append(sse / a.shape[1])
        if want_hat:
            tail = a > p[:, None]
            z = torch.where(tail, p[:, None], 0.0)
            s = torch.where(tail, ((m - p) / L)[:, None], (p / L)[:, None])
            v = ((a - z) / s).round_().clamp_(max=L) * s + z
            hats.append((torch.sign(w.double()).reshape(v.shape) * v).reshape(-1))
    got = {name: torch.cat(v) for name, v in found.items()}
    if case["kind"] == "search":
        got["k_star"] = None
    hat = torch.cat(hats) if want_hat else None
    return dict(got, codes=None, flags=None, w_hat=hat)
