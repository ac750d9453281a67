"""Timed cases of the library's main paths, through the entry points of `paper_2109_03513_amd`.

The cases follow a program's day: it calibrates weights (the aligner over a caller's grid,
then the projection), quantizes activations with a plan, contracts codes (GEMM, packed fully
connected layer, convolutions with their fused epilogues, depthwise and pointwise layers, a
network stem) and runs a whole ResNet18 forward pass replayed as a HIP graph.

    listed()             the named cases
    draw(rng)            one more case from the same ranges
    prepare(case, seed)  inputs, plans, workspaces and output buffers, on the GPU
    run(state)           one pass
    work(case)           bytes and operations the pass cannot do without
    tolerance(case)      how far another correct implementation may be off
    exact(case, seed)    what run() returns, from plain torch in 64 bits

Formats are (n, k_sig) as in include/esb.h.  Everything the library returns here is fixed by
its definition to the bit (integers, codes, correctly rounded fp32 operations in a stated
order), except the aligner's fp64 objective.
"""
import math

import torch

from paper_2109_03513_amd import esb, resnet18, workloads

G = 64           # candidate scales of every aligner search


def listed():
    return [
        # the classifier's input of ResNet18 at batch 64: the smallest quantization of a
        # forward, all latency
        dict(name="quantize_features", kind="quantize", len=64 * 512, n=5, ks=3, dist="relu"),
        # a 56x56x64 activation at batch 64: the largest layer input of that forward
        dict(name="quantize_activation", kind="quantize", len=64 * 56 * 56 * 64, n=5, ks=3,
             dist="relu"),
        # weights of a fully connected layer (9216 -> 4096), calibrated once per model: the
        # aligner over a grid given as is, with its objective, then the codes
        dict(name="calibrate_fc_weights", kind="calibrate", len=4096 * 9216, n=3, ks=1),
        # a large square product of 4-bit codes
        dict(name="gemm_4096_e2m1", kind="gemm", M=4096, N=4096, K=4096, nA=4, ksA=2, nB=4, ksB=2,
             layout="nk"),
        # a product with ragged rows and columns (tokens or positions that fill no tile),
        # 5-bit codes
        dict(name="gemm_ragged", kind="gemm", M=1999, N=1000, K=2048, nA=5, ksA=3, nB=5, ksB=3,
             layout="nk"),
        # AlexNet's first fully connected layer at batch 128 with its weights packed once
        dict(name="fc_packed_b128", kind="fc", M=128, N=4096, K=9216, nA=3, ksA=2, nB=3, ksB=1),
        # one image through a 64-channel 3x3 layer: single-request latency
        dict(name="conv3x3_b1", kind="conv", N=1, H=56, W=56, C=64, K=64, R=3, stride=1, n=4, ks=2,
             post="plain"),
        # ResNet18's first stage at batch 64: the second convolution of a block (residual, ReLU
        # and the next layer's maximum in the epilogue)
        dict(name="conv3x3_l1_b64", kind="conv", N=64, H=56, W=56, C=64, K=64, R=3, stride=1, n=5,
             ks=3, post="residual"),
        # ResNet18's last stage at batch 64 with fixed scales: the epilogue hands over codes
        dict(name="conv3x3_l4_b64", kind="conv", N=64, H=7, W=7, C=512, K=512, R=3, stride=1, n=5,
             ks=3, post="codes"),
        # MobileNetV2's inverted residual at 56x56, batch 32, fixed scales: pointwise 24 -> 144,
        # depthwise 3x3, pointwise 144 -> 24
        dict(name="mobile_block_b32", kind="mobile", N=32, side=56, C=24, expand=6, n=5, ks=3),
        # a 7x7 / stride 2 stem with its ReLU and max pool on 224x224 RGB, batch 64
        dict(name="stem_b64", kind="stem", N=64, side=224, n=5, ks=3),
        # the whole network at batch 64, every layer quantized by its own search on the device
        dict(name="resnet18_b64", kind="resnet18", N=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["quantize", "quantize", "calibrate", "gemm", "gemm", "fc", "conv", "conv",
                       "conv", "mobile", "stem", "resnet18"])
    fmt = rng.choice([(5, 3), (5, 3), (4, 2), (3, 2), (6, 3)])
    if kind == "quantize":
        return dict(kind=kind, len=_log(rng, 1 << 12, 64 * 56 * 56 * 64), n=fmt[0], ks=fmt[1],
                    dist=rng.choice(["relu", "normal"]))
    if kind == "calibrate":
        n, ks = rng.choice([(3, 1), (4, 2), (5, 3)])
        return dict(kind=kind, len=_log(rng, 1 << 12, 4096 * 9216), n=n, ks=ks)
    if kind == "gemm":
        M, N = _log(rng, 16, 4096), _log(rng, 64, 4096)
        K = rng.choice([_log(rng, 64, 4096), 64 * _log(rng, 1, 64)])
        return dict(kind=kind, M=M, N=N, K=K, nA=fmt[0], ksA=fmt[1], nB=fmt[0], ksB=fmt[1],
                    layout=rng.choice(["nk", "nk", "nk", "kn"]))
    if kind == "fc":
        (nA, ksA), (nB, ksB) = rng.choice([((3, 2), (3, 1)), ((4, 2), (4, 2)), ((4, 2), (3, 2))])
        return dict(kind=kind, M=_log(rng, 1, 256), N=_log(rng, 512, 4608),
                    K=32 * _log(rng, 16, 288), nA=nA, ksA=ksA, nB=nB, ksB=ksB)
    if kind == "conv":
        # a network's layers: channels grow as the side shrinks
        H = rng.randint(7, 56)
        top = max(1, min(8, 448 // H // 2 if H > 14 else 8))
        C, K = 64 * rng.randint(1, top), 64 * rng.randint(1, top)
        if rng.random() < 0.25:
            C, K = 16 * rng.randint(1, 4 * top), 8 * rng.randint(2, 8 * top)
        n, ks = rng.choice([(5, 3), (5, 3), (4, 2)])
        stride = rng.choice([1, 1, 1, 2])
        return dict(kind=kind, N=_log(rng, 1, 64), H=H, W=max(7, H + rng.randint(-3, 3)), C=C, K=K,
                    R=rng.choice([3, 3, 1]), stride=stride, n=n, ks=ks,
                    post=rng.choice(["plain", "relu", "residual", "codes"]))
    if kind == "mobile":
        C = 8 * rng.randint(2, 12)
        return dict(kind=kind, N=_log(rng, 1, 32), side=rng.randint(7, 56 if C <= 32 else 28), C=C,
                    expand=6, n=5, ks=3)
    if kind == "stem":
        return dict(kind=kind, N=_log(rng, 1, 64), side=rng.randint(64, 224), n=5, ks=3)
    return dict(kind="resnet18", N=rng.randint(1, 64))


# ---- the format, in plain torch -------------------------------------------------------------


def _magnitudes(n, ks):
    """(value, code) of the non-negative codes, ascending by value."""
    k = ks - 1
    top = (1 << (n - 1 - k)) - 1
    both = []
    for m in range(1 << (n - 1)):
        e, f = m >> k, (m & ((1 << k) - 1)) / (1 << k)
        both.append((f if e == top else 2.0 ** e * (1 + f), m))
    both.sort()
    return both


def _cmax(n, ks):
    return _magnitudes(n, ks)[-1][0]


def _values_of(codes, n, ks):
    """q of each code, float64."""
    table = torch.zeros(256, dtype=torch.float64)
    for v, m in _magnitudes(n, ks):
        for c in range(m, 256, 1 << n):
            table[c] = v
            table[c | (1 << (n - 1))] = -v
    return table.to(codes.device)[codes.long()]


def _nearest(x, alpha, n, ks):
    """(index of the nearest magnitude) of fl32(x / alpha); alpha: a device scalar."""
    mags = [v for v, _ in _magnitudes(n, ks)]
    mids = torch.tensor([(a + b) / 2 for a, b in zip(mags, mags[1:])], dtype=torch.float32,
                        device=x.device)
    return torch.bucketize((x / alpha).abs(), mids, right=True)


def _codes_of(x, alpha, n, ks):
    """The codes of x under the device scalar alpha."""
    mag = torch.tensor([m for _, m in _magnitudes(n, ks)], dtype=torch.uint8, device=x.device)
    i = _nearest(x, alpha, n, ks)
    sign = ((x < 0) & (i > 0)).to(torch.uint8) << (n - 1)
    return mag[i] | sign


def _aligned(x, n, ks, grid):
    """(alpha, D) of the aligner's search: sums in 64 bits, the least index of the least D."""
    q = torch.tensor([v for v, _ in _magnitudes(n, ks)], dtype=torch.float64, device=x.device)
    D = torch.zeros(grid.numel(), dtype=torch.float64, device=x.device)
    for j in range(grid.numel()):
        for part in x.reshape(-1).split(1 << 24):
            a = grid[j:j + 1]
            d = part.abs().double() - a.double() * q[_nearest(part, a, n, ks)]
            D[j] += (d * d).sum()
    return grid[D.argmin()].reshape(1), D


def _planned_grid(n, ks, xmax):
    """The candidates 2^E c_j, E the binary exponent of the device scalar xmax."""
    f = torch.from_numpy(workloads.maxabs_grid_factors(_cmax(n, ks), G)).to(xmax.device)
    _, E = torch.frexp(xmax)
    return torch.ldexp(f, E)


def _conv64(xq, wq, stride, pad):
    """Cross-correlation of NHWC xq with KRSC wq (groups = C when wq has one channel and more
    filters than that share no channel), float64."""
    N, H, W, C = xq.shape
    K, R, S, Cg = wq.shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    xp = torch.zeros((N, H + 2 * pad, W + 2 * pad, C), dtype=torch.float64, device=xq.device)
    xp[:, pad:pad + H, pad:pad + W] = xq
    acc = torch.zeros((N, P, Q, K), dtype=torch.float64, device=xq.device)
    for r in range(R):
        for s in range(S):
            tap = xp[:, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride]
            if Cg == 1 and C > 1:
                acc += tap * wq[:, r, s, 0]
            else:
                acc += (tap.reshape(-1, C) @ wq[:, r, s].t().contiguous()).reshape(acc.shape)
    return acc


def _y32(acc, aX, aW):
    """fl32(s fl32(acc)) for acc in units of q: a power of two away from the integer sums."""
    return acc.float() * (aX * aW)


# ---- inputs ---------------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, shape, std=1.0):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std


def _operand(g, shape, n, ks, relu):
    """Codes of normal (weights) or rectified normal (activations) data clipped at 3 sigma, and
    their scale."""
    x = _normal(g, shape)
    alpha = torch.full((1,), 3.0 / _cmax(n, ks), dtype=torch.float32, device="cuda")
    return _codes_of(x.relu() if relu else x, alpha, n, ks), alpha


def _out_alpha(red, n, ks):
    """A scale for outputs that sum `red` products of rectified and normal unit data: C at three
    standard deviations."""
    return torch.full((1,), 3.0 * math.sqrt(red / 2) / _cmax(n, ks), dtype=torch.float32,
                      device="cuda")


def _bytes(n):
    return torch.empty(max(int(n), 1), dtype=torch.uint8, device="cuda")


def _pads(c):
    return c["R"] // 2


def _conv_out(c):
    p = _pads(c)
    return esb.conv_out_hw(c["H"], c["W"], c["R"], c["R"], (c["stride"],) * 2, (p, p))


def _resnet_inputs(c, seed):
    g = _gen(seed)
    shapes = [(name, (cout, k, k, cin), k * k * cin)
              for name, cin, cout, k, _, _ in workloads.RESNET18_CONVS] + [("fc", (1000, 512), 512)]
    weights = {name: _normal(g, shape, math.sqrt(2.0 / fan)) for name, shape, fan in shapes}
    return weights, _normal(g, (c["N"], 224, 224, 3))


def _inputs(c, seed):
    """The tensors of a case, from the seed alone."""
    g, kind = _gen(seed), c["kind"]
    if kind == "quantize":
        x = _normal(g, (c["len"],), 0.5 + (seed % 7))
        return dict(x=x.relu_() if c["dist"] == "relu" else x)
    if kind == "calibrate":
        return dict(x=_normal(g, (c["len"],), 0.01))
    if kind in ("gemm", "fc"):
        A, aA = _operand(g, (c["M"], c["K"]), c["nA"], c["ksA"], True)
        shape = (c["K"], c["N"]) if c.get("layout") == "kn" else (c["N"], c["K"])
        B, aB = _operand(g, shape, c["nB"], c["ksB"], False)
        return dict(A=A, aA=aA, B=B, aB=aB)
    n, ks = c["n"], c["ks"]
    if kind == "conv":
        x, aX = _operand(g, (c["N"], c["H"], c["W"], c["C"]), n, ks, True)
        w, aW = _operand(g, (c["K"], c["R"], c["R"], c["C"]), n, ks, False)
        d = dict(x=x, aX=aX, w=w, aW=aW)
        red = c["R"] * c["R"] * c["C"]
        if c["post"] == "residual":
            P, Q = _conv_out(c)
            d["residual"] = _normal(g, (c["N"], P, Q, c["K"]), math.sqrt(red / 2)).relu_()
        if c["post"] == "codes":
            d["aY"] = _out_alpha(red, n, ks)
        return d
    if kind == "mobile":
        C, E = c["C"], c["C"] * c["expand"]
        x, aX = _operand(g, (c["N"], c["side"], c["side"], C), n, ks, True)
        w1, aW1 = _operand(g, (E, 1, 1, C), n, ks, False)
        w2, aW2 = _operand(g, (E, 3, 3, 1), n, ks, False)
        w3, aW3 = _operand(g, (C, 1, 1, E), n, ks, False)
        a1 = _out_alpha(C, n, ks)
        return dict(x=x, aX=aX, w1=w1, aW1=aW1, w2=w2, aW2=aW2, w3=w3, aW3=aW3, a1=a1,
                    a2=a1 * math.sqrt(9.0 / 2))
    if kind == "stem":
        x, aX = _operand(g, (c["N"], c["side"], c["side"], 3), n, ks, False)
        w, aW = _operand(g, (64, 7, 7, 3), n, ks, False)
        return dict(x=x, aX=aX, w=w, aW=aW)
    raise ValueError(kind)


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "resnet18":
        weights, x = _resnet_inputs(c, seed)
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            model = resnet18.ResNet18ESB({k: v.cpu().numpy() for k, v in weights.items()}, c["N"],
                                         stream=stream)
            model.forward(x)
            stream.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                logits = model.forward(x)
        torch.cuda.current_stream().wait_stream(stream)
        return dict(case=c, model=model, x=x, graph=graph, logits=logits)
    s = dict(case=c, **_inputs(c, seed))
    if kind == "quantize":
        n, ks = c["n"], c["ks"]
        factors = torch.from_numpy(workloads.maxabs_grid_factors(_cmax(n, ks), G)).cuda()
        s["plan"] = esb.esb_dda_plan(n, ks, factors)
        s["xmax"] = s["x"].abs().max().reshape(1)
        s["ws"] = _bytes(esb.esb_dda_workspace_size(c["len"], n, ks, G))
        s["alpha"] = torch.empty(1, dtype=torch.float32, device="cuda")
        s["codes"] = torch.empty_like(s["x"], dtype=torch.uint8)
    elif kind == "calibrate":
        s["grid"] = torch.from_numpy(workloads.scale_grid(0.01, G)).cuda()
        s["ws"] = _bytes(esb.esb_dda_workspace_size(c["len"], c["n"], c["ks"], G))
        s["alpha"] = torch.empty(1, dtype=torch.float32, device="cuda")
        s["D"] = torch.empty(G, dtype=torch.float64, device="cuda")
        s["codes"] = torch.empty_like(s["x"], dtype=torch.uint8)
    elif kind in ("gemm", "fc"):
        size = (esb.esb_gemm_workspace_size if kind == "gemm"
                else esb.esb_gemm_packed_workspace_size)
        s["ws"] = _bytes(size(c["M"], c["N"], c["K"], c["nA"], c["ksA"], c["nB"], c["ksB"]))
        s["y"] = torch.empty((c["M"], c["N"]), dtype=torch.float32, device="cuda")
        if kind == "fc":
            s["packed"] = esb.esb_pack(s["B"], c["nB"], c["ksB"])
    elif kind == "conv":
        p, P, Q = _pads(c), *_conv_out(c)
        s["ws"] = _bytes(esb.esb_conv2d_workspace_size(
            s["x"].shape, s["w"].shape, c["n"], c["ks"], c["n"], c["ks"],
            stride=(c["stride"],) * 2, pad=(p, p)))
        kind_of_y = torch.uint8 if c["post"] == "codes" else torch.float32
        s["y"] = torch.empty((c["N"], P, Q, c["K"]), dtype=kind_of_y, device="cuda")
        s["absmax"] = torch.zeros(1, dtype=torch.float32, device="cuda")
    elif kind == "mobile":
        N, side, C, E = c["N"], c["side"], c["C"], c["C"] * c["expand"]
        n, ks = c["n"], c["ks"]
        need = max(esb.esb_conv2d_workspace_size((N, side, side, i), (o, 1, 1, i), n, ks, n, ks)
                   for i, o in ((C, E), (E, C)))
        s["ws"] = _bytes(need)
        s["c1"], s["c2"] = (torch.empty((N, side, side, E), dtype=torch.uint8, device="cuda")
                            for _ in range(2))
        s["y"] = torch.empty((N, side, side, C), dtype=torch.float32, device="cuda")
    elif kind == "stem":
        P, _ = esb.conv_out_hw(c["side"], c["side"], 7, 7, (2, 2), (3, 3))
        PP, _ = esb.conv_out_hw(P, P, 3, 3, (2, 2), (1, 1))
        s["ws"] = _bytes(esb.esb_conv2d_relu_maxpool_workspace_size(
            s["x"].shape, s["w"].shape, c["n"], c["ks"], c["n"], c["ks"]))
        s["y"] = torch.empty((c["N"], PP, PP, 64), dtype=torch.float32, device="cuda")
        s["absmax"] = torch.zeros(1, dtype=torch.float32, device="cuda")
    return s


# ---- one pass -------------------------------------------------------------------------------


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "resnet18":
        s["graph"].replay()
        return [s["logits"]]
    if kind == "quantize":
        esb.esb_quantize_planned(s["x"], c["n"], c["ks"], s["plan"], G, s["xmax"],
                                 alpha_out=s["alpha"], codes=s["codes"], workspace=s["ws"],
                                 want_D=False)
        return [s["alpha"], s["codes"]]
    if kind == "calibrate":
        esb.esb_dda_align(s["x"], c["n"], c["ks"], s["grid"], alpha_out=s["alpha"], D_out=s["D"],
                          workspace=s["ws"])
        esb.esb_project(s["x"], s["alpha"], c["n"], c["ks"], codes=s["codes"])
        return [s["alpha"], s["D"], s["codes"]]
    if kind == "gemm":
        esb.esb_gemm(s["A"], c["nA"], c["ksA"], s["aA"], s["B"], c["nB"], c["ksB"], s["aB"],
                     b_layout=esb.ESB_B_KN if c["layout"] == "kn" else esb.ESB_B_NK, y=s["y"],
                     want_acc=False, workspace=s["ws"])
        return [s["y"]]
    if kind == "fc":
        esb.esb_gemm_packed(s["A"], c["nA"], c["ksA"], s["aA"], s["packed"], c["nB"], c["ksB"],
                            s["aB"], s["ws"], y=s["y"], want_acc=False)
        return [s["y"]]
    n, ks = c["n"], c["ks"]
    if kind == "conv":
        st, pd = (c["stride"],) * 2, (_pads(c),) * 2
        if c["post"] == "plain":
            esb.esb_conv2d(s["x"], n, ks, s["aX"], s["w"], n, ks, s["aW"], stride=st, pad=pd,
                           y=s["y"], want_acc=False, workspace=s["ws"])
            return [s["y"]]
        if c["post"] == "codes":
            esb.esb_conv2d_post(s["x"], n, ks, s["aX"], s["w"], n, ks, s["aW"], s["aY"], n, ks,
                                relu=True, stride=st, pad=pd, codes=s["y"], workspace=s["ws"])
            return [s["y"]]
        esb.esb_conv2d_post(s["x"], n, ks, s["aX"], s["w"], n, ks, s["aW"], None, n, ks,
                            residual=s.get("residual"), relu=True, stride=st, pad=pd,
                            want_codes=False, y=s["y"], absmax=s["absmax"], workspace=s["ws"])
        return [s["y"], s["absmax"]]
    if kind == "mobile":
        E = c["C"] * c["expand"]
        esb.esb_conv2d_post(s["x"], n, ks, s["aX"], s["w1"], n, ks, s["aW1"], s["a1"], n, ks,
                            relu=True, codes=s["c1"], workspace=s["ws"])
        esb.esb_conv2d_post(s["c1"], n, ks, s["a1"], s["w2"], n, ks, s["aW2"], s["a2"], n, ks,
                            relu=True, pad=(1, 1), groups=E, codes=s["c2"])
        esb.esb_conv2d(s["c2"], n, ks, s["a2"], s["w3"], n, ks, s["aW3"], y=s["y"],
                       want_acc=False, workspace=s["ws"])
        return [s["c1"], s["c2"], s["y"]]
    if kind == "stem":
        esb.esb_conv2d_relu_maxpool(s["x"], n, ks, s["aX"], s["w"], n, ks, s["aW"], y=s["y"],
                                    absmax=s["absmax"], workspace=s["ws"])
        return [s["y"], s["absmax"]]
    raise ValueError(kind)


# ---- what a pass cannot do without ----------------------------------------------------------


def work(case):
    c, kind = case, case["kind"]
    if kind in ("quantize", "calibrate"):
        return dict(bytes=5.0 * c["len"], flops=0.0)
    if kind in ("gemm", "fc"):
        b = c["N"] * c["K"] / (2 if kind == "fc" else 1)
        return dict(bytes=c["M"] * c["K"] + b + 4.0 * c["M"] * c["N"],
                    flops=2.0 * c["M"] * c["N"] * c["K"])
    if kind == "conv":
        P, Q = _conv_out(c)
        out = c["N"] * P * Q * c["K"]
        red = c["R"] * c["R"] * c["C"]
        per = {"plain": 4, "relu": 4, "residual": 8, "codes": 1}[c["post"]]
        return dict(bytes=c["N"] * c["H"] * c["W"] * c["C"] + c["K"] * red + float(per) * out,
                    flops=2.0 * out * red)
    if kind == "mobile":
        px, C, E = c["N"] * c["side"] ** 2, c["C"], c["C"] * c["expand"]
        return dict(bytes=px * (C + 4.0 * E + 4 * C) + 2 * C * E + 9 * E,
                    flops=2.0 * px * (2 * C * E + 9 * E))
    if kind == "stem":
        P = (c["side"] - 1) // 2 + 1
        PP = (P - 1) // 2 + 1
        return dict(bytes=c["N"] * (3.0 * c["side"] ** 2 + 4 * 64 * PP * PP) + 147 * 64,
                    flops=2.0 * c["N"] * P * P * 64 * 147)
    ops = 2.0 * 1000 * 512
    weights = 1000 * 512
    for name, cin, cout, k, st, pd in workloads.RESNET18_CONVS:
        side = resnet18.input_side(name)
        P, Q = esb.conv_out_hw(side, side, k, k, (st, st), (pd, pd))
        ops += 2.0 * P * Q * cout * k * k * cin
        weights += cout * k * k * cin
    return dict(bytes=c["N"] * (4.0 * 224 * 224 * 3 + 4000) + weights, flops=ops * c["N"])


def tolerance(case):
    # D's fp64 sums in another order differ by a few 1e-13 relative; alpha and the codes are the
    # same as long as no two candidates' D lie that close
    return dict(rel=1e-12, max=1e-11) if case["kind"] == "calibrate" else "exact"


# ---- the same in 64 bits --------------------------------------------------------------------


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "resnet18":
        return _exact_resnet18(c, seed)
    s = _inputs(c, seed)
    if kind in ("quantize", "calibrate"):
        n, ks = c["n"], c["ks"]
        grid = (_planned_grid(n, ks, s["x"].abs().max().reshape(1)) if kind == "quantize"
                else torch.from_numpy(workloads.scale_grid(0.01, G)).cuda())
        alpha, D = _aligned(s["x"], n, ks, grid)
        codes = _codes_of(s["x"], alpha, n, ks)
        return [alpha, codes] if kind == "quantize" else [alpha, D, codes]
    if kind in ("gemm", "fc"):
        A, B = _values_of(s["A"], c["nA"], c["ksA"]), _values_of(s["B"], c["nB"], c["ksB"])
        acc = A @ (B if c.get("layout") == "kn" else B.t().contiguous())
        return [acc * (s["aA"].double() * s["aB"].double())]
    n, ks = c["n"], c["ks"]
    xq = _values_of(s["x"], n, ks)
    if kind == "conv":
        acc = _conv64(xq, _values_of(s["w"], n, ks), c["stride"], _pads(c))
        if c["post"] == "codes":
            return [_codes_of(_y32(acc, s["aX"], s["aW"]).relu(), s["aY"], n, ks)]
        y = acc * (s["aX"].double() * s["aW"].double())
        if c["post"] == "plain":
            return [y]
        if c["post"] == "residual":
            y = y + s["residual"].double()
        y = y.relu()
        return [y, y.max().reshape(1)]
    if kind == "mobile":
        c1 = _codes_of(_y32(_conv64(xq, _values_of(s["w1"], n, ks), 1, 0), s["aX"],
                            s["aW1"]).relu(), s["a1"], n, ks)
        c2 = _codes_of(_y32(_conv64(_values_of(c1, n, ks), _values_of(s["w2"], n, ks), 1, 1),
                            s["a1"], s["aW2"]).relu(), s["a2"], n, ks)
        acc = _conv64(_values_of(c2, n, ks), _values_of(s["w3"], n, ks), 1, 0)
        return [c1, c2, acc * (s["a2"].double() * s["aW3"].double())]
    acc = _conv64(xq, _values_of(s["w"], n, ks), 2, 3)
    y = _pool64((acc * (s["aX"].double() * s["aW"].double())).relu())
    return [y, y.max().reshape(1)]


def _pool64(z):
    """3x3 / stride 2 / pad 1 max pool of rectified NHWC values."""
    N, P, Q, K = z.shape
    zp = torch.zeros((N, P + 2, Q + 2, K), dtype=z.dtype, device=z.device)
    zp[:, 1:-1, 1:-1] = z
    PP, QQ = (P - 1) // 2 + 1, (Q - 1) // 2 + 1
    taps = [zp[:, r:r + 2 * PP - 1:2, s:s + 2 * QQ - 1:2] for r in range(3) for s in range(3)]
    out = taps[0]
    for t in taps[1:]:
        out = torch.maximum(out, t)
    return out


def _exact_resnet18(c, seed):
    """The network layer by layer: exact sums, the fp32 roundings that its definition puts
    between layers, the logits in 64 bits."""
    n, ks = resnet18.N_BITS, resnet18.K_SIG
    weights, x = _resnet_inputs(c, seed)

    def quantized(t):
        t = t.contiguous()
        alpha, _ = _aligned(t, n, ks, _planned_grid(n, ks, t.abs().max().reshape(1)))
        return _values_of(_codes_of(t, alpha, n, ks), n, ks), alpha

    shape = {name: (st, pd) for name, _, _, _, st, pd in workloads.RESNET18_CONVS}
    wq = {name: quantized(w) for name, w in weights.items()}

    def conv(name, q):
        return _y32(_conv64(q[0], wq[name][0], *shape[name]), q[1], wq[name][1])

    a = _pool64(conv("conv1", quantized(x)).relu())
    for stage in (1, 2, 3, 4):
        for blk in (0, 1):
            p = "l%d.%d." % (stage, blk)
            q = quantized(a)
            mid = quantized(conv(p + "c1", q).relu())
            short = conv(p + "ds", q) if p + "ds" in wq else a
            a = (conv(p + "c2", mid) + short).relu()
    feat = a.double().sum(dim=(1, 2)).div(a.shape[1] * a.shape[2]).float()
    q = quantized(feat)
    return [(q[0] @ wq["fc"][0].t().contiguous()) * (q[1].double() * wq["fc"][1].double())]
