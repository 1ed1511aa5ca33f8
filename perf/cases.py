"""The work a user of this library has it do, as cases that can be timed and compared.

Every case is one pass through the public entry points of ``paper_2104_08314_amd.api`` on a layer
(or a chain of layers) of the kind the library is written for: non-pointwise convolution layers of
image networks on post-ReLU activation maps, fp32, one map per call or a batch.  Operations:

  layer    encoding + convolution of a layer in one call, how a layer runs at inference time
  encode   the encoding alone (with the previous layer's bias and ReLU on the way in, or without)
  conv     the convolution alone, over a map that was encoded before
  im2col   the dense comparator, fp32 or bf16 (weights converted per call or prepared once)
  chain    the convolution layers of a network one after the other, a method per layer

``listed()`` names twelve of them, ``draw()`` gives more of the same ranges: 16 to 512 channels and
kernels, maps of 7 to 64 rows and columns (up to 224 for a first layer of three channels), the
kernel shapes of residual and inception networks, 40 to 85 % zeros, 1 to 32 maps per call.
"""
import math
import statistics

import torch

from paper_2104_08314_amd import api

# kh, kw, stride, pad_h, pad_w of the layers in use (residual networks: 3 x 3 with stride 1 and 2;
# inception networks: 5 x 5, 1 x n and n x 1 layers padded so that the map keeps its size)
KERNELS = {
    "3x3": (3, 3, 1, 1, 1), "3x3s2": (3, 3, 2, 1, 1), "5x5": (5, 5, 1, 2, 2),
    "1x7": (1, 7, 1, 0, 3), "7x1": (7, 1, 1, 3, 0), "1x3": (1, 3, 1, 0, 1), "3x1": (3, 1, 1, 1, 0),
    "7x7s2": (7, 7, 2, 3, 3),
}
MAX_ELEMENTS = 32 * 128 * 56 * 56      # of an input: 32 maps of 128 channels at 56 x 56
MAX_FLOPS = 2 * 32 * 128 * 128 * 9 * 56 * 56
MAX_CHAIN_FLOPS = 1.2e11


def _layer(name, op, C, H, W, K, kernel, **more):
    case = {"name": name, "op": op, "C": C, "H": H, "W": W, "K": K, "kernel": kernel, "n": 1, "method": "cpo",
            "zeros": 0.6, "clustered": False, "dead": 0.05, "in_bits": 32, "relu": False, "layout": "chw", "precision": 0}
    case.update(more)
    return case


def _chain(name, **more):
    case = {"name": name, "op": "chain", "width": 64, "size": 56, "stages": 4, "depth": "3463", "n": 1, "methods": "cpo",
            "precision": 0}
    case.update(more)
    return case


def listed():
    return [
        # the smallest layer of the workloads: launches and host time count
        _layer("layer-cpo-16@28-x1", "layer", 16, 28, 28, 16, "3x3", zeros=0.5, dead=0.125),
        # the headline layer: one VGG-style map per call
        _layer("layer-cpo-128@56-x1", "layer", 128, 56, 56, 128, "3x3", zeros=0.6, dead=0.0),
        # a deep residual layer, clustered zeros, CPS with a compact map
        _layer("layer-cps-256@14-x1", "layer", 256, 14, 14, 256, "3x3", method="cps", zeros=0.7, clustered=True, dead=0.1,
               in_bits=16),
        # a strided layer between two stages, a small batch
        _layer("layer-cpo-128@56s2-x8", "layer", 128, 56, 56, 256, "3x3s2", n=8, zeros=0.65, clustered=True, dead=0.0),
        # a 1 x 7 layer of an inception network, CPS, a batch
        _layer("layer-cps-1x7-192@17-x16", "layer", 192, 17, 17, 192, "1x7", n=16, method="cps", zeros=0.7),
        # encoding alone, a serving batch
        _layer("encode-cpo-128@56-x32", "encode", 128, 56, 56, 128, "3x3", n=32, zeros=0.6, dead=0.0),
        # convolution alone over an encoded batch, 5 x 5
        _layer("conv-cpo-5x5-64@27-x32", "conv", 64, 27, 27, 192, "5x5", n=32, zeros=0.5, dead=0.0),
        # the dense comparator, as the per-layer selection times it
        _layer("im2col-f32-128@56-x1", "im2col", 128, 56, 56, 128, "3x3", zeros=0.6, dead=0.0),
        # the same layer as a bf16 product with prepared weights, a serving batch
        _layer("im2col-bf16-128@56-x32", "im2col", 128, 56, 56, 128, "3x3", n=32, zeros=0.6, dead=0.0, precision=2),
        # a network's first layer: dense images, channel-last as decoders deliver them
        _layer("im2col-f32-stem-x16", "im2col", 3, 224, 224, 64, "7x7s2", n=16, zeros=0.0, dead=0.0, layout="hwc"),
        # sixteen 3 x 3 layers of a residual network, one image, CPO everywhere
        _chain("chain-cpo-x1"),
        # the same network on a serving batch, the method the selection picks: CPO on the sparse
        # deep layers, im2col before them
        _chain("chain-selected-x32", n=32, methods="selected"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        op = rng.choices(["layer", "encode", "conv", "im2col", "chain"], [35, 15, 15, 20, 15])[0]
        n = 1 if rng.random() < 0.4 else _log_int(rng, 2, 32)
        if op == "chain":
            stages = rng.randint(2, 4)
            case = _chain("", width=_log_int(rng, 32, 64), size=_log_int(rng, 24, 60), stages=stages,
                          depth="".join(str(rng.randint(2, 4)) for _ in range(stages)), n=n,
                          methods=rng.choice(["cpo", "cps", "selected", "im2col"]))
            del case["name"]
            if _chain_flops(case) <= MAX_CHAIN_FLOPS:
                return case
            continue
        kernel = rng.choices(list(KERNELS), [45, 15, 10, 7, 7, 3, 3, 10])[0]
        if kernel == "7x7s2":        # a first layer: three dense channels
            size = _log_int(rng, 96, 224)
            C, H, W, K = 3, size, size + rng.choice([0, 0, -5, 8]), rng.choice([32, 64, 64, 96])
            W = min(W, 224)
        else:
            H = _log_int(rng, 7, 60)
            W = H if rng.random() < 0.7 else max(7, min(60, H + rng.randint(-6, 6)))
            C, K = _log_int(rng, 16, 512), _log_int(rng, 16, 512)
            if rng.random() < 0.5:   # most networks keep to multiples of 16
                C, K = (C + 15) // 16 * 16, (K + 15) // 16 * 16
        case = _layer("", op, C, H, W, K, kernel, n=n, method=rng.choice(["cpo", "cps"]),
                      zeros=0.0 if C == 3 else round(rng.uniform(0.4, 0.85), 3), clustered=C > 3 and rng.random() < 0.3,
                      dead=0.0 if C == 3 else rng.choice([0.0, 0.05, 0.1]), in_bits=rng.choice([32, 32, 16]),
                      relu=op in ("encode", "im2col") and C > 3 and rng.random() < 0.4,
                      layout="hwc" if rng.random() < (0.5 if C == 3 else 0.1) else "chw",
                      precision=rng.choice([0, 0, 1, 2, 2]) if op == "im2col" else 0)
        del case["name"]
        if n * C * H * W <= MAX_ELEMENTS and _dense_flops(case) <= MAX_FLOPS:
            return case


def _shape(case):
    kh, kw, stride, pad_h, pad_w = KERNELS[case["kernel"]]
    return (case["C"], case["H"], case["W"], case["K"], kh, kw, stride, pad_h, pad_w,
            api.LAYOUT_HWC if case["layout"] == "hwc" else api.LAYOUT_CHW)


def _out_size(case):
    kh, kw, stride, pad_h, pad_w = KERNELS[case["kernel"]]
    return (case["H"] + 2 * pad_h - kh) // stride + 1, (case["W"] + 2 * pad_w - kw) // stride + 1


def _dense_flops(case):
    kh, kw = KERNELS[case["kernel"]][:2]
    Oh, Ow = _out_size(case)
    return 2.0 * case["n"] * case["K"] * case["C"] * kh * kw * Oh * Ow


# ---- inputs --------------------------------------------------------------------------------------

def _ppf(p):
    return statistics.NormalDist().inv_cdf(p)


def _field(case, gen):
    """A standard normal field per channel; clustered: blurred (sigma 2 px), unit variance again."""
    n, C, H, W = case["n"], case["C"], case["H"], case["W"]
    x = torch.randn((n, C, H, W), generator=gen, device="cuda")
    if case["clustered"]:
        def blur(size):
            at = torch.arange(size, device="cuda", dtype=torch.float32)
            g = torch.exp(-0.5 * ((at[:, None] - at[None, :]) / 2.0) ** 2)
            return g / g.square().sum(0, keepdim=True).sqrt()
        x = (x.reshape(-1, W) @ blur(W)).reshape(n * C, H, W).transpose(1, 2).reshape(-1, H) @ blur(H)
        x = x.reshape(n * C, W, H).transpose(1, 2).reshape(n, C, H, W).contiguous()
    return x


def _dead_channels(count, C, gen):
    return torch.randperm(C, generator=gen, device="cuda")[:count]


def _input(case, gen):
    """(map, bias): the activated map and None, or the sums before bias and ReLU and the bias."""
    x, z, C = _field(case, gen), case["zeros"], case["C"]
    dead = _dead_channels(int(case["dead"] * C), C, gen)
    bias = None
    if z > 0.0:
        shift = _ppf(1.0 - z)
        if case["relu"]:
            bias = shift + 0.1 * torch.randn(C, generator=gen, device="cuda")
            bias[dead] = -8.0
        else:
            x = torch.relu_(x.add_(shift))
            x[:, dead] = 0.0
    if case["layout"] == "hwc":
        x = x.permute(0, 2, 3, 1).contiguous()
    return x, bias


def _he_weights(K, C, kh, kw, gen):
    return torch.randn((K, C, kh, kw), generator=gen, device="cuda") * math.sqrt(2.0 / (C * kh * kw))


def _map_outputs(m):
    """The streams, the side band and the stream lengths of every map (the last two header words are
    the library's own in device memory).  Filled once, so that what lies behind a stream's end is
    the same for everybody."""
    for t in (m.ptr, m.da, m.ind, m.chan_off):
        t.zero_()
    return {"ptr": m.ptr, "da": m.da, "in": m.ind, "chan_off": m.chan_off, "lengths": m.hdr.view(-1, 8)[:, :6]}


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "chain":
        return _prepare_chain(case, gen)
    shape, n = _shape(case), case["n"]
    x, bias = _input(case, gen)
    w = _he_weights(case["K"], case["C"], shape[4], shape[5], gen)
    buf = api.LayerBuffers(shape, n_images=n, in_bits=case["in_bits"])
    state = {"case": case, "shape": shape, "x": x, "bias": bias, "w": w, "buf": buf}
    if case["op"] == "im2col":
        if case["precision"] == 2:
            api.im2col_prepare_weights_bf16(w, shape, buf.wb)
            state["w"] = buf.wb
        return state
    m = buf.cpo if case["method"] == "cpo" else buf.cps
    state["map"] = m
    if case["op"] in ("layer", "conv"):
        api.cpoconv_prepare_weights(w, shape, buf.wt)
    if case["op"] in ("layer", "encode"):
        state["streams"] = _map_outputs(m)
    else:
        (api.cpo_encode_batch if case["method"] == "cpo" else api.cps_encode_batch)(x, shape, m, buf.scratch)
    return state


# ---- chains: stages of 3 x 3 layers, the first layer of every stage but the first halves the map --

def _chain_layers(case):
    """(C, size, K, stride) of every layer."""
    layers, C, size = [], case["width"], case["size"]
    for s in range(case["stages"]):
        K = case["width"] << s
        for i in range(int(case["depth"][s])):
            stride = 2 if s > 0 and i == 0 else 1
            layers.append((C, size, K, stride))
            C, size = K, (size - 1) // stride + 1
    return layers


def _chain_zeros(case):
    """Zero fraction in front of every layer: 40 % to 85 % over the depth of the network."""
    L = len(_chain_layers(case))
    return [0.40 + 0.45 * i / max(L - 1, 1) for i in range(L)]


def _chain_flops(case):
    return sum(2.0 * case["n"] * K * C * 9 * ((size - 1) // s + 1) ** 2 for C, size, K, s in _chain_layers(case))


def _chain_methods(case):
    code = {"cpo": api.ALGO_CPO, "cps": api.ALGO_CPS, "im2col": api.ALGO_IM2COL}
    if case["methods"] == "selected":
        return [code["cpo"] if z >= 0.66 and s == 1 else code["im2col"]
                for z, (_, _, _, s) in zip(_chain_zeros(case), _chain_layers(case))]
    return [code[case["methods"]]] * len(_chain_layers(case))


def _relu_moment(mean, sd):
    """E[max(0, X)^2] of X ~ N(mean, sd^2)."""
    t = statistics.NormalDist()
    return (mean * mean + sd * sd) * t.cdf(mean / sd) + mean * sd * t.pdf(mean / sd)


def _prepare_chain(case, gen):
    layers, zeros = _chain_layers(case), _chain_zeros(case)
    C, size = layers[0][:2]
    x = torch.relu_(torch.randn((case["n"], C, size, size), generator=gen, device="cuda").add_(_ppf(1.0 - zeros[0])))
    weights, biases, shapes = [], [], []
    mean, sd = _ppf(1.0 - zeros[0]), 1.0
    for i, (C, size, K, stride) in enumerate(layers):
        shapes.append((C, size, size, K, 3, 3, stride, 1))
        weights.append(_he_weights(K, C, 3, 3, gen))
        if i == 0:
            biases.append(None)
            continue
        # with He-normal weights the sums are close to N(0, 2 E[a^2]) of the input a
        sd = math.sqrt(2.0 * _relu_moment(mean, sd))
        mean = sd * _ppf(1.0 - zeros[i])
        b = mean + 0.1 * sd * torch.randn(C, generator=gen, device="cuda")
        b[_dead_channels(int(0.05 * C), C, gen)] = -8.0 * sd
        biases.append(b)
    chain = api.Chain(shapes, weights, biases, [b is not None for b in biases], _chain_methods(case), n_images=case["n"],
                      precision=case["precision"])
    return {"case": case, "x": x, "chain": chain}


# ---- one pass ------------------------------------------------------------------------------------

def run(state):
    case = state["case"]
    op, x = case["op"], state["x"]
    if op == "chain":
        state["chain"].forward(x)
        return state["chain"].outs
    shape, buf, n, cps = state["shape"], state["buf"], case["n"], case["method"] == "cps"
    if op == "layer":
        (api.cps_encode_conv if cps else api.cpo_encode_conv)(x, shape, state["map"], buf.wt, buf.out, buf.scratch)
        return {"streams": state["streams"], "out": buf.out}
    if op == "encode":
        if case["relu"]:
            (api.cps_encode_relu if cps else api.cpo_encode_relu)(x, state["bias"], shape, state["map"], buf.scratch)
        elif n == 1:
            (api.cps_encode if cps else api.cpo_encode)(x, shape, state["map"], buf.scratch)
        else:
            (api.cps_encode_batch if cps else api.cpo_encode_batch)(x, shape, state["map"], buf.scratch)
        return state["streams"]
    if op == "conv":
        if n == 1:
            (api.cps_conv if cps else api.cpo_conv)(state["map"], shape, buf.wt, buf.out, buf.scratch)
        else:
            (api.cps_conv_batch if cps else api.cpo_conv_batch)(state["map"], shape, buf.wt, buf.out, buf.scratch)
        return buf.out
    if case["relu"]:
        api.im2col_conv_relu(x, state["bias"], shape, n, state["w"], buf.lowered, buf.out, case["precision"])
    elif n == 1:
        api.im2col_conv(x, shape, state["w"], buf.lowered, buf.out, case["precision"])
    else:
        api.im2col_conv_batch(x, shape, n, state["w"], buf.lowered, buf.out, case["precision"])
    return buf.out


# ---- what a pass cannot do without ---------------------------------------------------------------

def work(case):
    """Bytes: every input read once, every output written once.  Flops: the multiply-adds of the NZEs
    for a sparse method, of every element for the dense one."""
    if case["op"] == "chain":
        layers, zeros, methods = _chain_layers(case), _chain_zeros(case), _chain_methods(case)
        flops, nbytes = 0.0, 4.0 * case["n"] * layers[0][0] * layers[0][1] ** 2
        for (C, size, K, s), z, m in zip(layers, zeros, methods):
            out = case["n"] * K * ((size - 1) // s + 1) ** 2
            flops += 2.0 * out * C * 9 * (1.0 if m == api.ALGO_IM2COL else 1.0 - z)
            nbytes += 4.0 * (K * C * 9 + out)
        return {"bytes": nbytes, "flops": flops}
    kh, kw = KERNELS[case["kernel"]][:2]
    n, elements = case["n"], case["n"] * case["C"] * case["H"] * case["W"]
    Oh, Ow = _out_size(case)
    live = 1.0 - int(case["dead"] * case["C"]) / case["C"]
    nnz = elements * live * (1.0 - case["zeros"])
    streams = nnz * (4 + case["in_bits"] // 8) + 4.0 * n * live * api.cpoconv_sizes(_shape(case)).ptr_cap
    weights, out = 4.0 * case["K"] * case["C"] * kh * kw, 4.0 * n * case["K"] * Oh * Ow
    dense = _dense_flops(case)
    sparse = dense * nnz / elements
    return {"layer": {"bytes": 4.0 * elements + streams + weights + out, "flops": sparse},
            "encode": {"bytes": 4.0 * elements + streams, "flops": 0.0},
            "conv": {"bytes": streams + weights + out, "flops": sparse},
            "im2col": {"bytes": 4.0 * elements + weights * (0.5 if case["precision"] == 2 else 1.0) + out,
                       "flops": dense}}[case["op"]]


def tolerance(case):
    if case["op"] == "encode":
        return "exact"               # values are copied, indices counted
    if case["precision"] != 0:
        return {"rel": 1e-2}         # operands rounded to bf16, sums in fp32
    return {"rel": 1e-5}             # fp32 sums; streams are whole numbers and copied values
