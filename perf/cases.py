"""Performance cases of the ternary inference and training library.

Each case is one pass of something a program built on this library does, called through the
binding or the ResNet-18 harness exactly as such a program calls them: weights, tables, plans
and buffers are prepared once, a pass takes fp32 inputs and leaves its outputs on the GPU.
The sizes are those of the repository's own configurations, benchmark and tests (ResNet-18's
ternary layers, the GEMM configurations, MobileNet's and AlexNet's layer shapes), or generic
odd sizes.

Kinds of case
  conv                one ternary conv layer: ternarize + pack the fp32 input, conv with the
                      reparameterizing epilogue (ReLU, BN)
  layers              the 19 ternary conv layers of ResNet-18, each with its own pack
  trunk               the same layers chained as the network's trunk, activations handed
                      over as codes (TernaryResNet18.trunk)
  gemm                ternarize + pack the activation rows, GEMM with the fused epilogue
  mobilenet           MobileNet's 13 depthwise + 13 pointwise layers as a chain
  weight_only_layers  the 19 layer shapes with ternary weights and fp32 activations
  weight_only_gemm    GEMM with ternary weights and fp32 activations
  backward            training: gradients of the reparameterized activation (layer 1's tensor)
                      and of the ternary weights of all 19 layers
"""
import math

import torch

from paper_1912_02057_amd import binding as B
from paper_1912_02057_amd import workloads as wl
from paper_1912_02057_amd.resnet18 import TernaryResNet18

DEV = "cuda:0"
FORMATS = {"fp4": B.RTN_CODE_FP4, "i8": B.RTN_CODE_I8, "planes": B.RTN_CODE_BITPLANE}
CODE_BITS = {"fp4": 4, "i8": 8, "planes": 2}

# channels in, input height, stride of the depthwise conv, channels out of the pointwise conv
MOBILENET = ([(32, 112, 1, 64), (64, 112, 2, 128), (128, 56, 1, 128), (128, 56, 2, 256), (256, 28, 1, 256),
              (256, 28, 2, 512)] + [(512, 14, 1, 512)] * 5 + [(512, 14, 2, 1024), (1024, 7, 1, 1024)])


def listed():
    return [
        # the latency of one layer on one image: two launches
        dict(name="conv_one_image", kind="conv", fmt="fp4", batch=1, C=64, H=56, W=56, O=64, k=3, stride=1, pad=1),
        # AlexNet's 5x5 layer on int8 codes: image sides and pixel counts that are odd
        dict(name="conv_5x5_ragged_i8", kind="conv", fmt="i8", batch=7, C=96, H=27, W=27, O=256, k=5, stride=1, pad=2),
        # the benchmark's headline: every ternary layer of ResNet-18 by itself, serving batch
        dict(name="layers_b256", kind="layers", fmt="fp4", batch=256),
        # the whole ternary trunk at the serving batch ...
        dict(name="trunk_b256", kind="trunk", fmt="fp4", batch=256),
        # ... and for a single image, where launches and latency count
        dict(name="trunk_one_image", kind="trunk", fmt="fp4", batch=1),
        # the GEMM configuration of the benchmark
        dict(name="gemm_4096", kind="gemm", fmt="fp4", M=4096, N=4096, K=4096, bn=False),
        # the largest point of the benchmark's GEMM sweep
        dict(name="gemm_16384x8192", kind="gemm", fmt="fp4", M=16384, N=8192, K=8192, bn=False),
        # a layer of odd sizes on int8 codes, with ReLU and BN in the epilogue
        dict(name="gemm_ragged_i8", kind="gemm", fmt="i8", M=1000, N=1003, K=2187, bn=True),
        # the paper's own 2-bit storage
        dict(name="gemm_4096_planes", kind="gemm", fmt="planes", M=4096, N=4096, K=4096, bn=False),
        # depthwise-separable network at the serving batch
        dict(name="mobilenet_b256", kind="mobilenet", fmt="fp4", batch=256),
        # 2-bit weights, 32-bit activations (the rows of the paper's table with full-precision activations)
        dict(name="weight_only_layers_b256", kind="weight_only_layers", batch=256),
        # one training step's quantizer gradients
        dict(name="backward_b256", kind="backward", batch=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["conv"] * 4 + ["gemm"] * 4 +
                      ["layers", "trunk", "mobilenet", "weight_only_layers", "weight_only_gemm", "backward"])
    if kind == "conv":
        while True:
            k = rng.choice([1, 3, 3, 5])
            H = _log_int(rng, 7, 112)
            c = dict(kind=kind, fmt=rng.choice(["fp4", "i8"]), batch=_log_int(rng, 1, 256), C=_log_int(rng, 24, 1024),
                     H=H, W=H + rng.choice([0, 0, 1, 3]), O=_log_int(rng, 24, 1024), k=k, stride=rng.choice([1, 1, 2]),
                     pad=k // 2)
            w = work(c)
            if w["flops"] <= 2e11 and w["bytes"] <= 6e8:
                return c
    if kind == "gemm":
        while True:
            c = dict(kind=kind, fmt=rng.choice(["fp4", "fp4", "i8", "planes"]), M=_log_int(rng, 1, 16384),
                     N=_log_int(rng, 64, 8192), K=_log_int(rng, 64, 8192), bn=rng.random() < 0.5)
            if rng.random() < 0.3:      # sizes of real layers are often multiples of 64
                c["N"], c["K"] = (c["N"] + 63) // 64 * 64, (c["K"] + 63) // 64 * 64
            if c["fmt"] != "planes" or work(c)["flops"] <= 4e11:
                return c
    if kind == "weight_only_gemm":
        while True:
            c = dict(kind=kind, M=_log_int(rng, 1, 8192), N=_log_int(rng, 64, 8192), K=_log_int(rng, 64, 8192))
            if work(c)["flops"] <= 4e11:
                return c
    c = dict(kind=kind, batch=_log_int(rng, 1, 256))
    if kind in ("layers", "trunk", "mobilenet"):
        c["fmt"] = rng.choice(["fp4", "fp4", "i8"])
    return c


# ---- inputs ---------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, n, lo, hi):
    return torch.rand(n, generator=g, device=DEV) * (hi - lo) + lo


def _filters(g, shape, fmt):
    """He-initialised weights ternarized at 0.7 mean|w| per filter: codes and their sums."""
    w = torch.randn(shape, generator=g, device=DEV) * math.sqrt(2.0 / math.prod(shape[1:]))
    d = (0.7 * w.reshape(shape[0], -1).abs().mean(1)).contiguous()
    return B.ternarize_pack(w, -d, d, fmt)


def _bn(g, n):
    return _uniform(g, n, 0.5, 1.5), torch.randn(n, generator=g, device=DEV) * 0.2


def _code_tensor(n, h, w, channels, fmt):
    kp = B.padded_k(channels, fmt)
    if fmt == B.RTN_CODE_I8:
        return torch.empty((n, h, w, kp), dtype=torch.int8, device=DEV)
    return torch.empty((n, h, w, kp // 2), dtype=torch.uint8, device=DEV)


def _conv_layer(g, fmt, batch, C, H, W, O, k, stride, pad, x=True, bn=None):
    """A layer as a program keeps it: weight codes, constant table, buffers; and its input."""
    OH, OW = B.conv_out_hw(H, W, k, k, stride, pad)
    cw, sw = _filters(g, (O, C, k, k), fmt)
    scale, shift = _bn(g, O) if bn is None else bn
    aa = 0.5 + float(torch.rand(1, generator=g, device=DEV))
    ep = B.Epilogue(aa, 0.1, _uniform(g, O, 0.5, 1.5), _uniform(g, O, -0.2, 0.2), None, sw, relu=True,
                    bn_scale=scale, bn_shift=shift)
    return dict(fmt=fmt, geo=(batch, C, H, W, O, k, k, stride, pad), cw=cw, ep=ep,
                ws=B.conv2d_prepare_constants(C, O, k, k, pad, ep), codes=_code_tensor(batch, H, W, C, fmt),
                y=torch.empty((batch, O, OH, OW), dtype=torch.float32, device=DEV), delta=0.56,
                x=torch.randn((batch, C, H, W), generator=g, device=DEV) if x else None)


def _run_conv(l, x):
    B.ternarize_pack(x, -l["delta"], l["delta"], l["fmt"], codes=l["codes"], want_sum=False)
    return B.ternary_conv2d(l["codes"], l["cw"], *l["geo"], ep=l["ep"], y_out=l["y"], workspace=l["ws"], fmt=l["fmt"])[1]


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    fmt = FORMATS[case["fmt"]] if "fmt" in case else None
    if kind == "conv":
        return dict(kind=kind, layer=_conv_layer(g, fmt, *[case[n] for n in ("batch", "C", "H", "W", "O", "k", "stride", "pad")]))
    if kind == "layers":
        return dict(kind=kind, layers=[_conv_layer(g, fmt, case["batch"], s.C, s.H, s.H, s.O, s.k, s.stride, s.pad)
                                       for s in wl.resnet18_ternary_layers()])
    if kind == "trunk":
        # the trunk's input is the stem's output: ReLU and max-pool, so non-negative
        x = torch.randn((case["batch"], 64, 56, 56), generator=g, device=DEV).abs_()
        return dict(kind=kind, net=TernaryResNet18(wl.resnet18_network_params(int(seed) % 65536), case["batch"], DEV, fmt), x=x)
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        x = torch.randn((M, K), generator=g, device=DEV)
        w = torch.randn((N, K), generator=g, device=DEV)
        d = (0.7 * w.abs().mean(1)).contiguous()
        cw, sw = B.ternarize_pack(w, -d, d, fmt)
        sa = torch.empty(M, dtype=torch.int32, device=DEV)
        scale, shift = _bn(g, N) if case["bn"] else (None, None)
        ep = B.Epilogue(_uniform(g, M, 0.5, 1.5), _uniform(g, M, -0.2, 0.2), _uniform(g, N, 0.5, 1.5),
                        _uniform(g, N, -0.2, 0.2), sa, sw, relu=case["bn"], bn_scale=scale, bn_shift=shift)
        shape = {B.RTN_CODE_FP4: (M, B.padded_k(K, fmt) // 2), B.RTN_CODE_I8: (M, B.padded_k(K, fmt)),
                 B.RTN_CODE_BITPLANE: (2, M, B.padded_k(K, fmt) // 64)}[fmt]
        dtype = {B.RTN_CODE_FP4: torch.uint8, B.RTN_CODE_I8: torch.int8, B.RTN_CODE_BITPLANE: torch.int64}[fmt]
        return dict(kind=kind, fmt=fmt, size=(M, N, K), x=x, cw=cw, sa=sa, ep=ep,
                    codes=torch.empty(shape, dtype=dtype, device=DEV),
                    y=torch.empty((M, N), dtype=torch.float32, device=DEV))
    if kind == "mobilenet":
        batch, layers = case["batch"], []
        for C, H, stride, O in MOBILENET:
            OH = (H - 1) // stride + 1
            # the BN affine returns each layer's output to about zero mean and unit variance
            # (a dot product of K terms, 36 % of them non-zero, then ReLU)
            bn = lambda n, K: (_uniform(g, n, 0.9, 1.1) / (0.58 * math.sqrt(0.36 * K)),
                               torch.randn(n, generator=g, device=DEV) * 0.1 - 0.69)
            wd = torch.randn((C, 9), generator=g, device=DEV) * 0.3
            cwd, _ = B.ternarize_pack(wd, -0.16, 0.16, want_sum=False)
            scale, shift = bn(C, 9)
            epd = B.Epilogue(1.1, 0.1, _uniform(g, C, 0.8, 1.2), None, None, None, relu=True, bn_scale=scale, bn_shift=shift)
            layers.append(dict(geo=(batch, C, H, H, 3, 3, stride, 1), cwd=cwd, epd=epd,
                               codes=_code_tensor(batch, H, H, C, B.RTN_CODE_I8),
                               yd=torch.empty((batch, C, OH, OH), dtype=torch.float32, device=DEV),
                               pw=_conv_layer(g, fmt, batch, C, OH, OH, O, 1, 1, 0, x=False, bn=bn(O, C))))
        return dict(kind=kind, layers=layers, x=torch.randn((batch, 32, 112, 112), generator=g, device=DEV))
    if kind == "weight_only_layers":
        batch, layers = case["batch"], []
        for s in wl.resnet18_ternary_layers():
            cw, _ = _filters(g, (s.O, s.C, s.k, s.k), B.RTN_CODE_I8)
            scale, shift = _bn(g, s.O)
            layers.append(dict(
                sh=s, prep=B.weight_conv2d_prepare(cw, s.C, s.O, s.k, s.k, s.pad, _uniform(g, s.O, 0.5, 1.5), scale, shift),
                x=torch.randn((batch, s.C, s.H, s.H), generator=g, device=DEV),
                y=torch.empty((batch, s.O, s.OH, s.OH), dtype=torch.float32, device=DEV),
                ws=torch.empty(B.lib().rtn_weight_conv2d_workspace_bytes(batch, s.C, s.H, s.H, s.O, s.k, s.k, s.pad),
                               dtype=torch.uint8, device=DEV)))
        return dict(kind=kind, layers=layers)
    if kind == "weight_only_gemm":
        M, N, K = case["M"], case["N"], case["K"]
        w = torch.randn((N, K), generator=g, device=DEV)
        d = (0.7 * w.abs().mean(1)).contiguous()
        cw, _ = B.ternarize_pack(w, -d, d, want_sum=False)
        return dict(kind=kind, size=(M, N, K), x=torch.randn((M, K), generator=g, device=DEV), alpha=_uniform(g, N, 0.5, 1.5),
                    prep=B.weight_gemm_prepare(cw, N, K), y=torch.empty((M, N), dtype=torch.float32, device=DEV),
                    ws=torch.empty(B.lib().rtn_weight_gemm_workspace_bytes(M, N, K), dtype=torch.uint8, device=DEV))
    assert kind == "backward", kind
    shape = (case["batch"], 64, 56, 56)
    a = torch.randn(shape, generator=g, device=DEV)
    filters = []
    for s in wl.resnet18_ternary_layers():
        O, K = s.O, s.K
        filters.append(dict(w=torch.randn((O, K), generator=g, device=DEV) * 0.6, g=torch.randn((O, K), generator=g, device=DEV),
                            kw=_uniform(g, O, 0.7, 1.7), bw=torch.randn(O, generator=g, device=DEV) * 0.1,
                            alpha=_uniform(g, O, 0.2, 1.2), dw=torch.empty((O, K), device=DEV),
                            sums=torch.empty((O, 3), dtype=torch.float64, device=DEV)))
    # gradients with a mean, so that the sums over them do not cancel to noise
    return dict(kind=kind, a=a, g=torch.randn(shape, generator=g, device=DEV) + 0.25 * a + 0.1, da=torch.empty_like(a),
                sums=torch.empty(2, dtype=torch.float64, device=DEV), filters=filters,
                ws=torch.empty(B.lib().rtn_activation_backward_workspace_bytes(a.numel()), dtype=torch.uint8, device=DEV))


# ---- one pass ---------------------------------------------------------------------------------
def run(state):
    kind = state["kind"]
    if kind == "conv":
        return _run_conv(state["layer"], state["layer"]["x"])
    if kind == "layers":
        return [_run_conv(l, l["x"]) for l in state["layers"]]
    if kind == "trunk":
        net = state["net"]
        net.trunk(state["x"])
        # the output of every block (and shortcut conv), and the codes of the last one
        return [l["y"] for l in net.L if l["y"] is not None] + [net.last_codes]
    if kind == "gemm":
        M, N, K = state["size"]
        B.ternarize_pack(state["x"], -0.56, 0.56, state["fmt"], codes=state["codes"], sum_t=state["sa"])
        return B.ternary_gemm(state["codes"], state["cw"], M, N, K, fmt=state["fmt"], ep=state["ep"], y_out=state["y"])[1]
    if kind == "mobilenet":
        x = state["x"]
        for l in state["layers"]:
            B.ternarize_pack(x, -0.5, 0.5, codes=l["codes"], want_sum=False)
            B.ternary_depthwise_conv2d(l["codes"], l["cwd"], *l["geo"], ep=l["epd"], y_out=l["yd"])
            x = _run_conv(l["pw"], l["yd"])
        return [l["pw"]["y"] for l in state["layers"]]
    if kind == "weight_only_layers":
        return [B.ternary_weight_conv2d(l["x"], None, l["sh"].O, l["sh"].k, l["sh"].k, l["sh"].stride, l["sh"].pad, relu=True,
                                        y_out=l["y"], workspace=l["ws"], prepared=l["prep"]) for l in state["layers"]]
    if kind == "weight_only_gemm":
        M, N, K = state["size"]
        return B.ternary_weight_gemm(state["x"], None, M, N, K, state["alpha"], y_out=state["y"], workspace=state["ws"],
                                     prepared=state["prep"])
    out = list(B.activation_backward(state["a"], state["g"], -0.5, 0.5, 0.9, grad_in=state["da"], sums=state["sums"],
                                     workspace=state["ws"]))
    for f in state["filters"]:
        out += B.weight_backward(f["w"], f["g"], -0.5, 0.5, f["kw"], f["bw"], f["alpha"], grad_w=f["dw"], sums=f["sums"])
    return out


# ---- what a pass cannot do without --------------------------------------------------------------
def _conv_work(batch, C, H, W, O, k, stride, pad, w_bits, hand_over):
    """fp32 input and output, filters of w_bits; hand_over: code bytes per input element that the
    pack writes and the conv reads."""
    OH, OW = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    nbytes = batch * C * H * W * (4 + 2 * hand_over) + O * C * k * k * w_bits / 8 + batch * O * OH * OW * 4.0
    return nbytes, 2.0 * batch * O * OH * OW * C * k * k


def work(case):
    kind, b, f = case["kind"], 0.0, 0.0
    bits = CODE_BITS[case["fmt"]] if "fmt" in case else 0
    if kind == "conv":
        b, f = _conv_work(case["batch"], case["C"], case["H"], case["W"], case["O"], case["k"], case["stride"], case["pad"],
                          bits, bits / 8)
    elif kind in ("layers", "weight_only_layers"):
        for s in wl.resnet18_ternary_layers():
            db, df = _conv_work(case["batch"], s.C, s.H, s.H, s.O, s.k, s.stride, s.pad, bits or 2, bits / 8)
            b, f = b + db, f + df
    elif kind == "trunk":
        # every tensor handed from one call to the next is written once and read once: codes between the convs
        # (the shortcut conv shares conv1's), the fp32 shortcut into a block tail, each block's fp32 output
        sh, n, cb = wl.resnet18_ternary_layers(), case["batch"], bits / 8
        b = n * 64 * 56 * 56 * (4 + cb)
        for i1, i2, ids in wl.resnet18_block_topology():
            mid, out = n * sh[i1].O * sh[i1].OH ** 2, n * sh[i2].O * sh[i2].OH ** 2
            b += n * sh[i1].C * sh[i1].H ** 2 * cb + 2 * mid * cb + out * (4 + 4 + cb) + (0 if ids is None else 4 * out)
            for i in (i1, i2, ids):
                if i is not None:
                    b, f = b + sh[i].O * sh[i].K * cb, f + 2.0 * sh[i].macs(n)
    elif kind in ("gemm", "weight_only_gemm"):
        M, N, K = case["M"], case["N"], case["K"]
        b, f = M * K * (4 + 2 * bits / 8) + N * K * (bits or 2) / 8 + M * N * 4.0, 2.0 * M * N * K
    elif kind == "mobilenet":
        for C, H, stride, O in MOBILENET:
            n, OH = case["batch"], (H - 1) // stride + 1
            b += n * C * H * H * (4 + 1 + 1) + n * C * OH * OH * 4.0 + C * 9
            f += 2.0 * n * C * OH * OH * 9
            db, df = _conv_work(n, C, OH, OH, O, 1, 1, 0, bits, bits / 8)
            b, f = b + db, f + df
    else:
        n = case["batch"] * 64 * 56 * 56 + sum(s.O * s.K for s in wl.resnet18_ternary_layers())
        b, f = 12.0 * n, 6.0 * n
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("weight_only_layers", "weight_only_gemm"):
        # fp32 accumulation of up to 3 * 4608 exact products, in any order (7.9e-7 against float64)
        return {"rel": 3e-6}
    if kind == "backward":
        # the gradients are single fp32 products; the sums are formed in double
        return {"rel": 1e-11}
    # integer sums, the epilogue in double, one rounding to fp32 (2.5e-8 against float64)
    return {"rel": 1e-7}
