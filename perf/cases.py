"""Performance cases of the convolution passes: what a training or serving program has the library do, through
the public entry points of paper_1911_10175_amd, on tensors resident on the GPU.

A case is one layer: its geometry (N, C, K, H, W, the square filter R, stride, pad), the zero fraction of the
activations (px) and of the output gradients (pdy), the passes taken ("train": FWD, BWI and BWW one after the
other as a training step takes them; "fwd", "bwi", "bww": one pass) and the form of the entry points: "skip"
(st_conv_fwd / bwi / bww, zero-skipping), "auto" (st_conv_*_auto, which pick the form on the device) or "dense"
(st_conv_*_dense).  The inputs are those of stgen, drawn on the GPU: x = max(0, z - t), dy = Gaussian times a
Bernoulli mask, He-normal filters, all in the library's blocked layouts.
"""
import math
from statistics import NormalDist

import torch

import paper_1911_10175_amd as st

B = 16                                              # channel block of the layouts


def _case(name, form, passes, N, C, K, H, W, R, stride, pad, px, pdy):
    return {"name": name, "form": form, "passes": passes, "N": N, "C": C, "K": K, "H": H, "W": W, "R": R,
            "stride": stride, "pad": pad, "px": px, "pdy": pdy}


def listed():
    return [
        # the smallest layer (16 -> 16 @8, one image): launches and latency only
        _case("tiny_train_skip", "skip", "train", 1, 16, 16, 8, 8, 3, 1, 1, 0.5, 0.5),
        # the VGG16 conv3_2 layer at minibatch 16, 60 / 50 % zeros, zero-skipping entry points
        _case("vgg3_2_train_skip", "skip", "train", 16, 256, 256, 56, 56, 3, 1, 1, 0.6, 0.5),
        # the layers of a VGG16 training step, first to last, by a program that leaves the form to the library:
        # the largest images with the fewest channels
        _case("vgg1_2_train_auto", "auto", "train", 32, 64, 64, 224, 224, 3, 1, 1, 0.5, 0.5),
        # early in training, when ReLU leaves few zeros; channel counts that differ
        _case("vgg3_1_train_auto_30", "auto", "train", 32, 128, 256, 56, 56, 3, 1, 1, 0.3, 0.3),
        # the most channels
        _case("vgg4_2_train_auto", "auto", "train", 32, 512, 512, 28, 28, 3, 1, 1, 0.5, 0.5),
        # late layers of a trained network: small images, many zeros
        _case("vgg5_1_train_auto_70", "auto", "train", 32, 512, 512, 14, 14, 3, 1, 1, 0.7, 0.7),
        # the 1x1 layers of a ResNet-50 bottleneck, bound by memory (56 x 56) and by arithmetic (7 x 7)
        _case("resnet2_1b_train_auto", "auto", "train", 32, 256, 64, 56, 56, 1, 1, 0, 0.4, 0.5),
        _case("resnet5_3_train_auto", "auto", "train", 32, 512, 2048, 7, 7, 1, 1, 0, 0.5, 0.5),
        # a down-sampling layer
        _case("resnet3_2r_train_auto", "auto", "train", 32, 128, 128, 56, 56, 3, 2, 1, 0.5, 0.5),
        # a basic block under batch normalisation: its gradients hold no zeros, the program takes the dense forms
        _case("resnet3_2_train_dense", "dense", "train", 32, 128, 128, 28, 28, 3, 1, 1, 0.5, 0.0),
        # channel counts and image sides that are no multiple of any tile
        _case("ragged_train_auto", "auto", "train", 3, 80, 48, 37, 53, 3, 1, 1, 0.5, 0.5),
        # one image through a late layer: serving latency
        _case("vgg5_3_serve_auto", "auto", "fwd", 1, 512, 512, 14, 14, 3, 1, 1, 0.5, 0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A layer of the same ranges: 3x3 at stride 1 (most), 1x1, 3x3 at stride 2; any form, any passes."""
    limit = max(_dense_flops(c) for c in listed())
    while True:
        kind = rng.choice(["3x3", "3x3", "3x3", "1x1", "3x3s2"])
        R, stride, pad = {"3x3": (3, 1, 1), "1x1": (1, 1, 0), "3x3s2": (3, 2, 1)}[kind]
        H = _log_int(rng, 7, 224)
        W = H if rng.random() < 0.6 else _log_int(rng, 7, 224)
        top = 2048 if kind == "1x1" else 512
        C, K = (B * _log_int(rng, 1, top // B) for _ in range(2))
        form = rng.choice(["auto", "auto", "auto", "skip", "dense"])
        passes = rng.choice(["train", "train", "fwd", "bwi", "bww"])
        c = _case("", form, passes, _log_int(rng, 1, 32), C, K, H, W, R, stride, pad,
                  round(rng.uniform(0.0, 0.9), 2), round(rng.uniform(0.0, 0.9), 2))
        del c["name"]
        # activations that fit beside two other states, and no more work than the largest listed case
        if _dense_flops(c) <= limit and c["N"] * max(C, K) * H * W * 4 <= 1 << 30:
            return c


def _desc(c):
    return st.ConvDesc(c["N"], c["C"], c["K"], c["H"], c["W"], c["R"], c["R"], c["stride"], c["stride"], c["pad"], c["pad"])


def _passes(c):
    return ("fwd", "bwi", "bww") if c["passes"] == "train" else (c["passes"],)


def _dense_flops(c):
    return _desc(c).flops * len(_passes(c))


def work(c):
    """Every tensor of a pass once; the products whose tested operand is not zero (all of them in a dense form)."""
    d = _desc(c)
    x, y, w = c["N"] * c["C"] * c["H"] * c["W"], c["N"] * c["K"] * d.OH * d.OW, c["C"] * c["K"] * c["R"] ** 2
    zeros = {"fwd": c["px"], "bwi": c["pdy"], "bww": max(c["px"], c["pdy"])}
    flops = sum(d.flops * (1.0 if c["form"] == "dense" else 1.0 - zeros[p]) for p in _passes(c))
    return {"bytes": 4 * (x + y + w) * len(_passes(c)), "flops": flops}


def _entry(form, p):
    return getattr(st, "st_conv_" + p + {"skip": "", "auto": "_auto", "dense": "_dense"}[form])


def _workspace_bytes(c, p):
    base = {"fwd": st.ST_PASS_FWD, "bwi": st.ST_PASS_BWI, "bww": st.ST_PASS_BWW}[p]
    auto = {"fwd": st.ST_PASS_FWD_AUTO, "bwi": st.ST_PASS_BWI_AUTO, "bww": st.ST_PASS_BWW_AUTO}[p]
    return st.st_conv_workspace_bytes(_desc(c), auto if c["form"] == "auto" else base, c["form"] == "dense")


def _inputs(c, seed):
    d = _desc(c)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    passes = _passes(c)
    x = w = dy = None
    if "fwd" in passes or "bww" in passes:
        x = torch.randn((c["N"], c["C"] // B, c["H"], c["W"], B), device="cuda", generator=g)
        if c["px"] > 0:
            x = torch.relu_(x.sub_(NormalDist().inv_cdf(c["px"])))
    if "fwd" in passes or "bwi" in passes:
        w = torch.randn((c["K"] // B, c["C"] // B, c["R"], c["R"], B, B), device="cuda", generator=g)
        w.mul_(math.sqrt(2.0 / (c["C"] * c["R"] ** 2)))
    if "bwi" in passes or "bww" in passes:
        shape = (c["N"], c["K"] // B, d.OH, d.OW, B)
        dy = torch.randn(shape, device="cuda", generator=g)
        if c["pdy"] > 0:
            dy.mul_(torch.rand(shape, device="cuda", generator=g) >= c["pdy"])
    return x, w, dy


def prepare(c, seed):
    d = _desc(c)
    x, w, dy = _inputs(c, seed)
    # one workspace, used by the passes in turn on one stream
    need = max(_workspace_bytes(c, p) for p in _passes(c))
    ws = torch.empty((need + 3) // 4, device="cuda") if need else None
    calls, out = [], {}
    for p in _passes(c):
        a, b, shape = {"fwd": (x, w, (c["N"], c["K"] // B, d.OH, d.OW, B)),
                       "bwi": (dy, w, (c["N"], c["C"] // B, c["H"], c["W"], B)),
                       "bww": (x, dy, (c["K"] // B, c["C"] // B, c["R"], c["R"], B, B))}[p]
        name = {"fwd": "y", "bwi": "dx", "bww": "dw"}[p]
        out[name] = torch.empty(shape, device="cuda")
        calls.append((_entry(c["form"], p), a, b, out[name]))
    return {"desc": d, "calls": calls, "ws": ws, "out": out}


def run(state):
    stream = torch.cuda.current_stream()
    for fn, a, b, o in state["calls"]:
        fn(state["desc"], a, b, o, state["ws"], stream)
    return state["out"]


def tolerance(c):
    # sums of 32-bit products in another order: the entry points are 1e-7 to 6e-7 off the 64-bit result over the
    # listed layers, so two of them differ by up to about 8e-7; four times that
    return {"rel": 3e-6}


def exact(c, seed):
    """The passes in 64 bits, one matrix product per filter tap."""
    d = _desc(c)
    x, w, dy = _inputs(c, seed)
    N, C, K, H, W, R, s, pad = (c[k] for k in ("N", "C", "K", "H", "W", "R", "stride", "pad"))
    OH, OW = d.OH, d.OW
    Hp, Wp = H + 2 * pad, W + 2 * pad

    def plain(t):                                   # [N][c/16][h][w][16] -> [c][N][h][w] in 64 bits
        return t.double().permute(1, 4, 0, 2, 3).reshape(t.shape[1] * B, t.shape[0], t.shape[2], t.shape[3])

    def blocked(t):                                 # the inverse
        return t.reshape(t.shape[0] // B, B, *t.shape[1:]).permute(2, 0, 3, 4, 1).contiguous()

    def tap(t, v, u):                               # the samples a tap meets
        return t[:, :, v:v + s * (OH - 1) + 1:s, u:u + s * (OW - 1) + 1:s]

    xp = torch.nn.functional.pad(plain(x), (pad, pad, pad, pad)) if x is not None else None
    dyf = plain(dy).reshape(K, -1) if dy is not None else None
    wf = w.double().permute(2, 3, 0, 5, 1, 4).reshape(R, R, K, C) if w is not None else None
    res = {}
    for p in _passes(c):
        if p == "fwd":
            y = torch.zeros((K, N * OH * OW), dtype=torch.float64, device="cuda")
            for v in range(R):
                for u in range(R):
                    y += wf[v, u] @ tap(xp, v, u).reshape(C, -1)
            res["y"] = blocked(y.reshape(K, N, OH, OW))
        elif p == "bwi":
            dxp = torch.zeros((C, N, Hp, Wp), dtype=torch.float64, device="cuda")
            for v in range(R):
                for u in range(R):
                    tap(dxp, v, u).add_((wf[v, u].t() @ dyf).reshape(C, N, OH, OW))
            res["dx"] = blocked(dxp[:, :, pad:pad + H, pad:pad + W])
        else:
            dw = torch.empty((R, R, K, C), dtype=torch.float64, device="cuda")
            for v in range(R):
                for u in range(R):
                    dw[v, u] = dyf @ tap(xp, v, u).reshape(C, -1).t()
            res["dw"] = dw.reshape(R, R, K // B, B, C // B, B).permute(2, 4, 0, 1, 5, 3).contiguous()
    return res
