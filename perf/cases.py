"""What a user of this package has it do, as measurable cases.

The sizes are the five layer configurations of the benchmark, the other layers
of the same networks (ResNet-50's four stages and its classifier, MobileNetV2's
pointwise pairs, the 7x7 RGB stem, the keyword-spotting CNN), and batches from
one sample to a server's.  A case is a dict of plain values; "kind" names the
program:

  linear      int8 linear layer with bias and k-WTA on a sparse input
  gsc         the int8 keyword-spotting CNN, dense input to logits
  conv3x3     fp32 3x3 layer with k-WTA on a sparse input (dense output)
  block       fp32 1x1 then 3x3, k-WTA after each
  bottleneck  fp32 1x1, 3x3, 1x1: k-WTA after the first two, sums of the last
  pointwise   int8 1x1 expand with bias and k-WTA, 1x1 project (sums)
  stem        int8 7x7/2 RGB stem with block-complementary kernels
  head        fp32 classifier on a sparse feature vector

The chains run as a serving program runs them: a Network packed once, its
forward pass recorded into a HIP graph over a static input, one replay a pass.
The stem and the head are single library calls.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2112_13896_amd import ops
from paper_2112_13896_amd.network import Network


def listed():
    return [
        # one request of a small int8 classifier: two launches, all latency
        dict(name="linear_b16", kind="linear", batch=16, d_in=512, d_out=64, n=8, nnz=64, k=16),
        # a streaming word: one image, latency
        dict(name="gsc_b1", kind="gsc", batch=1),
        # the benchmark's batch, one image per compute unit
        dict(name="gsc_b256", kind="gsc", batch=256),
        # offline scoring, a ragged number of words
        dict(name="gsc_b1900", kind="gsc", batch=1900),
        # ResNet-50 stage 1, 56x56
        dict(name="res1_3x3_b32", kind="conv3x3", batch=32, size=56, ch=64, stride=1, n=8, nnz=7,
             k=8),
        # stage 2's entry: stride 2, 56x56 -> 28x28, an odd batch
        dict(name="res2_3x3s2_b13", kind="conv3x3", batch=13, size=56, ch=128, stride=2, n=8,
             nnz=16, k=16),
        # stage 3's block as the benchmark has it
        dict(name="res3_block_b64", kind="block", batch=64, size=14, c_in=1024, ch=256, n=16,
             nnz=102, k=26),
        # a whole stage-4 bottleneck at 7x7, wide layers over few pixels
        dict(name="res4_bneck_b32", kind="bottleneck", batch=32, size=7, c_in=2048, ch=512, n=16,
             nnz=205, k=51),
        # MobileNetV2's 96-channel pair as the benchmark has it
        dict(name="mbv2_96_b128", kind="pointwise", batch=128, size=14, ch=96, n=8, nnz=12, k=72),
        # its 160-channel pair at 7x7: few pixels, long rows
        dict(name="mbv2_160_b32", kind="pointwise", batch=32, size=7, ch=160, n=8, nnz=20, k=120),
        # the RGB stem on full-size images
        dict(name="stem_b32", kind="stem", batch=32, size=224),
        # the classifier after global pooling
        dict(name="head_b64", kind="head", batch=64, d_in=2048, d_out=1000, n=8, nnz=205),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("linear", "gsc", "conv3x3", "conv3x3", "block", "bottleneck", "pointwise",
                       "pointwise", "stem", "head"))
    while True:
        c = _draw_kind(rng, kind)
        w = work(c)
        # the two dense-input programs are bounded by their listed sizes, the others by these
        if kind in ("gsc", "stem") or (w["bytes"] <= 9e7 and w["flops"] <= 2.5e8):
            return c


def _draw_kind(rng, kind):
    if kind == "linear":
        n = rng.choice((4, 8, 16))
        d_in, d_out = n * _log_int(rng, 192 // n, 2048 // n), n * _log_int(rng, 64 // n, 1536 // n)
        return dict(kind=kind, batch=_log_int(rng, 1, 512), d_in=d_in, d_out=d_out, n=n,
                    nnz=max(1, int(d_in * rng.uniform(0.08, 0.2))),
                    k=max(1, int(d_out * rng.uniform(0.08, 0.25))))
    if kind == "gsc":
        return dict(kind=kind, batch=_log_int(rng, 1, 1900))
    if kind == "conv3x3":
        ch, size = rng.choice(((64, 56), (128, 28), (128, 56), (256, 14), (256, 28), (512, 7),
                               (512, 14)))
        act = rng.choice((0.1, 0.125))
        return dict(kind=kind, batch=_log_int(rng, 1, 64), size=size + rng.choice((-1, 0, 0, 1, 3)),
                    ch=ch, stride=rng.choice((1, 1, 2)), n=rng.choice((8, 16)),
                    nnz=int(ch * act), k=int(ch * act))
    if kind == "block":
        ch, size = rng.choice(((64, 56), (128, 28), (256, 14)))
        return dict(kind=kind, batch=_log_int(rng, 1, 64), size=size + rng.choice((-1, 0, 0, 1)),
                    c_in=4 * ch, ch=ch, n=rng.choice((8, 16)), nnz=int(0.4 * ch), k=int(0.1 * ch))
    if kind == "bottleneck":
        ch, size = rng.choice(((64, 56), (128, 28), (256, 14), (512, 7)))
        return dict(kind=kind, batch=_log_int(rng, 1, 32), size=size + rng.choice((-1, 0, 0, 1)),
                    c_in=4 * ch, ch=ch, n=rng.choice((8, 16)), nnz=int(0.4 * ch), k=int(0.1 * ch))
    if kind == "pointwise":
        ch, size = rng.choice(((24, 56), (32, 28), (64, 14), (96, 14), (160, 7)))
        return dict(kind=kind, batch=_log_int(rng, 1, 128), size=size + rng.choice((-1, 0, 0, 1)),
                    ch=ch, n=8, nnz=max(3, ch // 8), k=6 * ch // 8)
    if kind == "stem":
        return dict(kind=kind, batch=_log_int(rng, 1, 32), size=rng.randint(97, 224))
    n = rng.choice((4, 8, 16))
    d_in = n * _log_int(rng, 512 // n, 2048 // n)
    return dict(kind="head", batch=_log_int(rng, 1, 256), d_in=d_in,
                d_out=n * _log_int(rng, 96 // n, 1024 // n), n=n,
                nnz=int(d_in * rng.uniform(0.08, 0.2)))


# ---------------------------------------------------------------- inputs
def _layer(kind, c_in, c_out, n, kh=1, stride=1, pad=0, pool=1, k=None, shift=None,
           dense_input=False):
    return SimpleNamespace(name=f"{kind}{kh}x{kh}_{c_in}_{c_out}", kind=kind, c_in=c_in,
                           c_out=c_out, n=n, kh=kh, kw=kh, stride=stride, pad=pad, pool=pool, k=k,
                           shift=shift, dense_input=dense_input)


def _layers(case):
    """(layers, input shape per sample, whether int8, whether biased) of a chain."""
    kind = case["kind"]
    if kind == "linear":
        return [_layer("linear", case["d_in"], case["d_out"], case["n"], k=case["k"])], \
            (case["d_in"],), True, True
    if kind == "gsc":
        return [_layer("conv", 1, 64, 1, kh=5, pool=2, k=8, shift=11, dense_input=True),
                _layer("conv", 64, 64, 16, kh=5, pool=2, k=8, shift=9),
                _layer("linear", 1600, 1500, 20, k=75, shift=9),
                _layer("linear", 1500, 12, 1)], (32, 32, 1), True, False
    s = case["size"]
    if kind == "conv3x3":
        c = case["ch"]
        return [_layer("conv", c, c, case["n"], kh=3, stride=case["stride"], pad=1, k=case["k"])], \
            (s, s, c), False, False
    if kind in ("block", "bottleneck"):
        c, n, k = case["ch"], case["n"], case["k"]
        ls = [_layer("conv", case["c_in"], c, n, k=k), _layer("conv", c, c, n, kh=3, pad=1, k=k)]
        if kind == "bottleneck":
            ls.append(_layer("conv", c, case["c_in"], n))
        return ls, (s, s, case["c_in"]), False, False
    if kind == "pointwise":
        c = case["ch"]
        return [_layer("conv", c, 6 * c, case["n"], k=case["k"], shift=9),
                _layer("conv", 6 * c, c, case["n"])], (s, s, c), True, True
    raise ValueError(kind)


def _weights(gen, c_out, r, n, int8, block=1):
    """Dense [c_out][r] weights in complementary sets: for every set a random
    permutation of the r / block slots is cut into n nearly equal pieces, one
    per kernel.  int8: uniform non-zero; fp32: N(0, 2 n / r)."""
    nb, G, dev = r // block, c_out // n, gen.device
    order = torch.rand((G, nb), generator=gen, device=dev).argsort(dim=1)
    owner = torch.empty_like(order)
    piece = (torch.arange(nb, device=dev) * n // nb).expand(G, nb)
    owner.scatter_(1, order, piece)                       # kernel of the set that owns the block
    owner = owner.repeat_interleave(block, dim=1)
    mask = owner[:, None, :] == torch.arange(n, device=dev)[None, :, None]
    if int8:
        v = torch.randint(1, 128, (G, n, r), generator=gen, device=dev, dtype=torch.int32)
        v *= 2 * torch.randint(0, 2, (G, n, r), generator=gen, device=dev, dtype=torch.int32) - 1
        w = torch.where(mask, v, 0).to(torch.int8)
    else:
        v = torch.randn((G, n, r), generator=gen, device=dev) * math.sqrt(2.0 * n / r)
        v = torch.where(v == 0, 1e-3, v)
        w = torch.where(mask, v, 0.0)
    return w.reshape(c_out, r)


def _sparse(gen, rows, c, nnz, int8):
    """[rows][c] activations with nnz non-zeros per row at uniform places:
    int8 uniform in 1..127, fp32 |N(0, 1)| (a k-WTA's winners after a ReLU)."""
    dev = gen.device
    at = torch.rand((rows, c), generator=gen, device=dev).topk(nnz, dim=1).indices
    if int8:
        v = torch.randint(1, 128, (rows, nnz), generator=gen, device=dev, dtype=torch.int32)
        x = torch.zeros((rows, c), dtype=torch.int8, device=dev)
        return x.scatter_(1, at, v.to(torch.int8))
    v = torch.randn((rows, nnz), generator=gen, device=dev).abs() + 1e-6
    return torch.zeros((rows, c), device=dev).scatter_(1, at, v)


def _inputs(case, seed):
    """(x, [W], [bias or None]): all made from the seed, on the GPU."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind, b = case["kind"], case["batch"]
    if kind == "stem":
        s = case["size"]
        x = torch.randint(-127, 128, (b, s, s, 3), generator=gen, device="cuda",
                          dtype=torch.int32).to(torch.int8)
        return x, [_weights(gen, 64, 147, 4, True, block=3)], [None]
    if kind == "head":
        x = _sparse(gen, b, case["d_in"], case["nnz"], False)
        W = _weights(gen, case["d_out"], case["d_in"], case["n"], False)
        return x, [W], [torch.randn(case["d_out"], generator=gen, device="cuda")]
    layers, shape, int8, biased = _layers(case)
    Ws = [_weights(gen, s.c_out, s.kh * s.kw * s.c_in, s.n, int8) for s in layers]
    bs = [torch.randint(-1000, 1001, (s.c_out,), generator=gen, device="cuda",
                        dtype=torch.int32) if biased else None for s in layers]
    if kind == "gsc":
        x = torch.randint(-127, 128, (b,) + shape, generator=gen, device="cuda",
                          dtype=torch.int32).to(torch.int8)
    else:
        rows = b * int(np.prod(shape[:-1]))
        x = _sparse(gen, rows, shape[-1], case["nnz"], int8).reshape((b,) + shape)
    return x, Ws, bs


def prepare(case, seed):
    x, Ws, bs = _inputs(case, seed)
    if case["kind"] == "stem":
        aug, kidb, _ = ops.pack_blocks(Ws[0].cpu().numpy(), 4, 3)
        return dict(kind="stem", x=x, aug=ops.aug_to_device(aug), kidb=torch.from_numpy(kidb).cuda(),
                    out=torch.empty((case["batch"], (case["size"] - 1) // 2 + 1,
                                     (case["size"] - 1) // 2 + 1, 64), dtype=torch.int32,
                                    device="cuda"))
    if case["kind"] == "head":
        aug, _ = ops.pack(Ws[0].cpu().numpy(), case["n"])
        return dict(kind="head", x=x, aug=ops.aug_to_device(aug), n=case["n"], bias=bs[0],
                    ws=ops.workspace(0, x.dtype, case["batch"], case["d_in"], x.device),
                    out=torch.empty((case["batch"], case["d_out"]), device="cuda"))
    layers, shape, _, _ = _layers(case)
    net = Network(layers, [w.cpu().numpy() for w in Ws],
                  [None if t is None else t.cpu().numpy() for t in bs], shape, case["batch"],
                  device="cuda", keep_sums=False)
    net.forward(x)                                        # the kernels are loaded before a capture
    return dict(kind="net", net=net, x=x, graph=net.capture(x), out=net.out[-1])


def run(state):
    if state["kind"] == "stem":
        return ops.conv2d_dense_blocks(state["x"], state["aug"], state["kidb"], 7, 7, 4, stride=2,
                                       pad=3, out=state["out"])
    if state["kind"] == "head":
        return ops.linear(state["x"], state["aug"], state["n"], state["bias"], ws=state["ws"],
                          out=state["out"])
    state["graph"].replay()
    return state["out"]


# ---------------------------------------------------------------- costs
def _taps(size, kh, stride, pad):
    """(output positions, (position, tap) pairs inside the map) along one axis."""
    out = (size + 2 * pad - kh) // stride + 1
    return out, sum(1 for o in range(out) for t in range(kh) if 0 <= o * stride + t - pad < size)


def work(case):
    """Dense input, packed tables (value and Kernel ID per slot) and output
    once each; 2 operations per (non-zero, set) pair under a window."""
    kind, b = case["kind"], case["batch"]
    if kind == "stem":
        s = case["size"]
        o, t = _taps(s, 7, 2, 3)
        return dict(bytes=b * s * s * 3 + 147 * 16 * 2 + b * o * o * 64 * 4,
                    flops=2 * b * t * t * 3 * 16)
    if kind == "head":
        G = case["d_out"] // case["n"]
        return dict(bytes=4 * b * case["d_in"] + 8 * case["d_in"] * G + 4 * b * case["d_out"],
                    flops=2 * b * case["nnz"] * G)
    layers, shape, int8, _ = _layers(case)
    esz, asz = (2, 1) if int8 else (8, 4)
    size = shape[0] if len(shape) == 3 else 1
    nnz = case.get("nnz", 1)
    byts = b * int(np.prod(shape)) * asz
    flops = 0
    for i, s in enumerate(layers):
        G = s.c_out // s.n
        byts += s.kh * s.kw * s.c_in * G * esz
        if s.kind == "linear":
            per = nnz if i == 0 else nnz * size * size
            flops += 2 * b * per * G
            size = 1
        else:
            o, t = _taps(size, s.kh, s.stride, s.pad)
            flops += 2 * b * t * t * nnz * G
            size = o // s.pool
        nnz = s.k
    byts += b * size * size * layers[-1].c_out * 4
    return dict(bytes=byts, flops=flops)


# ---------------------------------------------------------------- accuracy
def tolerance(case):
    """Integer chains are exact.  fp32 results are sums of up to a few thousand
    products, and a k-WTA keeps or drops them unchanged: over twelve seeds of
    each fp32 case the sums are within 5e-8 .. 8e-8 of 64 bits (2-norm), no
    value further off than 1e-6.  (Now and then - one such run in sixty - a
    k-WTA's k-th and (k+1)-th sums are so close that rounding decides.)"""
    if case["kind"] in ("linear", "gsc", "pointwise", "stem"):
        return "exact"
    return dict(rel=4e-7, max=8e-6)


def _conv64(x, W, spec):
    """Plain float64 NHWC convolution, one matrix product per tap."""
    b, h, w, c = x.shape
    W = W.double().reshape(spec.c_out, spec.kh, spec.kw, c)
    x = torch.nn.functional.pad(x, (0, 0, spec.pad, spec.pad, spec.pad, spec.pad))
    o = (h + 2 * spec.pad - spec.kh) // spec.stride + 1
    span = (o - 1) * spec.stride + 1
    y = torch.zeros((b * o * o, spec.c_out), dtype=torch.float64, device=x.device)
    for ky in range(spec.kh):
        for kx in range(spec.kw):
            v = x[:, ky:ky + span:spec.stride, kx:kx + span:spec.stride].reshape(-1, c)
            y += v @ W[:, ky, kx].t().contiguous()
    return y.reshape(b, o, o, spec.c_out)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("linear", "gsc", "pointwise", "stem"):    # whole numbers, compared exactly
        return None
    x, Ws, bs = _inputs(case, seed)
    cur = x.double()
    if kind == "head":
        return cur @ Ws[0].double().t().contiguous() + bs[0].double()
    for spec, W in zip(_layers(case)[0], Ws):
        cur = _conv64(cur, W, spec)
        if spec.k is not None:
            at = cur.topk(spec.k, dim=-1).indices
            cur = torch.zeros_like(cur).scatter_(-1, at, cur.gather(-1, at))
    return cur
