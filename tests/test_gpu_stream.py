"""The fp32 layer with its table streamed through LDS (mrs_stream_f32) where its
tiles, table pieces and lists end: 4, 8 and 16 lanes of 8 and 16 channels a
pixel, one and two sets a lane, blocks of one and of several whole taps and
channel ranges of a tap, a last block that is not full, lists of more than
the 32 entries loaded ahead, empty and full pixels, stride 2, a last tile of
a few pixels, k = 0 and k = c_out, k-WTA units.  Sums within tolerance of the
oracle, winners the exact top-k of the kernel's own sums; and sums, dense
outputs and lists the same bits as the table-block kernel's, which takes the
same layer when y is not 16-byte aligned.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import cs_oracle as o
from paper_2112_13896_amd import ops
from tests.gpu_util import assert_f32_close, check_kwta_f32, dev, host

pytestmark = pytest.mark.gpu

# (b, h, w, c_in), non-zeros, kh, stride, pad, c_out, n, k, unit, blocks of the table
CASES = [
    ((2, 7, 7, 256), 26, 3, 1, 1, 256, 16, 26, 256, 9),     # 16 lanes x 16, one tap a block
    ((1, 9, 5, 1024), 102, 1, 1, 0, 256, 16, 26, 256, 4),   # channel ranges of one tap
    ((1, 9, 5, 1024), 700, 1, 1, 0, 256, 16, 0, 256, 4),    # long lists, k = 0
    ((2, 9, 9, 128), 16, 3, 2, 1, 128, 8, 16, 128, 5),      # two taps a block, the last of one
    ((2, 6, 7, 128), 100, 3, 1, 1, 256, 8, 256, 256, 9),    # two sets a lane, k = c_out
    ((1, 6, 6, 256), 40, 3, 1, 1, 256, 8, 25, 256, 18),     # two sets, two ranges a tap
    ((1, 5, 6, 512), 50, 3, 1, 1, 64, 16, 6, 64, 5),        # 4 lanes x 16
    ((2, 6, 5, 256), 30, 3, 1, 1, 128, 16, 12, 64, 5),      # 8 lanes, units of 64
    ((3, 3, 3, 384), 0, 3, 1, 1, 128, 8, 5, 128, 18),       # empty input: the bias wins
]


@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
@pytest.mark.parametrize("form", ["dense", "lists"])
def test_streamed_table_layer(case, form):
    shape, nnz, kh, stride, pad, c_out, n, k, unit, nblocks = case
    r = np.random.default_rng(sum(shape) + c_out + k)
    b, h, w, c = shape
    x = np.zeros((b * h * w, c), np.float32)
    for i in range(len(x)):
        m = (nnz, nnz // 3, 0, min(c, 2 * nnz))[i % 4]
        x[i, r.permutation(c)[:m]] = r.normal(size=m)
    R, G = kh * kh * c, c_out // n
    W = np.zeros((G, n, R), np.float32)
    np.put_along_axis(W, r.integers(0, n, (G, 1, R)), r.normal(size=(G, 1, R)).astype(np.float32),
                      axis=1)
    W = W.reshape(c_out, R)
    bias = r.normal(size=c_out).astype(np.float32)
    aug = ops.aug_to_device(ops.pack(W, n)[0])
    plan = ops.mrs_plan(torch.float32, c, shape, kh, kh, stride, pad, c_out, n, 1, k)
    assert plan["path"] == "blocks" and plan["table_blocks"] == nblocks, plan
    idx, lv, cnt = ops.compact(dev(x))
    ho, wo = ops.conv_out(h, kh, stride, pad), ops.conv_out(w, kh, stride, pad)
    rows = b * ho * wo
    cap = ops.list_capacity(k * (c_out // unit)) if form == "lists" else None

    def layer(y, keep=True):
        args = (idx, lv, cnt, shape, aug, kh, kh, n, stride, pad, dev(bias))
        if unit < c_out:
            return ops.mrs_kwta_units_conv2d(*args, k=k, unit=unit, y=y, keep_sums=keep, cap=cap)[1]
        return ops.mrs_kwta_conv2d(*args, k=k, y=y, keep_sums=keep, cap=cap)[1]

    def dense(res):
        if form == "dense":
            return host(res).reshape(rows, c_out)
        gi, gv, gc = (host(t) for t in res)
        d = np.zeros((rows, c_out), np.float32)
        for i in range(rows):
            ii = gi[i, :gc[i]].view(np.uint16)
            assert (np.diff(ii.astype(int)) > 0).all()
            d[i, ii] = gv[i, :gc[i]]
        return d

    y = torch.empty((b, ho, wo, c_out), device="cuda")
    got = dense(layer(y))
    assert np.array_equal(dense(layer(torch.empty_like(y), keep=False)), got)
    ref = o.conv2d_nhwc(x.reshape(shape), W.reshape(c_out, kh, kh, c), stride, pad, bias)
    S = o.abs_sum_conv(x.reshape(shape), W.reshape(c_out, kh, kh, c), stride, pad) + np.abs(bias)
    acc = host(y).reshape(rows, c_out)
    assert_f32_close(acc, ref.reshape(rows, c_out), S.reshape(rows, c_out), "sums")
    win = o.kwta_winners(acc.reshape(-1, unit), k).reshape(rows, c_out)
    full = np.where(win, acc, np.float32(0))
    assert np.array_equal(got, full)
    check_kwta_f32(acc.reshape(-1, unit), full.reshape(-1, unit), ref.reshape(-1, unit),
                   S.reshape(-1, unit), k)
    if nnz:
        # the table-block kernel: the same sums, and so the same winners
        off = torch.empty(y.numel() + 1, device="cuda")[1:].view(y.shape)
        if unit == c_out:
            other = dense(layer(off))
            assert np.array_equal(other.view(np.uint32), got.view(np.uint32))
        else:
            ops.mrs_conv2d(idx, lv, cnt, shape, aug, kh, kh, n, stride, pad, dev(bias), out=off)
        assert torch.equal(off.view(torch.int32), y.view(torch.int32))
    # the sums alone
    y2 = ops.mrs_conv2d(idx, lv, cnt, shape, aug, kh, kh, n, stride, pad, dev(bias))
    assert torch.equal(y2.view(torch.int32), y.view(torch.int32))


# (b, h, w, c_in), non-zeros, stride, pad, c_out, n; in slices: how many, parts of a list;
# the kernel that adds the sums a k-WTA follows
WIDE_CASES = [
    ((2, 8, 8, 64), 20, 1, 0, 512, 16, (2, 2), "fused"),
    ((1, 1, 127, 64), 64, 1, 0, 512, 16, (2, 2), "fused"),       # a short last tile, full lists
    ((1, 8, 12, 36), 9, 1, 0, 768, 8, (3, 2), "fused"),          # two sets a lane
    ((2, 14, 14, 128), 12, 1, 0, 512, 16, (2, 4), "fused"),      # four parts in pairs
    ((3, 9, 9, 8), 5, 1, 1, 512, 16, (2, 1), "fused"),           # padding, one part
    ((4, 14, 14, 128), 12, 2, 0, 1024, 16, (4, 2), "tiled"),     # stride 2
    ((1, 14, 14, 256), 120, 1, 0, 1024, 16, (4, 4), "tiled"),    # four parts in order, long lists
    ((1, 14, 14, 128), 40, 1, 0, 512, 8, (2, 2), "tiled"),
    ((1, 5, 7, 64), 30, 1, 0, 1536, 16, (6, 1), "tiled"),
    ((1, 9, 9, 512), 50, 1, 0, 1024, 16, None, "tiled"),         # the table takes two blocks
    ((3, 9, 9, 64), 8, 1, 0, 384, 16, None, "fused"),            # not a multiple of 256
    ((3, 9, 9, 64), 8, 1, 0, 512, 4, None, "fused"),             # sets of four
]


@pytest.mark.parametrize("case", WIDE_CASES, ids=[str(i) for i in range(len(WIDE_CASES))])
def test_wide_sums_in_slices(case):
    """Sums of a 1x1 layer of more than 256 channels, which go in slices of 256:
    within tolerance of the oracle, and the bits of the sums that the layer with
    a k-WTA keeps (cs_mrs_kwta_conv2d: "cs_mrs_conv2d followed by k-WTA"), which
    run on the fused or the table-slice kernel."""
    shape, nnz, stride, pad, c_out, n, wide, kept_path = case
    r = np.random.default_rng(sum(shape) + c_out + n)
    b, h, w, c = shape
    x = np.zeros((b * h * w, c), np.float32)
    for i in range(len(x)):
        m = (nnz, nnz // 3, 0, min(c, 2 * nnz), 1, c)[i % 6]
        x[i, r.permutation(c)[:m]] = r.normal(size=m)
    W = np.zeros((c_out // n, n, c), np.float32)
    np.put_along_axis(W, r.integers(0, n, (c_out // n, 1, c)),
                      r.normal(size=(c_out // n, 1, c)).astype(np.float32), axis=1)
    W = W.reshape(c_out, c)
    bias = r.normal(size=c_out).astype(np.float32)
    plan = [ops.mrs_plan(torch.float32, c, shape, 1, 1, stride, pad, c_out, n, 1, k)
            for k in (-1, c_out // 16)]
    assert plan[1]["path"] == kept_path and plan[1]["kwta"] == "separate", plan
    if wide is None:
        assert plan[0]["path"] == kept_path, plan
    else:
        assert (plan[0]["slices"], plan[0]["list_parts"]) == wide, plan
        assert plan[0]["select"] == 9 and plan[0]["table_blocks"] == 1, plan
    idx, lv, cnt = ops.compact(dev(x))
    aug = ops.aug_to_device(ops.pack(W, n)[0])
    args = (idx, lv, cnt, shape, aug, 1, 1, n, stride, pad)
    W4 = W.reshape(c_out, 1, 1, c)
    ref = o.conv2d_nhwc(x.reshape(shape), W4, stride, pad, bias)
    S = o.abs_sum_conv(x.reshape(shape), W4, stride, pad) + np.abs(bias)
    got = ops.mrs_conv2d(*args, dev(bias))
    assert_f32_close(host(got).reshape(-1, c_out), ref.reshape(-1, c_out), S.reshape(-1, c_out),
                     "sums")
    for bd in (dev(bias), None):
        got = ops.mrs_conv2d(*args, bd)
        kept = ops.mrs_kwta_conv2d(*args, bd, k=c_out // 16)[0]
        assert torch.equal(got.view(torch.int32).flatten(), kept.view(torch.int32).flatten())
        whole = ops.conv2d(dev(x.reshape(shape)), aug, 1, 1, n, stride, pad, bd)
        assert torch.equal(whole.view(torch.int32).flatten(), kept.view(torch.int32).flatten())
