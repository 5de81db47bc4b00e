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
