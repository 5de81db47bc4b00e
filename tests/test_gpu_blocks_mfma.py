"""The matrix-core form of the block-CS dense-input layer (cs_conv2d_dense_blocks
for whole 16-channel tiles and windows up to 7x7) at the edges of its tiles:
one to four contraction steps, one to four 16-channel tiles a workgroup and
several channel slices, 1 to 4 input channels, odd and even strides, tiles of
one, two and four output rows, output rows and columns that end inside a tile,
several tiles across a row and several tiles of a workgroup one after another,
images whose last pixel ends the input (each case's plan is asserted).
int32 sums equal the oracle's dense convolution bit for bit; an output that is
not 16-byte aligned, or a channel count off the tiles, takes the routed kernel
and gives the same bits.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import cs_oracle as o
from paper_2112_13896_amd import ops
from tests.gpu_util import dev, host
from tests.test_gpu_dense_blocks import int8_block_weights

pytestmark = pytest.mark.gpu

# (b, h, w, c_in), kh, stride, pad, c_out, n, bias, and the plan: rows of a tile, tiles
# across, tiles, workgroups of a slice, slices, steps
CASES = [
    ((1, 5, 5, 3), 5, 1, 2, 16, 4, True, (1, 1, 5, 5, 1, 3)),
    ((2, 9, 17, 4), 3, 1, 1, 48, 4, False, (1, 1, 18, 18, 3, 1)),     # 17 columns
    ((1, 6, 33, 1), 1, 1, 0, 64, 4, True, (1, 1, 6, 6, 1, 1)),        # 4 bytes past the last pixel
    ((2, 7, 3, 2), 3, 3, 1, 32, 1, True, (1, 1, 6, 6, 1, 1)),         # output narrower than the window
    ((2, 30, 31, 3), 7, 2, 3, 128, 8, False, (1, 1, 30, 30, 2, 4)),
    ((1, 23, 300, 3), 7, 2, 3, 64, 4, True, (1, 1, 12, 12, 1, 4)),    # a wide row in one tile
    ((300, 8, 8, 3), 7, 2, 3, 64, 4, False, (2, 1, 600, 600, 1, 4)),
    ((1, 11, 11, 3), 5, 1, 2, 64, 16, True, (1, 1, 11, 11, 1, 3)),    # stride 1, 20-word tap rows
    ((1, 9, 1190, 3), 7, 2, 3, 64, 4, True, (1, 4, 20, 20, 1, 4)),    # the last tile across is short
    ((130, 7, 7, 3), 3, 1, 1, 64, 4, True, (2, 1, 520, 520, 1, 1)),   # the last two rows: one
    ((40, 100, 36, 3), 7, 2, 3, 64, 4, False, (4, 1, 520, 520, 1, 4)),   # the last four rows: two
    ((260, 6, 6, 3), 3, 1, 1, 48, 4, True, (4, 1, 520, 341, 3, 1)),   # a second tile for 179 of 341
    ((3, 40, 1480, 2), 3, 1, 1, 80, 4, False, (1, 2, 240, 204, 5, 1)),   # two across, some two each
]


@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
def test_matrix_core_blocks_match_oracle(case):
    shape, kh, stride, pad, c_out, n, has_bias, plan = case
    pl = ops.conv2d_dense_blocks_plan(shape, kh, kh, c_out, n, stride, pad)
    assert (pl["rows"], pl["segments"], pl["tiles"], pl["workgroups"], pl["slices"],
            pl["steps"]) == plan, pl
    r = np.random.default_rng(sum(shape) + 10 * c_out + kh)
    x = r.integers(-128, 128, size=shape).astype(np.int8)
    W = int8_block_weights(r, c_out, kh, kh, shape[3], n)
    bias = r.integers(-2**31, 2**31, size=c_out).astype(np.int32) if has_bias else None
    aug, kidb, _ = ops.pack_blocks(W.reshape(c_out, -1), n, shape[3])
    args = (dev(x), ops.aug_to_device(aug), dev(kidb), kh, kh, n, stride, pad,
            None if bias is None else dev(bias))
    y = ops.conv2d_dense_blocks(*args)
    ref = o.conv2d_nhwc(x, W, stride, pad, None)
    if bias is not None:
        ref = ref + bias.astype(np.int64)
    ref = ref.astype(np.int64).astype(np.int32)                   # sums wrap modulo 2^32
    assert np.array_equal(host(y), ref)
    # the routed kernel, taken when the output is not 16-byte aligned
    off = torch.empty(y.numel() + 1, dtype=torch.int32, device="cuda")[1:].view(y.shape)
    assert np.array_equal(host(ops.conv2d_dense_blocks(*args, out=off)), ref)
