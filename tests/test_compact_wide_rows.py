"""The vectorised compaction where two rows of 17 to 32 vectors share a
wavefront (groups of 32 lanes): the lane arithmetic as a CPU model (every load
inside the input and every list position inside its row, the lists equal to the
rows' non-zeros), and on the GPU against the oracle's compaction around the
edges of the groups and of the one-row passes beyond them."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import cs_oracle as o
from tests.test_compact_addresses import put


def rows_of_nonzeros(rows, c, dtype, seed):
    r = np.random.default_rng(seed)
    x = np.zeros((rows, c), dtype=dtype)
    for i in range(rows):
        nnz = (0, 1, c // 10, c)[i % 4]                    # empty, one, sparse, full
        at = r.choice(c, size=nnz, replace=False)
        x[i, at] = r.integers(1, 100, size=nnz) if dtype == np.int8 else r.normal(size=nnz)
    return x


@pytest.mark.parametrize("rows,c,dtype", [(7, 128, np.float32), (5, 68, np.float32),
                                          (9, 512, np.int8), (1, 272, np.int8)])
def test_two_rows_per_wavefront_model(rows, c, dtype):
    E = 16 // np.dtype(dtype).itemsize
    NL, lg = c // E, 5
    assert 16 < NL <= 32
    x = rows_of_nonzeros(rows, c, dtype, rows + c)
    idx = np.full((rows, c), -1, dtype=np.int64)
    val = np.zeros((rows, c), dtype=dtype)
    cnt = np.full(rows, -1, dtype=np.int64)
    loads = []
    blocks = (-(-rows // 2) + 3) // 4                      # two rows a wavefront, four of them
    for w in range(4 * blocks):
        for r0 in range(2 * w, rows, 8 * blocks):
            q, nl, rows_of, vi_of = {}, np.zeros(64, dtype=np.int64), {}, {}
            for lane in range(64):
                row, p = r0 + (lane >> lg), lane & 31
                if row < rows and p < NL:
                    a = row * c + p * E
                    assert 0 <= a and a + E <= rows * c
                    loads.append(a)
                    q[lane] = x.reshape(-1)[a:a + E]
                    nl[lane] = int((q[lane] != 0).sum())
                    rows_of[lane], vi_of[lane] = row, p
            tot = put(nl, q, q, vi_of, np.zeros(64, dtype=np.int64), lg, rows_of, idx, val, c, E)
            for lane in (0, 32):
                if r0 + (lane >> lg) < rows:
                    cnt[r0 + (lane >> lg)] = tot[lane]
    assert sorted(loads) == list(range(0, rows * c, E))
    for i, (ii, vv) in enumerate(o.compact_rows(x)):
        assert cnt[i] == len(ii)
        assert np.array_equal(idx[i, :cnt[i]], ii) and np.array_equal(val[i, :cnt[i]], vv)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,c,dtype", [
    (31, 68, np.float32), (30, 96, np.float32), (1001, 128, np.float32),   # 17, 24, 32 vectors
    (13, 132, np.float32), (9, 256, np.float32), (9, 260, np.float32),     # 33, 64, 65
    (6, 1024, np.float32), (6, 1028, np.float32), (5, 2052, np.float32),   # 256, 257, 513
    (40, 272, np.int8), (33, 512, np.int8), (7, 528, np.int8), (3, 8192, np.int8),
])
def test_compaction_matches_oracle(rows, c, dtype):
    from paper_2112_13896_amd import ops
    from tests.gpu_util import dev, host
    x = rows_of_nonzeros(rows, c, dtype, rows + c)
    idx, val, cnt = (host(t) for t in ops.compact(dev(x)))
    for i, (ii, vv) in enumerate(o.compact_rows(x)):
        assert cnt[i] == len(ii)
        assert np.array_equal(idx[i, :cnt[i]].view(np.uint16), ii)
        assert np.array_equal(val[i, :cnt[i]], vv)
