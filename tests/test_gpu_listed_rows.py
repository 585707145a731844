"""Appends of few rows, whose destinations the host lists, on both sides of the limits (lists of 32 and of 64 rows; more go by the
sequence metadata), with sequences that get none, and the window's ring with rows that leave it in the same call: every byte of the
pools against an enumeration of the rows."""
import numpy as np
import pytest
import torch

from paper_2603_22910_amd import binding as ek

pytestmark = pytest.mark.gpu
H_KV, D_HEAD, M = 4, 64, 64
D = H_KV * D_HEAD
DEV = "cuda:0"


def rows_of(batch, total):
    """`total` new rows over the sequences, none for every third while there are others."""
    n = np.zeros(batch, dtype=np.int32)
    takers = [b for b in range(batch) if b % 3 != 1] or [0]
    for i in range(total):
        n[takers[i % len(takers)]] += 1
    return n


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("batch,total", [(1, 1), (5, 31), (32, 32), (40, 33), (64, 64), (1, 65), (3, 128), (150, 31), (150, 63), (1, 32)])
def test_listed_rows(batch, total, dtype):
    n_sink, n_recent = 2, 5
    n_new = rows_of(batch, total)
    before = np.array([(7 * b) % 11 for b in range(batch)], dtype=np.int32)
    caps = (before + n_new + 3).astype(np.int32)
    starts = np.concatenate([[0], np.cumsum(caps)[:-1]]).astype(np.int64)
    pool = int(caps.sum())
    g = torch.Generator(device=DEV)
    g.manual_seed(total * 1000 + batch)
    new = [torch.randn(total, D, generator=g, device=DEV).to(dtype) for _ in range(2)]
    shape = ek.make_shape(8, H_KV, D_HEAD, M, "bf16" if dtype == torch.bfloat16 else "f32")
    first = np.concatenate([[0], np.cumsum(n_new)[:-1]])
    for width in (D, M):
        k, v = (torch.randn(pool, width, generator=g, device=DEV).to(dtype) for _ in range(2))
        want = [k.clone(), v.clone()]
        for b in range(batch):
            at = int(starts[b] + before[b])
            for w, src in zip(want, new):
                w[at:at + n_new[b]] = src[first[b]:first[b] + n_new[b], :width]
        cache = ek.LayerCache(k, v, width, pool, list(starts), list(before), list(caps))
        ek.cache_append(shape, cache, new[0], new[1], n_new)
        torch.cuda.synchronize()
        assert torch.equal(k, want[0]) and torch.equal(v, want[1])
        assert list(cache.seq_len) == list(before + n_new)
    win = [torch.randn(batch, n_sink + n_recent, D, generator=g, device=DEV).to(dtype) for _ in range(2)]
    want = [w.clone() for w in win]
    for b in range(batch):
        for i in range(n_new[b]):            # in order: a later row overwrites what leaves the ring
            p = int(before[b]) + i
            row = p if p < n_sink else n_sink + (p - n_sink) % n_recent
            for w, src in zip(want, new):
                w[b, row] = src[first[b] + i]
    ek.window_append(shape, win[0], win[1], n_sink, n_recent, before, new[0], new[1], n_new)
    torch.cuda.synchronize()
    assert torch.equal(win[0], want[0]) and torch.equal(win[1], want[1])
