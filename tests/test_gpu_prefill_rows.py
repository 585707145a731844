"""GPU parity of the twelve-wave prefill attention: blocks of 384 (query, head) rows of a KV head and the shares of their
keys, at the edges of both; every output element against the fp64 oracle."""
import pytest
import torch

from paper_2603_22910_amd import binding as ek
from paper_2603_22910_amd import synth

import oracle_ref as ref
from test_gpu_parity import check, host, make_dw

pytestmark = pytest.mark.gpu

CASES = [                                # H_q, H_kv, d, m, tokens, queries
    (8, 2, 64, 64, 2100, 16),            # 64 rows of a block: ten of its waves only copy; 11 shares of 3 tiles
    (8, 2, 64, 64, 6200, 96),            # exactly one block of rows; 32 shares
    (8, 2, 64, 64, 2100, 97),            # four rows in the second block
    (6, 2, 128, 128, 1500, 129),         # three heads per KV head: rows 384 + 3
    (4, 4, 64, 64, 1100, 390),           # one head per KV head
    (4, 2, 64, 64, 1024, 1024),          # whole chunk, split: shares past the diagonal of the early blocks
    (2, 2, 128, 128, 1500, 1030),        # more than 1024 queries behind cached tokens
    (10, 2, 64, 0, 1029, 7),             # five heads, blocks of 35 rows
]


def run(H_q, H_kv, d, m, plen, pq):
    w = synth.Workload("prefill_rows", "bf16", H_q, H_kv, d, m, seed=81, seq_lens=(8,), prefill_len=plen, prefill_q=pq)
    inp = synth.generate(w)
    return inp, make_dw(inp, 0)


@pytest.mark.parametrize("H_q,H_kv,d,m,plen,pq", CASES)
def test_rows_and_shares(H_q, H_kv, d, m, plen, pq):
    inp, dw = run(H_q, H_kv, d, m, plen, pq)
    out, lse = dw.prefill()
    torch.cuda.synchronize()
    o_ref, l_ref = ref.prefill_ref(inp)
    check(host(out), o_ref, "bf16", f"{H_q} {H_kv} {d} {m} {plen} {pq}")
    assert abs(host(lse) - l_ref).max() <= 2e-2


@pytest.mark.parametrize("plen,pq", [(6200, 16), (1500, 1030)])
def test_least_workspace(plen, pq):
    """The number of shares follows from the workspace's size: nothing is written past its end, from the least one that is accepted to
    one just short of what the launch would use, and with all of it that tail is written."""
    inp, dw = run(8, 2, 64, 64, plen, pq)
    o_ref = ref.prefill_ref(inp)[0]
    full, need, lo = dw.workspace, dw.workspace.numel(), 0
    while need - lo > 256:
        mid = (need + lo) // 512 * 256
        dw.workspace = full[:mid]
        try:
            dw.prefill()
            need = mid
        except ek.EchoKVError:
            lo = mid
    assert need < full.numel()

    def tail_written(size, begin):
        full[begin:] = 0xA5
        dw.workspace = full[:size]
        dw.out_prefill.fill_(float("nan"))
        out, _ = dw.prefill()
        torch.cuda.synchronize()
        check(host(out), o_ref, "bf16", f"workspace {size} of {full.numel()}")
        return not bool((full[begin:] == 0xA5).all())

    assert tail_written(full.numel(), need)
    for eighth in range(8):
        size = need + (full.numel() - need) * eighth // 2048 * 256
        assert not tail_written(size, size), size
