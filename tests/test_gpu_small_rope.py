"""GPU parity of the rotary scores in the kernel for small decode problems (bf16): two and four token blocks per workgroup, heads of 64 and
128, group sizes, sequence ends inside and at the edges of a block; every output element against the fp64 oracle."""
import pytest
import torch

from paper_2603_22910_amd import synth

import oracle_ref as ref
from test_gpu_parity import check, host, make_dw

pytestmark = pytest.mark.gpu

CASES = [                                # H_q, H_kv, d, m, lengths
    (8, 2, 128, 128, (31, 32, 33, 1)),   # tiles of 32 tokens
    (3, 3, 128, 0, (17, 64)),            # one query head per KV head
    (6, 2, 128, 64, (200,)),             # three; a split head
    (8, 2, 64, 64, (15, 16, 47, 300)),   # heads of 64, an odd last head
    (6, 6, 64, 0, (129,)),
    (16, 16, 128, 0, (700, 63, 65)),     # more than 240 workgroups of 32: tiles of 64
    (32, 8, 128, 512, (4000,)),
    (32, 32, 64, 512, (900, 1)),
]


@pytest.mark.parametrize("window", [None, (4, 16)])
@pytest.mark.parametrize("H_q,H_kv,d,m,lens", CASES)
def test_small_rotary_scores(H_q, H_kv, d, m, lens, window):
    inp = synth.generate(synth.Workload("small_rope", "bf16", H_q, H_kv, d, m, seed=82, seq_lens=lens))
    dw = make_dw(inp, 0)
    rope = synth.rope_tables(d, max(lens))
    win = None
    if window:
        wk, wv = synth.window_rows(inp, *window)
        win = (wk, wv, *window)
    out, lse = dw.decode_ex(rope, win)
    torch.cuda.synchronize()
    o_ref, l_ref = ref.decode_paper_ref(inp, rope, win)
    check(host(out), o_ref, "bf16", f"{H_q} {H_kv} {d} {m} {lens} {window}")
    assert abs(host(lse) - l_ref).max() <= 2e-2
