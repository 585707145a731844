"""GPU parity of the prefill path's rotary embedding: predicted keys rotated on their way out of the predictor
product, whatever the number of its workgroups, retained keys by workgroups of the product's launch, also where no head is
predicted; every output element against the fp64 oracle."""
import pytest
import torch

from paper_2603_22910_amd import synth

import oracle_ref as ref
from test_gpu_parity import check, host, make_dw

pytestmark = pytest.mark.gpu

CASES = [                                # H_q, H_kv, d, m, tokens, queries
    (4, 2, 128, 128, 15104, 9),          # 59 token tiles x 1 column tile, twice: 118 workgroups
    (4, 2, 128, 128, 15105, 9),          # 120: one row in the last tile
    (8, 4, 64, 64, 15300, 5),            # heads of 64, 192 predicted dims
    (12, 6, 64, 0, 7700, 33),            # no retained head; the second column tile is half empty
    (4, 2, 64, 128, 700, 70),            # no predicted head: the launch rotates retained keys only
    (4, 4, 128, 256, 5, 5),
    (4, 2, 128, 128, 16, 16),            # rows are stored in blocks of 16 as far as the tile's tokens go
    (4, 2, 128, 128, 17, 9),
    (4, 2, 64, 0, 272, 20),
    (4, 2, 64, 0, 273, 20),
]


@pytest.mark.parametrize("H_q,H_kv,d,m,plen,pq", CASES)
def test_prefill_rope_routes(H_q, H_kv, d, m, plen, pq):
    w = synth.Workload("prefill_rope", "bf16", H_q, H_kv, d, m, seed=76, seq_lens=(8,), prefill_len=plen, prefill_q=pq)
    inp = synth.generate(w)
    dw = make_dw(inp, 0)
    rope = synth.rope_tables(d, plen)
    out, _ = dw.prefill_ex(rope)
    torch.cuda.synchronize()
    o_ref, _ = ref.prefill_paper_ref(inp, rope)
    check(host(out), o_ref, "bf16", f"{H_q} {H_kv} {d} {m} {plen} {pq}")


@pytest.mark.parametrize("plen,pq", [(3700, 385), (4500, 800), (6000, 1023)])
def test_prefill_key_shares_below_the_limit(plen, pq):
    """Two and three query blocks of 32 heads: fewer key shares than the workspace has room for."""
    w = synth.Workload("prefill_shares", "bf16", 32, 4, 64, 64, seed=77, seq_lens=(8,), prefill_len=plen, prefill_q=pq)
    inp = synth.generate(w)
    out, _ = make_dw(inp, 0).prefill()
    torch.cuda.synchronize()
    o_ref, _ = ref.prefill_ref(inp)
    check(host(out), o_ref, "bf16", f"{plen} {pq}")
