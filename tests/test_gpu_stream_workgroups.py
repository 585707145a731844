"""GPU parity of the streaming workgroups behind the predictor product's: retained heads and window of a
decode call on the kernel for large problems, and retained heads' scores and window of the value-absorbed mode.  Chunk
counts on both sides of multiples of 8 (their order changes there), every way the query heads of a KV head
are grouped, rows of 64 and 128 dims, a layer whose heads are all retained, streams in launches of their own, by chunks or head after head; every output element against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2603_22910_amd import binding as ek
from paper_2603_22910_amd import synth

import oracle_ref as ref
from test_gpu_parity import check, host, make_dw

pytestmark = pytest.mark.gpu

# H_q, H_kv, d, m, lengths.  Chunks of 128 tokens up to 256 workgroups, of 512 up to 1024, then longer ones.
CASES = [
    (8, 4, 128, 128, (1100, 129, 1)),         # G = 2, 12 chunks: 8 and 4
    (8, 4, 128, 128, (4500, 600, 1)),         # 42 chunks: 40 and 2
    (12, 4, 64, 64, (900, 31)),               # G = 3: one query head at a time, 9 chunks
    (12, 4, 64, 64, (4100, 31)),              # 34 chunks
    (16, 4, 64, 128, (1024,)),                # G = 4, two retained heads, 8 chunks, no tail
    (16, 4, 64, 128, (4096,)),                # 32 chunks x 2 heads
    (32, 4, 128, 256, (257, 255)),            # G = 8: two groups per KV head
    (8, 8, 64, 512, (17000, 70)),             # every head retained; 134 chunks x 8 heads are too many: 35 of 512 tokens, 280 workgroups
    (16, 4, 64, 128, (17000, 70)),            # 134 x 2: just over one round, 35 x 2
    (28, 4, 128, 384, (25000, 70)),           # G = 7: 50 chunks x 21 are too many, 26 of 1024 tokens
    (56, 8, 128, 768, (300,) * 128),          # G = 7, 256 tiles: no unit idle, the streams ahead of the product, head after head
    (24, 8, 64, 384, (512,) * 127 + (500,)),  # G = 3: the same by chunks
    (32, 4, 128, 384, (500,) * 128),          # G = 8: only with the window and rotary tables
    (8, 8, 128, 896, (500,) * 128),           # G = 1, G = 2: 256 tiles and many retained rows, by chunks
    (16, 8, 128, 896, (500,) * 128),
    (16, 8, 64, 448, (500,) * 128),
]


@pytest.mark.parametrize("flags", [pytest.param(ek.FLAG_STAGED, id="fused"), pytest.param(ek.FLAG_ABSORB_V, id="absorb_v")])
@pytest.mark.parametrize("extras", [pytest.param(False, id="plain"), pytest.param(True, id="rope+window")])
@pytest.mark.parametrize("H_q,H_kv,d,m,lens", CASES)
def test_streams_against_the_oracle(H_q, H_kv, d, m, lens, extras, flags):
    inp = synth.generate(synth.Workload("streams", "bf16", H_q, H_kv, d, m, seed=73, seq_lens=lens))
    dw = make_dw(inp, flags)
    if extras:
        rope = synth.rope_tables(d, max(lens))
        window = (*synth.window_rows(inp, 4, 24), 4, 24)
        out, lse = dw.decode_ex(rope, window)
        o_ref, l_ref = ref.decode_paper_ref(inp, rope, window)
    else:
        out, lse = dw.decode()
        o_ref, l_ref = ref.decode_ref(inp)
    torch.cuda.synchronize()
    check(host(out), o_ref, "bf16", f"{H_q} {H_kv} {d} {m} {lens}")
    assert np.abs(host(lse) - l_ref).max() <= 2e-2
