"""GPU parity of the score and value epilogues of the kernel for large problems at every number of query heads per KV head: scores without
rotary tables and value sums of up to two on the vector unit, of more on the matrix pipe four at a time, so 3, 5, 6 and 7 leave a part of the last four
unused (scores with tables: the fused kernel's on the matrix pipe for any number, the score kernel's by the same rule as without); heads of 64
and 128, weights row-major and packed, a column tile that is not full, behind a full one or alone, with even and odd numbers of k-tiles, slots of which one
wave's half or all of it lies past the end; every output element against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2603_22910_amd import binding as ek
from paper_2603_22910_amd import synth

import oracle_ref as ref
from test_gpu_parity import PACKED, check, host, make_dw

pytestmark = pytest.mark.gpu

# d, query heads per KV head, KV heads, m: three / five predicted heads are 1.5 / 1.25 column tiles
CASES = [(128, g, 4, 128) for g in range(1, 9)] + [(64, g, 6, 64) for g in range(1, 5)]
HALVES = [(128, g, 3, 64) for g in (1, 3, 8)] + [(128, 4, 3, 256), (64, 2, 4, 128), (64, 4, 3, 64)]      # 7 k-tiles (the split head is rebuilt); one tile
LENS = (300, 64, 65, 129, 1)


@pytest.mark.parametrize("extras", [pytest.param(False, id="plain"), pytest.param(True, id="rope+window")])
@pytest.mark.parametrize("flags", [pytest.param(ek.FLAG_STAGED, id="fused"), pytest.param(ek.FLAG_STAGED | PACKED, id="packed"),
                                   pytest.param(ek.FLAG_ABSORB_V, id="absorb_v")])
@pytest.mark.parametrize("d,G,H_kv,m", CASES + HALVES)
def test_group_sizes(d, G, H_kv, m, flags, extras):
    if flags & PACKED and m % d:
        pytest.skip("packed weights: whole heads only")
    inp = synth.generate(synth.Workload("groups", "bf16", H_kv * G, H_kv, d, m, seed=91, seq_lens=LENS))
    dw = make_dw(inp, flags)
    if flags & PACKED:
        dw.W_K, dw.W_V = dw.W_K_packed, dw.W_V_packed
    if extras:
        rope = synth.rope_tables(d, max(LENS))
        window = (*synth.window_rows(inp, 2, 5), 2, 5)
        out, lse = dw.decode_ex(rope, window)
        o_ref, l_ref = ref.decode_paper_ref(inp, rope, window)
    else:
        out, lse = dw.decode()
        o_ref, l_ref = ref.decode_ref(inp)
    torch.cuda.synchronize()
    check(host(out), o_ref, "bf16", f"{d} {G}")
    assert np.abs(host(lse) - l_ref).max() <= 2e-2
