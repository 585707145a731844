"""GPU parity of the score and value epilogues of the kernel for large problems at every number of query heads per KV head: up to two on
the vector unit, beyond on the matrix pipe four at a time, so 3, 5, 6 and 7 leave a part of the last four unused; heads of 64 and 128, a
column tile that is not full, slots of which one wave's half or all of it lies past the end; every output element against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2603_22910_amd import binding as ek
from paper_2603_22910_amd import synth

import oracle_ref as ref
from test_gpu_parity import check, host, make_dw

pytestmark = pytest.mark.gpu

CASES = [(128, g) for g in range(1, 9)] + [(64, g) for g in range(1, 5)]      # d, query heads per KV head
LENS = (300, 64, 65, 129, 1)


@pytest.mark.parametrize("extras", [pytest.param(False, id="plain"), pytest.param(True, id="rope+window")])
@pytest.mark.parametrize("flags", [pytest.param(ek.FLAG_STAGED, id="fused"), pytest.param(ek.FLAG_ABSORB_V, id="absorb_v")])
@pytest.mark.parametrize("d,G", CASES)
def test_group_sizes(d, G, flags, extras):
    H_kv = 4 if d == 128 else 6                                    # three / five predicted heads: 1.5 / 1.25 column tiles
    inp = synth.generate(synth.Workload("groups", "bf16", H_kv * G, H_kv, d, d, seed=91, seq_lens=LENS))
    dw = make_dw(inp, flags)
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
