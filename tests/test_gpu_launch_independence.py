"""The fused product's sums of a sequence are the same bits whatever other sequences the call decodes ahead of it or behind it."""
import pytest
import torch

from paper_2603_22910_amd import binding as ek
from paper_2603_22910_amd import synth

from test_gpu_parity import make_dw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [pytest.param(ek.FLAG_STAGED, id="row-major"), pytest.param(ek.FLAG_STAGED | ek.FLAG_W_PACKED, id="packed")])
@pytest.mark.parametrize("H_kv,d", [(8, 64), (11, 128)])          # 8 and 22 steps over the input dims, 2 and 6 column tiles
def test_bits_of_a_sequence_do_not_depend_on_the_others(H_kv, d, mode):
    inp = synth.generate(synth.Workload("order", "bf16", H_kv, H_kv, d, 0, seed=83, seq_lens=(900, 600, 2000)))
    dw = make_dw(inp, ek.FLAG_STAGED, out_dtype="f32")
    if mode & ek.FLAG_W_PACKED:
        dw.pack_weights()
    q, anchor, target = dw.q, dw.anchor, dw.target

    def decode(first, n):
        dw.q, dw.anchor, dw.target = q[first:first + n], anchor.view(first, n), target.view(first, n)
        out, lse = dw.decode()
        return out[1 - first].clone(), lse[1 - first].clone()

    alone = decode(1, 1)
    for first, n in ((0, 2), (1, 2), (0, 3)):                     # one ahead, one behind, both
        for a, b in zip(decode(first, n), alone):
            assert torch.equal(a, b), (first, n)
