"""GPU parity of the small-problem decode kernel and of the rule that sends a call to it: lengths on
both sides of its tile sizes (16, 32 and 64 tokens) and of the workgroup counts at which the tile
size or the kernel changes, every output element against the fp64 oracle; and the fall-back to
the large kernel when the workspace holds only that one's partials."""
import numpy as np
import pytest
import torch

from paper_2603_22910_amd import binding as ek
from paper_2603_22910_amd import synth
from paper_2603_22910_amd.harness import DeviceWorkload

import oracle_ref as ref
from test_gpu_parity import PACKED, check, host, make_dw

pytestmark = pytest.mark.gpu

# H_q, H_kv, d, m, dtype, lengths.  Column tiles: 128 columns (fp32: one head).
CASES = [
    (8, 4, 128, 128, "bf16", (31, 32, 33, 1)),          # 3 column tiles, edges of a 32-token tile
    (8, 4, 128, 128, "bf16", (2560,)),                  # 240 workgroups: the last with 32-token tiles
    (8, 4, 128, 128, "bf16", (2561,)),                  # the first with 64-token tiles
    (8, 4, 128, 128, "bf16", (14976,)),                 # 702 of at most 704 workgroups: slower than the 256 x 256 kernel
    (8, 4, 128, 128, "bf16", (15000, 64, 65)),          # over it
    (10, 5, 64, 128, "bf16", (65, 129, 3)),             # three predicted heads of 64: half of the last tile is empty
    (16, 2, 128, 64, "bf16", (200, 63)),                # split head (r = 64), G = 8
    (4, 1, 64, 0, "bf16", (100,)),                      # d_in = 64: fewer steps than waves, the 256 x 256 kernel
    (4, 2, 64, 0, "bf16", (100,)),                      # d_in = 128: one step for each wave
    (8, 8, 64, 256, "f32", (15, 16, 17, 1)),            # 4 column tiles, edges of a 16-token tile
    (8, 8, 64, 256, "f32", (1024,)),                    # 256 workgroups: the last with 16-token tiles
    (8, 8, 64, 256, "f32", (1025, 700)),
    (2, 2, 64, 64, "f32", (196608, 31)),                # 6145 workgroups of at most 6144: the 256 x 256 kernel
    (6, 3, 128, 128, "f32", (40, 33)),
]
EXTRAS = [pytest.param(False, id="plain"), pytest.param(True, id="rope+window")]


@pytest.mark.parametrize("packed", [pytest.param(0, id="row-major"), pytest.param(PACKED, id="packed")])
@pytest.mark.parametrize("extras", EXTRAS)
@pytest.mark.parametrize("H_q,H_kv,d,m,dtype,lens", CASES)
def test_small_decode_against_the_oracle(H_q, H_kv, d, m, dtype, lens, extras, packed):
    if packed and (dtype != "bf16" or m % d or extras):
        pytest.skip("packed weights: whole heads of a bf16 layer")
    w = synth.Workload("small", dtype, H_q, H_kv, d, m, seed=71, seq_lens=lens)
    inp = synth.generate(w)
    dw = make_dw(inp, packed)
    if extras:
        rope = synth.rope_tables(d, max(lens))
        window = (*synth.window_rows(inp, 4, 24), 4, 24)
        out, lse = dw.decode_ex(rope, window)
        o_ref, l_ref = ref.decode_paper_ref(inp, rope, window)
    else:
        out, lse = dw.decode()
        o_ref, l_ref = ref.decode_ref(inp)
    torch.cuda.synchronize()
    check(host(out), o_ref, dtype, f"{w} {lens}")
    assert np.abs(host(lse) - l_ref).max() <= (1e-5 if dtype == "f32" else 2e-2)


def test_workspace_of_the_large_kernel_alone_is_still_accepted():
    w = synth.Workload("small_ws", "bf16", 8, 4, 128, 128, seed=72, seq_lens=(600,))
    inp = synth.generate(w)
    dw = DeviceWorkload(inp)
    a256 = lambda x: (x + 255) // 256 * 256
    slots = (600 + 127) // 128 + 1                      # one partial per 128 tokens, one for the window
    need = a256(slots * 8 * 128 * 4) + a256(slots * 8 * 2 * 4)
    dw.workspace = dw.workspace[:need]
    out, lse = dw.decode(); torch.cuda.synchronize()
    o_ref, l_ref = ref.decode_ref(inp)
    check(host(out), o_ref, "bf16", "workspace without room for 32-token partials")
    dw.workspace = dw.workspace[:need - 256]
    with pytest.raises(ek.EchoKVError) as e:
        dw.decode()
    assert e.value.code == ek.ERR_WORKSPACE


ROUTES = [                                       # H_q, H_kv, d, m, lengths, tokens per partial: 32, 64 or (256 x 256 kernel) 128
    (8, 4, 128, 128, (2560,), 32),
    (8, 4, 128, 128, (2561,), 64),
    (8, 4, 128, 128, (10880,), 64),              # 510 workgroups: two rounds
    (8, 4, 128, 128, (10881,), 128),             # 513
    (8, 8, 128, 896, (3200,) * 8, 128),          # 400, each unit streams seven retained heads as well
    (8, 8, 128, 768, (1600,) * 8, 64),           # 400, six retained heads of half as many tokens
]


@pytest.mark.parametrize("H_q,H_kv,d,m,lens,tok", ROUTES)
def test_kernel_taken(H_q, H_kv, d, m, lens, tok):
    """Which kernel ran, by how many partials it left in the workspace."""
    inp = synth.generate(synth.Workload("small_route", "bf16", H_q, H_kv, d, m, seed=80, seq_lens=lens))
    dw = DeviceWorkload(inp)
    dw.workspace.fill_(0xA5)
    out, _ = dw.decode()
    torch.cuda.synchronize()
    o_ref, _ = ref.decode_ref(inp)
    check(host(out), o_ref, "bf16", f"{H_q} {H_kv} {d} {m} {lens}")
    end = int((dw.workspace != 0xA5).nonzero().max()) + 1
    slots = sum(-(-L // tok) for L in lens)      # and one per sequence for a window, not written here
    want = ((slots + len(lens)) * H_q * d * 4 + 255) // 256 * 256 + slots * H_q * 8
    assert want - 8 < end <= want


LARGE_F32 = [                                    # H_q, H_kv, d, m, lengths
    (4, 2, 128, 128, (300, 129, 1)),             # G = 2
    (16, 4, 128, 128, (257, 70)),                # G = 4, three predicted heads: two column tiles, the second half empty
    (16, 4, 64, 64, (256, 255, 128)),            # G = 4, heads of 64
    (7, 7, 64, 64, (513, 31)),                   # six predicted heads of 64: both halves of a tile and a second tile
    (8, 2, 128, 64, (200, 140)),                 # split head
    (8, 4, 128, 0, (130,)),                      # nothing retained
]


@pytest.mark.parametrize("extras", EXTRAS)
@pytest.mark.parametrize("H_q,H_kv,d,m,lens", LARGE_F32)
def test_large_fp32_kernel_on_short_sequences(H_q, H_kv, d, m, lens, extras):
    """The fp32 256 x 256 kernel, which only very long sequences reach by themselves."""
    inp = synth.generate(synth.Workload("large_f32", "f32", H_q, H_kv, d, m, seed=81, seq_lens=lens))
    dw = DeviceWorkload(inp, flags=ek.FLAG_STAGED)
    if extras:
        rope = synth.rope_tables(d, max(lens))
        window = (*synth.window_rows(inp, 4, 24), 4, 24)
        out, lse = dw.decode_ex(rope, window)
        o_ref, l_ref = ref.decode_paper_ref(inp, rope, window)
    else:
        out, lse = dw.decode()
        o_ref, l_ref = ref.decode_ref(inp)
    torch.cuda.synchronize()
    check(host(out), o_ref, "f32", f"{H_q} {H_kv} {d} {m} {lens}")
    assert np.abs(host(lse) - l_ref).max() <= 1e-5
