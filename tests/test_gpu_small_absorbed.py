"""GPU parity of the absorbed modes on short sequences: the 32-token score kernel (edges of its tiles, partial
128-dim stages, fewer stages than waves, the grid size at which it ends), value splits below 1024 tokens with and
without statistics of their own, their number, and the plan that a workspace without room for them falls back to."""
import numpy as np
import pytest
import torch

from paper_2603_22910_amd import binding as ek
from paper_2603_22910_amd import synth
from paper_2603_22910_amd.harness import DeviceWorkload

import oracle_ref as ref
from test_gpu_parity import check, host, make_dw

pytestmark = pytest.mark.gpu

CASES = [                                      # H_q, H_kv, d, m, lengths
    (8, 4, 128, 128, (31, 32, 33, 129)),       # edges of 32-token tiles and of slots
    (6, 3, 64, 64, (100, 1)),                  # D = 192, m = 64: two partial stages of three
    (40, 5, 128, 64, (200,)),                  # 40 query heads: the second block of 32 is mostly empty
    (2, 2, 64, 64, (8192,)),                   # 256 workgroups of the 32-token kernel: one round
    (2, 2, 64, 64, (8193,)),
    (2, 2, 64, 64, (12288,)),                  # 384: its last grid
    (2, 2, 64, 64, (12289,)),
    (8, 8, 128, 512, (20,) * 128 + (65,)),     # 129 sequences, two launch groups, one 32-token workgroup each but the last
    (40, 5, 128, 128, (25,) * 40 + (130,)),    # blocks of heads; the queries of 41 sequences are over 1 MB
    (32, 8, 128, 512, (1500, 700)),            # several splits of 128 tokens per sequence
]
MODES = [pytest.param(ek.FLAG_ABSORBED, id="absorbed"), pytest.param(ek.FLAG_ABSORB_V, id="absorb_v")]


@pytest.mark.parametrize("flags", MODES)
@pytest.mark.parametrize("H_q,H_kv,d,m,lens", CASES)
def test_short_absorbed_against_the_oracle(H_q, H_kv, d, m, lens, flags):
    inp = synth.generate(synth.Workload("absorbed", "bf16", H_q, H_kv, d, m, seed=74, seq_lens=lens))
    out, lse = make_dw(inp, flags).decode()
    torch.cuda.synchronize()
    o_ref, l_ref = ref.decode_ref(inp)
    check(host(out), o_ref, "bf16", f"{H_q} {H_kv} {d} {m} {lens}")
    assert np.abs(host(lse) - l_ref).max() <= 2e-2


@pytest.mark.parametrize("flags", MODES)
def test_sums_of_few_and_many_value_workgroups(flags):
    """Up to 256 workgroups of the value pass each wave adds up a quarter of the heads, past that the sums meet in a tree: the same bits.
    Three column tiles: 255 workgroups of 85 sequences, 258 of 86."""
    inp = synth.generate(synth.Workload("absorbed_sums", "bf16", 8, 4, 128, 128, seed=84, seq_lens=tuple(100 + i % 29 for i in range(86))))
    dw = DeviceWorkload(inp, out_dtype="f32", flags=flags)
    many = dw.decode()[0].clone()
    check(host(many), ref.decode_ref(inp)[0], "bf16", "86 sequences")
    dw.anchor, dw.target = dw.anchor_all.view(0, 85), dw.target_all.view(0, 85)
    few = dw.decode()[0]
    assert torch.equal(few[:85], many[:85])


@pytest.mark.parametrize("flags", MODES)
def test_workspace_of_splits_of_1024_tokens_is_still_accepted(flags):
    H_q, D, m, L, nseq = 16, 1024, 512, 1500, 2
    inp = synth.generate(synth.Workload("absorbed_ws", "bf16", H_q, 8, 128, m, seed=75, seq_lens=(L,) * nseq))
    dw = DeviceWorkload(inp, flags=flags)
    a256 = lambda x: (x + 255) // 256 * 256
    d_in, slots, splits, pad = D + m, nseq * 12, nseq * 2, 32            # 12 slots of 128 and 2 splits of 1024 tokens each
    need = (a256(nseq * pad * d_in * 2) + a256(pad * slots * 128 * 4) + a256(splits * pad * 2 * 4) + a256(splits * pad * d_in * 4)
            + a256(nseq * H_q * d_in * 4) + a256(6 * nseq * H_q * 128 * 4) + a256(nseq * H_q * 2 * 4)
            + a256(nseq * H_q * 128 * 4) + a256(nseq * H_q * 2 * 4))
    dw.workspace = dw.workspace[:need]
    out, lse = dw.decode()
    torch.cuda.synchronize()
    o_ref, _ = ref.decode_ref(inp)
    check(host(out), o_ref, "bf16", "workspace without room for splits of 128 tokens")
    dw.workspace = dw.workspace[:need - 256]
    with pytest.raises(ek.EchoKVError) as e:
        dw.decode()
    assert e.value.code == ek.ERR_WORKSPACE


def workspace_end(H_q, d, d_in, lens, splits):
    """Bytes of workspace that a call with `splits` splits of the value pass writes up to."""
    a256 = lambda x: (x + 255) // 256 * 256
    n, pad, slots = len(lens), (H_q + 31) // 32 * 32, sum((L + 127) // 128 for L in lens)
    slices = max(1, min(64, d_in // 256))
    slices = -(-d_in // (-(-(-(-d_in // slices)) // 64) * 64))
    return (a256(n * pad * d_in * 2) + a256(pad * slots * 512) + a256(splits * pad * 8) + a256(splits * pad * d_in * 4)
            + a256(n * H_q * d_in * 4) + a256(slices * n * H_q * d * 4) + n * H_q * 8)


SPLITS = [                                       # H_q, H_kv, m, sequences, length, tokens per split
    (64, 8, 896, 16, 700, 1024),                 # one split each: 256 workgroups already, no launch to join them
    (64, 8, 896, 16, 1000, 1024),
    (32, 8, 512, 16, 1000, 512),
    (32, 8, 512, 2, 1500, 128),
    (64, 8, 896, 4, 700, 256),                   # few predicted dims: only the absorbed plan asks for workspace
    (32, 8, 512, 1, 128, 128),                   # one split that works out its own statistics
]


@pytest.mark.parametrize("more", [pytest.param(0, id="asked"), pytest.param(64 << 20, id="larger")])
@pytest.mark.parametrize("H_q,H_kv,m,n,L,ts", SPLITS)
def test_tokens_per_split(H_q, H_kv, m, n, L, ts, more):
    """The same in the workspace that was asked for and in a larger one."""
    inp = synth.generate(synth.Workload("absorbed_splits", "bf16", H_q, H_kv, 128, m, seed=79, seq_lens=(L,) * n))
    dw = DeviceWorkload(inp, flags=ek.FLAG_ABSORBED)
    dw.workspace = torch.full((dw.workspace.numel() + more,), 0xA5, dtype=torch.uint8, device=dw.dev)
    out, _ = dw.decode()
    torch.cuda.synchronize()
    o_ref, _ = ref.decode_ref(inp)
    check(host(out), o_ref, "bf16", f"{H_q} {H_kv} {m} {n} {L}")
    end = int((dw.workspace != 0xA5).nonzero().max()) + 1
    want = workspace_end(H_q, 128, H_kv * 128 + m, (L,) * n, n * -(-L // ts))
    assert want - 8 < end <= want
