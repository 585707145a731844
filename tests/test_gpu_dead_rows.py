"""What rows hold that stand for no token must not reach the output of a decode call: NaN in window rows that no position has filled, and
an infinite value in the last row of a sequence, which the streaming workgroups read again in place of rows past the end of their
chunk (0 times infinity is not 0).  Every way the query heads of a KV head share a pass, rows of 64 and 128 dims, both dtypes."""
import numpy as np
import pytest
import torch

from paper_2603_22910_amd import binding as ek
from paper_2603_22910_amd import synth

import oracle_ref as ref
from test_gpu_parity import TOL, check, host, make_dw

pytestmark = pytest.mark.gpu

LAYERS = [(4, 4, 128), (8, 4, 128), (16, 4, 128), (32, 4, 128), (12, 4, 128), (16, 4, 64), (8, 4, 64), (4, 4, 64)]      # H_q, H_kv, d
MODES = [pytest.param("bf16", 0, id="small"), pytest.param("bf16", ek.FLAG_STAGED, id="large"), pytest.param("bf16", ek.FLAG_UNFUSED, id="unfused"),
         pytest.param("bf16", ek.FLAG_ABSORB_V, id="absorb_v"), pytest.param("f32", 0, id="f32")]


@pytest.mark.parametrize("use_rope", [pytest.param(False, id="plain"), pytest.param(True, id="rope")])
@pytest.mark.parametrize("dtype,flags", MODES)
@pytest.mark.parametrize("H_q,H_kv,d", LAYERS)
def test_window_rows_without_a_token(H_q, H_kv, d, dtype, flags, use_rope):
    n_sink, n_recent, lens = 4, 24, (3, 1, 11, 200)              # only the last one fills its window
    inp = synth.generate(synth.Workload("dead", dtype, H_q, H_kv, d, 2 * d, seed=17, seq_lens=lens))
    win = synth.window_rows(inp, n_sink, n_recent)
    for b, n in enumerate(lens):
        held = [p if p < n_sink else n_sink + (p - n_sink) % n_recent for p in range(n)]
        empty = [r for r in range(n_sink + n_recent) if r not in held]
        for w in win:
            w[b, empty] = float("nan")
    window = (*win, n_sink, n_recent)
    rope = synth.rope_tables(d, max(lens)) if use_rope else None
    out, lse = make_dw(inp, flags).decode_ex(rope, window)
    torch.cuda.synchronize()
    o_ref, l_ref = ref.decode_paper_ref(inp, rope, window)
    check(host(out), o_ref, dtype, f"{H_q} {H_kv} {d}")
    assert np.abs(host(lse) - l_ref).max() <= (1e-5 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("use_rope", [pytest.param(False, id="plain"), pytest.param(True, id="rope")])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H_q,H_kv,d", LAYERS)
def test_row_read_again_past_the_end(H_q, H_kv, d, dtype, use_rope):
    """Every head retained: the rows go through the streaming workgroups alone, and one infinite value makes one dim of one KV head infinite."""
    inp = synth.generate(synth.Workload("dead", dtype, H_q, H_kv, d, H_kv * d, seed=18, seq_lens=(130, 1, 77)))
    for b in range(3):
        inp.V_r[inp.seq_start[b] + inp.seq_len[b] - 1, d + 5] = float("inf")
    rope = synth.rope_tables(d, 130) if use_rope else None
    dw = make_dw(inp, 0)
    out, _ = dw.decode_ex(rope, None) if use_rope else dw.decode()
    torch.cuda.synchronize()
    got, (want, _) = host(out), ref.decode_paper_ref(inp, rope) if use_rope else ref.decode_ref(inp)
    assert np.isposinf(want).any() and not np.isnan(want).any()
    assert (np.isposinf(got) == np.isposinf(want)).all()
    fin = np.isfinite(want)
    assert np.abs(got[fin] - want[fin]).max() <= TOL[dtype][0]


def poison(dw, inp):
    """NaN in every pool row outside the sequences and all over the workspace."""
    outside = torch.ones(inp.pool_tokens, dtype=torch.bool)
    for s, n in zip(inp.seq_start, inp.seq_len):
        outside[s:s + n] = False
    for t in (dw.K_a, dw.V_a, dw.K_r, dw.V_r):
        t[outside.to(t.device)] = float("nan")
    dw.workspace.fill_(255)


@pytest.mark.parametrize("use_rope", [pytest.param(False, id="plain"), pytest.param(True, id="rope+window")])
@pytest.mark.parametrize("dtype,flags", MODES + [pytest.param("bf16", ek.FLAG_ABSORBED, id="absorbed")])
@pytest.mark.parametrize("H_q,H_kv,d", [(4, 4, 128), (16, 4, 128), (8, 4, 64)])
@pytest.mark.parametrize("lens", [(300, 65, 1, 200), (1500, 1030)])
def test_pool_rows_outside_the_sequences(lens, H_q, H_kv, d, dtype, flags, use_rope):
    if use_rope and flags == ek.FLAG_ABSORBED:
        pytest.skip("absorbed decode: position-free keys only")
    inp = synth.generate(synth.Workload("dead", dtype, H_q, H_kv, d, 2 * d, seed=19, seq_lens=lens))
    dw = make_dw(inp, flags)
    poison(dw, inp)
    if use_rope:
        rope, window = synth.rope_tables(d, max(lens)), (*synth.window_rows(inp, 4, 24), 4, 24)
        out, lse = dw.decode_ex(rope, window)
        o_ref, l_ref = ref.decode_paper_ref(inp, rope, window)
    else:
        out, lse = dw.decode()
        o_ref, l_ref = ref.decode_ref(inp)
    torch.cuda.synchronize()
    check(host(out), o_ref, dtype, f"{H_q} {H_kv} {d} {lens}")
    assert np.abs(host(lse) - l_ref).max() <= (1e-5 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("use_rope", [pytest.param(False, id="plain"), pytest.param(True, id="rope")])
@pytest.mark.parametrize("dtype,plen,pq", [("bf16", 300, 70), ("bf16", 1500, 33), ("bf16", 1300, 1030), ("f32", 200, 19)])
@pytest.mark.parametrize("H_q,H_kv,d", [(4, 4, 128), (16, 4, 128), (8, 4, 64)])
def test_prefill_beside_unused_rows(H_q, H_kv, d, dtype, plen, pq, use_rope):
    inp = synth.generate(synth.Workload("dead", dtype, H_q, H_kv, d, 2 * d, seed=20, seq_lens=(8,), prefill_len=plen, prefill_q=pq))
    dw = make_dw(inp, 0)
    poison(dw, inp)
    rope = synth.rope_tables(d, plen) if use_rope else None
    out, _ = dw.prefill_ex(rope) if use_rope else dw.prefill()
    torch.cuda.synchronize()
    o_ref, _ = ref.prefill_paper_ref(inp, rope) if use_rope else ref.prefill_ref(inp)
    check(host(out), o_ref, dtype, f"{H_q} {H_kv} {d} {plen} {pq}")
