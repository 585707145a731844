"""Prefill chunks split over the keys: fewer key shares than a workspace of eight has room for cost no precision."""
import pytest
import torch

from paper_2603_22910_amd import synth
from paper_2603_22910_amd.harness import DeviceWorkload, error_metrics

import oracle_ref as ref
from test_gpu_parity import host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("plen,pq", [(7680, 500), (7680, 390)])
def test_probabilities_do_not_depend_on_the_shares_taken(plen, pq):
    """Eight possible shares of 15 key tiles of 64; five shares are taken of 500 queries (11 blocks of 384 rows per KV head), seven of 390
    (9 blocks).  Keys of one of the eight have one score, so that its probabilities are exactly 1 relative to its own reference; relative
    to the reference of a longer share they would be rounded to bf16, 2^-9 of them.  (A share that begins inside one of the eight has the
    same reference there: how other scores would round in it is not seen.)  What is left are fp32 sums of 7680 terms: 1e-5, the
    tolerance of fp32 inputs."""
    w = synth.Workload("shares", "bf16", 32, 4, 64, 256, seed=78, seq_lens=(8,), prefill_len=plen, prefill_q=pq)
    inp = synth.generate(w)                     # m = D: nothing is predicted, the keys are the stored ones
    rows = inp.rows(inp.n_decode)
    level = torch.tensor([0.9, -3.3, 5.1, 2.7, -7.7, 1.3, -2.1, 6.1])
    k = torch.zeros(plen, 4, 64)
    k[:, :, 0] = level[torch.arange(plen) // (15 * 64)][:, None]
    inp.K_r[rows] = k.view(plen, 256).to(inp.K_r.dtype)
    inp.q_prefill[:, :, 0] = 1.0
    out, lse = DeviceWorkload(inp, out_dtype="f32").prefill()
    torch.cuda.synchronize()
    o_ref, l_ref = ref.prefill_ref(inp)
    mx, rl = error_metrics(host(out), o_ref)
    print(f"[parity] max_abs={mx:.3e} rel_l2={rl:.3e}", flush=True)
    assert mx <= 1e-5 and rl <= 1e-5
    assert abs(host(lse) - l_ref).max() <= 1e-4
