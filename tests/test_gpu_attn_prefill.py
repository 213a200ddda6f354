"""Prefill attention where its workgroups number fewer than, as many as and
more than multiples of the eight compute dies they are dealt to: every
(sequence, head, query block) has to be taken exactly once (also with several
groups of pairs per die), and prompts around 32 tokens, the edge of the short form.  A sequence's
output does not depend on the others, so the bits are those of the sequence
alone; one sequence is held against the oracle (tolerance: probabilities
rounded to fp16 before P V)."""
import numpy as np
import pytest

from oracle import gqa_attention
from paper_2504_03664_amd import binding as B
from paper_2504_03664_amd.binding import DeviceBuffer as DB

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,P,H,Hkv,D", [(5, 17, 1, 1, 64), (8, 128, 1, 1, 128), (3, 129, 4, 2, 64),
                                         (3, 400, 7, 7, 128), (2, 600, 13, 13, 64),
                                         (9, 260, 8, 1, 128), (11, 129, 32, 8, 64), (5, 129, 63, 63, 64),
                                         (2, 770, 16, 8, 64),
                                         (3, 31, 8, 8, 128), (2, 32, 8, 2, 64), (2, 33, 5, 5, 128)])
def test_attn_prefill_every_block_once(b, P, H, Hkv, D):
    print(f"attn_prefill blocks b={b} P={P} H={H}/{Hkv} D={D}", flush=True)
    rng = np.random.default_rng(P + b + H)
    q = (rng.standard_normal((b, P, H * D)) * 0.3).astype(np.float16)
    kc = rng.standard_normal((P, b, Hkv * D)).astype(np.float16)
    vc = rng.standard_normal((P, b, Hkv * D)).astype(np.float16)

    def run(rows):
        k, v = (np.ascontiguousarray(x[:, rows]) for x in (kc, vc))
        dq, dk, dv = DB.from_array(q[rows]), DB.from_array(k), DB.from_array(v)
        do = DB.from_array(np.full(q[rows].shape, np.nan, np.float16))
        B.pipo_op_attn_prefill_gqa(dq.ptr, dk.ptr, dv.ptr, do.ptr, len(rows), P, H, Hkv, D)
        B.pipo_dev_synchronize()
        return do.to_array(np.uint16, q[rows].shape)

    got = run(list(range(b)))
    for i in range(b):
        assert np.array_equal(got[i], run([i])[0])
    want = gqa_attention(q[-1].astype(np.float64), kc[:, -1].astype(np.float64),
                         vc[:, -1].astype(np.float64), H, Hkv)
    assert np.abs(got[-1].view(np.float16) - want).max() <= 8e-3 * max(1.0, np.abs(want).max())
