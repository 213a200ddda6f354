"""Grouped-query decode attention at the edges of its shares: fewer keys than
waves, shares that end inside a 32-key block, four- and eight-wave
workgroups, splits, large scores, and a cache off 16-byte alignment; against
the oracle's attention.  Tolerance: fp16 output (2^-11) and hardware exp2."""
import numpy as np
import pytest

from oracle import gqa_attention
from paper_2504_03664_amd import binding as B
from paper_2504_03664_amd.binding import DeviceBuffer as DB

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,T,H,Hkv,D,scale,shift", [
    (1, 1, 2, 1, 128, 0.3, 0), (1, 7, 8, 1, 64, 0.3, 0), (2, 33, 16, 2, 128, 0.3, 0),
    (1, 257, 8, 4, 128, 30.0, 0), (3, 255, 12, 6, 64, 30.0, 0), (1, 2049, 8, 2, 128, 0.3, 0),
    (65, 40, 16, 4, 64, 0.3, 0), (33, 130, 32, 8, 128, 0.3, 0),
    (2, 100, 8, 2, 128, 0.3, 1), (33, 65, 32, 8, 64, 0.3, 1)])
def test_attn_decode_gqa_edges(b, T, H, Hkv, D, scale, shift):
    print(f"gqa edges b={b} T={T} H={H}/{Hkv} D={D} scale={scale} shift={shift}", flush=True)
    rng = np.random.default_rng(T * 7 + b + H)
    dkv = Hkv * D
    q = (rng.standard_normal((b, H * D)) * scale).astype(np.float16)
    kc = rng.standard_normal((T, b, dkv)).astype(np.float16)
    vc = rng.standard_normal((T, b, dkv)).astype(np.float16)
    pad = np.zeros(shift, np.float16)
    dk, dv = (DB.from_array(np.concatenate([pad, x.reshape(-1)])) for x in (kc, vc))
    dq, do = DB.from_array(q), DB(b * H * D * 2)
    ws_bytes = B.pipo_op_attn_decode_gqa_workspace_bytes(b, H, Hkv, D, T - 1)
    outs = []
    for n in {0, ws_bytes}:
        ws = DB(n) if n else None
        B.pipo_op_attn_decode_gqa(dq.ptr, dk.ptr + 2 * shift, dv.ptr + 2 * shift, do.ptr, b, H, Hkv,
                                  D, T - 1, B.PIPO_KV_FP16, ws.ptr if ws else None, n)
        B.pipo_dev_synchronize()
        outs.append(do.to_array(np.float16, (b, H * D)).astype(np.float64))
    for got in outs:
        for i in range(b):
            want = gqa_attention(q[i:i + 1].astype(np.float64), kc[:, i].astype(np.float64),
                                 vc[:, i].astype(np.float64), H, Hkv)[0]
            assert np.abs(got[i] - want).max() <= 2e-3 * max(1.0, np.abs(want).max())
