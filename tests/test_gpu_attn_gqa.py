"""Grouped-query decode attention at the edges of its shares: fewer keys than
waves, shares that end inside a 32-key block, four- and eight-wave
workgroups, splits, large scores, and a cache off 16-byte alignment; against
the oracle's attention.  Tolerance: fp16 output (2^-11) and hardware exp2."""
import numpy as np
import pytest

from oracle import dequant_int4_g64, gqa_attention, quant_kv_int4_g64
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


def _run(q, kc, vc, H, Hkv, D, fmt=B.PIPO_KV_FP16, split=True):
    """kc, vc: [T][b][...] rows as the cache holds them"""
    T, b = kc.shape[:2]
    dq, dk, dv, do = DB.from_array(q), DB.from_array(kc), DB.from_array(vc), DB(b * H * D * 2)
    n = B.pipo_op_attn_decode_gqa_workspace_bytes(b, H, Hkv, D, T - 1) if split else 0
    ws = DB(n) if n else None
    B.pipo_op_attn_decode_gqa(dq.ptr, dk.ptr, dv.ptr, do.ptr, b, H, Hkv, D, T - 1, fmt,
                              ws.ptr if ws else None, n)
    B.pipo_dev_synchronize()
    return do.to_array(np.float16, (b, H * D))


@pytest.mark.parametrize("gap", [14, 17.5, 20, 23.5])
@pytest.mark.parametrize("T,D,split", [(200, 64, False), (8192, 128, True), (8192, 128, False)])
def test_attn_decode_gqa_small_probabilities(gap, T, D, split):
    """A key of value 0 in every 32 and a long tail `gap` below its score, of
    value 1000 or 50 000: the output is the tail's alone.  Tolerance: an fp16
    output (2^-11) and what 22 bits of each probability and the fp32 exp2 of
    an argument of 35 (2^-19 from rounding it) leave, twice over."""
    print(f"gqa tail gap={gap} T={T} D={D} split={split}", flush=True)
    H, Hkv = 8, 2
    q = np.zeros((1, H * D), np.float16)
    q[:, ::D] = 1
    kc = np.zeros((T, 1, Hkv * D), np.float16)
    vc = np.zeros((T, 1, Hkv * D), np.float16)
    vc[:] = 1000 if gap < 20 else 50000
    kc[:, :, ::D] = -gap
    kc[::32, :, ::D] = 0
    vc[::32] = 0
    got = _run(q, kc, vc, H, Hkv, D, split=split).astype(np.float64)
    want = gqa_attention(q.astype(np.float64), kc[:, 0].astype(np.float64),
                         vc[:, 0].astype(np.float64), H, Hkv)
    assert want.min() > 2.0 ** -14  # (a normal fp16 number)
    assert np.abs(got / want - 1).max() <= 2.0 ** -11 + 2 * (2.0 ** -22 + 2.0 ** -19)


@pytest.mark.parametrize("T,split", [(5, False), (70, False), (600, True), (600, False)])
@pytest.mark.parametrize("D", [64, 128])
def test_attn_decode_gqa_infinite_values(T, D, split):
    """An infinite value gives its sign in its own dimension and nothing else:
    for the last key (repeated past the end of a block), for one in the middle
    and for one whose score is 30 below the others; opposite infinities give
    NaN.  The other dimensions keep their bits."""
    print(f"gqa infinite values T={T} D={D} split={split}", flush=True)
    H, Hkv = 8, 2
    rng = np.random.default_rng(T + D)
    q = (rng.standard_normal((1, H * D)) * 0.3).astype(np.float16)
    kc = rng.standard_normal((T, 1, Hkv * D)).astype(np.float16)
    vc = rng.standard_normal((T, 1, Hkv * D)).astype(np.float16)
    q[:, ::D] = 1
    low = T // 2 + 1
    kc[low, :, ::D] = -30
    plain = _run(q, kc, vc, H, Hkv, D, split=split)
    inf = vc.copy()
    inf[T - 1, 0, 3::D] = np.inf
    inf[T // 2, 0, 20::D] = -np.inf
    inf[low, 0, 37::D] = np.inf
    inf[0, 0, 41::D], inf[T - 1, 0, 41::D] = np.inf, -np.inf
    got = _run(q, kc, inf, H, Hkv, D, split=split).reshape(H, D)
    assert (got[:, 3] == np.inf).all() and (got[:, 20] == -np.inf).all()
    assert (got[:, 37] == np.inf).all() and np.isnan(got[:, 41]).all()
    keep = [i for i in range(D) if i not in (3, 20, 37, 41)]
    assert np.array_equal(got[:, keep].view(np.uint16),
                          plain.reshape(H, D)[:, keep].view(np.uint16))


@pytest.mark.parametrize("b,T,H,Hkv,D", [
    (1, 1, 8, 4, 64), (1, 7, 8, 2, 128), (2, 33, 16, 4, 64), (1, 257, 8, 4, 128),  # eight waves
    (65, 40, 16, 4, 64), (33, 130, 32, 8, 128), (33, 2050, 16, 8, 64),             # four
    (65, 33, 32, 8, 128), (129, 64, 16, 4, 64), (130, 65, 8, 4, 128),              # two, four
    (129, 7, 8, 4, 128), (129, 32, 16, 4, 64), (257, 1, 16, 4, 64)])               # one
def test_attn_decode_gqa_waves_and_int4(b, T, H, Hkv, D):
    """Every number of waves, with as many blocks and more, over fp16 rows
    against the oracle (the first and last sequence) and over INT4 rows against
    the fp16 kernel on the expanded rows, bit for bit."""
    print(f"gqa waves b={b} T={T} H={H}/{Hkv} D={D}", flush=True)
    rng = np.random.default_rng(T * 11 + b)
    dkv = Hkv * D
    q = (rng.standard_normal((b, H * D)) * 0.3).astype(np.float16)
    rows = []
    for _ in range(2):
        codes, sm = quant_kv_int4_g64(rng.standard_normal((T * b, dkv)).astype(np.float16))
        packed = np.concatenate([codes, np.ascontiguousarray(sm.reshape(T * b, -1)).view(np.uint8)],
                                axis=1).reshape(T, b, -1)
        rows.append((packed, dequant_int4_g64(codes, sm, np.float64).astype(np.float16)
                     .reshape(T, b, dkv)))
    (k4, kc), (v4, vc) = rows
    for split in (True, False):
        got = _run(q, kc, vc, H, Hkv, D, split=split)
        for i in (0, b - 1):
            want = gqa_attention(q[i:i + 1].astype(np.float64), kc[:, i].astype(np.float64),
                                 vc[:, i].astype(np.float64), H, Hkv)[0]
            assert np.abs(got[i] - want).max() <= 2e-3 * max(1.0, np.abs(want).max())
        got4 = _run(q, k4, v4, H, Hkv, D, fmt=B.PIPO_KV_INT4_G64, split=split)
        assert np.array_equal(got.view(np.uint16), got4.view(np.uint16))
