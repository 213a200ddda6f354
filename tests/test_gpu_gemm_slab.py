"""GEMM shapes at the edges of the dispatch (gemm.hip, gemm_plan): every slab
configuration with ragged rows, columns and chunk counts, K ranges with and
without room for their partials, and operands off the 16-byte alignment that
loads into LDS need.  Small integers, so every order of summation gives the
oracle's product exactly."""
import numpy as np
import pytest

from oracle import dequant_int4_g64
from paper_2504_03664_amd import binding as B
from paper_2504_03664_amd.binding import DeviceBuffer as DB
from test_gpu_ops import run_gemm

pytestmark = pytest.mark.gpu

DECODE = [(9, 5136, 384), (16, 8192, 128), (13, 80, 640),           # M <= 16
          (1, 8208, 384), (16, 12305, 128), (3, 81, 256),             # (odd N: row-major only)
          (17, 80, 640), (32, 80, 2048), (31, 8208, 128), (20, 16400, 128), (32, 24592, 256),
          (33, 80, 384), (64, 144, 2048), (50, 16400, 128), (64, 24592, 128),
          (65, 80, 640), (128, 144, 2048), (100, 16400, 128), (127, 16400, 384)]
PREFILL = [(129, 528, 2048), (130, 768, 3072), (200, 1040, 8192), (257, 4112, 1024),
           (300, 16400, 128), (1030, 528, 1152)]


def _case(M, N, K, w4):
    rng = np.random.default_rng(M * 31 + N + K + w4)
    X = rng.integers(-1, 2, (M, K)).astype(np.float64)
    if not w4:
        W = rng.integers(-2, 3, (N, K)).astype(np.float64)
        return X, W, None, X @ W.T
    codes = rng.integers(0, 16, (N, K))
    q = (codes[:, 0::2] | (codes[:, 1::2] << 4)).astype(np.uint8)
    sm = np.empty((N, K // 64, 2), np.float16)
    sm[..., 0] = rng.choice([0.5, 1.0], (N, K // 64))
    sm[..., 1] = rng.choice([-3.0, 0.0], (N, K // 64))
    return X, None, (q, sm), X @ dequant_int4_g64(q, sm, np.float64).T


@pytest.mark.parametrize("M,N,K", DECODE + PREFILL)
@pytest.mark.parametrize("w4", [False, True])
def test_gemm_plan_edges_exact(M, N, K, w4):
    X, W, q, want = _case(M, N, K, w4)
    rng = np.random.default_rng(N)
    init = rng.integers(-100, 100, (M, N)).astype(np.float64)
    bias = rng.integers(-8, 9, N).astype(np.float64)
    for frag in (False, True) if N % 16 == 0 else (False,):
        for ws in (True, False):
            print(f"gemm plan M={M} N={N} K={K} w4={w4} frag={frag} workspace={ws}", flush=True)
            got = run_gemm(X, W, bias, B.PIPO_EPI_ADD_F32, init, w4=q, workspace=ws, frag=frag)
            assert np.array_equal(got.astype(np.float64), init + want + bias)
    got = run_gemm(X, W, bias, B.PIPO_EPI_RELU_F16, w4=q, frag=N % 16 == 0)
    assert np.array_equal(got, np.maximum(want + bias, 0).astype(np.float16))


@pytest.mark.parametrize("M", [4, 16, 40, 128, 300])
@pytest.mark.parametrize("w4", [False, True])
def test_gemm_unaligned_operands_exact(M, w4):
    """X two bytes, or INT4 codes four bytes, past a 16-byte boundary."""
    N, K = 5136, 256
    X, W, q, want = _case(M, N, K, w4)
    print(f"gemm unaligned M={M} w4={w4}", flush=True)
    dO = DB(M * N * 4)
    if w4:
        dX, dsm = DB.from_array(X.astype(np.float16)), DB.from_array(q[1])
        dW = DB.from_array(np.concatenate([np.zeros(4, np.uint8), q[0].reshape(-1)]))
        B.pipo_op_gemm_w4(dX.ptr, dW.ptr + 4, dsm.ptr, None, dO.ptr, M, N, K, B.PIPO_EPI_F32)
    else:
        dX = DB.from_array(np.concatenate([np.zeros(1, np.float16),
                                           X.astype(np.float16).reshape(-1)]))
        dW = DB.from_array(W.astype(np.float16))
        B.pipo_op_gemm_f16(dX.ptr + 2, dW.ptr, None, dO.ptr, M, N, K, B.PIPO_EPI_F32)
    B.pipo_dev_synchronize()
    assert np.array_equal(dO.to_array(np.float32, (M, N)).astype(np.float64), want)


# (M, N, K, w4): a workspace with room for part of the K ranges, where other
# tiles take over: narrow ones in decode and where those would be too many;
# 128 x 128 tiles, big tiles with fewer ranges or none, and gemm_tiled in prefill
PARTIAL = [(20, 144, 16384, True), (20, 144, 16384, False), (32, 8320, 2048, False),
           (40, 144, 16384, True), (64, 144, 16384, False), (70, 80, 16384, True),
           (100, 144, 8448, False), (130, 8208, 1024, False), (130, 20496, 2048, False),
           (130, 10256, 2048, False), (300, 12304, 1024, False), (300, 12304, 384, False),
           (130, 528, 8192, True), (130, 528, 8192, False), (200, 1040, 1024, True)]


@pytest.mark.parametrize("M,N,K,w4", PARTIAL)
def test_gemm_partial_workspace_exact(M, N, K, w4):
    """All of the workspace that the query asks for, a half, a quarter and one
    byte less than that, and none."""
    X, W, q, want = _case(M, N, K, w4)
    full = B.pipo_op_gemm_workspace_bytes(M, N, K, B.PIPO_W_INT4_G64 if w4 else B.PIPO_W_FP16)
    dX, dO, dWs = DB.from_array(X.astype(np.float16)), DB(M * N * 4), DB(max(full, 16))
    for frag in (False, True):
        if w4:
            ops = [DB.from_array(x) for x in (B.pipo_pack_w4(*q) if frag else q)]
            call = B.pipo_op_gemm_w4_frag if frag else B.pipo_op_gemm_w4
        else:
            W16 = W.astype(np.float16)
            ops = [DB.from_array(B.pipo_pack_f16(W16) if frag else W16)]
            call = B.pipo_op_gemm_f16_frag if frag else B.pipo_op_gemm_f16
        for nbytes in sorted({full, full // 2, full // 4, max(full // 4 - 1, 0), 0}):
            print(f"gemm workspace {nbytes} of {full} M={M} N={N} K={K} w4={w4} frag={frag}",
                  flush=True)
            call(dX.ptr, *[o.ptr for o in ops], None, dO.ptr, M, N, K, B.PIPO_EPI_F32,
                 dWs.ptr if nbytes else None, nbytes)
            B.pipo_dev_synchronize()
            assert np.array_equal(dO.to_array(np.float32, (M, N)).astype(np.float64), want)


@pytest.mark.parametrize("M,N,K", [(20, 80, 2048), (32, 8320, 2048), (32, 24592, 256),
                                   (20, 144, 16384), (33, 80, 384), (64, 24592, 128),
                                   (64, 144, 16384), (65, 80, 640), (100, 16400, 128),
                                   (127, 144, 2048), (128, 144, 16384)])
@pytest.mark.parametrize("w4", [False, True])
def test_gemm_unaligned_decode_exact(M, N, K, w4):
    """Every decode configuration with X two bytes, W eight bytes or the
    (scale, min) pairs two bytes past their alignment, with K ranges and
    without."""
    X, W, q, want = _case(M, N, K, w4)
    full = B.pipo_op_gemm_workspace_bytes(M, N, K, B.PIPO_W_INT4_G64 if w4 else B.PIPO_W_FP16)
    dO, dWs = DB(M * N * 4), DB(max(full, 16))

    def shifted(x, nbytes):
        return DB.from_array(np.concatenate([np.zeros(nbytes, np.uint8),
                                             np.ascontiguousarray(x).view(np.uint8).reshape(-1)]))

    for frag in (False, True):
        if w4:
            mats = B.pipo_pack_w4(*q) if frag else q
            call = B.pipo_op_gemm_w4_frag if frag else B.pipo_op_gemm_w4
        else:
            W16 = W.astype(np.float16)
            mats = (B.pipo_pack_f16(W16) if frag else W16,)
            call = B.pipo_op_gemm_f16_frag if frag else B.pipo_op_gemm_f16
        for shifts in ((2, 0, 0), (0, 8, 0), (0, 0, 2))[:3 if w4 else 2]:
            dX = shifted(X.astype(np.float16), shifts[0])
            ops = [shifted(m, s) for m, s in zip(mats, shifts[1:])]
            for nbytes in {full, 0}:
                print(f"gemm unaligned {shifts} M={M} N={N} K={K} w4={w4} frag={frag} ws={nbytes}",
                      flush=True)
                call(dX.ptr + shifts[0], *[o.ptr + s for o, s in zip(ops, shifts[1:])], None,
                     dO.ptr, M, N, K, B.PIPO_EPI_F32, dWs.ptr if nbytes else None, nbytes)
                B.pipo_dev_synchronize()
                assert np.array_equal(dO.to_array(np.float32, (M, N)).astype(np.float64), want)


# both sides of the rules that choose the kernel from K and the number of
# workgroups: the streaming kernel's two groups, with chunks of 256 and of 128
# k; skinny or slab at M <= 16; K ranges of big and of 128 x 128 tiles, and
# tiles of 128 x 128 through registers; big INT4 tiles
RULES = [(17, 8208, 4096), (31, 8208, 4352), (20, 8199, 3968), (32, 4112, 8192), (20, 4112, 8704),
         (12, 4112, 2432), (9, 4112, 2560), (16, 4096, 3072), (3, 4096, 1536), (3, 4081, 1664),
         (16, 5136, 3072), (16, 5136, 2944),
         (300, 4112, 1024), (600, 4112, 2048), (600, 4112, 3200), (130, 1040, 2048),
         (1030, 4112, 128), (1030, 4112, 1152), (1030, 4112, 2560),
         (1030, 7424, 256)]


@pytest.mark.parametrize("M,N,K", RULES)
@pytest.mark.parametrize("w4", [False, True])
def test_gemm_rule_edges_exact(M, N, K, w4):
    X, W, q, want = _case(M, N, K, w4)
    for frag in (False, True) if N % 16 == 0 else (False,):
        for ws in (True, False):
            print(f"gemm rules M={M} N={N} K={K} w4={w4} frag={frag} workspace={ws}", flush=True)
            got = run_gemm(X, W, None, B.PIPO_EPI_F32, w4=q, workspace=ws, frag=frag)
            assert np.array_equal(got.astype(np.float64), want)


# (M, N, K): the layouts' kernels differ (skinny and slab, streaming and slab,
# tiles through registers and big ones), with one K range and several
SAME_BITS = [(1, 4112, 1664), (16, 4096, 2048), (12, 4112, 2560), (9, 12304, 256),
             (17, 16400, 1280), (20, 16400, 384), (31, 144, 16384), (32, 144, 14464), (20, 528, 28672),
             (32, 8208, 4096), (17, 12304, 4352), (24, 4112, 8192), (40, 4112, 8192),
             (300, 20496, 512), (300, 12304, 1536), (600, 4112, 1024), (520, 4112, 4096),
             (770, 4112, 3072), (300, 5136, 6144)]


@pytest.mark.parametrize("M,N,K", SAME_BITS)
@pytest.mark.parametrize("w4", [False, True])
def test_gemm_layouts_same_bits(M, N, K, w4):
    """Row-major W gives the bits of fragment order, with all of the workspace,
    with half of it and without: random operands, whose sums show an order."""
    rng = np.random.default_rng(M + N * 3 + K)
    X = rng.standard_normal((M, K)).astype(np.float16)
    wfmt = B.PIPO_W_INT4_G64 if w4 else B.PIPO_W_FP16
    if w4:
        q = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
        sm = np.stack([rng.uniform(0.5, 1, (N, K // 64)), rng.uniform(-9, -6, (N, K // 64))],
                      -1).astype(np.float16)
        mats = ((q, sm), B.pipo_pack_w4(q, sm))
        calls = (B.pipo_op_gemm_w4, B.pipo_op_gemm_w4_frag)
    else:
        W = rng.standard_normal((N, K), dtype=np.float32).astype(np.float16)
        mats = ((W,), (B.pipo_pack_f16(W),))
        calls = (B.pipo_op_gemm_f16, B.pipo_op_gemm_f16_frag)
    full = B.pipo_op_gemm_workspace_bytes(M, N, K, wfmt)
    dX, dWs = DB.from_array(X), DB(max(full, 16))
    dev = [[DB.from_array(m) for m in ms] for ms in mats]
    dO = DB(M * N * 4)
    for nbytes in sorted({full, full // 2, 0}):
        print(f"gemm layouts M={M} N={N} K={K} w4={w4} workspace={nbytes} of {full}", flush=True)
        out = []
        for call, ops in zip(calls, dev):
            call(dX.ptr, *[o.ptr for o in ops], None, dO.ptr, M, N, K, B.PIPO_EPI_F32,
                 dWs.ptr if nbytes else None, nbytes)
            B.pipo_dev_synchronize()
            out.append(dO.to_array(np.uint32, (M, N)))
        assert np.array_equal(*out)
