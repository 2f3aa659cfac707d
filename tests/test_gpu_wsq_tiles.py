"""The weights-SQ layer on both tiles of its kernel (128 and 256 tokens), one to several banks (fewer than the ring holds,
and more), ragged edges, aligned and unaligned rows of Y; and the activation quantiser at the edges of the row lengths it
keeps in registers.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle.wsq as W
import paper_2512_05409_amd as sq
from gpu_util import Guarded, dev
from test_gpu_wsq import case, consumer_order
from workloads import pack_int4

pytestmark = pytest.mark.gpu


# banks of 64: 256-token tiles where they make one full round of 256 (8 x 31); 9 x 29 are two, hardly begun, and go to the
# smaller tile.  Banks of 128: up to 256 of the smaller tiles, more of them in pairs on a compute unit (one, two and three
# banks), the 256-token tiles where they are one round of rows of 768 channels or more
@pytest.mark.parametrize("M,K,N,bank,pad", [(2100, 64, 3700, 64, 0), (2100, 320, 3650, 64, 3), (2048, 128, 4129, 128, 8),
                                            (1999, 384, 4200, 128, 3), (2000, 64, 3900, 64, 0),
                                            (2041, 320, 3850, 64, 3), (600, 256, 6600, 128, 3), (513, 768, 6700, 128, 8),
                                            (1, 64, 20, 64, 0), (40, 640, 260, 128, 8), (128, 256, 128, 64, 0),
                                            (129, 448, 300, 64, 3)])
@pytest.mark.parametrize("out_dtype", [sq.SQ_OUT_F32, sq.SQ_OUT_BF16])
def test_weights_sq_tiles(M, K, N, bank, pad, out_dtype):
    print(f"wsq tiles M={M} K={K} N={N} bank={bank} pad={pad} out={out_dtype}", flush=True)
    topk = bank // 8
    wb, xb, d = case(700 + M + K + N, M, K, N)
    codes, scale = W.quantize_activations(xb, 8)
    prod = W.gemm(codes, scale, W.encode_weights(wb, bank, topk, 8, 4, d=d))
    p = sq.params(M, K, N, bank, topk, out_dtype=out_dtype)
    ws = sq.WeightSQ(p)
    sq.sq_wsq_encode(p, dev(wb), ws, hinv_diag=dev(d))
    pre = torch.empty(sq.sq_wsq_prepack_bytes(p), dtype=torch.uint8, device="cuda")
    sq.sq_wsq_prepack(p, ws, pre)
    f32 = out_dtype == sq.SQ_OUT_F32
    ldy = N + pad
    y = Guarded(M * ldy * (4 if f32 else 2), torch.int32 if f32 else torch.int16)
    y.t.fill_(0x5A5A)
    wsb = Guarded(sq.sq_wsq_linear_workspace_bytes(p), torch.uint8)
    sq.sq_wsq_linear(p, dev(xb), ws, pre, y.t, wsb.t, act_bits=8, ldy=ldy)
    torch.cuda.synchronize()
    y.check()
    wsb.check()
    got = y.host(np.uint32 if f32 else np.uint16).reshape(M, ldy)
    assert np.array_equal(got[:, :N], prod.y32.view(np.uint32) if f32 else prod.ybf16)
    assert (got[:, N:] == 0x5A5A).all(), "written past a row"


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("K", [64, 4096, 4160, 8192, 8256, 16384, 16448])
def test_activation_quantiser_row_lengths(K, bits):
    print(f"quantize act K={K} bits={bits}", flush=True)
    M = 3
    _, xb, _ = case(900 + K, M, K, 4)
    xb[1] = 0
    codes, scale = W.quantize_activations(xb, bits)
    p = sq.params(M, K, 64)
    a8, sa = Guarded(M * K, torch.int8), Guarded(M * 4, torch.float32)
    sq.sq_quantize_act(p, dev(xb), a8.t, sa.t, bits=bits)
    torch.cuda.synchronize()
    a8.check()
    sa.check()
    assert np.array_equal(a8.host(np.int8).reshape(M, K), consumer_order(codes))
    assert np.array_equal(sa.host(np.uint32), scale.view(np.uint32))


@pytest.mark.parametrize("M,K,N,bank", [(1, 64, 70, 64), (64, 320, 300, 64), (33, 128, 129, 128), (50, 384, 260, 128), (2, 256, 33000, 128)])
@pytest.mark.parametrize("special", ["tiny", "zero"])
def test_low_scales_below_the_image_s_range(M, K, N, bank, special):
    """Up to 64 tokens: low scales that the image, which holds them divided by 16, cannot (below 2^-122, down to the smallest
    subnormal; and zero).  Also in a single channel of a tile, and next to ordinary ones."""
    print(f"wsq tiny scales M={M} K={K} N={N} bank={bank} {special}", flush=True)
    rng = np.random.default_rng(M + K + N)
    G, topk = K // bank, bank // 8
    lo = rng.integers(-7, 8, size=(N, G, bank)).astype(np.int8)
    high = np.argsort(rng.random((N, G, bank)), -1)[..., :topk]
    np.put_along_axis(lo, high, -8, -1)
    hi_val = rng.integers(-127, 128, size=(N, G, topk)).astype(np.int8)
    s_lo = rng.uniform(0.01, 0.02, (N, G)).astype(np.float32)
    s_hi = rng.uniform(0.001, 0.002, (N, G)).astype(np.float32)
    rows = np.r_[5, 40:48, 64, 69]  # (tiles of 32 channels without one, with one, with several, and the ragged last one)
    exp = rng.integers(-149, -118, (len(rows), G))
    s_lo[rows] = 0 if special == "zero" else np.ldexp(rng.uniform(1, 2, (len(rows), G)), exp).astype(np.float32)
    s_hi[rows] = np.ldexp(rng.uniform(1, 2, (len(rows), G)), exp - 3).astype(np.float32)
    if special == "tiny":
        s_lo[rows[0]] = np.float32(2.0 ** -149)
    codes = rng.integers(-127, 128, size=(M, K)).astype(np.int8)
    scale = np.full(M, 2.0 ** 100, np.float32)
    scale[0] = 0.37
    prod = W.gemm(codes, scale, W.WeightSQ(N, K, bank, topk, 8, 4, lo.reshape(N, K), hi_val, s_lo, s_hi))
    p = sq.params(M, K, N, bank, topk, out_dtype=sq.SQ_OUT_F32)
    ws = sq.WeightSQ(p)
    ws.lo.copy_(dev(pack_int4(lo.reshape(N, K))).view(-1))
    ws.hi_val.copy_(dev(hi_val).view(-1))
    ws.scale_lo.copy_(dev(s_lo).view(-1))
    ws.scale_hi.copy_(dev(s_hi).view(-1))
    pre = torch.empty(sq.sq_wsq_prepack_bytes(p), dtype=torch.uint8, device="cuda")
    sq.sq_wsq_prepack(p, ws, pre)
    y = Guarded(M * N * 4, torch.float32)
    sq.sq_wsq_gemm(p, dev(consumer_order(codes)), dev(scale), ws, pre, y.t)
    torch.cuda.synchronize()
    y.check()
    assert np.array_equal(y.host(np.uint32).reshape(M, N), prod.y32.view(np.uint32))
