"""sq_gemm kernels that share K among the waves of a workgroup: the few-token kernel (every token count it has an
instantiation for, every channel width, K shorter than its waves, partial last steps, both parts of the reordered
static operands) and the tiles with two K groups (odd and even step counts, a missing and a partial last step); and the light
tile that takes their place where K is short.
Accumulators and outputs are compared with the oracle bit for bit, into buffers between guard bytes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_05409_amd as sq
from gpu_util import Guarded, dev
from test_gpu_parity import make_static_mask, random_case, run_gemm

pytestmark = pytest.mark.gpu


def check(M, K, N, bank, topk, mode):
    print(f"split K M={M} K={K} N={N} bank={bank} topk={topk} mode={mode}", flush=True)
    p = sq.params(M, K, N, bank, topk, mode=mode, out_dtype=sq.SQ_OUT_F32)
    bits, wq, sw = random_case(8000 + M + K + N, M, K, N, outliers=min(6, K // 16))
    mask = pre = None
    if mode == sq.SQ_STATIC:
        mask = make_static_mask(K, bank, topk, seed=K + N)
        pre = torch.empty(sq.sq_weight_prepack_bytes(p), dtype=torch.uint8, device="cuda")
        sq.sq_weight_prepack(p, dev(wq), mask, dev(mask), pre)
    if mode == sq.SQ_DYNAMIC_TIED:
        prod = oracle.gemm_tied(oracle.encode_tied(bits, bank, topk), wq, sw)
    else:
        enc = oracle.encode(bits, bank, topk, static_mask=mask)
        prod = oracle.gemm(enc, wq, sw)
        y, alo, ahi = run_gemm(p, enc, wq, sw, sq.SQ_OUT_F32, prepacked=pre, static_mask=mask)
        assert np.array_equal(alo, prod.acc_lo), "acc_lo"
        assert np.array_equal(ahi, prod.acc_hi), "acc_hi"
        assert np.array_equal(y.view(np.uint32), prod.y32.view(np.uint32)), "fp32 output"
    # the whole call (static mode: with the reordered low part), bf16 rows at an odd distance
    p.out_dtype = sq.SQ_OUT_BF16
    ldy = N + 3
    y16 = Guarded(M * ldy * 2, torch.int16)
    y16.t.fill_(0x5A5A)
    ws = Guarded(sq.sq_linear_workspace_bytes(p), torch.uint8)
    md = None if mask is None else dev(mask)
    sq.sq_linear(p, dev(bits), sq.weight(dev(wq), dev(sw), pre), y16.t, ws.t, static_mask=md, ldy=ldy)
    torch.cuda.synchronize()
    y16.check()
    ws.check()
    got = y16.host(np.uint16).reshape(M, ldy)
    assert np.array_equal(got[:, :N], prod.ybf16), "bf16 output"
    assert (got[:, N:] == 0x5A5A).all(), "written past a row"


# N decides the channels per workgroup: one tile of 16 up to 4096 channels, one more per 4096 after that
@pytest.mark.parametrize("M", [1, 8, 9, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("mode", [sq.SQ_DYNAMIC, sq.SQ_STATIC, sq.SQ_DYNAMIC_TIED])
def test_few_tokens_token_counts(M, mode):
    assert sq.sq_gemm_variant(sq.params(M, 2048, 301, 64, 8, mode=mode)) == "few_tokens"
    check(M, 2048, 301, 64, 8, mode)


@pytest.mark.parametrize("N", [4097, 8193, 12300, 16500, 20500, 24600, 28690])
@pytest.mark.parametrize("M,mode", [(7, sq.SQ_DYNAMIC), (11, sq.SQ_STATIC), (27, sq.SQ_DYNAMIC_TIED), (30, sq.SQ_STATIC)])
def test_few_tokens_channel_widths(M, N, mode):
    K = 512 if M <= 16 else 8192  # (short K with more tokens: the light tile)
    assert sq.sq_gemm_variant(sq.params(M, K, N, 64, 8, mode=mode)) == "few_tokens"
    check(M, K, N, 64, 8, mode)


@pytest.mark.parametrize("K,bank,topk", [(64, 64, 32), (192, 64, 32), (1088, 32, 16), (1152, 128, 32), (5504, 64, 16)])
@pytest.mark.parametrize("M,mode", [(5, sq.SQ_DYNAMIC), (20, sq.SQ_STATIC), (40, sq.SQ_DYNAMIC)])
def test_few_tokens_channel_tails(M, K, bank, topk, mode):
    check(M, K, 130, bank, topk, mode)


TILE_SHAPES = [(65, 1088, 70), (130, 1152, 515), (100, 1216, 260), (333, 1280, 300), (64, 1152, 8200), (40, 1408, 12300),
               (200, 2112, 8000), (300, 2240, 4095), (130, 2048, 515), (200, 4096, 8000)]


@pytest.mark.parametrize("M,K,N,mode", [s + (m,) for s in TILE_SHAPES for m in (sq.SQ_DYNAMIC, sq.SQ_STATIC)]
                         + [s + (sq.SQ_DYNAMIC_TIED,) for s in TILE_SHAPES if s[1] & (s[1] - 1) == 0])
def test_tiles_with_two_k_groups(M, K, N, mode):
    assert sq.sq_gemm_variant(sq.params(M, K, N, 64, 32, mode=mode)) in ("tile64x64", "tile64x128")
    check(M, K, N, 64, 32, mode)


# the 64 x 64 tile with one K group: one to eight steps, the last one partial or not
LIGHT_SHAPES = [(65, 64, 70), (130, 128, 515), (100, 192, 260), (40, 384, 12300), (300, 320, 4095), (30, 256, 28690),
                (64, 512, 20000), (500, 960, 4000)]


@pytest.mark.parametrize("M,K,N,mode", [s + (m,) for s in LIGHT_SHAPES for m in (sq.SQ_DYNAMIC, sq.SQ_STATIC)]
                         + [s + (sq.SQ_DYNAMIC_TIED,) for s in LIGHT_SHAPES if s[1] in (256, 512)])
def test_light_tile(M, K, N, mode):
    assert sq.sq_gemm_variant(sq.params(M, K, N, 64, 32, mode=mode)) == "tile64x64_light"
    check(M, K, N, 64, 32, mode)


# the 128 x 256 tile with padded and unaligned rows of Y (8 x 32 of its tiles: one round over the chip)
@pytest.mark.parametrize("mode", [sq.SQ_DYNAMIC, sq.SQ_STATIC])
def test_large_tile_rows_of_y(mode):
    assert sq.sq_gemm_variant(sq.params(1000, 256, 8100, 64, 8, mode=mode)) == "tile128x256"
    check(1000, 256, 8100, 64, 8, mode)
