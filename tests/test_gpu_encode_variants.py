"""The dynamic encoders for calls past the few-bank kernel's range: the streaming kernel (power-of-two bank counts) and the
general one, in every format, with two scales and tied, in every precision pair, with padded rows of X and with the
matrix-core image -- against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_05409_amd as sq
from gpu_util import Guarded, GuardedAct, assert_encoding_equal, dev
from test_gpu_encode_few import FORMATS, image_of
from test_gpu_parity import random_case

pytestmark = pytest.mark.gpu


def sample(M, n):
    rows = np.r_[0:4, np.random.default_rng(M + n).integers(0, M, n), M - 1]  # the first four: ties, zeros, all equal
    return np.unique(rows[rows < M])


def check(kernel, M, K, bank, topk, tied=False, pair=(8, 4), pad=0, rows=None):
    print(f"encode {kernel} M={M} K={K} bank={bank} topk={topk} tied={tied} {pair} pad={pad}", flush=True)
    p = sq.params(M, K, 64, bank, topk, mode=sq.SQ_DYNAMIC_TIED if tied else sq.SQ_DYNAMIC, h_high=pair[0], h_low=pair[1])
    assert sq.sq_encode_variant(p) == kernel
    bits, _, _ = random_case(6100 + M + K + bank + topk, M=M, K=K, N=8, outliers=min(6, K // 16))
    rows = np.arange(M) if rows is None else rows
    if pair != (8, 4):
        enc = oracle.encode_pair(bits[rows], bank, topk, *pair)
    else:
        enc = (oracle.encode_tied if tied else oracle.encode)(bits[rows], bank, topk)
    x = np.full((M, K + pad), 0x7F80, np.uint16)  # +inf between the rows: never read as data
    x[:, :K] = bits
    act = GuardedAct(p)
    image = Guarded(M * K, torch.int8)
    act.hi_dense = image.t
    sq.sq_encode(p, dev(x), act, ldx=K + pad)
    torch.cuda.synchronize()
    act.check()
    image.check()
    assert_encoding_equal(act, enc, rows=rows)
    assert np.array_equal(image.host(np.int8).reshape(M, K)[rows], image_of(enc, len(rows), K, tied)), "image"


@pytest.mark.parametrize("bank,topk", FORMATS)
@pytest.mark.parametrize("tied", [False, True])
@pytest.mark.parametrize("M,K,pad", [(8311, 512, 0), (4200, 1024, 24)])
def test_streaming_formats(M, K, pad, bank, topk, tied):
    check("streaming", M, K, bank, topk, tied, pad=pad, rows=sample(M, 150) if tied else None)


@pytest.mark.parametrize("bank,topk", FORMATS)
@pytest.mark.parametrize("M,K,pad", [(2100, 1152, 0), (8311, 384, 8)])
def test_general_formats(M, K, pad, bank, topk):
    check("general", M, K, bank, topk, pad=pad)


@pytest.mark.parametrize("pair", [(8, 3), (8, 2), (4, 2)])
@pytest.mark.parametrize("kernel,M,K,bank,topk", [
    ("streaming", 3, 16384, 64, 8), ("streaming", 3, 8192, 32, 4), ("streaming", 4200, 512, 64, 32), ("streaming", 4200, 512, 32, 16),
    ("streaming", 4200, 1024, 128, 16), ("general", 3, 16448, 64, 8), ("general", 5, 11008, 32, 2), ("general", 2100, 1152, 128, 32),
    ("general", 4200, 320, 64, 16)])
def test_precision_pairs(kernel, M, K, bank, topk, pair):
    check(kernel, M, K, bank, topk, pair=pair, rows=sample(M, 12))
