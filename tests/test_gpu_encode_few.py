"""The encoder for few banks (several lanes per bank): every format, with the matrix-core image, two scales and tied, odd
bank counts, several rows per wave (with lanes to spare and without, the last wave not full), rows that fill its eight
waves, the last calls of its rule and the first past it -- against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_05409_amd as sq
from gpu_util import Guarded, GuardedAct, assert_encoding_equal, dev
from test_gpu_parity import random_case
from workloads import unpack_int4

pytestmark = pytest.mark.gpu

FORMATS = [(32, 2), (32, 4), (32, 8), (32, 16), (64, 4), (64, 8), (64, 16), (64, 32), (128, 8), (128, 16), (128, 32)]


def image_of(enc, M, K, tied):
    """High codes at their channels (tied: 16 x the low codes elsewhere), per 8 channels the even ones first."""
    bits = (enc.mask[:, :, None] >> np.arange(32, dtype=np.uint32)) & 1
    high = bits.reshape(M, K).astype(bool)
    full = (16 * unpack_int4(enc.d_lo).astype(np.int16)).astype(np.int8) if tied else np.zeros((M, K), np.int8)
    full[high] = enc.hi_val.reshape(-1)
    return full.reshape(M, K // 8, 4, 2).transpose(0, 1, 3, 2).reshape(M, K)


def check(M, K, bank, topk, tied=False):
    print(f"encode few M={M} K={K} bank={bank} topk={topk} tied={tied}", flush=True)
    bits, _, _ = random_case(600 + M + K + bank + topk, M=M, K=K, N=8, outliers=min(6, K // 16))
    enc = oracle.encode_tied(bits, bank, topk) if tied else oracle.encode(bits, bank, topk)
    p = sq.params(M, K, 64, bank, topk, mode=sq.SQ_DYNAMIC_TIED if tied else sq.SQ_DYNAMIC)
    act = GuardedAct(p)
    image = Guarded(M * K, torch.int8)
    act.hi_dense = image.t
    sq.sq_encode(p, dev(bits), act)
    torch.cuda.synchronize()
    act.check()
    image.check()
    assert_encoding_equal(act, enc)
    assert np.array_equal(image.host(np.int8).reshape(M, K), image_of(enc, M, K, tied)), "image"


@pytest.mark.parametrize("bank,topk", FORMATS)
@pytest.mark.parametrize("tied", [False, True])
def test_formats(bank, topk, tied):
    check(5, 1024, bank, topk, tied)


@pytest.mark.parametrize("M,K,bank,topk", [(1, 64, 64, 8), (4, 192, 64, 8), (3, 5120, 64, 32), (200, 11008, 128, 16),
                                           (256, 8192, 64, 8), (257, 8192, 64, 8), (2, 8256, 64, 8), (520, 4096, 128, 8),
                                           (2048, 512, 64, 8), (2049, 512, 64, 16)])
def test_shapes(M, K, bank, topk):
    check(M, K, bank, topk)


@pytest.mark.parametrize("K,bank,topk", [(64, 64, 32), (64, 32, 16), (128, 128, 8), (192, 64, 8), (192, 64, 32), (256, 128, 32),
                                         (320, 32, 16), (512, 32, 16), (576, 64, 8), (640, 128, 16), (1024, 128, 32),
                                         (1152, 64, 32), (2048, 64, 32)])
@pytest.mark.parametrize("M", [1, 3, 67, 301])
def test_rows_that_share_a_wave(M, K, bank, topk):
    assert sq.sq_encode_variant(sq.params(M, K, 64, bank, topk)) == "few_banks"
    check(M, K, bank, topk)
    if K // bank & (K // bank - 1) == 0:
        check(M, K, bank, topk, tied=True)


# the rule: eight waves per compute unit (256 of them), four where two lanes share a bank; short rows share waves
@pytest.mark.parametrize("M,K,bank,topk", [(2048, 1024, 64, 8), (4096, 512, 64, 8), (1024, 2048, 64, 32), (2048, 1024, 64, 32),
                                           (256, 4096, 64, 32), (256, 8192, 64, 32)])
def test_ends_of_the_rule(M, K, bank, topk):
    for m, kernel in ((M, "few_banks"), (M + 16, "streaming")):
        assert sq.sq_encode_variant(sq.params(m, K, 64, bank, topk)) == kernel
    check(M, K, bank, topk)
