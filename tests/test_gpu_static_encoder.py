"""The row-staged static encoder at the edges of its instantiations (rows that just fit and just do not fit a number of
pieces per thread, one and two row buffers), with few rows and with several rows per workgroup, banks whose low channels
do not come in whole pieces, and both forms of the low part at once -- bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_05409_amd as sq
from gpu_util import Guarded, GuardedAct, assert_encoding_equal, dev
from test_gpu_parity import compact_low, make_static_mask, random_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,bank,topk", [
    (1, 64, 64, 32), (2, 512, 64, 4), (9, 4096, 64, 8), (9, 4160, 64, 32), (5, 8192, 128, 2), (5, 8256, 64, 32),
    (3, 12288, 64, 16), (3, 12352, 64, 32), (3, 16384, 32, 1), (3, 16448, 64, 32), (2, 32768, 64, 8), (2, 34816, 128, 16),
    (2100, 512, 64, 8), (5000, 64, 32, 16), (9, 576, 64, 32), (4500, 1024, 128, 16), (7, 1024, 32, 1), (9, 1088, 64, 32), (1700, 8192, 128, 32), (1601, 11008, 64, 16), (600, 34816, 128, 4)])
@pytest.mark.parametrize("low", ["compact", "dense", "both"])
def test_static_encoder(M, K, bank, topk, low):
    print(f"static encoder M={M} K={K} bank={bank} topk={topk} low={low}", flush=True)
    bits, _, _ = random_case(900 + M + K, M, K, N=8, outliers=min(6, K // 16))
    mask = make_static_mask(K, bank, topk, seed=K + topk)
    enc = oracle.encode(bits, bank, topk, static_mask=mask)
    p = sq.params(M, K, 64, bank, topk, mode=sq.SQ_STATIC)
    md = dev(mask)
    act = GuardedAct(p, static_mask=md)
    compact = Guarded(sq.sq_lo_compact_bytes(p), torch.uint8)
    if low != "dense":
        act.lo_compact = compact.t
    d_lo = act.d_lo
    if low == "compact":
        act.d_lo = None
    sq.sq_encode(p, dev(bits), act, static_mask=md)
    torch.cuda.synchronize()
    act.check()
    compact.check()
    if low != "dense":
        assert np.array_equal(compact.host(np.uint8).reshape(M, -1), compact_low(enc)), "lo_compact"
    act.d_lo = d_lo if low != "compact" else dev(enc.d_lo).view(-1)
    assert_encoding_equal(act, enc)
