"""The storage conversions over whole rows: several rows per workgroup with a last group that is not full, one long row per
workgroup, streams at every kind of byte offset, against the oracle's streams and back; and the calls on either side of the
size from which packing goes through the image of whole rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_05409_amd as sq
from gpu_util import Guarded, GuardedAct, dev
from test_gpu_parity import make_static_mask, random_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_high,h_low", [(8, 4), (8, 3), (4, 2)])
@pytest.mark.parametrize("M,K,bank,topk", [(1, 64, 64, 8), (130, 64, 32, 8), (37, 512, 64, 16), (5, 8128, 64, 32),
                                           (3, 8192, 128, 8), (2, 16384, 32, 2), (2, 65536, 128, 32),
                                           (33, 576, 64, 4), (7, 320, 32, 2)])  # (8/3): low sections that end in half a byte
@pytest.mark.parametrize("form,offset", [("dynamic", 0), ("dynamic", 13), ("static", 3), ("sentinel", 0), ("sentinel", 6)])
def test_storage_rows(M, K, bank, topk, h_high, h_low, form, offset):
    if form == "static" and (K // bank * topk) % 32:
        topk = 32 if bank == 64 else 16  # whole groups of 32 high channels
    if form == "static" and (K // bank * topk) % 32:
        bank, topk = 64, 32
    print(f"storage rows ({h_high}/{h_low}) {form} M={M} K={K} bank={bank} topk={topk} offset={offset}", flush=True)
    bits, _, _ = random_case(5200 + M + K + h_low + bank, M=M, K=K, N=8, outliers=4)
    mask = make_static_mask(K, bank, topk, seed=K + 1) if form == "static" else None
    enc = oracle.encode_pair(bits, bank, topk, h_high, h_low, static_mask=mask)
    sentinel = form == "sentinel"
    want = (oracle.pack_storage_sentinel if sentinel else oracle.pack_storage)(enc, h_high, h_low)
    p = sq.params(M, K, 64, bank, topk, mode=sq.SQ_STATIC if mask is not None else sq.SQ_DYNAMIC, h_high=h_high, h_low=h_low)
    row = (sq.sq_storage_row_bytes_sentinel if sentinel else sq.sq_storage_row_bytes)(p)
    md = None if mask is None else dev(mask)
    act = sq.Act(p, static_mask=md)
    act.d_lo.copy_(dev(enc.d_lo).view(-1))
    act.hi_val.copy_(dev(enc.hi_val).view(-1))
    if mask is None:
        act.mask.copy_(dev(enc.mask).view(-1))
    buf = Guarded(offset + M * row + 5, torch.uint8)
    buf.t.fill_(0xC3)
    packed = buf.t[offset:offset + M * row]
    (sq.sq_pack_storage_sentinel if sentinel else sq.sq_pack_storage)(p, act, packed)
    torch.cuda.synchronize()
    buf.check()
    got = buf.host(np.uint8)
    assert np.array_equal(got[offset:offset + M * row].reshape(M, row), want)
    assert (got[:offset] == 0xC3).all() and (got[offset + M * row:] == 0xC3).all(), "written outside the stream"
    back = GuardedAct(p, static_mask=md)
    for t in (back.d_lo, back.hi_val) + ((back.mask,) if sentinel else ()):
        t.fill_(0x5A)
    if form == "dynamic":
        back.mask.copy_(act.mask)
    (sq.sq_unpack_storage_sentinel if sentinel else sq.sq_unpack_storage)(p, packed, back)
    torch.cuda.synchronize()
    back.check()
    assert torch.equal(back.d_lo, act.d_lo) and torch.equal(back.hi_val, act.hi_val)
    if sentinel:
        assert torch.equal(back.mask, act.mask)


# the last call that packs byte by byte and the first that packs whole rows (every form and rule: sentinel 2^19 channels, 2^18
# with short codes; explicit 2^17, 2^19 where half of the channels are high; banks of 128 and short codes always whole rows)
@pytest.mark.parametrize("form,h_high,h_low,K,bank,topk,M", [
    ("sentinel", 8, 4, 4096, 64, 8, 128), ("sentinel", 4, 2, 1024, 32, 4, 256), ("sentinel", 8, 3, 11008, 64, 8, 47),
    ("dynamic", 8, 4, 512, 64, 8, 256), ("dynamic", 8, 4, 8192, 64, 32, 64), ("dynamic", 8, 4, 576, 64, 4, 227),
    ("static", 8, 4, 1024, 32, 16, 512), ("dynamic", 8, 4, 1024, 128, 32, 3), ("dynamic", 8, 3, 1024, 64, 8, 3)])
def test_ways_of_packing(form, h_high, h_low, K, bank, topk, M):
    for m in (M, M + 1):
        test_storage_rows(m, K, bank, topk, h_high, h_low, form, 5)
