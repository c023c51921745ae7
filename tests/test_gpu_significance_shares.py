"""The significance update's deal of pages to workgroups: tables with fewer pages than the
grid gives them workgroups, with more than a workgroup's twelve (several workgroups), and
so many tables that each has one workgroup for a long table's pages."""
import numpy as np
import pytest
import torch
from test_gpu_significance import _compare, _step

from gpu_util import dev_cache_from_oracle, layouts, t
from oracle import oracle as orc
from paper_2412_03131_amd import diffkv as dk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,gq,lens", [
    (3, 2, 4, (191, 193, 400)),   # 12, 13 and 25 pages
    (7, 1, 5, (0, 1, 16, 17, 180, 200, 900)),
    (1025, 8, 1, (700, 3)),       # 8200 tables: one workgroup each
])
def test_pages_dealt_to_workgroups(B, Hkv, gq, lens):
    rng = np.random.default_rng(B)
    new_len = np.zeros(B, np.int32)
    new_len[:len(lens)] = lens
    rows = int(new_len.sum())
    k = (rng.standard_normal((rows, Hkv, 128)) * 2).astype(np.float16).view(np.uint16)
    v = rng.standard_normal((rows, Hkv, 128)).astype(np.float16).view(np.uint16)
    score = (rng.random((rows, Hkv)) * 0.01).astype(np.float32)
    quota = np.zeros((B, Hkv, 2), np.int32)
    quota[:, :, 0] = new_len[:, None]
    quota[:, ::2, 0] //= 2
    quota[:, ::2, 1] = new_len[:, None] - quota[:, ::2, 0]
    Lo, Ld = layouts(max_seq_len=1024)
    pages = int((-(-quota // 16)).sum()) + 64
    oc = orc.Cache(Lo, pages, B, Hkv, ring=rng.permutation(pages))
    orc.quantize_append(oc, new_len, k, v, score, quota=quota)
    assert oc.status[0] == 0
    dc = dev_cache_from_oracle(Ld, oc)
    q = rng.standard_normal((B, gq * Hkv, 128)).astype(np.float16).view(np.uint16)
    print("case: significance pages dealt, B=%d" % B, flush=True)
    _step(dc, oc, q)
    assert _compare(dc, oc, "B=%d" % B) == rows * Hkv


def test_lengths_past_the_table_stay_in_its_row():
    """Section lengths of more pages than the table has slots: the row's own pages are read, nothing
    past it (the neighbouring table's entries), and the neighbours' scores are as ever."""
    rng = np.random.default_rng(3)
    B, Hkv, gq = 3, 1, 2
    new_len = np.array([40, 60, 90], np.int32)
    rows = int(new_len.sum())
    k = rng.standard_normal((rows, Hkv, 128)).astype(np.float16).view(np.uint16)
    v = rng.standard_normal((rows, Hkv, 128)).astype(np.float16).view(np.uint16)
    score = (rng.random((rows, Hkv)) * 0.01).astype(np.float32)
    quota = np.zeros((B, Hkv, 2), np.int32)
    quota[:, 0, 0] = new_len
    Lo, Ld = layouts(max_seq_len=112)  # 8 slots per table
    oc = orc.Cache(Lo, 32, B, Hkv, ring=rng.permutation(32))
    orc.quantize_append(oc, new_len, k, v, score, quota=quota)
    dc = dev_cache_from_oracle(Ld, oc)
    before = dc.pool.cpu().numpy().copy()
    dc.len[0, 0] = 16 * 5000
    q = rng.standard_normal((B, gq * Hkv, 128)).astype(np.float16).view(np.uint16)
    lse = torch.full((B, gq * Hkv), 3.0, dtype=torch.float32, device="cuda")
    print("case: significance, lengths past the table", flush=True)
    dk.update_significance(dc, t(q), 1.0 / np.sqrt(128.0), lse)
    torch.cuda.synchronize()
    got = dc.pool.cpu().numpy()
    # the same update of the neighbours alone, table 0 empty
    dc.pool.copy_(torch.from_numpy(before))
    dc.len[0] = 0
    dk.update_significance(dc, t(q), 1.0 / np.sqrt(128.0), lse)
    torch.cuda.synchronize()
    want = dc.pool.cpu().numpy()
    others = oc.table[1:][oc.table[1:] >= 0]
    assert np.array_equal(got[others], want[others])
    assert not np.array_equal(got[others], before[others])


@pytest.mark.parametrize("B,Hkv,gq,lens", [
    (30, 8, 4, (9000, 300, 70)),   # 240 tables with room for 577 pages: between one and two times the usual
    (70, 8, 1, (20000, 30)),       # 560 tables, one long: twice the usual
])
def test_long_tables_among_short_ones(B, Hkv, gq, lens):
    rng = np.random.default_rng(B)
    new_len = np.full(B, 5, np.int32)
    new_len[:len(lens)] = lens
    rows = int(new_len.sum())
    k = (rng.standard_normal((rows, Hkv, 128)) * 2).astype(np.float16).view(np.uint16)
    v = rng.standard_normal((rows, Hkv, 128)).astype(np.float16).view(np.uint16)
    score = (rng.random((rows, Hkv)) * 0.01).astype(np.float32)
    quota = np.zeros((B, Hkv, 2), np.int32)
    quota[:, :, 0] = new_len[:, None] // 2
    quota[:, :, 1] = new_len[:, None] - quota[:, :, 0]
    Lo, Ld = layouts(max_seq_len=max(lens) + 200)
    pages = int((-(-quota // 16)).sum()) + 64
    oc = orc.Cache(Lo, pages, B, Hkv, ring=rng.permutation(pages))
    orc.quantize_append(oc, new_len, k, v, score, quota=quota)
    dc = dev_cache_from_oracle(Ld, oc)
    q = rng.standard_normal((B, gq * Hkv, 128)).astype(np.float16).view(np.uint16)
    print("case: significance, long among short, B=%d" % B, flush=True)
    _step(dc, oc, q)
    assert _compare(dc, oc, "B=%d" % B) == rows * Hkv
