"""Classing of prompts longer than a tile (4096 tokens): a table's tiles dealt to several
workgroups, to fewer than there are tiles, and to one.  Quota form with ties at the cuts
that cross tiles, threshold form, recent windows across a tile's edge; bit-exact."""
import numpy as np
import pytest
from gpu_util import assert_state_equal, dev_cache_from_oracle, layouts, t

from oracle import oracle as orc
from paper_2412_03131_amd import diffkv as dk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,lens,window", [
    (2, 1, (4096, 13001), 0),        # one tile; four workgroups
    (3, 2, (4097, 8192, 12288), 5),  # tiles' edges, a window inside the last tile
    (1, 1, (8200,), 4100),           # a window over two tiles
    (100, 2, (9000, 3, 40), 1),      # 200 tables: two workgroups for three tiles
    (300, 1, (5000, 700), 0),        # 300 tables: one workgroup for two tiles
])
@pytest.mark.parametrize("form", ["quota", "threshold"])
def test_tiles(B, Hkv, lens, window, form):
    rng = np.random.default_rng(B * 10 + Hkv)
    new_len = np.zeros(B, np.int32)
    new_len[:len(lens)] = lens
    rows = int(new_len.sum())
    k = rng.standard_normal((rows, Hkv, 128)).astype(np.float16).view(np.uint16)
    v = rng.standard_normal((rows, Hkv, 128)).astype(np.float16).view(np.uint16)
    score = (np.round(rng.random((rows, Hkv)) * 40) / 40).astype(np.float32) * np.float32(2.0 / max(lens))  # many ties
    quota = None
    if form == "quota":
        hi = (new_len[:, None] * rng.uniform(0.1, 0.5, (B, Hkv))).astype(np.int32)
        lo = (new_len[:, None] * rng.uniform(0.1, 0.4, (B, Hkv))).astype(np.int32)
        quota = np.stack([hi, lo], axis=2).astype(np.int32)
    Lo, Ld = layouts(max_seq_len=max(lens) + 16)
    pages = int((new_len // 16 + 2).sum()) * Hkv
    oc = orc.Cache(Lo, pages, B, Hkv, ring=rng.permutation(pages))
    dc = dev_cache_from_oracle(Ld, oc)
    print("case: classify tiles B=%d Hkv=%d %s window=%d" % (B, Hkv, form, window), flush=True)
    orc.quantize_append(oc, new_len, k, v, score, quota=quota, alpha_h=1.2, alpha_l=0.4, window=window)
    dk.quantize_append(dc, t(new_len), t(k), t(v), t(score), quota=None if quota is None else t(quota), alpha_h=1.2,
                       alpha_l=0.4, window=window, total_new=rows, max_new=int(new_len.max()))
    assert oc.status[0] == 0
    assert_state_equal(dc, oc, what="tiles")
