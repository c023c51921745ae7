"""Balanced attention in shares of a table's own (few tables, or short ones), and the
one-attempt claim of the arrival words.

The share rule is modelled here on the host (units, quantum, ranges) to check that the
ranges of every table cover its pages once and fit the workgroups; on the GPU, tables at
the edges of the rule (one range, two, the merge's chunk sizes and one more, many) are
compared with the oracle.
"""
import math
import random

import numpy as np
import pytest
from test_arrival_protocol import CB, MASK, Word, arrive_count, start_word

HI, LO, SEG = 3, 6, 50


def page_at_unit(x, ph, np_):
    if x <= 0:
        return 0
    x -= SEG
    if x <= 0:
        return 1 if np_ > 0 else 0
    xh = HI * ph
    p = -(-x // HI) if x <= xh else ph + -(-(x - xh) // LO)
    return min(p, np_)


def quantum_of(tabs, T, W, waves):
    """The range length of tables [(ph, pl)], or None where the list is cut."""
    pus = [HI * a + LO * b for a, b in tabs if a + b]
    total, held = sum(pus) + SEG * len(pus), len(pus)
    little = T < W and total * T <= SEG * W * (W - T)
    fit = total - SEG * T <= W * waves * HI
    if not little and (T > W or not fit):
        return None
    part = lambda p, n: -(-p // n)
    tries = [waves * HI if fit else part(total - SEG * T, W - T // 2)]
    if little:
        tries += [part(sum(pus), W - held // 2)] * fit + [part(sum(pus), W - held)]
    for q in tries:
        if sum(-(-p // q) for p in pus) <= W:
            return q if pus else None
    return None


def ranges_of(ph, pl, quantum):
    pu = HI * ph + LO * pl
    n = -(-pu // quantum)
    cut = [0] + [SEG + c * pu // n for c in range(1, n + 1)]
    return [(page_at_unit(cut[c], ph, ph + pl), page_at_unit(cut[c + 1], ph, ph + pl)) for c in range(n)]


def test_own_shares_cover_every_page_once():
    """Every page lies in one range, the ranges fit the workgroups, and no range holds more than one
    page per wave (the length of a wave's chain, on which the error depends) where such ranges
    fit, nor more page units than a workgroup's part where every table wastes a range."""
    rng = random.Random(5)
    checked = longer = 0
    for _ in range(6000):
        W, waves = rng.choice(((512, 8), (256, 12)))
        T = int(math.exp(rng.uniform(0, math.log(W))))
        top = int(math.exp(rng.uniform(0, math.log(3000))))
        tabs = [(rng.randint(0, top), rng.randint(0, top)) for _ in range(T)]
        q = quantum_of(tabs, T, W, waves)
        if q is None:
            continue
        checked += 1
        assert sum(-(-(HI * a + LO * b) // q) for a, b in tabs) <= W
        total = sum(SEG + HI * a + LO * b for a, b in tabs if a + b)
        if q > waves * HI:
            longer += 1
            held = sum(a + b > 0 for a, b in tabs)
            assert sum(-(-(HI * a + LO * b) // (waves * HI)) for a, b in tabs) > W
            assert q <= (total - SEG * held) / (W - held) + 1
        for a, b in tabs:
            if a + b == 0:
                continue
            r = ranges_of(a, b, q)
            assert r[0][0] == 0 and r[-1][1] == a + b
            assert all(x[1] == y[0] and x[0] < x[1] for x, y in zip(r, r[1:]))
            assert q > waves * HI or all(0 < x[1] - x[0] <= waves for x in r)
    assert checked > 500 and longer > 100


def claim_once(w, tag):
    """arrive_peek, then arrive_claim_once: one exchange, whatever its outcome."""
    old = w.v
    yield  # the load
    if (old >> CB) != tag:
        yield  # the compare-and-swap
        if w.v == old:
            w.v = tag << CB


def test_one_attempt_claim_loses_no_arrival():
    rng = random.Random(6)
    for _ in range(3000):
        tag, n = rng.randrange(1 << 44), rng.randint(1, 12)
        w = Word(start_word(rng.randrange(3), tag, rng))
        if (w.v >> CB) == tag:
            continue
        gens = [arrive_count(w, tag) for _ in range(n)] + [claim_once(w, tag)]
        res, live = [None] * (n + 1), list(range(n + 1))
        while live:
            i = rng.choice(live)
            try:
                next(gens[i])
            except StopIteration as e:
                res[i] = e.value
                live.remove(i)
        assert sorted(res[:n]) == list(range(1, n + 1))
        assert w.v == (tag << CB) | n and n <= MASK


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hkv,gq,layout,lens", [
    (1, 1, 1, 0, (9000,)),                      # one table in many ranges
    (1, 3, 4, 0, (128, )),                      # about one page per wave: one range or two
    (2, 2, 5, 3, (1, 700)),                     # a token alone beside a table of a few ranges
    (3, 1, 8, 0, (2600, 300, 0)),               # twelve waves, an empty table
    (5, 1, 7, 1, (33, 500, 1100, 1700, 2300)),  # one to eight ranges, 8-bit values
    (4, 2, 3, 2, (1900, 900, 450, 60)),
    (2, 4, 8, 0, (9000, 7000)),                 # ranges longer than a page per wave
    (16, 8, 4, 0, (2000, 1800, 1500, 40)),      # the same with tables of one to four ranges
    (2, 4, 6, 3, (6000, 0)),                    # with empty tables
])
def test_own_shares_match_oracle(B, Hkv, gq, layout, lens):
    import torch
    from gpu_util import assert_attention_close, dev_cache_from_oracle, layouts, t

    from oracle import oracle as orc
    from paper_2412_03131_amd import diffkv as dk

    kw = [dict(), dict(v_bits=(8, 2)), dict(v_bits=(2, 1)), dict(tokens_per_page=(16, 16))][layout]
    rng = np.random.default_rng(91 + layout)
    new_len = np.array(lens * (B // len(lens)), np.int32)
    rows = int(new_len.sum())
    k = rng.standard_normal((rows, Hkv, 128)).astype(np.float16).view(np.uint16)
    v = rng.standard_normal((rows, Hkv, 128)).astype(np.float16).view(np.uint16)
    score = rng.random((rows, Hkv)).astype(np.float32)
    quota = np.stack([(new_len[:, None] * rng.uniform(0.2, 0.6, (B, Hkv))).astype(np.int32) + 1,
                      (new_len[:, None] * rng.uniform(0.1, 0.4, (B, Hkv))).astype(np.int32)], axis=2)
    Lo, Ld = layouts(max_seq_len=max(lens) + 16, **kw)
    pages = int((quota // 16 + 2).sum()) + 8
    oc = orc.Cache(Lo, pages, B, Hkv, ring=rng.permutation(pages))
    orc.quantize_append(oc, new_len, k, v, score, quota=quota)
    assert oc.status[0] == 0
    q = rng.standard_normal((B, gq * Hkv, 128)).astype(np.float16).view(np.uint16)
    scale = 1.0 / np.sqrt(128.0)
    ref, ref_lse = orc.attention(oc, q, scale)
    dc = dev_cache_from_oracle(Ld, oc)
    first = None
    for splits in (0, -1):
        print("case: own shares B=%d Hkv=%d gq=%d layout=%d splits=%d" % (B, Hkv, gq, layout, splits), flush=True)
        out, lse = dk.decode_attention(dc, t(q), scale, num_splits=splits)
        torch.cuda.synchronize()
        assert_attention_close(out.cpu().numpy(), lse.cpu().numpy(), ref, ref_lse, "own shares")
        first = first if first is not None else (out, lse)
        assert torch.equal(out, first[0]) and torch.equal(lse, first[1])


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hkv,gq,pages", [(6, 8, 4, 80), (1, 1, 1, 8), (3, 8, 8, 96), (16, 8, 4, 32)])
def test_own_shares_hold_a_page_per_wave(B, Hkv, gq, pages):
    """Tables of high pages only, a multiple of the workgroup's waves (8, or 12 at GQ 8) each, whose
    ranges fit the device: the shares are then num_splits = pages / waves equal ranges, merged in the
    same order, so the results are the same bits.  With longer shares they are not."""
    import torch
    from gpu_util import dev_cache_from_oracle, layouts, t

    from oracle import oracle as orc
    from paper_2412_03131_amd import diffkv as dk

    rng = np.random.default_rng(pages)
    n = pages * 16
    new_len = np.full(B, n, np.int32)
    k = rng.standard_normal((B * n, Hkv, 128)).astype(np.float16).view(np.uint16)
    v = rng.standard_normal((B * n, Hkv, 128)).astype(np.float16).view(np.uint16)
    score = rng.random((B * n, Hkv)).astype(np.float32)
    quota = np.tile(np.array([n, 0], np.int32), (B, Hkv, 1))
    Lo, Ld = layouts(max_seq_len=n + 16)
    oc = orc.Cache(Lo, B * Hkv * pages + 8, B, Hkv, ring=rng.permutation(B * Hkv * pages + 8))
    orc.quantize_append(oc, new_len, k, v, score, quota=quota)
    assert oc.status[0] == 0
    dc = dev_cache_from_oracle(Ld, oc)
    q = rng.standard_normal((B, gq * Hkv, 128)).astype(np.float16).view(np.uint16)
    waves = 12 if gq == 8 else 8
    got = []
    for splits in (-1, pages // waves):
        print("case: page per wave B=%d gq=%d splits=%d" % (B, gq, splits), flush=True)
        got.append(dk.decode_attention(dc, t(q), 1.0 / np.sqrt(128.0), num_splits=splits))
        torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
