"""Page jobs of the append, one wave or one workgroup per page: fresh and continued pages with the job's
slots starting and ending anywhere (each lane row's first and last slot, one slot, a whole
page), every page format, and groups at the quantizer's edges.  Bit-exact against the oracle."""
import numpy as np
import pytest
from gpu_util import assert_state_equal, dev_cache_from_oracle, layouts, t

from oracle import oracle as orc
from paper_2412_03131_amd import diffkv as dk

pytestmark = pytest.mark.gpu

LAYOUTS = [dict(), dict(v_bits=(8, 2)), dict(v_bits=(2, 1)), dict(tokens_per_page=(16, 16))]


def edge_values(rng, rows, Hkv):
    """Groups of 32: plain, constant, ranges whose scale rounds to zero or a subnormal, signed
    zeros, the largest finite values, and quotients at or next to half-integers."""
    x = rng.standard_normal((rows, Hkv, 4, 32)).astype(np.float32)
    kind = rng.integers(0, 8, (rows, Hkv, 4))
    x[kind == 1] = np.float32(1.5)
    tiny = rng.integers(0, 40, x.shape).astype(np.float32) * np.float32(2.0 ** -24)
    x[kind == 2] = tiny[kind == 2]
    x[kind == 3] = np.where(rng.random(x.shape) < 0.5, np.float32(-0.0), np.float32(0.0))[kind == 3]
    x[kind == 4] = np.where(rng.random(x.shape) < 0.5, np.float32(-65504), np.float32(65504))[kind == 4]
    grid = rng.integers(0, 511, x.shape).astype(np.float32) * np.float32(0.5)
    grid[..., 0], grid[..., 1] = 0.0, 255.0
    x[kind == 5] = grid[kind == 5]
    grid = rng.integers(0, 31, x.shape).astype(np.float32) * np.float32(0.25) - np.float32(2.0)
    grid[..., 0], grid[..., 1] = -2.0, 5.5
    x[kind == 6] = grid[kind == 6]
    return x.astype(np.float16).view(np.uint16).reshape(rows, Hkv, 128)


@pytest.mark.parametrize("layout", range(4))
# few jobs, a workgroup each; a wave each, the plan in every workgroup; and planned once
@pytest.mark.parametrize("B,Hkv", [(5, 3), (70, 8), (70, 15)])
def test_page_jobs_bitexact(layout, B, Hkv):
    rng = np.random.default_rng(300 + layout)
    Lo, Ld = layouts(max_seq_len=192, **LAYOUTS[layout])
    pages = B * Hkv * 16
    oc = orc.Cache(Lo, pages, B, Hkv, ring=rng.permutation(pages))
    oc.pool[:] = rng.integers(0, 256, oc.pool.shape, dtype=np.uint8)  # free pages hold old bytes
    dc = dev_cache_from_oracle(Ld, oc)
    for step, most in enumerate((40, 3, 17, 1, 35, 5)):
        new_len = rng.integers(0, most + 1, B).astype(np.int32)
        new_len[0] = most
        rows = int(new_len.sum())
        k, v = edge_values(rng, rows, Hkv), edge_values(rng, rows, Hkv)
        score = rng.random((rows, Hkv)).astype(np.float32)
        hi = (new_len[:, None] * rng.random((B, Hkv))).astype(np.int32)
        lo = ((new_len[:, None] - hi) * rng.choice([0.0, 0.5, 1.0], (B, Hkv))).astype(np.int32)
        quota = np.stack([hi, lo], axis=2).astype(np.int32)
        print("case: page jobs layout=%d B=%d step=%d" % (layout, B, step), flush=True)
        orc.quantize_append(oc, new_len, k, v, score, quota=quota)
        dk.quantize_append(dc, t(new_len), t(k), t(v), t(score), quota=t(quota), total_new=rows, max_new=most)
        assert oc.status[0] == 0
        assert_state_equal(dc, oc, what="layout %d step %d" % (layout, step))


@pytest.mark.parametrize("shift", [1, 2, 3, 4, 7])
def test_rows_of_any_alignment(shift):
    """k and v that start `shift` fp16 values past a 16-byte boundary (a slice of a larger buffer)."""
    import torch
    rng = np.random.default_rng(shift)
    Lo, Ld = layouts(max_seq_len=192)
    B, Hkv = 3, 2
    pages = B * Hkv * 16
    oc = orc.Cache(Lo, pages, B, Hkv, ring=rng.permutation(pages))
    dc = dev_cache_from_oracle(Ld, oc)
    for step, most in enumerate((70, 1, 19)):
        new_len = np.array([most, most // 2, 1], np.int32)
        rows = int(new_len.sum())
        k, v = edge_values(rng, rows, Hkv), edge_values(rng, rows, Hkv)
        score = rng.random((rows, Hkv)).astype(np.float32)
        quota = np.repeat(np.stack([new_len // 2, new_len - new_len // 2], 1)[:, None], Hkv, 1).astype(np.int32)

        def shifted(x):
            buf = torch.zeros(x.size + 16, dtype=torch.int16, device="cuda")
            out = buf[shift:shift + x.size].view(x.shape)
            out.copy_(t(x))
            assert out.data_ptr() % 16 == 2 * shift
            return out

        print("case: page jobs shift=%d step=%d" % (shift, step), flush=True)
        orc.quantize_append(oc, new_len, k, v, score, quota=quota)
        dk.quantize_append(dc, t(new_len), shifted(k), shifted(v), t(score), quota=t(quota), total_new=rows,
                           max_new=most)
        assert oc.status[0] == 0
        assert_state_equal(dc, oc, what="shift %d step %d" % (shift, step))


def model_group(x, bits):
    """(scale, zero, codes) of one group: NaN ignored in the extremes, NaN quotients code 0."""
    with np.errstate(all="ignore"):
        f = x.astype(np.float32) + np.float32(0)
        ok = f[~np.isnan(f)]
        mn, mx = (ok.min(), ok.max()) if ok.size else (np.float32(np.nan),) * 2
        lb = np.float32(2 ** bits - 1)
        s, z = ((mx - mn) / lb).astype(np.float16), mn.astype(np.float16)
        if s == 0:
            return s, z, np.zeros(f.size, np.int64)
        q = np.rint((f - z.astype(np.float32)) / s.astype(np.float32))
        q[np.isnan(q)] = 0
        return s, z, np.clip(q, 0, lb).astype(np.int64)


def codes_of(seg, count, bits):
    """`count` codes of `bits` bits from a segment's rows of bytes, lowest first."""
    return np.unpackbits(seg, axis=-1, bitorder="little")[..., :count * bits].reshape(*seg.shape[:-1], count, bits) @ \
        (1 << np.arange(bits))


@pytest.mark.parametrize("layout", range(4))
def test_infinities_and_nan(layout):
    """Groups with infinities and NaN: an infinity makes the scale infinite and every code 0, NaN counts
    in no extreme and gets code 0, and the groups beside them are untouched by either."""
    import torch
    rng = np.random.default_rng(40 + layout)
    Lo, Ld = layouts(max_seq_len=192, **LAYOUTS[layout])
    n = 24
    k, v = (rng.standard_normal((n, 1, 4, 32)).astype(np.float16) for _ in range(2))
    for x in (k, v):
        kind = rng.integers(0, 8, (n, 1, 4))
        at = rng.random(x.shape) < 0.1
        for i, values in enumerate(((np.inf,), (-np.inf,), (np.nan,), (np.inf, -np.inf, np.nan))):
            pick = at & (kind == i)[..., None]
            x[pick] = rng.choice(values, int(pick.sum())).astype(np.float16)
        x[kind == 4] = np.float16(np.nan)
    score = np.arange(n, 0, -1).astype(np.float32)[:, None]
    new_len = np.array([n], np.int32)
    half = n // 2  # one page per section
    quota = np.array([[[half, half]]], np.int32)
    dc = dk.Cache(Ld, 8, 1, 1)
    bits = lambda x: torch.from_numpy(x.view(np.int16).reshape(n, 1, 128).copy()).cuda()
    print("case: page jobs, infinities and NaN, layout=%d" % layout, flush=True)
    dk.quantize_append(dc, t(new_len), bits(k), bits(v), t(score), quota=t(quota), total_new=n, max_new=n)
    torch.cuda.synchronize()
    assert int(dc.status.cpu()[0]) == 0
    table, pool = dc.page_table.cpu().numpy()[0], dc.pool.cpu().numpy()
    for sec in (0, 1):
        T, kb, vb = Ld.tokens_per_page[sec], Ld.k_bits[sec], Ld.v_bits[sec]
        page = pool[table[0] if sec == 0 else table[-1]]
        chunks = kb  # 128 * kb / 128 chunks of 16 bytes per token
        kc = codes_of(page[Ld.off_kcode[sec]:][:chunks * T * 16].reshape(chunks, T, 16), 128 // kb, kb)
        kc = kc.transpose(1, 0, 2).reshape(T, 128)
        vc = codes_of(page[Ld.off_vcode[sec]:][:128 * T * vb // 8].reshape(128, T * vb // 8), T, vb).T
        km = page[Ld.off_kmeta[sec]:][:T * 16].view(np.float16).reshape(T, 4, 2)
        vm = page[Ld.off_vmeta[sec]:][:T * 16].view(np.float16).reshape(4, T, 2)
        for slot in range(half):
            for g in range(4):
                for x, b, code, meta in ((k, kb, kc, km[slot, g]), (v, vb, vc, vm[g, slot])):
                    s, z, want = model_group(x[sec * half + slot, 0, g], b)
                    assert np.array_equal(np.array([s, z]), meta, equal_nan=True), (sec, slot, g, s, z, meta)
                    assert np.array_equal(code[slot, 32 * g:32 * g + 32], want), (sec, slot, g)
