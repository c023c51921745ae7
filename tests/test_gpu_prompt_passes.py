"""Prompt-phase significance where its two passes branch: query segments of the column
pass (fewer stages than segments, one segment, a sum over several), pairs no multiple of
eight with empty blocks between, head groups of the row pass, and
logits that jump past what the row pass's running max absorbs.  Against the oracle,
with the tolerance of fp32 logits (relative 5e-5)."""
import numpy as np
import pytest
from test_gpu_prompt_significance import LD, SCALE, _close, _draw, _lse_numpy

from gpu_util import t
from oracle import oracle as orc
from paper_2412_03131_amd import diffkv as dk

pytestmark = pytest.mark.gpu


def _run(new_len, q, k, lse=None):
    import torch
    got = dk.prompt_significance(LD, t(new_len), t(q).view(torch.float16), t(k).view(torch.float16), SCALE,
                                 lse=None if lse is None else t(lse))
    torch.cuda.synchronize()
    return got.cpu().numpy()


@pytest.mark.parametrize("lens,Hkv,g", [
    ((31,), 1, 1),                         # fewer stages than segments
    ((33, 0, 255, 256, 257), 3, 7),        # head groups of 4 + 3, block edges
    ((700,), 2, 8),                        # two head groups, several stages per segment
    ((5, 130, 1, 64, 97) * 5, 9, 2),       # 225 pairs, no multiple of eight
    ((129,) * 260, 8, 1),                  # 2080 key blocks: one segment
])
def test_segments_and_queues(lens, Hkv, g):
    rng = np.random.default_rng(len(lens) * 100 + Hkv * 10 + g)
    new_len = np.array(lens, np.int32)
    q, k = _draw(rng, new_len, Hkv * g, Hkv)
    print("case: prompt passes %s x%d Hkv=%d g=%d" % (lens[:5], len(lens), Hkv, g), flush=True)
    want = orc.prompt_significance(new_len, q, k, SCALE)
    _close(_run(new_len, q, k), want, "rows computed")
    _close(_run(new_len, q, k, _lse_numpy(new_len[new_len > 0], q, k)), want, "rows given")


@pytest.mark.parametrize("step", [0.9, 1.3, 2.2, 4.0])
def test_logits_that_jump(step):
    """Every 40 keys the logits rise by about 16, 24, 40 or 72 (23 to 104 in log2, beyond the
    raise threshold of 8, and past 127, where the first sum overflows, over two steps)."""
    rng = np.random.default_rng(7)
    new_len = np.array([230], np.int32)
    q = (np.ones((230, 3, 128)) * 1.5 + rng.standard_normal((230, 3, 128)) * 0.01).astype(np.float16)
    level = (np.arange(230) // 40 - 3)[:, None, None]
    k = (np.ones((230, 1, 128)) * level * step + rng.standard_normal((230, 1, 128)) * 0.05).astype(np.float16)
    q, k = q.view(np.uint16), k.view(np.uint16)
    print("case: jumping logits, step %g" % step, flush=True)
    # logits reach 200: fp32 sums of 128 products of about 18 are off by up to 1e-4 in the exponent's unit
    got, want = _run(new_len, q, k), orc.prompt_significance(new_len, q, k, SCALE)
    assert np.all(np.abs(got - want) <= 5e-4 * np.abs(want) + 1e-30), np.abs(got / np.maximum(want, 1e-30) - 1).max()
