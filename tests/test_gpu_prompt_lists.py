"""Prompt significance's lists of work items: more items than workgroups, with one long prompt among
many short ones (groups of unequal size, lists of unequal length, pairs no multiple of eight, a
search over more than 64 groups), and the workspace's end, behind which nothing is written."""
import numpy as np
import pytest
from test_gpu_prompt_passes import _run
from test_gpu_prompt_significance import LD, SCALE, _close, _draw, _lse_numpy

from gpu_util import t
from oracle import oracle as orc
from paper_2412_03131_amd import diffkv as dk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,Hkv,g", [
    ((600,) + (3, 0, 1) * 600, 8, 1),         # 14408 pairs: 226 groups per list
    ((2, 70, 5) * 40 + (900,) + (17,) * 500, 7, 3),  # a long prompt in the middle
    ((1, 2) * 300 + (1100, 513), 5, 8),       # two head groups, the long ones last
])
def test_more_items_than_workgroups(lens, Hkv, g):
    rng = np.random.default_rng(len(lens))
    new_len = np.array(lens, np.int32)
    q, k = _draw(rng, new_len, Hkv * g, Hkv)
    print("case: prompt lists B=%d Hkv=%d g=%d" % (len(lens), Hkv, g), flush=True)
    want = orc.prompt_significance(new_len, q, k, SCALE)
    _close(_run(new_len, q, k), want, "rows computed")
    _close(_run(new_len, q, k, _lse_numpy(new_len[new_len > 0], q, k)), want, "rows given")


@pytest.mark.parametrize("lens,Hkv,g", [
    ((1,), 1, 1), ((31,), 1, 8), ((2000,), 1, 1), ((2000,), 8, 1), ((257,) * 7, 5, 7), ((300,) * 63, 8, 2),
    ((300,) * 64, 8, 2), ((4000, 10, 1), 3, 8), ((256,) * 255, 4, 1), ((256,) * 256, 4, 1), ((40,) * 300, 7, 1),
])
def test_nothing_behind_the_workspace(lens, Hkv, g):
    import torch
    new_len = np.array(lens, np.int32)
    n = int(new_len.sum())
    need = dk.workspace_size(dk.OP_PROMPT_SIGNIFICANCE, LD, len(lens), Hkv * g, Hkv, n)
    buf = torch.full((need + 65536,), 0xA5, dtype=torch.uint8, device="cuda")
    q = torch.zeros((n, Hkv * g, 128), dtype=torch.float16, device="cuda")
    k = torch.zeros((n, Hkv, 128), dtype=torch.float16, device="cuda")
    print("case: prompt workspace %s x%d Hkv=%d g=%d" % (lens[:3], len(lens), Hkv, g), flush=True)
    got = dk.prompt_significance(LD, t(new_len), q, k, SCALE, ws=buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0xA5).all())
    # equal logits: query j gives each of its j + 1 keys the same
    off = 0
    for m in lens:
        w = np.cumsum((1.0 / np.arange(1, m + 1))[::-1])[::-1] / np.arange(m, 0, -1)
        assert np.allclose(got[off:off + m].cpu().numpy(), w[:, None], rtol=1e-5)
        off += m
