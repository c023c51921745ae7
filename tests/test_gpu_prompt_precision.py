"""Prompt significance with rows computed by the call: the error against 64 bits.  The bounds are
what the 16x16-tile kernel before this one showed on the same inputs; results are
deterministic."""
import numpy as np
import pytest
from test_gpu_prompt_significance import LD, SCALE

from gpu_util import t
from paper_2412_03131_amd import diffkv as dk

pytestmark = pytest.mark.gpu


def _exact(new_len, q, k):
    q, k = q.astype(np.float64), k.astype(np.float64)
    out, r = np.zeros(k.shape[:2]), 0
    g = q.shape[1] // k.shape[1]
    for n in new_len:
        for h in range(k.shape[1]):
            s = np.einsum("qtd,kd->tqk", q[r:r + n, h * g:(h + 1) * g], k[r:r + n, h]) * SCALE
            s = np.where(np.tril(np.ones((n, n), bool)), s, -np.inf)
            p = np.exp(s - s.max(2, keepdims=True))
            p /= p.sum(2, keepdims=True)
            out[r:r + n, h] = p.max(0).sum(0) / np.arange(n, 0, -1)
        r += n
    return out


@pytest.mark.parametrize("lens,Hkv,g,bound", [
    ((300, 223), 4, 4, 3.25e-7),
    ((900, 700), 2, 8, 3.77e-7),
    ((1500,), 2, 3, 3.99e-7),
])
def test_error_against_64_bits(lens, Hkv, g, bound):
    import torch
    rng = np.random.default_rng(sum(lens))
    n = sum(lens)
    q = rng.standard_normal((n, Hkv * g, 128)).astype(np.float16)
    k = rng.standard_normal((n, Hkv, 128)).astype(np.float16)
    k[:, :, :4] *= np.float16(10)
    new_len = np.array(lens, np.int32)
    print("case: prompt precision %s g=%d" % (lens, g), flush=True)
    got = dk.prompt_significance(LD, t(new_len), t(q), t(k), SCALE)
    torch.cuda.synchronize()
    want = _exact(lens, q, k)
    err = np.linalg.norm(got.cpu().numpy().astype(np.float64) - want) / np.linalg.norm(want)
    print("error %.4e" % err, flush=True)
    assert err <= bound
