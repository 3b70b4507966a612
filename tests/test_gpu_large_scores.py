"""Attention whose scores are far beyond those of a trained model: queries and keys in the
thousands and scales around one give score x log2(e) up to 2^34, where a unit in the last place of
an fp32 score is more than the logarithm of fp16's range.  The inputs are finite, so the outputs are
those of the oracle: the softmax falls on the tokens with the largest score, and tokens of equal
codes share it."""
import numpy as np
import pytest
import torch

import paper_2405_03917_amd as cq
from oracle import cq_oracle as O

from gpu_util import check_attention, codes_to_cache, dev

pytestmark = pytest.mark.gpu

BASE = 10000.0
# largest |score| log2(e), about
MAGNITUDES = [2.0 ** 18, 2.0 ** 23, 2.0 ** 26, 2.0 ** 28, 2.0 ** 30, 2.0 ** 34]


def _case(seed, c, b, hq, hkv, B, m, T, distinct):
    rng = np.random.default_rng(seed)
    fmt = cq.CQFormat(c, b, 128, hkv)
    ck = (2000.0 * rng.standard_normal((fmt.groups, 1 << b, c))).astype(np.float16)
    cv = rng.standard_normal((fmt.groups, 1 << b, c)).astype(np.float16)
    kc = rng.integers(0, 1 << b, size=(B, T, fmt.groups)).astype(np.uint16)
    if distinct:                                             # tokens that share their key and with it the weight
        kc = kc[:, rng.integers(0, distinct, size=T)]
    vc = rng.integers(0, 1 << b, size=(B, T, fmt.groups)).astype(np.uint16)
    q = (2000.0 * rng.standard_normal((B, m, hq, 128))).astype(np.float16)
    return fmt, q, kc, vc, ck, cv


def _scale(magnitude, sign=1.0):
    # the largest of some thousand products of 128 channels is about 4 sqrt(128) 2000^2
    return float(sign * magnitude / (4.0 * 128 ** 0.5 * 2000.0 ** 2 * 1.4426950408889634))


def _reference(q, kc, vc, ck, cv, scale, hkv, rope_base=None):
    """Outputs of the oracle, and which rows are decided: the largest score is ahead of every other
    score by more than fp32 scores can err.  (A score is a sum of 128 products, rounded once or twice:
    2^-20 of the largest is ample; a lead of 64 leaves the others no weight.)"""
    B, m, hq, d = q.shape
    T = kc.shape[1]
    ref, clear = np.empty((B, m, hq, d)), np.empty((B, m, hq), dtype=bool)
    for j in range(m):
        n = T - m + 1 + j
        ref[:, j], s = O.attention(np.ascontiguousarray(q[:, j]), kc, vc, ck, cv, scale, hkv, want_scores=True,
                                   seq_lens=np.full(B, n, dtype=np.int32), rope_base=rope_base)
        s = s[:, :, :n]
        top = s.max(-1, keepdims=True)
        lead = (top - np.where(s < top, s, -np.inf).max(-1, keepdims=True))[..., 0]
        clear[:, j] = lead > np.maximum(64.0, 2.0 ** -20 * np.abs(s).max(-1))
    assert clear.mean() > 0.9
    return ref, clear


def _check(out, ref, clear):
    torch.cuda.synchronize()
    check_attention(out.cpu().numpy().reshape(ref.shape)[clear], ref[clear])


@pytest.mark.parametrize("magnitude", MAGNITUDES)
@pytest.mark.parametrize("c,hq", [(8, 8), (8, 4), (4, 6), (4, 4), (2, 4)])
def test_grouped_decode_over_rotated_keys(c, hq, magnitude):
    hkv, B, T = 2, 2, 700
    fmt, q, kc, vc, ck, cv = _case(c, c, 8, hq, hkv, B, 1, T, 0)
    t_cap = -(-T // 64) * 64
    rope = cq.RopeTable(BASE, t_cap)
    kcache, vcache = codes_to_cache(kc, fmt, t_cap), codes_to_cache(vc, fmt, t_cap)
    scale = _scale(magnitude)
    ref, clear = _reference(q, kc, vc, ck, cv, scale, hkv, BASE)
    for split in (t_cap, 256):
        _check(cq.cq_decode_attention_rope(dev(q[:, 0]), kcache, vcache, dev(ck), dev(cv), scale, fmt, T, t_cap, rope,
                                           tokens_per_split=split), ref, clear)


@pytest.mark.parametrize("magnitude,sign", [(x, 1.0) for x in MAGNITUDES] + [(2.0 ** 30, -1.0)])
@pytest.mark.parametrize("c,m,hq", [(8, 5, 2), (8, 6, 8), (4, 5, 2), (4, 16, 4), (8, 3, 2), (8, 4, 2), (4, 3, 2), (4, 4, 2)])
def test_chunks_of_few_rows(c, m, hq, magnitude, sign):
    hkv, B, T = 2, 2, 500
    fmt, q, kc, vc, ck, cv = _case(10 + c + m, c, 8, hq, hkv, B, m, T, 40)
    t_cap = -(-T // 64) * 64
    kcache, vcache = codes_to_cache(kc, fmt, t_cap), codes_to_cache(vc, fmt, t_cap)
    scale = _scale(magnitude, sign)
    ref, clear = _reference(q, kc, vc, ck, cv, scale, hkv)
    for split in (0, 256, t_cap):
        _check(cq.cq_chunk_attention(dev(q), kcache, vcache, dev(ck), dev(cv), scale, fmt, T, t_cap, tokens_per_split=split), ref, clear)


@pytest.mark.parametrize("magnitude,sign", [(x, 1.0) for x in MAGNITUDES] + [(2.0 ** 30, -1.0)])
@pytest.mark.parametrize("c,b", [(8, 8), (4, 8), (2, 8), (8, 10)])
@pytest.mark.parametrize("rope", [False, True])
def test_chunks_of_many_rows(rope, c, b, magnitude, sign):
    hq, hkv, B, T = 4, 2, 2, 500
    for m in (50, 70):                                       # 100 and 140 rows: four wavefronts and eight
        fmt, q, kc, vc, ck, cv = _case(30 + c + m, c, b, hq, hkv, B, m, T, 0 if rope else 40)
        t_cap = -(-T // 64) * 64
        args = (dev(q), codes_to_cache(kc, fmt, t_cap), codes_to_cache(vc, fmt, t_cap), dev(ck), dev(cv))
        scale = _scale(magnitude, sign)
        ref, clear = _reference(q, kc, vc, ck, cv, scale, hkv, BASE if rope else None)
        for split in (64, 256, t_cap):
            if rope:
                out = cq.cq_chunk_attention_rope(*args, scale, fmt, T, t_cap, cq.RopeTable(BASE, t_cap), tokens_per_split=split)
            else:
                out = cq.cq_chunk_attention(*args, scale, fmt, T, t_cap, tokens_per_split=split)
            _check(out, ref, clear)
