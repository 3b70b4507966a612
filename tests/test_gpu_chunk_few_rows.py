"""Chunks of three and four rows per KV head (CQ-8c8b, CQ-4c8b): their own kernel against the oracle where it can go
wrong: a last tile that only the last rows see, wavefronts and splits without a visible token, ragged lengths down to
the chunk itself, more items than workgroups, scores that grow along the context, pages."""
import math

import numpy as np
import pytest
import torch

import paper_2405_03917_amd as cq
from oracle import cq_oracle as O

from gpu_util import codes_to_cache, dev
from test_gpu_chunk import _case, _check
from test_gpu_decode_pairs import _pools

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [8, 4])
@pytest.mark.parametrize("m,T,split,hkv,data", [(3, 257, 0, 2, "plain"), (4, 258, 0, 1, "plain"), (4, 1025, 256, 2, "plain"), (3, 1091, 320, 1, "growing"),
                                                (4, 640, 640, 200, "plain")])
def test_few_rows_match_the_oracle(c, m, T, split, hkv, data):
    B = 5
    fmt, q, kc, vc, ck, cv = _case(m + T, c, 8, hkv, hkv, B, m, T)
    if data == "growing":                     # (scores rise by a few hundred binades: the reference moves with them)
        ck = np.broadcast_to((np.arange(256) / 32.0)[None, :, None], ck.shape).astype(np.float16)
        kc[:] = (np.arange(T) * 256 // T).astype(np.uint16)[None, :, None]
        q = np.abs(q)
    t_cap = -(-T // 64) * 64
    lens = np.array([T, m, T - 1, T // 2, min(T, 66)], dtype=np.int32)
    k1, v1 = codes_to_cache(kc, fmt, t_cap), codes_to_cache(vc, fmt, t_cap)
    scale = 1.0 / math.sqrt(128)
    a = (dev(ck), dev(cv), scale, fmt, T)
    outs = []
    for sl in (None, lens):
        sld = None if sl is None else dev(sl)
        out = cq.cq_chunk_attention(dev(q), k1, v1, *a, t_cap, seq_lens=sld, tokens_per_split=split)
        heads = slice(0, hkv) if hkv <= 2 else slice(0, 3)      # (a KV head's rows do not depend on the others)
        groups = slice(0, heads.stop * 128 // c)
        ref = O.chunk_attention(np.ascontiguousarray(q[:, :, heads]), kc[:, :, groups], vc[:, :, groups], ck[groups], cv[groups], scale,
                                heads.stop, seq_lens=sl)
        _check(np.ascontiguousarray(out.cpu().numpy()[:, :, heads]), ref)
        outs.append(out)
    (kp, vp), pages, _ = _pools(fmt, k1.view(B, -1), v1.view(B, -1), B, t_cap // 64, T)
    got = cq.cq_chunk_attention_paged(dev(q), kp.view(-1), vp.view(-1), *a, pages, seq_lens=dev(lens), tokens_per_split=split)
    assert torch.equal(got.view(torch.int16), outs[1].view(torch.int16))
