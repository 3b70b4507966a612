"""Grouped queries with two query heads per workgroup (large batches): the same results as the kernel for one head,
which serves each sequence by itself (a batch too small for pairs), and the oracle's."""
import math

import numpy as np
import pytest
import torch

import paper_2405_03917_amd as cq
from oracle import cq_oracle as O

from gpu_util import check_attention, codes_to_cache, dev

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)


def _problem(seed, c, b, hq, hkv, B, t, data="plain"):
    fmt = cq.CQFormat(c, b, 128, hkv)
    rng = np.random.default_rng(seed)
    G, K = fmt.groups, 1 << b
    ck = rng.standard_normal((G, K, c)).astype(np.float16)
    cv = rng.standard_normal((G, K, c)).astype(np.float16)
    q = rng.standard_normal((B, hq, 128)).astype(np.float16)
    kc = rng.integers(0, K, size=(B, t, G)).astype(np.uint16)
    vc = rng.integers(0, K, size=(B, t, G)).astype(np.uint16)
    if data != "plain":                       # scores that grow (or shrink) by a few hundred binades along the context
        ck = np.broadcast_to((np.arange(K) * (8.0 / K))[None, :, None], ck.shape).astype(np.float16)
        ramp = (np.arange(t) * K // t).astype(np.uint16)
        kc[:] = (ramp if data == "growing" else ramp[::-1])[None, :, None]
        # (one head of each pair falls while the other grows: their bins are rescaled apart)
        q = (0.3 * np.abs(q) * np.where(np.arange(hq) % 2, 1, -1 if data == "opposed" else 1)[None, :, None]).astype(np.float16)
    return fmt, ck, cv, q, kc, vc


def _attend(fmt, ck, cv, q, kcache, vcache, t, t_cap, lens, split):
    return cq.cq_decode_attention(q, kcache, vcache, ck, cv, SCALE, fmt, t, t_cap, seq_lens=lens, tokens_per_split=split)


def _close(pairs, single):
    """Both round fp32 values that differ by some 1e-6 of the largest weight's terms to fp16: one unit in the last place."""
    p, s = pairs.float(), single.float()
    floor = 1e-3 * s.abs().amax(-1, keepdim=True)
    assert torch.isfinite(p).all()
    assert ((p - s).abs() <= 2.0 ** -10 * torch.maximum(s.abs(), floor)).all()


@pytest.mark.parametrize("c,b", [(8, 8), (4, 8), (2, 8), (8, 10)])
@pytest.mark.parametrize("hq,hkv,B,t,split,data", [
    (32, 8, 16, 1, 0, "plain"), (32, 8, 16, 64, 0, "plain"), (32, 8, 16, 65, 0, "plain"), (16, 8, 32, 1000, 0, "plain"),
    (32, 8, 16, 1025, 1088, "plain"), (32, 8, 16, 2049, 0, "plain"), (12, 2, 85, 300, 0, "plain"),
    (16, 4, 8, 900, 256, "plain"), (4, 2, 15, 2100, 128, "plain"),
    (4, 1, 128, 8192, 8192, "growing"), (4, 1, 128, 8000, 8192, "opposed"), (4, 1, 128, 8192, 8192, "shrinking"),
    (2, 1, 256, 20000, 20032, "growing"), (2, 1, 256, 20000, 20032, "opposed")])
def test_pairs_equal_single_heads(c, b, hq, hkv, B, t, split, data):
    if split > 16384 and (b == 10 or c == 2):
        split = 8192                          # (the longest splits of formats that walk one chunk)
    distinct = min(B, 6)                      # sequences that differ; the others repeat them
    fmt, ck, cv, q, kc, vc = _problem(t + c, c, b, hq, hkv, distinct, t, data)
    t_cap = (t + 63) // 64 * 64
    k1, v1 = codes_to_cache(kc, fmt, t_cap), codes_to_cache(vc, fmt, t_cap)
    at = torch.arange(B, device="cuda") % distinct
    kcache = k1.view(distinct, -1)[at].flatten()
    vcache = v1.view(distinct, -1)[at].flatten()
    lens1 = torch.tensor([t, max(1, t - 1), max(1, t // 2), max(1, t // 3), 1, t], dtype=torch.int32, device="cuda")[:distinct]
    ckd, cvd, qd = dev(ck), dev(cv), dev(q)
    out = _attend(fmt, ckd, cvd, qd[at].contiguous(), kcache, vcache, t, t_cap, lens1[at].contiguous(), split)
    for n in range(distinct):
        step = k1.numel() // distinct
        one = _attend(fmt, ckd, cvd, qd[n:n + 1], k1[n * step:(n + 1) * step], v1[n * step:(n + 1) * step], t, t_cap, lens1[n:n + 1],
                      split if split else cq.cq_decode_default_split(fmt, B, hq, t))
        rows = out[n::distinct]
        assert torch.equal(rows, rows[:1].expand_as(rows))
        _close(rows[:1], one)
    n = min(2, distinct - 1)
    ln = int(lens1[n])
    if ln <= 2048:
        check_attention(out[n].cpu().numpy(), O.attention(q[n:n + 1], kc[n:n + 1, :ln], vc[n:n + 1, :ln], ck, cv, SCALE, hkv)[0])


@pytest.mark.parametrize("c,b", [(8, 8), (4, 8), (2, 8), (8, 10)])
@pytest.mark.parametrize("t,split", [(1, 0), (64, 0), (700, 256)])
def test_the_fused_step_of_pairs_and_of_layers(c, b, t, split):
    """cq_decode_step of pairs equals cq_encode_kv then cq_decode_attention, and cq_decode_step_layers of the same
    layers equals both, bit for bit."""
    hq, hkv, B, n_layers = 32, 8, 16, 2
    t_cap = (t + 63) // 64 * 64
    layers, want = [], []
    for l in range(n_layers):
        fmt, ck, cv, q, kc, vc = _problem(50 + l + t, c, b, hq, hkv, B, t)
        rng = np.random.default_rng(l)
        xk, xv = (dev(rng.standard_normal((B, fmt.channels)).astype(np.float16)) for _ in range(2))
        k0, v0 = codes_to_cache(kc, fmt, t_cap), codes_to_cache(vc, fmt, t_cap)
        ckd, cvd, qd = dev(ck), dev(cv), dev(q)
        k1, v1 = k0.clone(), v0.clone()
        cq.cq_encode_kv(xk[:, None], xv[:, None], ckd, cvd, fmt, k1, v1, t - 1, t_cap)
        ref = _attend(fmt, ckd, cvd, qd, k1, v1, t, t_cap, None, split)
        k2, v2 = k0.clone(), v0.clone()
        out = cq.cq_decode_step(qd, xk, xv, k2, v2, ckd, cvd, SCALE, fmt, t, t_cap, tokens_per_split=split)
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
        assert torch.equal(k2, k1) and torch.equal(v2, v1)
        layers.append(dict(q=qd, x_k_new=xk, x_v_new=xv, k_codes=k0.clone(), v_codes=v0.clone(), k_centroids=ckd, v_centroids=cvd,
                           out=torch.empty_like(qd)))
        want.append((ref, k1, v1))
    cq.cq_decode_step_layers(cq.LayerTable(layers, fmt, t_cap), SCALE, t, tokens_per_split=split)
    torch.cuda.synchronize()
    for lay, (ref, k1, v1) in zip(layers, want):
        assert torch.equal(lay["out"].view(torch.int16), ref.view(torch.int16))
        assert torch.equal(lay["k_codes"], k1) and torch.equal(lay["v_codes"], v1)


def _pools(fmt, k1, v1, B, tiles, seed):
    """The caches of `distinct` sequences as pools for B sequences (sequence n holds what n % distinct does) on permuted
    pages, a table with a row stride of its own, and the pages that no sequence has."""
    distinct = k1.shape[0]
    n_pages = B * tiles + 5
    perm = torch.from_numpy(np.random.default_rng(seed).permutation(n_pages)).cuda()
    wide = torch.full((B, tiles + 3), -7, dtype=torch.int32, device="cuda")
    wide[:, :tiles] = perm[:B * tiles].view(B, tiles).int()
    pools = []
    for cache in (k1, v1):
        tiles_of = cache.view(distinct, fmt.n_kv_heads, tiles, -1).transpose(1, 2)          # [n, tile, head, bytes]
        pool = torch.full((n_pages, fmt.n_kv_heads, tiles_of.shape[-1]), 0xA5, dtype=torch.uint8, device="cuda")
        pool[perm[:B * tiles]] = tiles_of[torch.arange(B, device="cuda") % distinct].reshape(B * tiles, fmt.n_kv_heads, -1)
        pools.append(pool)
    return pools, cq.PageTable(wide[:, :tiles], n_pages), perm[B * tiles:]


# (16 wavefronts of at most 8 tiles, of 16 with 10-bit codes, make a chunk: 8192 or 16384 tokens)
PAGED = [(4, 1, 128, 8900, 8960, "growing"), (4, 1, 128, 8900, 8960, "opposed"), (4, 2, 64, 3000, 768, "plain"),
         (8, 2, 64, 130, 0, "plain"), (2, 1, 500, 700, 0, "plain"), (32, 8, 8, 2100, 1088, "plain")]


@pytest.mark.parametrize("c,b", [(8, 8), (4, 8), (2, 8), (8, 10)])
@pytest.mark.parametrize("hq,hkv,B,t,split,data", PAGED)
def test_pairs_over_pages_and_ragged_lengths(c, b, hq, hkv, B, t, split, data):
    """Paged attention of pairs equals the contiguous call bit for bit (splits of several chunks, several splits, splits
    beyond a sequence's end), and the paged fused step at ragged positions equals cq_encode_kv_paged, sequence by
    sequence, then the paged attention; pages of no sequence stay as they are."""
    if split > 8192 and c == 2:
        split = 4480                          # (CQ-2c8b walks one chunk)
    distinct = 5
    fmt, ck, cv, q, kc, vc = _problem(t + 7 * c, c, b, hq, hkv, distinct, t, data)
    tiles = (t + 63) // 64
    t_cap = tiles * 64
    assert cq.cq_probe_decode_plan(fmt, B, hq, t, split)[0] == 2 and cq.cq_probe_decode_plan(fmt, 1, hq, t, split)[0] == 1
    k1, v1 = (codes_to_cache(x, fmt, t_cap).view(distinct, -1) for x in (kc, vc))
    at = torch.arange(B, device="cuda") % distinct
    lens1 = torch.tensor([t, max(1, t // 3), 1, max(1, t - 64), max(1, t // 2)], dtype=torch.int32, device="cuda")
    lens = lens1[at].contiguous()
    ckd, cvd, qd = dev(ck), dev(cv), dev(q)[at].contiguous()
    (kp, vp), pages, unused = _pools(fmt, k1, v1, B, tiles, t)
    flat = lambda p: p.view(-1)

    for sl in (None, lens):
        got = cq.cq_decode_attention_paged(qd, flat(kp), flat(vp), ckd, cvd, SCALE, fmt, t, pages, seq_lens=sl, tokens_per_split=split)
        want = _attend(fmt, ckd, cvd, qd, k1[at].flatten(), v1[at].flatten(), t, t_cap, sl, split)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    for n in range(distinct):                 # (the kernel for one head, by itself)
        _close(got[n:n + 1], _attend(fmt, ckd, cvd, qd[n:n + 1], k1[n], v1[n], t, t_cap, lens1[n:n + 1],
                                     split if split else cq.cq_decode_default_split(fmt, B, hq, t)))

    rng = np.random.default_rng(t)
    xk, xv = (dev(rng.standard_normal((distinct, fmt.channels)).astype(np.float16))[at].contiguous() for _ in range(2))
    k2, v2 = kp.clone(), vp.clone()
    for n in range(B):
        row = cq.PageTable(pages.block_table[n:n + 1], pages.n_pages)
        cq.cq_encode_kv_paged(xk[n:n + 1, None], xv[n:n + 1, None], ckd, cvd, fmt, flat(k2), flat(v2), row, int(lens1[n % distinct]) - 1)
    want = cq.cq_decode_attention_paged(qd, flat(k2), flat(v2), ckd, cvd, SCALE, fmt, t, pages, seq_lens=lens, tokens_per_split=split)
    k3, v3 = kp.clone(), vp.clone()
    got = cq.cq_decode_step_paged(qd, xk, xv, flat(k3), flat(v3), ckd, cvd, SCALE, fmt, t, pages, seq_lens=lens, tokens_per_split=split)
    torch.cuda.synchronize()
    assert torch.isfinite(got.float()).all()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert torch.equal(k3, k2) and torch.equal(v3, v2)
    assert bool((k3[unused] == 0xA5).all()) and bool((v3[unused] == 0xA5).all())
    rows = got[1::distinct]
    assert torch.equal(rows, rows[:1].expand_as(rows))


@pytest.mark.parametrize("c,b", [(8, 8), (4, 8), (2, 8), (8, 10)])
def test_a_given_split_fixes_the_bits_of_ungrouped_heads_in_every_batch(c, b):
    hq = hkv = 8
    B, t, split = 64, 1500, 512
    fmt, ck, cv, q, kc, vc = _problem(c, c, b, hq, hkv, 3, t)
    t_cap = 1536
    k1, v1 = (codes_to_cache(x, fmt, t_cap).view(3, -1) for x in (kc, vc))
    at = torch.arange(B, device="cuda") % 3
    lens = torch.tensor([t, 700, 1], dtype=torch.int32, device="cuda")
    ckd, cvd, qd = dev(ck), dev(cv), dev(q)
    out = _attend(fmt, ckd, cvd, qd[at].contiguous(), k1[at].flatten(), v1[at].flatten(), t, t_cap, lens[at].contiguous(), split)
    for n in range(3):
        one = _attend(fmt, ckd, cvd, qd[n:n + 1], k1[n], v1[n], t, t_cap, lens[n:n + 1], split)
        assert torch.equal(out[n::3].view(torch.int16), one.expand_as(out[n::3]).contiguous().view(torch.int16))
