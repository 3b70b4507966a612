"""Grouped queries with four query heads per workgroup and both codebooks in LDS (enough long splits): the same results
as the kernel for one head, which serves each sequence by itself (a batch too small for quads), and the oracle's."""
import numpy as np
import pytest
import torch

import paper_2405_03917_amd as cq

from gpu_util import check_attention, codes_to_cache, dev
from test_gpu_decode_pairs import SCALE, _attend, _close, _pools, _problem
from test_gpu_large_scores import _case, _check, _reference, _scale

pytestmark = pytest.mark.gpu

# (query heads, KV heads, batch, t, split): the shortest contexts and the fewest items that go here, odd ends, two quads
# per KV head, more items than CUs (a workgroup walks several), splits that join and splits that do not
SHAPES = {8: [(4, 1, 140, 1, 0, "plain"), (8, 2, 70, 65, 0, "plain"), (4, 1, 140, 961, 0, "plain"), (8, 1, 70, 1024, 0, "plain"), (32, 8, 18, 1025, 0, "plain"),
              (4, 1, 300, 1000, 0, "plain"), (4, 1, 150, 2049, 1088, "plain"), (8, 2, 20, 4100, 1024, "growing"), (8, 2, 20, 4100, 1024, "opposed"),
              (4, 1, 140, 3000, 3008, "shrinking")],
          4: [(4, 1, 140, 1, 0, "plain"), (4, 1, 300, 65, 0, "plain"), (32, 8, 18, 1500, 0, "plain"), (4, 1, 140, 4161, 0, "plain"), (8, 2, 70, 4224, 0, "plain"),
              (4, 1, 150, 8500, 4288, "growing"), (4, 1, 36, 16800, 4224, "opposed")]}
LENS = lambda t: torch.tensor([t, max(1, t - 1), max(1, t // 2), 1, max(1, t - 64)], dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("c,hq,hkv,B,t,split,data", [(c, *s) for c in SHAPES for s in SHAPES[c]])
def test_quads_equal_single_heads_over_pages_and_in_the_fused_step(c, hq, hkv, B, t, split, data):
    """Attention of quads is that of the kernel for one head to a unit in the last place; over pages the same bits; and
    the fused step at ragged positions is cq_encode_kv, sequence by sequence, then the attention, bit for bit."""
    distinct = 5
    fmt, ck, cv, q, kc, vc = _problem(t + c, c, 8, hq, hkv, distinct, t, data)
    tiles = (t + 63) // 64
    t_cap = tiles * 64
    assert cq.cq_probe_decode_plan(fmt, B, hq, t, split)[0] == 4 and cq.cq_probe_decode_plan(fmt, 1, hq, t, split)[0] == 1
    k1, v1 = (codes_to_cache(x, fmt, t_cap).view(distinct, -1) for x in (kc, vc))
    at = torch.arange(B, device="cuda") % distinct
    lens1 = LENS(t)
    lens = lens1[at].contiguous()
    ckd, cvd, qd = dev(ck), dev(cv), dev(q)
    qb = qd[at].contiguous()
    kb, vb = k1[at].flatten(), v1[at].flatten()
    (kp, vp), pages, unused = _pools(fmt, k1, v1, B, tiles, t)
    one_split = split if split else cq.cq_decode_default_split(fmt, B, hq, t)
    for sl in (None, lens):
        out = _attend(fmt, ckd, cvd, qb, kb, vb, t, t_cap, sl, split)
        for n in range(distinct):
            one = _attend(fmt, ckd, cvd, qd[n:n + 1], k1[n], v1[n], t, t_cap, None if sl is None else lens1[n:n + 1], one_split)
            _close(out[n:n + 1], one)
            rows = out[n::distinct]
            assert torch.equal(rows, rows[:1].expand_as(rows))
        got = cq.cq_decode_attention_paged(qb, kp.view(-1), vp.view(-1), ckd, cvd, SCALE, fmt, t, pages, seq_lens=sl, tokens_per_split=split)
        assert torch.equal(got.view(torch.int16), out.view(torch.int16))

    rng = np.random.default_rng(t)
    xk, xv = (dev(rng.standard_normal((distinct, fmt.channels)).astype(np.float16)) for _ in range(2))
    k2, v2 = k1.clone(), v1.clone()
    for n in range(distinct):
        cq.cq_encode_kv(xk[n:n + 1, None], xv[n:n + 1, None], ckd, cvd, fmt, k2[n], v2[n], int(lens1[n]) - 1, t_cap)
    want = _attend(fmt, ckd, cvd, qb, k2[at].flatten(), v2[at].flatten(), t, t_cap, lens, split)
    k3, v3 = kb.clone(), vb.clone()
    xkb, xvb = xk[at].contiguous(), xv[at].contiguous()
    got = cq.cq_decode_step(qb, xkb, xvb, k3, v3, ckd, cvd, SCALE, fmt, t, t_cap, seq_lens=lens, tokens_per_split=split)
    assert torch.isfinite(got.float()).all()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert torch.equal(k3, k2[at].flatten()) and torch.equal(v3, v2[at].flatten())
    got = cq.cq_decode_step_paged(qb, xkb, xvb, kp.view(-1), vp.view(-1), ckd, cvd, SCALE, fmt, t, pages, seq_lens=lens, tokens_per_split=split)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert bool((kp[unused] == 0xA5).all()) and bool((vp[unused] == 0xA5).all())


@pytest.mark.parametrize("c,hq,hkv,B,t,split", [(8, 8, 2, 70, 1100, 0), (8, 8, 2, 20, 4100, 1024), (4, 4, 1, 140, 4161, 0)])
def test_the_layer_batched_step_of_quads_and_its_replays(c, hq, hkv, B, t, split):
    """cq_decode_step_layers equals the layers' own steps bit for bit, eagerly and from a captured graph."""
    t_cap = (t + 63) // 64 * 64
    layers, want = [], []
    for l in range(2):
        fmt, ck, cv, q, kc, vc = _problem(70 + l, c, 8, hq, hkv, 4, t)
        at = torch.arange(B, device="cuda") % 4
        rng = np.random.default_rng(l)
        xk, xv = (dev(rng.standard_normal((B, fmt.channels)).astype(np.float16)) for _ in range(2))
        k0, v0 = (codes_to_cache(x, fmt, t_cap).view(4, -1)[at].flatten() for x in (kc, vc))
        qb, ckd, cvd = dev(q)[at].contiguous(), dev(ck), dev(cv)
        k1, v1 = k0.clone(), v0.clone()
        want.append((cq.cq_decode_step(qb, xk, xv, k1, v1, ckd, cvd, SCALE, fmt, t, t_cap, tokens_per_split=split), k1, v1))
        layers.append(dict(q=qb, x_k_new=xk, x_v_new=xv, k_codes=k0, v_codes=v0, k_centroids=ckd, v_centroids=cvd, out=torch.empty_like(qb)))
    table = cq.LayerTable(layers, fmt, t_cap)
    ws = torch.empty(2 * cq.cq_decode_workspace_bytes(fmt, B, hq, t, split), dtype=torch.uint8, device="cuda")
    run = lambda: cq.cq_decode_step_layers(table, SCALE, t, tokens_per_split=split, workspace=ws)

    def check():
        torch.cuda.synchronize()
        for lay, (ref, k1, v1) in zip(layers, want):
            assert torch.equal(lay["out"].view(torch.int16), ref.view(torch.int16))
            assert torch.equal(lay["k_codes"], k1) and torch.equal(lay["v_codes"], v1)
            lay["out"].fill_(7.0)
    run()
    check()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for _ in range(3):
        ws.fill_(0xFF)
        graph.replay()
        check()


@pytest.mark.parametrize("c,t", [(8, 1000), (4, 4200)])
@pytest.mark.parametrize("magnitude,sign", [(2.0 ** 23, 1.0), (2.0 ** 28, -1.0), (2.0 ** 34, 1.0)])
def test_quads_of_large_scores(c, t, magnitude, sign):
    hq, hkv, B = 8, 2, 70
    fmt, q, kc, vc, ck, cv = _case(c, c, 8, hq, hkv, 2, 1, t, 40)
    t_cap = (t + 63) // 64 * 64
    scale = _scale(magnitude, sign)
    ref, clear = _reference(q, kc, vc, ck, cv, scale, hkv)
    at = torch.arange(B, device="cuda") % 2
    k, v = (codes_to_cache(x, fmt, t_cap).view(2, -1)[at].flatten() for x in (kc, vc))
    assert cq.cq_probe_decode_plan(fmt, B, hq, t)[0] == 4
    out = cq.cq_decode_attention(dev(q[:, 0])[at].contiguous(), k, v, dev(ck), dev(cv), scale, fmt, t, t_cap)
    _check(out[:2], ref, clear)


@pytest.mark.parametrize("c", [8, 4])
@pytest.mark.parametrize("qper,B,t,split", [(2, 2, 65, 0), (3, 3, 700, 128), (4, 150, 300, 0), (5, 2, 1, 0), (7, 3, 1500, 640), (4, 300, 130, 64)])
def test_rotated_keys_for_up_to_four_heads_equal_single_heads(c, qper, B, t, split):
    """The kernel for four heads against the one for a single head (which splits of more than 88 tiles take)."""
    hkv, distinct = 1, min(B, 3)
    fmt, ck, cv, q, kc, vc = _problem(t + qper, c, 8, qper * hkv, hkv, distinct, t)
    t_cap = 89 * 64
    rope = cq.RopeTable(10000.0, t_cap)
    at = torch.arange(B, device="cuda") % distinct
    k, v = (codes_to_cache(x, fmt, t_cap).view(distinct, -1)[at].flatten() for x in (kc, vc))
    lens = torch.tensor([t, max(1, t - 1), max(1, t // 3)], dtype=torch.int32, device="cuda")[:distinct][at].contiguous()
    a = (dev(q)[at].contiguous(), k, v, dev(ck), dev(cv), SCALE, fmt, t, t_cap, rope)
    out = cq.cq_decode_attention_rope(*a, seq_lens=lens, tokens_per_split=split)
    _close(out, cq.cq_decode_attention_rope(*a, seq_lens=lens, tokens_per_split=89 * 64))
    rows = out[::distinct]
    assert torch.equal(rows, rows[:1].expand_as(rows))


@pytest.mark.parametrize("c", [8, 4])
@pytest.mark.parametrize("qper,t,split", [(3, 300, 128), (4, 1500, 128), (2, 700, 64)])
def test_a_given_split_fixes_the_bits_over_rotated_keys_in_every_batch(c, qper, t, split):
    """Workgroups walk several splits of a large batch one after the other: each stays a partial of its own, as alone."""
    B, distinct = 700, 3
    fmt, ck, cv, q, kc, vc = _problem(t + c, c, 8, qper, 1, distinct, t)
    t_cap = (t + 63) // 64 * 64
    rope = cq.RopeTable(10000.0, t_cap)
    k1, v1 = (codes_to_cache(x, fmt, t_cap).view(distinct, -1) for x in (kc, vc))
    lens = torch.tensor([t, t // 3, 1], dtype=torch.int32, device="cuda")
    ckd, cvd, qd = dev(ck), dev(cv), dev(q)

    def run(at, sl):
        return cq.cq_decode_attention_rope(qd[at].contiguous(), k1[at].flatten(), v1[at].flatten(), ckd, cvd, SCALE, fmt, t, t_cap, rope,
                                           seq_lens=None if sl is None else sl[at].contiguous(), tokens_per_split=split)
    at = torch.arange(B, device="cuda") % distinct
    for sl in (None, lens):
        out = run(at, sl)
        for n in range(distinct):
            rows = out[n::distinct]
            assert torch.equal(rows.view(torch.int16), run(at[n:n + 1], sl).expand_as(rows).contiguous().view(torch.int16))


@pytest.mark.parametrize("c,t", [(8, 1000), (4, 4200)])
@pytest.mark.parametrize("rotated", [False, True])
def test_tokens_beyond_the_range_of_fp32_have_no_weight(c, t, rotated):
    """A tile whose every token scores -inf for some heads (finite operands, a scale that overflows) and the others score 0."""
    hq, hkv, B = 8, 2, 70
    fmt, ck, cv, q, kc, vc = _problem(c, c, 8, hq, hkv, 1, t)
    g = 64 // c - 1                           # (its last channel: the pair that turns slowest, not past a right angle here)
    ck[:], q[:], kc[:] = 0, 0, 0
    ck[g::fmt.groups // hkv, 1, c - 1] = -60000.0
    q[:, ::2, 63] = 1.0                       # (the odd heads score 0 everywhere)
    kc[:, :64] = 1
    t_cap = (t + 63) // 64 * 64
    at = torch.zeros(B, dtype=torch.long, device="cuda")
    k, v = (codes_to_cache(x, fmt, t_cap).view(1, -1)[at].flatten() for x in (kc, vc))
    a = (dev(q)[at].contiguous(), k, v, dev(ck), dev(cv), 1e34, fmt, t, t_cap)
    if rotated:
        out = cq.cq_decode_attention_rope(*a, cq.RopeTable(10000.0, t_cap))
    else:
        assert cq.cq_probe_decode_plan(fmt, B, hq, t)[0] == 4
        out = cq.cq_decode_attention(*a)
    vals = cv.astype(np.float64)[np.arange(fmt.groups), vc[0]].reshape(t, hkv, 128)
    want = np.empty((hq, 128))
    for h in range(hq):
        want[h] = vals[64 if h % 2 == 0 else 0:, h // (hq // hkv)].mean(0)
    check_attention(out.cpu().numpy(), np.broadcast_to(want, (B, hq, 128)))


@pytest.mark.parametrize("c", [8, 4])
@pytest.mark.parametrize("rotated,qper,hkv,B,t,split", [(True, 4, 1, 300, 700, 0), (True, 3, 1, 270, 700, 128), (True, 4, 2, 140, 130, 64), (True, 2, 1, 300, 1, 0),
                                                        (False, 4, 1, 300, 1000, 0), (False, 8, 2, 70, 700, 384)])
def test_the_fused_step_of_workgroups_with_several_items(c, rotated, qper, hkv, B, t, split):
    """Every item brings its own new rows (rows of a wider array) and its own search: cq_encode_kv, sequence by sequence, then
    the attention, bit for bit, with the same codes in the caches; also over pages."""
    distinct, hq = 7, qper * hkv
    fmt, ck, cv, q, kc, vc = _problem(t + c, c, 8, hq, hkv, distinct, t)
    tiles = (t + 63) // 64
    t_cap = tiles * 64
    k1, v1 = (codes_to_cache(x, fmt, t_cap).view(distinct, -1) for x in (kc, vc))
    at = torch.arange(B, device="cuda") % distinct
    lens1 = torch.tensor([t, max(1, t - 1), max(1, t // 2), 1, max(1, t - 64), max(1, t // 3), min(t, 65)], dtype=torch.int32, device="cuda")
    lens = lens1[at].contiguous()
    ckd, cvd, qd = dev(ck), dev(cv), dev(q)[at].contiguous()
    rng = np.random.default_rng(t)
    wide = dev(rng.standard_normal((distinct, 2 * fmt.channels + 8)).astype(np.float16))
    xk, xv = wide[:, :fmt.channels], wide[:, fmt.channels:2 * fmt.channels]
    k2, v2 = k1.clone(), v1.clone()
    for n in range(distinct):
        cq.cq_encode_kv(xk[n:n + 1, None], xv[n:n + 1, None], ckd, cvd, fmt, k2[n], v2[n], int(lens1[n]) - 1, t_cap)
    wide_b = wide[at].contiguous()
    xkb, xvb = wide_b[:, :fmt.channels], wide_b[:, fmt.channels:2 * fmt.channels]
    rope = (cq.RopeTable(10000.0, t_cap),) if rotated else ()
    attention, step, step_paged = ((cq.cq_decode_attention_rope, cq.cq_decode_step_rope, cq.cq_decode_step_rope_paged) if rotated
                                   else (cq.cq_decode_attention, cq.cq_decode_step, cq.cq_decode_step_paged))
    assert rotated or cq.cq_probe_decode_plan(fmt, B, hq, t, split)[0] == 4
    want = attention(qd, k2[at].flatten(), v2[at].flatten(), ckd, cvd, SCALE, fmt, t, t_cap, *rope, seq_lens=lens, tokens_per_split=split)
    assert torch.isfinite(want.float()).all()
    k3, v3 = k1[at].flatten(), v1[at].flatten()
    got = step(qd, xkb, xvb, k3, v3, ckd, cvd, SCALE, fmt, t, t_cap, *rope, seq_lens=lens, tokens_per_split=split)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert torch.equal(k3, k2[at].flatten()) and torch.equal(v3, v2[at].flatten())
    (kp, vp), pages, unused = _pools(fmt, k1, v1, B, tiles, t)
    got = step_paged(qd, xkb, xvb, kp.view(-1), vp.view(-1), ckd, cvd, SCALE, fmt, t, pages, *rope, seq_lens=lens, tokens_per_split=split)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    (k4, v4), _, _ = _pools(fmt, k2, v2, B, tiles, t)
    assert torch.equal(kp, k4) and torch.equal(vp, v4)


@pytest.mark.parametrize("c,T", [(8, 1500), (4, 700)])
def test_a_chunk_of_two_tokens_goes_to_quads_token_by_token(c, T):
    """Query rows two tokens apart, contexts shortened by a token: the bits of the single-token calls."""
    hq, hkv, B, m = 8, 2, 72, 2
    fmt, ck, cv, _, kc, vc = _problem(c, c, 8, hq, hkv, 4, T)
    t_cap = (T + 63) // 64 * 64
    assert all(cq.cq_probe_decode_plan(fmt, B, hq, t)[0] == 4 for t in (T, T - 1))
    at = torch.arange(B, device="cuda") % 4
    k, v = (codes_to_cache(x, fmt, t_cap).view(4, -1)[at].flatten() for x in (kc, vc))
    q = dev(np.random.default_rng(c).standard_normal((B, m, hq, 128)).astype(np.float16))
    lens = torch.tensor([T, 2, T // 2, 65], dtype=torch.int32, device="cuda")[at].contiguous()
    a = (k, v, dev(ck), dev(cv), SCALE, fmt)
    for sl in (None, lens):
        out = cq.cq_chunk_attention(q, *a, T, t_cap, seq_lens=sl)
        for j in range(m):
            back = m - 1 - j
            one = cq.cq_decode_attention(q[:, j].contiguous(), *a, T - back, t_cap, seq_lens=None if sl is None else sl - back)
            assert torch.equal(out[:, j].contiguous().view(torch.int16), one.view(torch.int16))


@pytest.mark.parametrize("seed", range(10))
def test_quads_of_drawn_sizes(seed):
    rng = np.random.default_rng(1000 + seed)
    c, hkv = (8, 4)[seed % 2], int(rng.choice([1, 2, 3, 8]))
    hq = 4 * hkv * int(rng.choice([1, 1, 2, 3]))
    B = int(rng.integers(-(-140 * 4 // hq), -(-140 * 4 // hq) + 40))
    t = int(rng.choice([int(rng.integers(1, 300)), int(rng.integers(300, 2500))]))
    split = int(rng.choice([0, 64 * int(rng.integers(1, 20))]))
    test_quads_equal_single_heads_over_pages_and_in_the_fused_step(c, hq, hkv, B, t, split, "plain")
