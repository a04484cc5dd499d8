"""Sizes where one kernel or one branch of a dispatch can go wrong: edges of tiles,
remainders, the smallest and largest of a range, against the fp64 oracle.  The bars are
those of parity.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_30519_amd import (SCORE_PROB, CompressedCache, PagedKVCache, omnimem_compress_chunk,
                                  omnimem_dense_attn, omnimem_gated_combine, omnimem_select_compressed,
                                  omnimem_sparse_attn, synth)
from parity import check_bf16, check_f32, check_lse, check_selection, say

pytestmark = pytest.mark.gpu
NAN = float("nan")


@pytest.fixture(scope="module")
def dev():
    d = torch.device("cuda:0")
    torch.cuda.set_device(d)
    return d


def make(dev, H, d, S, Lq, B, n, dtype, seed, nonresident=()):
    g = torch.Generator().manual_seed(seed)
    q = torch.randn(Lq, H, d, generator=g).to(dtype)
    k = torch.randn(n, S, H, d, generator=g).to(dtype)
    v = torch.randn(n, S, H, d, generator=g).to(dtype)
    cache = synth.page_layer(k.to(dev), v.to(dev), B, seed=seed, pad_value=NAN, nonresident=nonresident)
    return q, k, v, cache, synth.resident_mask(cache).numpy()


def check(got, ref, dtype, what):
    (out, lse), (o_ref, l_ref, hs, qs) = got, ref
    o, l = out.cpu().float().numpy()[qs, hs], lse.cpu().numpy()[hs, qs]
    (check_f32 if dtype == torch.float32 else check_bf16)(o, o_ref, what)
    check_lse(l, l_ref, what + " lse", 1e-5 if dtype == torch.float32 else 5e-3)


def random_lists(rng, H, R, K, nb):
    """Lists of every length from none to K, with padding, an id past the end and
    duplicates among their entries."""
    idx = rng.integers(0, nb, (H, R, K)).astype(np.int32)
    idx[rng.random((H, R, K)) < 0.1] = -1
    idx[rng.random((H, R, K)) < 0.03] = nb
    cnt = rng.integers(0, K + 1, (H, R)).astype(np.int32)
    cnt[0, 0], cnt[-1, -1] = 0, K
    return idx, cnt


def sparse_ref(q, k, v, B, idx, cnt, G, scale, resident):
    nb = k.shape[0] * -(-k.shape[1] // B)
    idx = np.where(idx >= nb, -1, idx).astype(np.int32)   # the oracle refuses ids past the end; both skip padding
    return oracle.sparse_attn(q, k, v, B, idx, cnt, G, scale, resident=resident)


# fp32: 32-row tiles (one row, one short of a tile, one over), 32-key tiles (a tail of 1,
# 32, 33 and 72 tokens), fewer key tiles than waves and more
@pytest.mark.parametrize("H,d,S,Lq,B,n,K,G", [(2, 64, 65, 31, 64, 3, 2, 31), (2, 128, 161, 33, 64, 4, 5, 33),
                                              (1, 128, 96, 1, 64, 2, 1, 1), (3, 64, 200, 130, 128, 5, 7, 65),
                                              (2, 128, 200, 70, 128, 5, 9, 15), (1, 64, 128, 64, 64, 20, 30, 32)])
def test_fp32_attention(dev, H, d, S, Lq, B, n, K, G):
    say(f"fp32 attention H={H} d={d} S={S} Lq={Lq} B={B} n={n} K={K} G={G}")
    q, k, v, cache, resident = make(dev, H, d, S, Lq, B, n, torch.float32, 3 * Lq + d, nonresident=[1])
    idx, cnt = random_lists(np.random.default_rng(Lq), H, -(-Lq // G), K, n * -(-S // B))
    qd, scale = q.to(dev), d ** -0.5
    got = omnimem_sparse_attn(cache, qd, torch.from_numpy(idx).to(dev), torch.from_numpy(cnt).to(dev), G, scale)
    check(got, sparse_ref(q, k, v, B, idx, cnt, G, scale, resident), torch.float32, "sparse")
    got = omnimem_dense_attn(cache, qd, 0, n, scale)
    check(got, oracle.dense_attn(q, k, v, B, 0, n, scale, resident=resident), torch.float32, "dense")


@pytest.mark.parametrize("d,n", [(64, 513), (128, 257)])
def test_fp32_attention_long(dev, d, n):
    """Block lists longer than one decoded stretch (one entry per thread), and scores whose
    running max jumps between blocks by hundreds."""
    say(f"fp32 attention long d={d} n={n}")
    q, k, v, _, _ = make(dev, 1, d, 64, 33, 64, n, torch.float32, n)
    k[3::50] *= 30.0
    cache = synth.page_layer(k.to(dev), v.to(dev), 64, seed=6)
    got = omnimem_dense_attn(cache, q.to(dev), 0, n, d ** -0.5)
    check_ref = oracle.dense_attn(q, k, v, 64, 0, n, d ** -0.5)
    (out, lse), (o_ref, l_ref, hs, qs) = got, check_ref
    # scores of up to ~150: their fp32 rounding (2^-24 relative) moves a probability by
    # 150 * 6e-8 = 9e-6 of itself, and outputs of up to 5 by as much again
    err = np.abs(out.cpu().numpy()[qs, hs] - o_ref).max()
    say(f"  max-abs {err:.2e}")
    assert err <= 1e-4
    assert np.allclose(lse.cpu().numpy()[hs, qs], l_ref, rtol=2e-6, atol=1e-5)


def test_fp32_more_groups_than_a_grid(dev):
    """Groups of one row are a workgroup each, 512 threads at d = 64, and a grid holds fewer
    than 2^32 threads (of more, a part runs): 70 groups more than one grid."""
    most = (2 ** 32 - 1) // 512
    Lq, n, scale = most + 70, 5, 0.125
    say(f"fp32 attention, {Lq} groups of one row")
    g = torch.Generator(device=dev).manual_seed(3)
    k, v = (torch.randn((n, 1, 64, 64), generator=g, device=dev) for _ in range(2))
    cache = PagedKVCache(k, v, torch.arange(n, dtype=torch.int32, device=dev).view(n, 1), 64)
    q = torch.randn((Lq, 1, 64), generator=g, device=dev)
    idx = torch.randint(0, n, (1, Lq, 1), generator=g, device=dev, dtype=torch.int32)
    out, lse = omnimem_sparse_attn(cache, q, idx, torch.ones((1, Lq), dtype=torch.int32, device=dev), 1, scale)
    torch.cuda.synchronize()
    rows = torch.cat([torch.arange(300), most - 200 + torch.arange(270),
                      torch.randint(0, Lq, (2000,), generator=torch.Generator().manual_seed(4))]).to(dev)
    block = idx[0, rows, 0].long()
    u = scale * (k[block, 0].double() * q[rows].double()).sum(-1)
    want = (torch.softmax(u, -1).unsqueeze(-1) * v[block, 0].double()).sum(1)
    check_f32(out[rows, 0].cpu().numpy(), want.cpu().numpy(), "sparse")
    check_lse(lse[0, rows].cpu().numpy(), torch.logsumexp(u, -1).cpu().numpy(), "lse", 1e-5)


def key_streams(shim, d, H, Lq, G, tiles):
    """How many key streams a bf16 call with groups of more than 32 rows gets on this GPU."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return shim.shim_key_streams(d, H * -(-Lq // G), min(G, Lq), tiles, cus)


# The bf16 kernels of larger groups in each of their key-stream counts: block lists of every
# length, in any order, with tail blocks of 8 tokens, padding, duplicates, non-resident
# blocks, scores that jump between blocks far above the running max, lists of more than one
# decoded stretch (256 entries, at d = 64 512) and of an odd number of tiles.  Blocks of 128
# tokens are two tiles, each with a jump of its own, the second of a tail block 8 tokens.
@pytest.mark.parametrize("B", [64, 128])
@pytest.mark.parametrize("d,H,Lq,G,K,streams", [(128, 2, 300, 130, 25, 2), (128, 2, 33, 33, 601, 2),
                                                (128, 2, 32000, 250, 25, 1), (128, 2, 32000, 250, 601, 1),
                                                (64, 2, 300, 130, 25, 4), (64, 3, 65, 65, 601, 4),
                                                (64, 8, 2100, 2100, 25, 2), (64, 8, 2100, 2100, 601, 2),
                                                (64, 2, 32000, 250, 25, 1), (64, 2, 32000, 250, 601, 1)])
def test_key_streams(dev, host_shim, d, H, Lq, G, K, streams, B):
    say(f"key streams d={d} H={H} Lq={Lq} G={G} K={K} B={B}: {streams}")
    S, n = 200, 5
    nb = n * -(-S // B)
    tiles = min(K, nb) * B // 64
    assert key_streams(host_shim, d, H, Lq, G, tiles) == streams == key_streams(host_shim, d, H, Lq, Lq, nb * B // 64)
    g = torch.Generator().manual_seed(d + K)
    u = torch.randn(H, d, generator=g)
    u = 3.0 * u / u.norm(dim=-1, keepdim=True)
    q = (u + 0.3 * torch.randn(Lq, H, d, generator=g)).to(torch.bfloat16)
    jump = torch.tensor([1.0, 40.0, 1.0, 0.5, 400.0, 2.0, 0.25, 60.0, 1.0, 3.0, 400.0, 1.0, 0.1, 8.0, 1.0, 50.0, 1.0, 0.3,
                         20.0, 1.0])
    tokens = torch.arange(S) // 64
    k = (u + 0.3 * torch.randn(n, S, H, d, generator=g)) * jump.view(n, 4)[:, tokens].view(n, S, 1, 1)
    k = k.to(torch.bfloat16)
    v = torch.randn(n, S, H, d, generator=g).to(torch.bfloat16)
    cache = synth.page_layer(k.to(dev), v.to(dev), B, seed=K, pad_value=NAN, nonresident=[2, 9])
    resident = synth.resident_mask(cache).numpy()
    R = -(-Lq // G)
    idx, cnt = random_lists(np.random.default_rng(K + d), H, R, K, nb)
    if R > 1:
        cnt[:, 1] = 1
        idx[:, 1, 0] = 3   # nothing but a tail block
    qd, scale = q.to(dev), d ** -0.5
    out, lse = omnimem_sparse_attn(cache, qd, torch.from_numpy(idx).to(dev), torch.from_numpy(cnt).to(dev), G, scale)
    dout, dlse = omnimem_dense_attn(cache, qd, 0, n, scale)
    rng = np.random.default_rng(7)
    m = 400
    hs, qs = rng.integers(0, H, m).astype(np.int32), rng.integers(0, Lq, m).astype(np.int32)
    qs[:50] = rng.integers(0, min(2 * G, Lq), 50)
    qs[50:70] = Lq - 1 - rng.integers(0, min(G, 70), 20)
    oi = np.where(idx >= nb, -1, idx).astype(np.int32)
    ref = oracle.sparse_attn(q, k, v, B, oi, cnt, G, scale, resident=resident, hs=hs, qs=qs)
    check((out, lse), ref, torch.bfloat16, "sparse")
    ref = oracle.dense_attn(q, k, v, B, 0, n, scale, resident=resident, hs=hs, qs=qs)
    check((dout, dlse), ref, torch.bfloat16, "dense")


# Block lists by rising and by falling scores, the highest in a full block or in a tail block
# (of 128 tokens: in its second tile, 64 or 8 keys), and one that starts with a tail block:
# with rising scores every tile but a stream's first must settle against a max of earlier
# tiles, and the last one decides the result.
@pytest.mark.parametrize("B", [64, 128])
@pytest.mark.parametrize("d,H,Lq,G,streams", [(128, 2, 32000, 250, 1), (128, 2, 300, 300, 2), (64, 2, 32000, 250, 1),
                                              (64, 8, 2100, 2100, 2), (64, 2, 300, 300, 4)])
def test_ordered_jumps(dev, host_shim, d, H, Lq, G, streams, B):
    S, n = 200, 5
    bpc = -(-S // B)
    nb, R, scale = n * bpc, -(-Lq // G), d ** -0.5
    assert key_streams(host_shim, d, H, Lq, G, nb * B // 64) == streams
    g = torch.Generator().manual_seed(d + B)
    u = torch.randn(H, d, generator=g)
    u = 3.0 * u / u.norm(dim=-1, keepdim=True)
    q = (u + 0.3 * torch.randn(Lq, H, d, generator=g)).to(torch.bfloat16)
    qd = q.to(dev)
    v = torch.randn(n, S, H, d, generator=g).to(torch.bfloat16)
    rng = np.random.default_rng(B)
    hs, qs = rng.integers(0, H, 300).astype(np.int32), rng.integers(0, Lq, 300).astype(np.int32)
    for where, top in (("full", 2 * bpc), ("tail", 3 * bpc - 1)):
        jump = torch.tensor([1.0, 40.0, 1.5, 0.5, 30.0, 2.0, 0.25, 60.0, 1.2, 3.0, 30.0, 0.7, 0.1, 8.0, 1.1, 50.0, 0.9, 0.3,
                             20.0, 5.0]).view(nb, B // 64).sort(dim=-1).values      # a factor for each tile
        jump[top] *= 400.0 / jump[top].max()
        k = (u + 0.3 * torch.randn(n, S, H, d, generator=g)) * jump.view(n, -1)[:, torch.arange(S) // 64].view(n, S, 1, 1)
        k = k.to(torch.bfloat16)
        cache = synth.page_layer(k.to(dev), v.to(dev), B, seed=B, pad_value=NAN)
        up = torch.argsort(jump[:, -1])
        first = torch.tensor([bpc - 1])
        for name, ids in (("rising", up), ("falling", up.flip(0)), ("tail first", torch.cat([first, up[up != bpc - 1]]))):
            say(f"ordered jumps d={d} H={H} Lq={Lq} G={G} B={B}: {streams}, top in a {where} block, {name}")
            idx = ids.to(torch.int32).view(1, 1, nb).expand(H, R, nb).contiguous()
            cnt = torch.full((H, R), nb, dtype=torch.int32)
            got = omnimem_sparse_attn(cache, qd, idx.to(dev), cnt.to(dev), G, scale)
            ref = oracle.sparse_attn(q, k, v, B, idx.numpy(), cnt.numpy(), G, scale, hs=hs, qs=qs)
            check(got, ref, torch.bfloat16, name)


# One key outweighs the rest of every row, in the last of eight tiles, by less than the 2^8
# that a lagging max would let pass: with the max of the tiles so far its P is 1, exact in
# bf16, and a row of O is scaled by nothing but its own rounding.
@pytest.mark.parametrize("H,Lq,streams", [(2, 300, 4), (8, 2100, 2), (2, 32000, 1)])
def test_d64_largest_weight(dev, host_shim, H, Lq, streams):
    say(f"d=64 largest weight H={H} Lq={Lq}: {streams}")
    assert key_streams(host_shim, 64, H, Lq, Lq, 8) == streams
    d, S, B, scale = 64, 512, 64, 0.125
    g = torch.Generator().manual_seed(Lq)
    q = torch.zeros(Lq, H, d)
    q[..., 0] = 28 + 13 * torch.rand(Lq, H, generator=g)       # the last tile's key at 5 to 7.4 log2 units
    k = torch.zeros(1, S, H, d)
    k[..., 0] = -2.0
    k[:, [5, 70, 150, 250], :, 0] = 0.0                        # the first tiles' max
    k[:, S - 20, :, 0] = 1.0
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    v = torch.randn(1, S, H, d, generator=g).to(torch.bfloat16)
    cache = synth.page_layer(k.to(dev), v.to(dev), B, seed=2)
    out, lse = omnimem_dense_attn(cache, q.to(dev), 0, 1, scale)
    rng = np.random.default_rng(Lq)
    hs, qs = rng.integers(0, H, 500).astype(np.int32), rng.integers(0, Lq, 500).astype(np.int32)
    ref = oracle.dense_attn(q, k, v, B, 0, 1, scale, hs=hs, qs=qs)
    check((out, lse), ref, torch.bfloat16, "dense")
    got, want = out.cpu().float().numpy()[qs, hs].astype(np.float64), ref[0]
    factor = (got * want).sum(-1) / (want * want).sum(-1) - 1.0
    rms = float(np.sqrt((factor ** 2).mean()))
    say(f"  rows scaled by {rms:.2e} rms")
    # O's rounding, at most 2^-8 and 1.6e-3 rms an element, leaves sqrt(3 / 64) of that in the
    # projection of 64 normal values (3.5e-4); a rounded largest P adds its own 1.6e-3
    assert rms <= 8e-4


# Probability scores over one, two and three 64-key tiles, exactly full and one key over,
# in both slice modes; what the compressed cache holds past the history is NaN.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d,n,G", [(128, 64, 200), (128, 65, 200), (128, 128, 70), (64, 129, 200), (64, 63, 70),
                                   (64, 64, 15), (128, 129, 15), (128, 1, 200)])
def test_prob_tiles(dev, d, n, G, dtype):
    say(f"prob tiles d={d} keys={n} G={G} {dtype}")
    H, S, B, Lq, K = 2, 64, 64, 200, 5
    q, k, v, cache, _ = make(dev, H, d, S, Lq, B, n, dtype, n + d)
    cc = CompressedCache.allocate(cache, n + 70)
    for t in (cc.k_mean, cc.k_pages, cc.v_pages) + ((cc.k_lo,) if cc.k_lo is not None else ()):
        t.fill_(NAN)
    for c in range(n):
        omnimem_compress_chunk(cache, c, cc)
    sel = omnimem_select_compressed(cache, cc, q.to(dev), K, G, 0, 0, d ** -0.5, score_mode=SCORE_PROB)
    kbar = k.double().mean(dim=1).permute(1, 0, 2).contiguous().numpy()
    ref = oracle.select_prob(q, kbar, n, 1, K, G, 0, 0, d ** -0.5, want_all_scores=True)
    idx, cnt, score = sel.idx.cpu().numpy(), sel.cnt.cpu().numpy(), sel.score.cpu().numpy()
    check_selection(idx, cnt, ref)
    for h in range(H):
        for r in range(idx.shape[1]):
            c = int(cnt[h, r])
            want = ref["all_scores"][h, r, idx[h, r, :c]]
            assert (np.abs(score[h, r, :c] - want) <= 1e-4 * want).all()


# Probability scores at the ends of the range: a scale of 1.5e9 over small scores, and scores
# that are all below -1e36 before a scale of 7e-35; every logit is about +-114, the spread as
# usual.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d,n,G", [(128, 70, 200), (64, 65, 200), (128, 70, 15)])
@pytest.mark.parametrize("exp,sign", [(-17, 1.0), (55, -1.0)])
def test_prob_score_range(dev, exp, sign, d, n, G, dtype):
    say(f"prob score range 2^{exp} d={d} keys={n} G={G} {dtype}")
    H, S, B, Lq, K = 2, 64, 64, 200, 5
    g = torch.Generator().manual_seed(n + d)
    u = torch.randn(H, d, generator=g)
    u = 36.0 * (d / 128) ** 0.25 * u / u.norm(dim=-1, keepdim=True)
    q = ((u + 0.3 * torch.randn(Lq, H, d, generator=g)) * 2.0 ** exp).to(dtype)
    k = ((sign * u + torch.randn(n, S, H, d, generator=g)) * 2.0 ** exp).to(dtype)
    scale = d ** -0.5 * 2.0 ** (-2 * exp)
    if exp > 0:
        assert float((q[:, 0].double() @ k[:, :, 0].double().flatten(0, 1).t().contiguous()).max()) < -1e36
    cache = synth.page_layer(k.to(dev), k.to(dev), B, seed=n)
    cc = CompressedCache.allocate(cache, n)
    for c in range(n):
        omnimem_compress_chunk(cache, c, cc)
    sel = omnimem_select_compressed(cache, cc, q.to(dev), K, G, 0, 0, scale, score_mode=SCORE_PROB)
    kbar = k.double().mean(dim=1).permute(1, 0, 2).contiguous().numpy()
    ref = oracle.select_prob(q, kbar, n, 1, K, G, 0, 0, scale, want_all_scores=True)
    idx, cnt, score = sel.idx.cpu().numpy(), sel.cnt.cpu().numpy(), sel.score.cpu().numpy()
    check_selection(idx, cnt, ref)
    want = np.take_along_axis(ref["all_scores"], idx.astype(np.int64), axis=2)
    # the usual bar, and the pooled keys' two bf16 pieces: 2^-17 of each of the d terms that
    # make up a logit of 114, at random
    bar = 1e-4 + 4 * 114 * 2.0 ** -17 * d ** -0.5
    say(f"  largest relative error {np.abs(score / want - 1).max():.2e}, bar {bar:.2e}")
    assert (np.abs(score - want) <= bar * want).all()


# A softmax over 16,384 pooled keys that are all alike but for the four largest: exponentials
# of 0.33 added one by one to a sum of a thousand lose the same part of themselves each time.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("G", [1, 100])
def test_prob_long_sum(dev, G, dtype):
    say(f"prob long sum G={G} {dtype}")
    n, Lq, scale = 16384, 20 * G, 0.125
    pages = torch.zeros((1, 1, 64, 64), dtype=dtype, device=dev)
    cache = PagedKVCache(pages, pages, torch.zeros((n, 1), dtype=torch.int32, device=dev), 64)
    cc = CompressedCache.allocate(cache, n)
    for t in (cc.k_mean, cc.k_pages, cc.v_pages) + ((cc.k_lo,) if cc.k_lo is not None else ()):
        t.zero_()
    top = [0, 4, 32, 36]          # one among the keys of each lane that holds a row
    cc.k_mean[0, top, 0] = 1.0
    cc.k_pages[0, 0, top, 0] = 1.0
    q = torch.zeros(Lq, 1, 64)
    q[:, 0, 0] = 8.5 + torch.arange(Lq) // G / 8.0     # a group's rows alike
    sel = omnimem_select_compressed(cache, cc, q.to(dtype).to(dev), 4, G, 0, 0, scale, score_mode=SCORE_PROB)
    assert (sel.idx.cpu() == torch.tensor(top, dtype=torch.int32)).all()
    p = 1.0 / (4 + (n - 4) * np.exp(-scale * q[:, 0, 0].double().numpy()))
    err = np.abs(sel.score.cpu().double().numpy()[0, :, 0] / p.reshape(-1, G).mean(-1) - 1.0).max()
    say(f"  largest relative error {err:.2e}")
    # a sum over the 256 tiles: 256 roundings of at most 2^-24, half of that on a growing sum,
    # and a few more of the exponentials, the log2 of the sum (up to 14) and the exponent
    assert err <= 1e-5


# Mean-logit scores from the pooled keys for one to four groups: 16 (d = 128) or 32 rows per
# wave, four waves per workgroup; every block selected, so that every score is compared.
@pytest.mark.parametrize("d,n,G", [(128, 1, 100), (128, 15, 100), (128, 16, 25), (128, 17, 34), (128, 65, 100),
                                   (64, 31, 100), (64, 33, 25), (64, 129, 50)])
def test_pooled_score_rows(dev, d, n, G):
    say(f"pooled score rows d={d} blocks={n} G={G}")
    H, S, B, Lq = 3, 64, 64, 100
    q, k, v, cache, resident = make(dev, H, d, S, Lq, B, n, torch.bfloat16, 5 * n + d, nonresident=[n // 2] if n > 2 else [])
    cc = CompressedCache.allocate(cache, n)
    for c in range(n):
        omnimem_compress_chunk(cache, c, cc)
    sel = omnimem_select_compressed(cache, cc, q.to(dev), n + 1, G, 0, 0, d ** -0.5)
    ref = oracle.select(q, k, B, n + 1, G, 0, 0, d ** -0.5, resident=resident, want_all_scores=True)
    idx, cnt, score = sel.idx.cpu().numpy(), sel.cnt.cpu().numpy(), sel.score.cpu().numpy()
    check_selection(idx, cnt, ref)
    want = np.where(ref["idx"] >= 0, ref["score"], 0.0)
    # fp32 sums of d products: d * 2^-24 of sum |q k| / sqrt(d), a few units here
    assert np.abs(np.where(np.isfinite(score), score, 0.0) - want).max() <= 2e-5


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
def test_gated_combine_rows(dev, dtype, d):
    """A workgroup takes 16, 32 or 64 rows (by d and dtype): one row, one less, as many and
    one more, written over a branch, with the rows behind the last left alone."""
    per = 256 * 2 * (16 // dtype.itemsize) // d
    for rows in (1, per - 1, per, per + 1):
        say(f"gated combine rows={rows} d={d} {dtype}")
        g = torch.Generator(device=dev).manual_seed(rows)
        full = [torch.randn((rows + 1, 1, d), generator=g, device=dev).to(dtype) for _ in range(3)]
        logits = torch.randn((rows, 1, 3), generator=g, device=dev)
        host_in = [x[:rows].cpu().float().numpy().astype(np.float64) for x in full]
        behind = full[1][rows:].clone()
        omnimem_gated_combine(*[x[:rows] for x in full], logits, out=full[1][:rows])
        torch.cuda.synchronize()
        want = oracle.gated_combine(*host_in, logits.cpu().numpy())
        # a few fp32 roundings of the terms, then the result's own
        bound = 8 * 2.0 ** -24 * oracle.gated_combine(*[np.abs(x) for x in host_in], logits.cpu().numpy())
        bound += np.abs(want) * (2.0 ** -24 if dtype == torch.float32 else 2.0 ** -8)
        assert (np.abs(full[1][:rows].cpu().float().numpy() - want) <= bound).all()
        assert torch.equal(full[1][rows:], behind)


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.float32, 64)])
def test_gated_combine_streamed(dev, dtype, d):
    """More than 320 MiB of branches are read past the caches: the same bits as calls over
    parts of the rows, out of place and over a branch."""
    rows = (320 << 20) // (3 * d * dtype.itemsize) + 77
    say(f"gated combine rows={rows} d={d} {dtype}")
    g = torch.Generator(device=dev).manual_seed(8)
    branches = [torch.randn((rows, 1, d), generator=g, device=dev).to(dtype) for _ in range(3)]
    logits = torch.randn((rows, 1, 3), generator=g, device=dev)
    parts = torch.cat([omnimem_gated_combine(*[b[i:i + 200000] for b in branches], logits[i:i + 200000])
                       for i in range(0, rows, 200000)])
    assert torch.equal(omnimem_gated_combine(*branches, logits), parts)
    omnimem_gated_combine(*branches, logits, out=branches[2])
    torch.cuda.synchronize()
    assert torch.equal(branches[2], parts)


@pytest.mark.parametrize("top_k", [3, 70])
def test_small_group_lists_past_count(dev, top_k):
    """The one-wave-per-group walk reads lists ahead of their counts: whatever stands past a
    count (ids in and out of range) changes nothing, over several groups a wave and lists
    longer than a wave's 64 entries."""
    say(f"entries past the count, top_k={top_k}")
    H, G, R, bpc, n = 3, 2, 1400, 5, 16
    _, _, _, cache, _ = make(dev, H, 64, 300, 1, 64, n, torch.bfloat16, 9)
    g = torch.Generator(device=dev).manual_seed(10)
    q = torch.randn((R * G - 1, H, 64), generator=g, device=dev).to(torch.bfloat16)
    idx = torch.rand((H, R, n * bpc), generator=g, device=dev).topk(top_k, dim=-1).indices.to(torch.int32)
    cnt = torch.randint(0, top_k + 1, (H, R), generator=g, device=dev, dtype=torch.int32)
    past = torch.arange(top_k, device=dev) >= cnt.unsqueeze(-1)
    want = omnimem_sparse_attn(cache, q, idx.masked_fill(past, -1), cnt, G, 0.125)
    for junk in (None, 2**31 - 1, -(2**31), n * bpc):
        lists = idx if junk is None else idx.masked_fill(past, junk)
        got = omnimem_sparse_attn(cache, q, lists, cnt, G, 0.125)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
