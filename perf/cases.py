"""The work this library is measured on: calls of its public entry points, over the
sizes that chunk-by-chunk video generation meets.

A case names one operation and its sizes.  `listed` holds the fixed ones, `draw` makes
more of the same ranges, `prepare` builds what a generation loop has in hand before the
call (paged caches, block lists, compressed history, workspace and output buffers),
`run` makes the call and `exact` computes the same outputs in fp64 with plain torch.

Sizes follow the repository's workloads: Wan2.1-1.3B-shaped layers (12 heads of 128) and
14B-shaped ones (40 heads), chunks of three latent frames of 1,560 tokens, 64- and
128-token blocks, one query group per chunk or per frame, or groups of 15 rows.  Inputs
are seeded random tensors: unit normal Q, K and V, a per-block key offset, and per
(head, group) a direction that its queries and its relevant blocks share, so that block
scores spread as they do when something is to be found.  Physical pages are shuffled.
"""
import math

import torch

from paper_2605_30519_amd import (SCORE_LOGIT, SCORE_PROB, CompressedCache, PagedKVCache, omnimem_cmp_attn,
                                  omnimem_compress_chunk, omnimem_dense_attn, omnimem_gated_combine, omnimem_select,
                                  omnimem_select_compressed, omnimem_select_workspace_bytes, omnimem_sparse_attn,
                                  select_params)
from paper_2605_30519_amd.omnimem import Selection, workspace_tensor

DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}
DEV = "cuda"

# op: step = select + sparse attention, select / select_pooled / select_prob = block
# selection (over all of K, over the compressed history, by probabilities), sparse =
# attention over given block lists, window = dense attention over the last `w` chunks,
# cmp = attention over the compressed history, compress = pooling of the newest chunk,
# combine = Eq. 1's gated fusion, layer = Eq. 1 whole.
# S = tokens per chunk (history and queries alike), n = cached chunks, B = block,
# K = top-K, G = rows per query group, E / T = excluded window and its threshold.


def _case(name, op, dtype="bf16", H=12, d=128, S=4680, n=20, B=64, K=64, G=0, E=1, T=3, w=1):
    c = {"op": op, "dtype": dtype, "H": H, "d": d, "S": S, "n": n, "B": B, "K": K, "G": G or S, "E": E, "T": T, "w": w}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest whole step: a two-head fp32 layer over short chunks, all launch latency
        _case("tiny_fp32_step", "step", "fp32", H=2, d=64, S=256, n=8, K=4),
        # the two halves of the usual step of one 1.3B-shaped layer at 20 cached chunks
        _case("select_1.3b_n20", "select"),
        _case("sparse_1.3b_n20", "sparse"),
        # the largest selection: a 14B-shaped layer at 60 chunks, one group per latent frame
        _case("select_14b_n60", "select", H=40, n=60, B=128, K=32, G=1560),
        # attention of one GPU's heads of that layer when eight GPUs share them
        _case("sparse_14b_5heads", "sparse", H=5, n=60, B=128, K=32, G=1560),
        # the small-group setting: 312 groups of 15 rows, four blocks each, three window chunks
        _case("select_g15_n20", "select", K=4, G=15, E=3),
        _case("sparse_g15_n20", "sparse", K=4, G=15, E=3),
        # selection from the compressed history: the mean-logit score in a long rollout, and
        # the probability score
        _case("select_pooled_n60", "select_pooled", n=60),
        _case("select_prob_n20", "select_prob"),
        # Eq. 1 whole, as a generation step runs it: pool the newest chunk, select from the
        # compressed history, the three branches, the gated fusion
        _case("layer_1.3b_n20", "layer"),
        # fp32 attention, one latent frame per chunk: reference and debugging runs
        _case("sparse_fp32_frame", "sparse", "fp32", S=1560, n=10, K=16),
        # the sliding-window branch with 64-wide heads
        _case("window_d64", "window", H=16, d=64, S=1560, n=6, w=3),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        op = rng.choice(["step", "select", "select", "sparse", "sparse", "sparse", "select_pooled", "select_prob", "layer",
                         "window", "window", "cmp", "compress", "combine"])
        S = rng.choice([1560, 4680, log(256, 4680), log(256, 4680)])
        B = rng.choice([64, 64, 128])
        n = log(3, 60)
        bpc = -(-S // B)
        small = rng.random() < 0.3
        G = rng.choice([15, 15, log(8, 64)]) if small else rng.choice([S, S, -(-S // 3), log(100, S) if S > 100 else S])
        E = rng.choice([0, 1, 1, 3])
        c = _case(None, op, rng.choice(["bf16", "bf16", "bf16", "bf16", "fp32"]), H=rng.choice([1, 2, 3, 5, 8, 12, 12, 16, 24, 40]),
                  d=rng.choice([128, 128, 64]), S=S, n=n, B=B, K=rng.choice([4, 4, log(2, 16)]) if small else rng.choice([16, 32, 64, log(4, 96)]),
                  G=G, E=E, T=3, w=rng.choice([1, 1, 2, 3]))
        if c["K"] > (n - E) * bpc or n - E < 3:
            continue
        nb = n * bpc
        f = work(c)
        groups = c["H"] * -(-S // G)
        pool = 2 * nb * c["H"] * B * c["d"] * (2 if c["dtype"] == "bf16" else 4)
        if pool > 6e9 or groups * nb > 6e7 or f["bytes"] > 2.9e9 or f["flops"] > (2.6e11 if c["dtype"] == "bf16" else 9e9):
            continue
        return c


# ------------------------------------------------------------------------- inputs


class _Inputs:
    pass


def _sizes(case):
    S, B = case["S"], case["B"]
    bpc = -(-S // B)
    R = -(-S // case["G"])
    ncand = (case["n"] - case["E"]) * bpc   # blocks outside the window (exclusion is active in every case)
    return bpc, R, case["n"] * bpc, ncand


def _inputs(case, seed, values):
    """q [S, H, d], logical blocks k (and v) [nb, H, B, d] with zeros past a chunk's end, and
    block lists [H, R, K]: per (head, group) a random set of blocks outside the window,
    ascending, on whose keys the group's direction is planted."""
    bpc, R, nb, ncand = _sizes(case)
    H, d, S, B, K, n = (case[k] for k in ("H", "d", "S", "B", "K", "n"))
    dt = DTYPES[case["dtype"]]
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    x = _Inputs()
    a = torch.randn((H, R, d), generator=g, device=DEV)
    a /= a.norm(dim=-1, keepdim=True)
    x.lists = torch.rand((H, R, ncand), generator=g, device=DEV).topk(K, dim=-1).indices.sort(dim=-1).values
    hit = torch.zeros((H, R, nb), device=DEV).scatter_(2, x.lists, 1.0)
    shift = 0.5 * torch.randn((H, nb, d), generator=g, device=DEV)
    shift += 0.5 * math.sqrt(d) * torch.matmul(hit.transpose(1, 2).contiguous(), a)
    del hit
    q = torch.randn((S, H, d), generator=g, device=DEV)
    q += a.permute(1, 0, 2)[torch.arange(S, device=DEV) // case["G"]]
    x.q = q.to(dt)
    x.k = torch.empty((nb, H, B, d), dtype=dt, device=DEV)
    x.v = torch.empty_like(x.k)
    pad = bpc * B - S
    for c in range(n):
        blocks = slice(c * bpc, (c + 1) * bpc)
        t = torch.randn((bpc, H, B, d), generator=g, device=DEV)
        t += shift[:, blocks].permute(1, 0, 2).unsqueeze(2)
        x.k[blocks] = t
        if values:
            x.v[blocks] = torch.randn((bpc, H, B, d), generator=g, device=DEV)
    if pad:
        x.k[bpc - 1::bpc, :, B - pad:] = 0
        if values:
            x.v[bpc - 1::bpc, :, B - pad:] = 0
    if case["op"] in ("combine", "layer"):
        x.gates = torch.randn((S, H, 3), generator=g, device=DEV)
    if case["op"] == "combine":
        x.branches = [torch.randn((S, H, d), generator=g, device=DEV).to(dt) for _ in range(3)]
    x.table = torch.randperm(nb, generator=g, device=DEV).to(torch.int32)
    return x


_VALUES = ("step", "sparse", "window", "layer", "cmp", "compress")


def prepare(case, seed):
    op, H, S, K, n = case["op"], case["H"], case["S"], case["K"], case["n"]
    bpc, R, nb, _ = _sizes(case)
    x = _inputs(case, seed, op in _VALUES)
    s = _Inputs()
    s.case, s.q, s.scale = case, x.q, 1.0 / math.sqrt(case["d"])
    if op == "combine":
        s.branches, s.gates, s.out = x.branches, x.gates, torch.empty_like(x.q)
        return s
    where = x.table.long()
    kp, vp = torch.empty_like(x.k), torch.empty_like(x.v)
    kp[where] = x.k
    if op in _VALUES:
        vp[where] = x.v
    s.cache = PagedKVCache(kp, vp, x.table.view(n, bpc), S)
    if op in ("select_pooled", "select_prob", "layer", "cmp", "compress"):
        s.cc = CompressedCache.allocate(s.cache, n)
        for c in range(n - 1 if op in ("layer", "compress") else n):  # these two pool the newest chunk themselves
            omnimem_compress_chunk(s.cache, c, s.cc)
    if op in ("step", "select", "select_pooled", "select_prob", "layer"):
        mode = SCORE_PROB if op == "select_prob" else SCORE_LOGIT
        p = select_params(K, case["G"], case["E"], case["T"], s.scale, mode)
        s.ws = workspace_tensor(omnimem_select_workspace_bytes(s.cache, S, p), DEV)
        # small groups: the ids alone, as the attention takes them
        score = torch.empty((H, R, K), device=DEV) if _scored(case) else None
        s.sel = Selection(torch.empty((H, R, K), dtype=torch.int32, device=DEV),
                          torch.empty((H, R), dtype=torch.int32, device=DEV), score, 0)
    if op == "sparse":
        s.idx = x.lists.to(torch.int32)
        s.cnt = torch.full((H, R), K, dtype=torch.int32, device=DEV)
    if op in ("step", "sparse", "window", "cmp", "layer"):
        s.out = torch.empty_like(x.q)
        s.lse = torch.empty((H, S), device=DEV)
    if op == "layer":
        s.gates = x.gates
        s.o_cmp, s.o_swa = torch.empty_like(x.q), torch.empty_like(x.q)
        s.lse_cmp, s.lse_swa = torch.empty_like(s.lse), torch.empty_like(s.lse)
    return s


def _scored(case):
    return case["op"] in ("select", "select_pooled", "select_prob") and case["G"] > 64


def run(s):
    c = s.case
    op, K, G, E, T, n = (c[k] for k in ("op", "K", "G", "E", "T", "n"))
    if op == "combine":
        return omnimem_gated_combine(*s.branches, s.gates, out=s.out)
    if op == "compress":
        omnimem_compress_chunk(s.cache, n - 1, s.cc)
        return _pooled(s.cc)
    if op == "layer":
        omnimem_compress_chunk(s.cache, n - 1, s.cc)
    if op in ("step", "select"):
        omnimem_select(s.cache, s.q, K, G, E, T, s.scale, workspace=s.ws, out=s.sel)
    elif op in ("select_pooled", "select_prob", "layer"):
        omnimem_select_compressed(s.cache, s.cc, s.q, K, G, E, T, s.scale, workspace=s.ws, out=s.sel,
                                  score_mode=SCORE_PROB if op == "select_prob" else SCORE_LOGIT)
    if op == "step":
        omnimem_sparse_attn(s.cache, s.q, s.sel.idx, s.sel.cnt, G, s.scale, out=s.out, lse=s.lse)
        return {"idx": s.sel.idx, "cnt": s.sel.cnt, "out": s.out, "lse": s.lse}
    if op in ("select", "select_pooled", "select_prob"):
        return {"idx": s.sel.idx, "cnt": s.sel.cnt, "score": s.sel.score}
    if op == "sparse":
        omnimem_sparse_attn(s.cache, s.q, s.idx, s.cnt, G, s.scale, out=s.out, lse=s.lse)
    elif op == "window":
        omnimem_dense_attn(s.cache, s.q, n - c["w"], n, s.scale, out=s.out, lse=s.lse)
    elif op == "cmp":
        omnimem_cmp_attn(s.cc, n, s.q, s.scale, out=s.out, lse=s.lse)
    elif op == "layer":
        omnimem_cmp_attn(s.cc, n, s.q, s.scale, out=s.o_cmp, lse=s.lse_cmp)
        omnimem_sparse_attn(s.cache, s.q, s.sel.idx, s.sel.cnt, G, s.scale, out=s.out, lse=s.lse)
        omnimem_dense_attn(s.cache, s.q, n - c["w"], n, s.scale, out=s.o_swa, lse=s.lse_swa)
        fused = omnimem_gated_combine(s.o_cmp, s.out, s.o_swa, s.gates)
        return {"fused": fused, "slc": s.out, "idx": s.sel.idx, "cnt": s.sel.cnt, **_pooled(s.cc)}
    return {"out": s.out, "lse": s.lse}


def _pooled(cc):
    return {"k_mean": cc.k_mean, "k_pooled": cc.k_pages, "v_pooled": cc.v_pages}


# ------------------------------------------------------------------ size and accuracy


def work(case):
    op, H, d, S, n, B, K = (case[k] for k in ("op", "H", "d", "S", "n", "B", "K"))
    bpc, R, nb, ncand = _sizes(case)
    eb = 2 if case["dtype"] == "bf16" else 4
    rows = S * H * d * eb                     # one [S, H, d] tensor
    block = S / bpc * H * d * eb              # an average block of every head, K or V
    lists = H * R * (K + 1) * 4 + (H * R * K * 4 if _scored(case) else 0)
    union = ncand * (1.0 - (1.0 - K / ncand) ** R)
    pooled = nb * H * d

    def attn(keys, blocks):                   # keys per row; blocks of K and V read
        return {"bytes": 2 * rows + 2 * blocks * block + H * S * 4, "flops": 4.0 * d * H * S * keys}

    parts = []
    if op in ("step", "select"):
        parts.append({"bytes": rows + ncand * block + lists, "flops": H * d * (S * ncand / bpc + S + 2.0 * R * ncand)})
    if op in ("select_pooled", "layer"):
        parts.append({"bytes": rows + ncand * H * d * 4 + lists, "flops": H * d * (S + 2.0 * R * ncand)})
    if op == "select_prob":
        parts.append({"bytes": rows + 4 * pooled + lists, "flops": 2.0 * d * H * S * nb})
    if op in ("step", "sparse", "layer"):
        a = attn(K * S / bpc, union)
        a["bytes"] += H * R * (K + 1) * 4
        parts.append(a)
    if op in ("window", "layer"):
        parts.append(attn(case["w"] * S, case["w"] * bpc))
    if op in ("cmp", "layer"):
        parts.append({"bytes": 2 * rows + 2 * pooled * eb + H * S * 4, "flops": 4.0 * d * H * S * nb})
    if op in ("compress", "layer"):
        parts.append({"bytes": 2 * rows + bpc * H * d * (4 + 2 * eb + (2 if eb == 2 else 0)), "flops": 2.0 * S * H * d})
    if op in ("combine", "layer"):
        parts.append({"bytes": 4 * rows + S * H * 12, "flops": 6.0 * S * H * d})
    return {k: float(sum(p[k] for p in parts)) for k in ("bytes", "flops")}


def tolerance(case):
    # whole numbers: a block whose score ties with the last selected one to within fp32
    # rounding may be exchanged for it
    op = case["op"]
    if op == "select_prob":
        # 5e-7 off fp64 at one group per chunk, and more for small groups, whose mean averages
        # less (the pooled keys are carried as two bf16 pieces)
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    if op in ("select", "select_pooled"):
        # 5e-8 off fp64; sums over thousands of rows in another order move them by about as much
        return {"rel": 1e-6, "max": 2e-5, "differ": 1e-3}
    if case["dtype"] == "fp32":
        # 5e-7 to 1e-6 off fp64
        return {"rel": 4e-6, "max": 1e-4, "differ": 1e-3}
    # 2.1e-3 to 2.8e-3 off fp64: the rounding of the bf16 results is 1.7e-3, that of P before
    # PV about as much
    return {"rel": 1e-2, "max": 0.1, "differ": 1e-3}


# ------------------------------------------------------------------------- fp64


def _attend(q, k, v, scale):
    """softmax(scale q k^T) v and its log-sum-exp, fp64."""
    u = torch.matmul(q, k.transpose(-1, -2).contiguous()) * scale
    lse = torch.logsumexp(u, dim=-1)
    return torch.matmul(torch.exp(u - lse.unsqueeze(-1)), v), lse


def _tokens(x, case, h, blocks):
    """fp64 keys, values [.., T, d] of head h's blocks [.., m], and the mask of real tokens."""
    bpc, B, S = -(-case["S"] // case["B"]), case["B"], case["S"]
    o = blocks % bpc
    real = o.unsqueeze(-1) * B + torch.arange(B, device=DEV) < S
    shape = (*blocks.shape[:-1], -1)
    k = x.k[:, h][blocks].double().reshape(*shape, case["d"])
    v = x.v[:, h][blocks].double().reshape(*shape, case["d"])
    return k, v, real.reshape(shape)


def _exact_lists(x, case, lists, scale):
    H, S, G, d = case["H"], case["S"], case["G"], case["d"]
    _, R, _, _ = _sizes(case)
    out = torch.zeros((S, H, d), dtype=torch.float64, device=DEV)
    lse = torch.zeros((H, S), dtype=torch.float64, device=DEV)
    keys = case["K"] * case["B"]
    step = max(1, min(R, int(6e7 / max(keys * d, keys * G))))
    for h in range(H):
        for r0 in range(0, R, step):
            rows = torch.arange(r0 * G, min((r0 + step) * G, S), device=DEV)
            k, v, real = _tokens(x, case, h, lists[h, r0:r0 + step])
            q = torch.zeros((k.shape[0] * G, d), dtype=torch.float64, device=DEV)
            q[:len(rows)] = x.q[rows, h].double()
            u = torch.matmul(q.view(-1, G, d), k.transpose(1, 2).contiguous()) * scale
            u.masked_fill_(~real.unsqueeze(1), -math.inf)
            m = torch.logsumexp(u, dim=-1)
            o = torch.matmul(torch.exp(u - m.unsqueeze(-1)), v)
            out[rows, h] = o.reshape(-1, d)[:len(rows)]
            lse[h, rows] = m.reshape(-1)[:len(rows)]
    return out, lse


def _exact_dense(q, k, v, scale):
    """q [S, H, d]; k, v [H, T, d]: every row over every token."""
    S, H, d = q.shape
    out = torch.zeros((S, H, d), dtype=torch.float64, device=DEV)
    lse = torch.zeros((H, S), dtype=torch.float64, device=DEV)
    for h in range(H):
        for r in range(0, S, 2048):
            out[r:r + 2048, h], lse[h, r:r + 2048] = _attend(q[r:r + 2048, h].double(), k[h].double(), v[h].double(), scale)
    return out, lse


def _block_means(x, case, what):
    bpc, _, nb, _ = _sizes(case)
    count = torch.full((nb,), case["B"], dtype=torch.float64, device=DEV)
    count[bpc - 1::bpc] = case["S"] - (bpc - 1) * case["B"]
    t = torch.empty((case["H"], nb, case["d"]), dtype=torch.float64, device=DEV)
    for c in range(case["n"]):
        b = slice(c * bpc, (c + 1) * bpc)
        t[:, b] = (what[b].double().sum(dim=2) / count[b].view(-1, 1, 1)).permute(1, 0, 2)
    return t


def _exact_select(x, case, kbar, scale):
    H, S, G, K = (case[k] for k in ("H", "S", "G", "K"))
    _, R, nb, ncand = _sizes(case)
    group = torch.arange(S, device=DEV) // G
    size = torch.bincount(group, minlength=R).double()
    score = torch.empty((H, R, nb), dtype=torch.float64, device=DEV)
    for h in range(H):
        q, kt = x.q[:, h].double(), kbar[h].t().contiguous()
        if case["op"] == "select_prob":
            s = torch.zeros((R, nb), dtype=torch.float64, device=DEV)
            for r in range(0, S, 2048):
                s.index_add_(0, group[r:r + 2048], torch.softmax(torch.matmul(q[r:r + 2048], kt) * scale, dim=-1))
            score[h] = s / size.unsqueeze(-1)
        else:
            qbar = torch.zeros((R, case["d"]), dtype=torch.float64, device=DEV).index_add_(0, group, q) / size.unsqueeze(-1)
            score[h] = torch.matmul(qbar, kt) * scale
    top = score[:, :, :ncand].topk(K, dim=-1).indices.sort(dim=-1).values
    return top, torch.gather(score, 2, top)


def exact(case, seed):
    op, n = case["op"], case["n"]
    bpc, R, nb, _ = _sizes(case)
    x = _inputs(case, seed, op in _VALUES)
    scale = 1.0 / math.sqrt(case["d"])
    dt = DTYPES[case["dtype"]]
    gate = torch.sigmoid(x.gates.double()) if op in ("combine", "layer") else None
    if op == "combine":
        return sum(gate[:, :, i:i + 1] * x.branches[i].double() for i in range(3))
    if op == "sparse":
        return dict(zip(("out", "lse"), _exact_lists(x, case, x.lists, scale)))
    if op in ("window", "layer"):
        first = (n - case["w"]) * bpc
        k = x.k[first:].permute(1, 0, 2, 3).reshape(case["H"], case["w"], bpc * case["B"], -1)[:, :, :case["S"]]
        v = x.v[first:].permute(1, 0, 2, 3).reshape(case["H"], case["w"], bpc * case["B"], -1)[:, :, :case["S"]]
        swa = _exact_dense(x.q, k.flatten(1, 2), v.flatten(1, 2), scale)
        if op == "window":
            return dict(zip(("out", "lse"), swa))
    kbar = _block_means(x, case, x.k)
    pooled = {}
    if op in ("cmp", "compress", "layer"):
        vbar = _block_means(x, case, x.v)
        # the compressed cache holds them rounded to the cache's type, 64 tokens a page
        kc, vc = kbar.to(dt), vbar.to(dt)
        cmp = _exact_dense(x.q, kc, vc, scale) if op != "compress" else None
        if op == "cmp":
            return dict(zip(("out", "lse"), cmp))
        pages = -(-nb // 64)

        def paged(t):
            p = torch.zeros((case["H"], pages * 64, case["d"]), dtype=torch.float64, device=DEV)
            p[:, :nb] = t
            return p.view(case["H"], pages, 64, -1).transpose(0, 1).contiguous()

        pooled = {"k_mean": kbar, "k_pooled": paged(kbar), "v_pooled": paged(vbar)}
        if op == "compress":
            return pooled
    if op in ("select", "select_pooled", "select_prob") and not _scored(case):
        return None  # whole numbers only
    top, score = _exact_select(x, case, kbar, scale)
    if op in ("select", "select_pooled", "select_prob"):
        return {"idx": None, "cnt": None, "score": score}
    out, lse = _exact_lists(x, case, top, scale)
    if op == "step":
        return {"idx": None, "cnt": None, "out": out, "lse": lse}
    fused = gate[:, :, 0:1] * cmp[0] + gate[:, :, 1:2] * out + gate[:, :, 2:3] * swa[0]
    return {"fused": fused, "slc": out, "idx": None, "cnt": None, **pooled}
