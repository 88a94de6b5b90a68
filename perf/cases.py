"""The work a user of this package has one GPU do, as measurable cases.

Each case is one pass through the public entry points of
``paper_2512_20968_amd`` with everything a caller already holds (inputs,
output buffers, workspaces) prepared before it:

  fwd         mesh_attn_tile_fwd of a whole tile
  noalloc     mesh_attn_tile_fwd_noalloc of a whole tile
  chunks      a whole tile as k_Q x k_KV chunk tasks (mesh_attn_chunk_fwd,
              float32 running partials)
  merge       mesh_attn_lse_merge of k partial results
  bwd         mesh_attn_tile_bwd of a whole tile
  bwd_chunks  a whole tile's gradients as k_Q x k_KV chunk tasks
              (mesh_attn_chunk_bwd accumulating into zeroed gradients)

A tile is nq Q partitions (first q0, step qs) times nkv KV partitions (first
kv0, step kvs; a step above 1 is the list KV Partition Rotation makes) of a
sequence of n partitions of P tokens.  ``outliers`` scales one token row per Q
and K partition by 8, the activations that stress the softmax range.
"""

import math

import torch

import paper_2512_20968_amd as ma


def _tile(name, kind, n, P, q, kv, hq, hkv, d, causal, layout=0, out="bf16",
          outliers=False, kq=1, kkv=1):
    c = dict(kind=kind, n=n, P=P, q0=q[0], nq=q[1], qs=q[2], kv0=kv[0],
             nkv=kv[1], kvs=kv[2], hq=hq, hkv=hkv, d=d, causal=causal,
             layout=layout, out=out, outliers=outliers, kq=kq, kkv=kkv)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: a test-sized tile, 1024 tokens in four
        # partitions, where launches and latency are all there is.
        _tile("fwd tiny", "fwd", 4, 256, (0, 2, 1), (0, 2, 1), 4, 4, 64,
              False),
        # The allocation-free forward as a serving loop calls it: an 8K
        # sequence on a 2 x 4 mesh with grouped heads.
        _tile("noalloc 8k gqa", "noalloc", 8, 1024, (2, 2, 1), (0, 4, 1), 8,
              2, 128, True),
        # One Q partition against a long KV footprint with few heads (heads
        # already split over other ranks): few, long work items.
        _tile("fwd few heads", "fwd", 64, 4096, (0, 1, 1), (16, 16, 1), 4, 1,
              128, False),
        # An ordinary training tile: 64K tokens over 16 GPUs, causal.
        _tile("fwd causal 64k", "fwd", 16, 4096, (4, 4, 1), (0, 8, 1), 32,
              32, 128, True),
        # The largest: one GPU's share of 1M tokens over 256 GPUs.
        _tile("fwd 1m gqa", "fwd", 256, 4096, (16, 16, 1), (32, 16, 1), 32,
              8, 128, False),
        # Striped causal layout, rotated KV list, odd counts of partitions
        # and heads, head dim 64, float32 partials for a later merge.
        _tile("fwd striped d64 ragged", "fwd", 13, 1280, (1, 5, 2), (0, 6, 2),
              21, 7, 64, True, layout=1, out="fp32"),
        # The causal 64K tile as 2 x 2 overlap chunk tasks.
        _tile("chunks causal 64k", "chunks", 16, 4096, (4, 4, 1), (0, 8, 1),
              32, 32, 128, True, out="fp32", kq=2, kkv=2),
        # The reduce-scatter fold of a 16 x 16 mesh, bf16 partials.
        dict(name="merge 16 bf16", kind="merge", parts=16, rows=4096,
             heads=32, d=128, inp="bf16", out="bf16", hidden=0.0),
        # A short fold of float32 partials of an odd number of rows, some
        # parts without a visible key.
        dict(name="merge 3 fp32 ragged", kind="merge", parts=3, rows=1535,
             heads=21, d=64, inp="fp32", out="fp32", hidden=0.1),
        # The training tile's backward.
        _tile("bwd causal 64k", "bwd", 16, 4096, (4, 4, 1), (0, 8, 1), 32,
              32, 128, True),
        # A small model's backward: 4K tokens, grouped heads, head dim 64.
        _tile("bwd 4k gqa d64", "bwd", 8, 512, (3, 3, 1), (0, 5, 1), 12, 4,
              64, True),
        # Backward as 2 x 2 overlap chunk tasks, striped, grouped heads.
        _tile("bwd chunks striped", "bwd_chunks", 8, 2048, (0, 3, 2),
              (1, 4, 2), 16, 4, 128, True, layout=1, kq=2, kkv=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_tile(rng, kind):
    P = 256 * _log(rng, 1, 16)
    nq, nkv = _log(rng, 1, 16), _log(rng, 1, 16)
    qs, kvs = rng.choice((1, 1, 2, 3)), rng.choice((1, 1, 2, 3))
    q0 = rng.randrange(0, 12)
    # Causal tiles of a mesh lie at or below the diagonal.
    causal = rng.random() < 0.6
    kv0 = rng.randrange(0, q0 + 1) if causal else rng.randrange(0, 12)
    n = max(q0 + nq * qs, kv0 + nkv * kvs) + rng.randrange(0, 9)
    group = rng.choice((1, 1, 2, 3, 4, 8))
    hkv = _log(rng, 1, 32)
    while hkv > 1 and hkv * group > 64:
        hkv -= 1
    kq = kkv = 1
    if kind in ("chunks", "bwd_chunks"):
        kq = rng.choice([x for x in (1, 2, 3, 4) if P % (256 * x) == 0])
        kkv = rng.choice([x for x in (2, 3, 4, 5, 6, 8)
                          if P % (128 * x) == 0 and P // x >= 128])
    out = "fp32" if kind == "chunks" else rng.choice(("bf16", "bf16", "fp32"))
    return _tile(None, kind, n, P, (q0, nq, qs), (kv0, nkv, kvs),
                 hkv * group, hkv, rng.choice((64, 128, 128)), causal,
                 layout=rng.randrange(2), out=out,
                 outliers=rng.random() < 0.25, kq=kq, kkv=kkv)


def draw(rng):
    kind = rng.choice(("fwd", "fwd", "fwd", "noalloc", "chunks", "merge",
                       "merge", "bwd", "bwd", "bwd_chunks"))
    if kind == "merge":
        while True:
            c = dict(kind="merge", parts=_log(rng, 2, 33),
                     rows=_log(rng, 100, 40000), heads=_log(rng, 1, 64),
                     d=rng.choice((64, 128)), inp=rng.choice(("bf16", "fp32")),
                     out=rng.choice(("bf16", "fp32")),
                     hidden=rng.choice((0.0, 0.0, 0.2)))
            if 2 ** 20 <= work(c)["bytes"] <= 2 ** 32:
                return c
    while True:
        c = _draw_tile(rng, kind)
        w = work(c)
        # At most the largest listed case's cost, at least the tiny tile's.
        if 2.5e8 <= w["flops"] <= 3e13 and w["bytes"] <= 2 ** 33:
            return c


# ---------------------------------------------------------------------------

def _lists(c):
    return ([c["q0"] + i * c["qs"] for i in range(c["nq"])],
            [c["kv0"] + i * c["kvs"] for i in range(c["nkv"])])


def _positions(c, idx, device="cpu"):
    """Global position of every row of a stacked buffer."""
    r = torch.arange(c["P"], device=device)
    if c["layout"] == 1:
        return torch.cat([r * c["n"] + p for p in idx])
    return torch.cat([r + p * c["P"] for p in idx])


def _pairs(c):
    """Visible (query, key) pairs of the tile, per query head."""
    q_idx, kv_idx = _lists(c)
    P = c["P"]
    if not c["causal"]:
        return len(q_idx) * len(kv_idx) * P * P
    full, diag, below = P * P, P * (P + 1) // 2, P * (P - 1) // 2
    total = 0
    for a in q_idx:
        for b in kv_idx:
            if c["layout"] == 1:
                total += diag if b <= a else below
            else:
                total += full if b < a else diag if a == b else 0
    return total


def work(c):
    if c["kind"] == "merge":
        row = c["rows"] * c["heads"]
        i, o = (2 if c[k] == "bf16" else 4 for k in ("inp", "out"))
        return {"bytes": row * (c["parts"] * (c["d"] * i + 4) + c["d"] * o + 4),
                "flops": row * c["parts"] * 2 * c["d"]}
    rq = c["nq"] * c["P"] * c["hq"] * c["d"]
    rk = c["nkv"] * c["P"] * c["hkv"] * c["d"]
    lse = c["nq"] * c["P"] * c["hq"] * 4
    if c["kind"] in ("bwd", "bwd_chunks"):
        # Q, O, dO, K, V and LSE in; float32 dQ, dK, dV out.
        return {"bytes": 3 * 2 * rq + 2 * 2 * rk + lse + 4 * rq + 8 * rk,
                "flops": 10 * c["d"] * c["hq"] * _pairs(c)}
    o = 4 if c["out"] == "fp32" else 2
    return {"bytes": 2 * rq + 4 * rk + o * rq + lse,
            "flops": 4 * c["d"] * c["hq"] * _pairs(c)}


def tolerance(c):
    # bf16 probabilities (and dS) carry 2^-9 of relative rounding each and a
    # bf16 result as much again: measured 1.2e-3 to 2.4e-3 against 64 bits.
    if c["kind"] == "merge":
        return {"rel": 1e-5 if c["out"] == "fp32" else 8e-3}
    return {"rel": 1e-2}


# ---------------------------------------------------------------------------

def _randn(shape, gen):
    return torch.randn(shape, generator=gen, device="cuda")


def _inputs(c, seed):
    """bf16 Q, K, V of the tile, N(0, 1), with the outlier rows."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rq, rk = c["nq"] * c["P"], c["nkv"] * c["P"]
    q = _randn((rq, c["hq"], c["d"]), g)
    k = _randn((rk, c["hkv"], c["d"]), g)
    v = _randn((rk, c["hkv"], c["d"]), g)
    if c["outliers"]:
        for x, parts in ((q, c["nq"]), (k, c["nkv"])):
            at = torch.randint(0, c["P"], (parts,), generator=g,
                               device="cuda")
            at += torch.arange(parts, device="cuda") * c["P"]
            x[at] *= 8.0
    return [x.to(torch.bfloat16) for x in (q, k, v)] + [g]


def _scale(c):
    return float(torch.tensor(c["d"], dtype=torch.float64).rsqrt().float())


def _scores(c, q, k, h, rows, qpos, kpos, dtype):
    """Masked scaled scores of head h and the query rows of a slice."""
    x = q[rows, h].to(dtype) @ k[:, h // (c["hq"] // c["hkv"])].to(dtype).T
    x *= _scale(c)
    if c["causal"]:
        x.masked_fill_(kpos[None, :] > qpos[rows, None], -math.inf)
    return x


def _row_slices(c, rows):
    step = max(256, 2 ** 28 // max(1, c["nkv"] * c["P"]))
    return [slice(a, min(rows, a + step)) for a in range(0, rows, step)]


def _attention(c, q, k, v, dtype):
    """O [rows][hq][d] and LSE [hq][rows] in dtype, by plain torch."""
    q_idx, kv_idx = _lists(c)
    qpos, kpos = (_positions(c, i, q.device) for i in (q_idx, kv_idx))
    rows = q.shape[0]
    o = torch.zeros(q.shape, dtype=dtype, device=q.device)
    lse = torch.empty((c["hq"], rows), dtype=dtype, device=q.device)
    for h in range(c["hq"]):
        vh = v[:, h // (c["hq"] // c["hkv"])].to(dtype)
        for s in _row_slices(c, rows):
            x = _scores(c, q, k, h, s, qpos, kpos, dtype)
            lse[h, s] = torch.logsumexp(x, dim=1)
            x -= lse[h, s].nan_to_num(neginf=0.0)[:, None]
            o[s, h] = x.exp_() @ vh
    return o, lse


def _chunk_of(x, parts, k, i):
    """Chunk i of k of every partition of a stacked buffer."""
    P = x.shape[0] // parts
    return (x.view(parts, k, P // k, *x.shape[1:])[:, i]
            .reshape(parts * (P // k), *x.shape[1:]).contiguous())


def prepare(c, seed):
    if c["kind"] == "merge":
        g = torch.Generator(device="cuda").manual_seed(seed)
        dt = {"bf16": torch.bfloat16, "fp32": torch.float32}
        shape = (c["parts"], c["rows"], c["heads"], c["d"])
        o = torch.empty(shape, dtype=dt[c["inp"]], device="cuda")
        for i in range(c["parts"]):
            o[i] = _randn(shape[1:], g)
        lse = _randn((c["parts"], c["heads"], c["rows"]), g) * 4.0 + 10.0
        if c["hidden"] > 0:
            lse[torch.rand(lse.shape, generator=g, device="cuda")
                < c["hidden"]] = -math.inf
        return dict(c=c, o=o, lse=lse,
                    o_out=torch.empty(shape[1:], dtype=dt[c["out"]],
                                      device="cuda"),
                    lse_out=torch.empty((c["heads"], c["rows"]),
                                        device="cuda"))
    q, k, v, g = _inputs(c, seed)
    q_idx, kv_idx = _lists(c)
    prob = dict(num_partitions=c["n"], partition_len=c["P"],
                num_q_heads=c["hq"], num_kv_heads=c["hkv"], head_dim=c["d"],
                causal=int(c["causal"]), layout=c["layout"],
                softmax_scale=_scale(c))
    st = dict(c=c, prob=prob, q_idx=q_idx, kv_idx=kv_idx, q=q, k=k, v=v)
    rows = q.shape[0]
    f32 = dict(dtype=torch.float32, device="cuda")

    def ws(size):
        return torch.empty(max(16, size(prob, c["nq"], c["nkv"])),
                           dtype=torch.uint8, device="cuda")

    if c["kind"] in ("fwd", "noalloc"):
        st["o"] = torch.empty_like(
            q, dtype=torch.float32 if c["out"] == "fp32" else torch.bfloat16)
        st["lse"] = torch.empty((c["hq"], rows), **f32)
        if c["kind"] == "fwd":
            st["ws"] = ws(ma.mesh_attn_fwd_workspace_size)
    elif c["kind"] == "chunks":
        rc = rows // c["kq"]
        st.update(
            q=[_chunk_of(q, c["nq"], c["kq"], i) for i in range(c["kq"])],
            k=[_chunk_of(k, c["nkv"], c["kkv"], j) for j in range(c["kkv"])],
            v=[_chunk_of(v, c["nkv"], c["kkv"], j) for j in range(c["kkv"])],
            o=[torch.empty((rc, c["hq"], c["d"]), **f32)
               for _ in range(c["kq"])],
            lse=[torch.empty((c["hq"], rc), **f32) for _ in range(c["kq"])],
            ws=ws(ma.mesh_attn_chunk_fwd_workspace_size))
    else:
        # The final O and LSE of the tile's rows, by plain torch in 32 bits.
        o, lse = _attention(c, q, k, v, torch.float32)
        o = o.to(torch.bfloat16)
        do = _randn(q.shape, g).to(torch.bfloat16)
        st.update(o=o, lse=lse, do=do, dq=torch.empty(q.shape, **f32),
                  dk=torch.empty(k.shape, **f32),
                  dv=torch.empty(v.shape, **f32))
        if c["kind"] == "bwd":
            st["ws"] = ws(ma.mesh_attn_bwd_workspace_size)
        else:
            kq, kkv = c["kq"], c["kkv"]
            for x in ("q", "o", "do", "dq"):
                st[x] = [_chunk_of(st[x], c["nq"], kq, i) for i in range(kq)]
            for x in ("k", "v", "dk", "dv"):
                st[x] = [_chunk_of(st[x], c["nkv"], kkv, j)
                         for j in range(kkv)]
            lt = lse.T.contiguous()
            st["lse"] = [_chunk_of(lt, c["nq"], kq, i).T.contiguous()
                         for i in range(kq)]
            st["ws"] = ws(ma.mesh_attn_chunk_bwd_workspace_size)
    return st


def run(s):
    c = s["c"]
    if c["kind"] == "merge":
        ma.mesh_attn_lse_merge(s["o"], s["lse"], s["o_out"], s["lse_out"])
        return {"o": s["o_out"], "lse": s["lse_out"]}
    tile = (s["prob"], s["q_idx"], s["kv_idx"])
    if c["kind"] == "fwd":
        ma.mesh_attn_tile_fwd(*tile, s["q"], s["k"], s["v"], s["o"], s["lse"],
                              ws=s["ws"])
        return {"o": s["o"], "lse": s["lse"]}
    if c["kind"] == "noalloc":
        ma.mesh_attn_tile_fwd_noalloc(*tile, s["q"], s["k"], s["v"], s["o"],
                                      s["lse"])
        return {"o": s["o"], "lse": s["lse"]}
    if c["kind"] == "chunks":
        for i in range(c["kq"]):
            for j in range(c["kkv"]):
                ma.mesh_attn_chunk_fwd(
                    *tile, (i, c["kq"], j, c["kkv"]), s["q"][i], s["k"][j],
                    s["v"][j], s["o"][i], s["lse"][i], accumulate=int(j > 0),
                    ws=s["ws"])
        return {"o": s["o"], "lse": s["lse"]}
    if c["kind"] == "bwd":
        ma.mesh_attn_tile_bwd(*tile, s["q"], s["k"], s["v"], s["o"], s["do"],
                              s["lse"], s["dq"], s["dk"], s["dv"],
                              ws=s["ws"])
    else:
        for x in ("dq", "dk", "dv"):
            for t in s[x]:
                t.zero_()
        for i in range(c["kq"]):
            for j in range(c["kkv"]):
                ma.mesh_attn_chunk_bwd(
                    *tile, (i, c["kq"], j, c["kkv"]), s["q"][i], s["k"][j],
                    s["v"][j], s["o"][i], s["do"][i], s["lse"][i],
                    s["dq"][i], s["dk"][j], s["dv"][j], accumulate=1,
                    ws=s["ws"])
    return {"dq": s["dq"], "dk": s["dk"], "dv": s["dv"]}


# ---------------------------------------------------------------------------

def _exact_bwd(c, q, k, v, o, lse, do):
    dt = torch.float64
    q_idx, kv_idx = _lists(c)
    qpos, kpos = (_positions(c, i, q.device) for i in (q_idx, kv_idx))
    dq = torch.zeros(q.shape, dtype=dt, device=q.device)
    dk = torch.zeros(k.shape, dtype=dt, device=q.device)
    dv = torch.zeros_like(dk)
    for h in range(c["hq"]):
        hk = h // (c["hq"] // c["hkv"])
        kh, vh = k[:, hk].to(dt), v[:, hk].to(dt)
        for s in _row_slices(c, q.shape[0]):
            p = _scores(c, q, k, h, s, qpos, kpos, dt)
            ls = lse[h, s].to(dt)
            p -= ls.masked_fill(ls == -math.inf, math.inf)[:, None]
            p.exp_()
            doh, qh = do[s, h].to(dt), q[s, h].to(dt)
            dv[:, hk] += p.T @ doh
            ds = doh @ vh.T
            ds -= (doh * o[s, h].to(dt)).sum(1)[:, None]
            ds *= p
            ds *= _scale(c)
            dq[s, h] = ds @ kh
            dk[:, hk] += ds.T @ qh
    return dq, dk, dv


def exact(c, seed):
    if c["kind"] == "merge":
        s = prepare(c, seed)
        lse = torch.logsumexp(s["lse"].double(), dim=0)
        o = torch.zeros(s["o"].shape[1:], dtype=torch.float64, device="cuda")
        ref = lse.masked_fill(lse == -math.inf, 0.0)
        for i in range(c["parts"]):
            w = (s["lse"][i].double() - ref).exp()
            o += w.T[:, :, None] * s["o"][i].double()
        return {"o": o, "lse": lse}
    # Masked pairs are computed too: 64-bit products at some 30 TFLOP/s.
    dense = (c["nq"] * c["P"]) * (c["nkv"] * c["P"]) * c["hq"] * c["d"]
    if dense * (10 if "bwd" in c["kind"] else 4) > 1.5e14:
        return None
    if "bwd" in c["kind"]:
        q, k, v, g = _inputs(c, seed)
        o, lse = _attention(c, q, k, v, torch.float32)
        do = _randn(q.shape, g).to(torch.bfloat16)
        dq, dk, dv = _exact_bwd(c, q, k, v, o.to(torch.bfloat16), lse, do)
        if c["kind"] == "bwd_chunks":
            dq = [_chunk_of(dq, c["nq"], c["kq"], i) for i in range(c["kq"])]
            dk, dv = ([_chunk_of(x, c["nkv"], c["kkv"], j)
                       for j in range(c["kkv"])] for x in (dk, dv))
        return {"dq": dq, "dk": dk, "dv": dv}
    q, k, v, _ = _inputs(c, seed)
    o, lse = _attention(c, q, k, v, torch.float64)
    if c["kind"] == "chunks":
        lt = lse.T.contiguous()
        o = [_chunk_of(o, c["nq"], c["kq"], i) for i in range(c["kq"])]
        lse = [_chunk_of(lt, c["nq"], c["kq"], i).T.contiguous()
               for i in range(c["kq"])]
    return {"o": o, "lse": lse}
