"""Tiles whose long work items are split over several workgroups (few items,
or a nearly empty last round), through the C ABI, against the float64 oracle:
every row and head.  A call whose workspace has no room for partial results
must give the whole-item result, and the allocation-free forward the bits of
the call with a full workspace."""

import dataclasses

import pytest
import torch

import oracle
import paper_2512_20968_amd as ma
from mesh_inputs import WORKLOADS, make_grad, make_qkv

from helpers import (check_fwd, check_grad, device_list_tiles, log,
                     oracle_backward_rows, to_np)

pytestmark = pytest.mark.gpu

_T = dataclasses.replace(WORKLOADS["tiny-nc"], num_partitions=16, seed=71)
# One round of equal pieces; causal with unequal rows, GQA and both layouts
# (rows without a visible key among them); KV heads a multiple of the XCD
# count; whole rounds with only the last rows cut; a piece count that leaves
# uneven XCD lanes.
FWD = [
    dataclasses.replace(_T, name="one-round", q_idx=[2],
                        kv_idx=list(range(9)), num_q_heads=3, num_kv_heads=1,
                        head_dim=128),
    dataclasses.replace(_T, name="causal-gqa", partition_len=512,
                        q_idx=[5, 0, 4], kv_idx=[0, 3, 5, 1, 4], causal=True,
                        num_q_heads=6, num_kv_heads=3),
    dataclasses.replace(_T, name="striped-gqa8", partition_len=512,
                        q_idx=[3, 0], kv_idx=[1, 3, 0, 2, 6], causal=True,
                        layout=1, num_q_heads=16, num_kv_heads=8,
                        head_dim=128, outliers=True),
    dataclasses.replace(_T, name="tail-rows", q_idx=list(range(9)),
                        kv_idx=list(range(4, 12)), num_q_heads=32,
                        num_kv_heads=4, head_dim=128),
    dataclasses.replace(_T, name="uneven-lanes", q_idx=[1, 7, 3],
                        kv_idx=[0, 2, 9, 3, 4, 5, 6, 8, 15], num_q_heads=7,
                        num_kv_heads=7, head_dim=128),
    # A list too long for the kernel arguments (copied to the workspace, or
    # built on the device by the allocation-free call).
    dataclasses.replace(_T, name="long-list", num_partitions=64,
                        q_idx=list(range(63, 3, -1)),
                        kv_idx=list(range(0, 60, 5)), causal=True, layout=1,
                        num_q_heads=1, num_kv_heads=1),
]


@pytest.mark.parametrize("cfg", FWD, ids=[c.name for c in FWD])
@pytest.mark.parametrize("out", [torch.bfloat16, torch.float32])
def test_split_forward(gpu, cfg, out):
    q, k, v, _ = make_qkv(cfg)
    qd, kd, vd = (t.to(gpu) for t in (q, k, v))
    prob = cfg.problem()
    need = ma.mesh_attn_fwd_workspace_size(prob, cfg.nq, cfg.nkv)

    def call(nbytes):
        o = torch.full(qd.shape, float("nan"), dtype=out, device=gpu)
        lse = torch.full((cfg.num_q_heads, qd.shape[0]), float("nan"),
                         device=gpu)
        if nbytes is None:
            ma.mesh_attn_tile_fwd_noalloc(prob, cfg.q_idx, cfg.kv_idx, qd, kd,
                                          vd, o, lse)
        else:
            ws = torch.empty(nbytes, dtype=torch.uint8, device=gpu)
            ma.mesh_attn_tile_fwd(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd, o,
                                  lse, ws=ws)
        torch.cuda.synchronize()
        return o, lse

    log(f"{cfg.name}: split, whole, allocation-free")
    o, lse = call(need)
    o1, lse1 = call(need - 256)
    o2, lse2 = call(None)
    assert torch.equal(o, o2) and torch.equal(lse, lse2)
    # The split took place: float32 sums in another order.
    assert not torch.equal(lse, lse1)
    ro, rl = oracle.tile_forward(prob, cfg.q_idx, cfg.kv_idx, to_np(q),
                                 to_np(k), to_np(v))
    check_fwd(f"{cfg.name} split", to_np(o), to_np(lse), ro, rl)
    check_fwd(f"{cfg.name} whole", to_np(o1), to_np(lse1), ro, rl)


@pytest.mark.parametrize("cfg", FWD[:3], ids=[c.name for c in FWD[:3]])
def test_split_forward_of_a_nan_key(gpu, cfg):
    """A key that is not a number: rows that see it get NaN in O and -inf in
    LSE, split or whole, and the others what they get without it."""
    q, k, v, _ = make_qkv(cfg)
    row = 3 * cfg.partition_len + 77
    k[row] = float("nan")
    qd, kd, vd = (t.to(gpu) for t in (q, k, v))
    prob = cfg.problem()
    need = ma.mesh_attn_fwd_workspace_size(prob, cfg.nq, cfg.nkv)
    qpos = oracle.problem_positions(prob, cfg.q_idx)
    kpos = oracle.problem_positions(prob, cfg.kv_idx)
    hit = torch.from_numpy(qpos >= (kpos[row] if cfg.causal else 0)).to(gpu)
    assert hit.any()
    for nbytes in (need, need - 256):
        o = torch.empty_like(qd)
        lse = torch.empty((cfg.num_q_heads, qd.shape[0]), device=gpu)
        ws = torch.empty(nbytes, dtype=torch.uint8, device=gpu)
        ma.mesh_attn_tile_fwd(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd, o, lse,
                              ws=ws)
        torch.cuda.synchronize()
        assert torch.isnan(o[hit]).all() and torch.isfinite(o[~hit]).all()
        assert torch.isneginf(lse[:, hit]).all(), nbytes
        if not hit.all():
            k2 = torch.where(torch.isnan(kd), 0.0, kd)
            o2, lse2 = torch.empty_like(o), torch.empty_like(lse)
            ma.mesh_attn_tile_fwd(prob, cfg.q_idx, cfg.kv_idx, qd, k2, vd, o2,
                                  lse2, ws=ws)
            assert torch.equal(o[~hit], o2[~hit])
            assert torch.equal(lse[:, ~hit], lse2[:, ~hit])


def test_long_list_noalloc_in_a_captured_graph(gpu):
    """The allocation-free forward whose list is built on the device, split and
    whole, captured and replayed three times with an eager call of the other
    tile (which rewrites the scratch arrays) before each replay."""
    split = next(c for c in FWD if c.name == "long-list")
    whole = dataclasses.replace(split, kv_idx=[60, 3], name="whole-list",
                                num_q_heads=5)
    calls = []
    for cfg in (split, whole):
        q, k, v, _ = make_qkv(cfg)
        qd, kd, vd = (t.to(gpu) for t in (q, k, v))
        o = torch.empty_like(qd)
        lse = torch.empty((cfg.num_q_heads, qd.shape[0]), device=gpu)

        def call(cfg=cfg, qd=qd, kd=kd, vd=vd, o=o, lse=lse):
            ma.mesh_attn_tile_fwd_noalloc(cfg.problem(), cfg.q_idx,
                                          cfg.kv_idx, qd, kd, vd, o, lse)
        call()
        torch.cuda.synchronize()
        calls.append((call, o, lse, o.clone(), lse.clone()))
    for i in (0, 1):
        call, o, lse, ref_o, ref_l = calls[i]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call()
        for rep in range(3):
            o.fill_(float("nan"))
            lse.fill_(float("nan"))
            calls[1 - i][0]()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(o, ref_o) and torch.equal(lse, ref_l), (i, rep)


@pytest.mark.parametrize("cfg", device_list_tiles(), ids=lambda c: c.name)
def test_device_built_lists_of_split_tiles(gpu, cfg):
    """The list that the allocation-free forward builds on the device against
    the host's: the same bits in every row, and the oracle's on some."""
    q, k, v, _ = make_qkv(cfg)
    qd, kd, vd = (t.to(gpu) for t in (q, k, v))
    prob = cfg.problem()
    res = []
    for fn in (ma.mesh_attn_tile_fwd, ma.mesh_attn_tile_fwd_noalloc):
        o = torch.full(qd.shape, float("nan"), device=gpu)
        lse = torch.full((cfg.num_q_heads, qd.shape[0]), float("nan"),
                         device=gpu)
        fn(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd, o, lse)
        torch.cuda.synchronize()
        res.append((o, lse))
    assert torch.equal(res[0][0], res[1][0])
    assert torch.equal(res[0][1], res[1][1])
    rows = list(range(0, qd.shape[0], qd.shape[0] // 61)) + [qd.shape[0] - 1]
    ro, rl = oracle.tile_forward(prob, cfg.q_idx, cfg.kv_idx, to_np(q),
                                 to_np(k), to_np(v), rows=rows, heads=[0])
    check_fwd(cfg.name, to_np(res[1][0][rows][:, :1]),
              to_np(res[1][1][:1, rows]), ro, rl)


@pytest.mark.parametrize("first", [64, 128])
def test_long_lists_that_differ_in_head_dim_only(gpu, first):
    """One tile at both head dims, whose cuts differ, through the cache of long
    lists: each gets the bits of its allocation-free forward (which has no
    cache), and the backward the oracle's gradients."""
    base = dataclasses.replace(
        _T, num_partitions=8, partition_len=4096, q_idx=[0, 1, 2, 3, 4],
        kv_idx=[0, 1] if first == 64 else [1, 0], num_q_heads=4,
        num_kv_heads=4, grad_seed=73)
    for d in (first, 192 - first):
        cfg = dataclasses.replace(base, head_dim=d)
        prob = cfg.problem()
        q, k, v, _ = make_qkv(cfg)
        do = make_grad(cfg)
        qd, kd, vd, dod = (t.to(gpu) for t in (q, k, v, do))
        o, o2 = (torch.empty_like(qd) for _ in range(2))
        lse, lse2 = (torch.empty((4, qd.shape[0]), device=gpu)
                     for _ in range(2))
        log(f"d = {d}: forward, allocation-free forward, backward")
        ma.mesh_attn_tile_fwd(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd, o, lse)
        ma.mesh_attn_tile_fwd_noalloc(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd,
                                      o2, lse2)
        torch.cuda.synchronize()
        assert torch.equal(o, o2) and torch.equal(lse, lse2)
        dq, dk, dv = (torch.full(t.shape, float("nan"), device=gpu)
                      for t in (qd, kd, vd))
        ma.mesh_attn_tile_bwd(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd, o, dod,
                              lse, dq, dk, dv)
        torch.cuda.synchronize()
        q_rows, kv_rows = [0, 4095, 9000, 20479], [0, 4095, 4096, 8191]
        rq, rk, rv, _ = oracle_backward_rows(
            prob, cfg.q_idx, cfg.kv_idx, q, k, v, do, [3], q_rows, kv_rows)
        for name, g, rows, r in (("dq", dq, q_rows, rq), ("dk", dk, kv_rows, rk),
                                 ("dv", dv, kv_rows, rv)):
            assert torch.isfinite(g).all()
            check_grad(f"d = {d} {name}", to_np(g[rows][:, [3]]), r)


# Tiles of a few short items (the waves of a workgroup split the keys): the
# longest that are, in one round of workgroups and in two, 64 and 16 KV blocks;
# items of fewer blocks than waves; rows and whole items without a visible key.
SHORT = [
    dataclasses.replace(_T, name="short-64", q_idx=[2],
                        kv_idx=list(range(15, -1, -1)), num_q_heads=32,
                        num_kv_heads=8),
    dataclasses.replace(_T, name="short-16", q_idx=[9, 2], kv_idx=[4, 11, 0, 1],
                        num_q_heads=32, num_kv_heads=4, head_dim=128),
    dataclasses.replace(_T, name="short-odd", q_idx=[9, 2], kv_idx=[4, 11],
                        num_q_heads=5, num_kv_heads=5, head_dim=128),
    dataclasses.replace(_T, name="short-causal", partition_len=512,
                        q_idx=[1, 0], kv_idx=[1], causal=True, num_q_heads=3,
                        num_kv_heads=1, outliers=True),
    dataclasses.replace(_T, name="short-striped", q_idx=[0, 3, 2],
                        kv_idx=[1, 3], causal=True, layout=1, num_q_heads=4,
                        num_kv_heads=2, head_dim=128),
    dataclasses.replace(_T, name="short-unseen", q_idx=[0, 5], kv_idx=[3],
                        causal=True, num_q_heads=2, num_kv_heads=2),
]


@pytest.mark.parametrize("cfg", SHORT, ids=[c.name for c in SHORT])
@pytest.mark.parametrize("out", [torch.bfloat16, torch.float32])
def test_short_forward(gpu, cfg, out):
    q, k, v, _ = make_qkv(cfg)
    qd, kd, vd = (t.to(gpu) for t in (q, k, v))
    prob = cfg.problem()
    res = []
    for noalloc in (False, True):
        o = torch.full(qd.shape, float("nan"), dtype=out, device=gpu)
        lse = torch.full((cfg.num_q_heads, qd.shape[0]), float("nan"),
                         device=gpu)
        fn = (ma.mesh_attn_tile_fwd_noalloc if noalloc
              else ma.mesh_attn_tile_fwd)
        fn(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd, o, lse)
        torch.cuda.synchronize()
        res.append((o, lse))
    assert torch.equal(res[0][0], res[1][0])
    assert torch.equal(res[0][1], res[1][1])
    ro, rl = oracle.tile_forward(prob, cfg.q_idx, cfg.kv_idx, to_np(q),
                                 to_np(k), to_np(v))
    check_fwd(cfg.name, to_np(res[0][0]), to_np(res[0][1]), ro, rl)


@pytest.mark.parametrize("P,d", [(1536, 128), (512, 64), (512, 128)])
def test_split_chunk_accumulation(gpu, P, d):
    """Chunk tasks of a causal tile, split (P = 1536) or short: the running
    (O, LSE) is folded with the partial results."""
    cfg = dataclasses.replace(_T, partition_len=P, num_partitions=6,
                              q_idx=[4, 1], kv_idx=[1, 0, 4], causal=True,
                              num_q_heads=2, num_kv_heads=1, head_dim=d)
    kq, kkv = 2, 2
    q, k, v, _ = make_qkv(cfg)
    prob = cfg.problem()
    P = cfg.partition_len

    def chunk(x, n, parts, i):
        c = P // n
        return (x.view(parts, n, c, *x.shape[1:])[:, i]
                .reshape(parts * c, *x.shape[1:]).contiguous())

    ro, rl = oracle.tile_forward(prob, cfg.q_idx, cfg.kv_idx, to_np(q),
                                 to_np(k), to_np(v))
    ws = torch.empty(ma.mesh_attn_chunk_fwd_workspace_size(prob, cfg.nq,
                                                           cfg.nkv),
                     dtype=torch.uint8, device=gpu)
    for i in range(kq):
        qd = chunk(q, kq, cfg.nq, i).to(gpu)
        o = torch.full(qd.shape, float("nan"), device=gpu)
        lse = torch.full((cfg.num_q_heads, qd.shape[0]), float("nan"),
                         device=gpu)
        for j in range(kkv):
            ma.mesh_attn_chunk_fwd(
                prob, cfg.q_idx, cfg.kv_idx, (i, kq, j, kkv), qd,
                chunk(k, kkv, cfg.nkv, j).to(gpu),
                chunk(v, kkv, cfg.nkv, j).to(gpu), o, lse,
                accumulate=int(j > 0), ws=ws)
        torch.cuda.synchronize()
        rows = [a * P + i * (P // kq) + r for a in range(cfg.nq)
                for r in range(P // kq)]
        check_fwd(f"chunk row {i}", to_np(o), to_np(lse), ro[rows],
                  rl[:, rows])


@pytest.mark.parametrize("P,d", [(1536, 128), (512, 64), (512, 128)])
def test_accumulation_into_special_values(gpu, P, d):
    """Accumulating chunk tasks, split or short: a row that sees no key of the
    chunk keeps its O, also where its stored LSE is -inf; a row whose stored
    LSE is NaN ends with NaN."""
    cfg = dataclasses.replace(_T, partition_len=P, num_partitions=6,
                              q_idx=[4, 0], kv_idx=[1, 3], causal=True,
                              num_q_heads=2, num_kv_heads=1, head_dim=d)
    q, k, v, _ = make_qkv(cfg)
    qd, kd, vd = (t.to(gpu) for t in (q, k, v))
    prob = cfg.problem()
    o = torch.full(qd.shape, 2.0, device=gpu)
    lse = torch.full((2, 2 * P), -float("inf"), device=gpu)
    lse[0, 5] = lse[1, P - 1] = float("nan")  # rows that see keys
    ma.mesh_attn_chunk_fwd(prob, cfg.q_idx, cfg.kv_idx, (0, 1, 0, 1), qd, kd,
                           vd, o, lse, accumulate=1)
    torch.cuda.synchronize()
    assert (o[P:] == 2.0).all() and torch.isneginf(lse[:, P:]).all()
    bad = torch.zeros((2, 2 * P), dtype=torch.bool, device=gpu)
    bad[0, 5] = bad[1, P - 1] = True
    assert torch.equal(torch.isnan(lse), bad)
    assert torch.equal(torch.isnan(o).all(-1), bad.T)
    ro, rl = oracle.tile_forward(prob, cfg.q_idx, cfg.kv_idx, to_np(q),
                                 to_np(k), to_np(v))
    good = ~bad[0].cpu().numpy() & ~bad[1].cpu().numpy()
    good[P:] = False
    check_fwd(f"d = {d}", to_np(o)[good], to_np(lse)[:, good], ro[good],
              rl[:, good])


# Backward: both passes split in one round; GQA whose pieces cross the walks
# over the group's heads; causal with rows and keys that see nothing; only the
# dK/dV side split (many query heads on one KV head); KV heads a multiple of
# the XCD count.
BWD = [
    dataclasses.replace(_T, name="both-sides", q_idx=[0, 2, 4],
                        kv_idx=[1, 3, 0], num_q_heads=2, num_kv_heads=2,
                        head_dim=128),
    dataclasses.replace(_T, name="gqa-walks", partition_len=384,
                        num_partitions=6, q_idx=[4, 1], kv_idx=[2, 0, 4],
                        causal=True, num_q_heads=6, num_kv_heads=2),
    dataclasses.replace(_T, name="one-kv-head", partition_len=512,
                        num_partitions=4, q_idx=[3, 0], kv_idx=[1],
                        causal=True, layout=1, num_q_heads=11,
                        num_kv_heads=1, head_dim=128),
    dataclasses.replace(_T, name="gqa8", q_idx=[3, 1, 5], kv_idx=[2, 3, 0, 1],
                        causal=True, num_q_heads=16, num_kv_heads=8,
                        outliers=True),
]


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("cfg", BWD, ids=[c.name for c in BWD])
def test_split_backward(gpu, cfg, accumulate):
    cfg = dataclasses.replace(cfg, grad_seed=72)
    q, k, v, _ = make_qkv(cfg)
    do = make_grad(cfg)
    prob = cfg.problem()
    ro, rl = oracle.tile_forward(prob, cfg.q_idx, cfg.kv_idx, to_np(q),
                                 to_np(k), to_np(v))
    refs = oracle.tile_backward(prob, cfg.q_idx, cfg.kv_idx, to_np(q),
                                to_np(k), to_np(v), to_np(do))[:3]
    qd, kd, vd, dod = (t.to(gpu) for t in (q, k, v, do))
    o = torch.from_numpy(ro).to(torch.bfloat16).to(gpu)
    lse = torch.from_numpy(rl).float().to(gpu)
    need = ma.mesh_attn_bwd_workspace_size(prob, cfg.nq, cfg.nkv)

    def call(nbytes):
        g = [torch.full(t.shape, 1.5 if accumulate else float("nan"),
                        device=gpu) for t in (qd, kd, vd)]
        ws = torch.empty(nbytes, dtype=torch.uint8, device=gpu)
        ma.mesh_attn_tile_bwd(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd, o, dod,
                              lse, *g, accumulate=accumulate, ws=ws)
        torch.cuda.synchronize()
        return [t - 1.5 if accumulate else t for t in g]

    log(f"{cfg.name}: split, split again, whole")
    split, again, whole = call(need), call(need), call(need - 256)
    assert all(torch.equal(a, b) for a, b in zip(split, again))
    # Split: float32 sums in another order.
    assert not torch.equal(split[1], whole[1])
    for name, s, w, r in zip(("dq", "dk", "dv"), split, whole, refs):
        check_grad(f"{cfg.name} {name} split", to_np(s), r)
        check_grad(f"{cfg.name} {name} whole", to_np(w), r)


_ADD = [BWD[0], BWD[2], BWD[3]]


@pytest.mark.parametrize("cfg", _ADD, ids=[c.name for c in _ADD])
def test_split_backward_accumulates_in_one_addition(gpu, cfg):
    """accumulate = 1 adds the sum of the partial gradients in one addition:
    exactly the stored value plus what accumulate = 0 gives, also where the
    stored value is much larger.  Whole items too, where scaling dK and dQ in
    the same rounding changes nothing (a scale that is a power of two)."""
    cfg = dataclasses.replace(cfg, grad_seed=74)
    q, k, v, _ = make_qkv(cfg)
    prob = cfg.problem()
    qd, kd, vd, dod = (t.to(gpu) for t in (q, k, v, make_grad(cfg)))
    o = torch.empty_like(qd)
    lse = torch.empty((cfg.num_q_heads, qd.shape[0]), device=gpu)
    ma.mesh_attn_tile_fwd(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd, o, lse)
    need = ma.mesh_attn_bwd_workspace_size(prob, cfg.nq, cfg.nkv)
    always = (0, 1, 2) if cfg.head_dim == 64 else (2,)
    for nbytes, exact in ((need, (0, 1, 2) if cfg.name == "both-sides"
                           else always), (need - 256, always)):
        res = []
        for accumulate in (0, 1):
            g = [torch.full(t.shape, 1000.0 * accumulate, device=gpu)
                 for t in (qd, kd, vd)]
            ws = torch.empty(nbytes, dtype=torch.uint8, device=gpu)
            ma.mesh_attn_tile_bwd(prob, cfg.q_idx, cfg.kv_idx, qd, kd, vd, o,
                                  dod, lse, *g, accumulate=accumulate, ws=ws)
            torch.cuda.synchronize()
            res.append(g)
        for i in exact:
            assert torch.equal(res[1][i], 1000.0 + res[0][i]), (nbytes, i)
