"""The library caches the long work lists of the tiles it has seen (at most
1024, those that do not fit the kernel arguments) in pinned host memory, which
kernels of a call read on the caller's stream.  These calls run more distinct
tiles than the cache holds, back to back with no synchronization, so evicted
lists' pinned buffers are recycled while kernels that read them may still be
queued; every result must still match the float64 oracle, and a tile seen again
after its eviction gives the same bits as the first time.  (That the lists are
long ones, and when a buffer may be recycled: test_library_plan_cache.py.)"""

import pytest
import torch

import oracle
import paper_2512_20968_amd as ma
from mesh_inputs import make_grad, make_qkv

from helpers import (check_fwd, check_grad, log, oracle_backward_rows,
                     plan_cache_tiles, run_fwd, to_np)

pytestmark = pytest.mark.gpu


def test_more_tiles_than_the_plan_cache_holds(gpu):
    cfg, kv_lists = plan_cache_tiles()
    prob = cfg.problem()
    q, k, v, _ = make_qkv(cfg)
    qd, kd, vd = (t.to(gpu) for t in (q, k, v))
    outs = [run_fwd(prob, cfg.q_idx, kv, qd, kd, vd) for kv in kv_lists]
    again = run_fwd(prob, cfg.q_idx, kv_lists[0], qd, kd, vd)
    torch.cuda.synchronize()
    log(f"{len(kv_lists)} distinct tiles run back to back")
    assert torch.equal(again[0], outs[0][0])
    assert torch.equal(again[1], outs[0][1])
    rows = list(range(0, 25600, 97)) + [25599]
    for i in list(range(0, len(kv_lists), 37)) + list(range(1090, 1100)):
        ro, rl = oracle.tile_forward(prob, cfg.q_idx, kv_lists[i], to_np(q),
                                     to_np(k), to_np(v), rows=rows, heads=[0])
        o, lse = outs[i]
        check_fwd(f"tile {i} {kv_lists[i]}", to_np(o[rows]),
                  to_np(lse[:, rows]), ro, rl)


def test_more_tiles_than_the_plan_cache_holds_backward(gpu):
    cfg, kv_lists = plan_cache_tiles()
    prob = cfg.problem()
    q, k, v, _ = make_qkv(cfg)
    do = make_grad(cfg)
    qd, kd, vd, dod = (t.to(gpu) for t in (q, k, v, do))
    ws = torch.empty(ma.mesh_attn_bwd_workspace_size(prob, 100, 2),
                     dtype=torch.uint8, device=gpu)

    def run(kv):
        o, lse = run_fwd(prob, cfg.q_idx, kv, qd, kd, vd)
        g = [torch.empty(t.shape, device=gpu) for t in (qd, kd, vd)]
        ma.mesh_attn_tile_bwd(prob, cfg.q_idx, kv, qd, kd, vd, o, dod, lse, *g,
                              ws=ws)
        return g

    outs = [run(kv) for kv in kv_lists]
    again = run(kv_lists[0])
    torch.cuda.synchronize()
    log(f"{len(kv_lists)} distinct tiles run back to back")
    assert all(torch.equal(a, b) for a, b in zip(again, outs[0]))
    q_rows, kv_rows = list(range(0, 25600, 997)), list(range(0, 512, 37))
    for i in (0, 300, 600, 1023, 1024, 1099):
        refs = oracle_backward_rows(prob, cfg.q_idx, kv_lists[i], q, k, v, do,
                                    [0], q_rows, kv_rows)[:3]
        for name, g, rows, r in zip(("dq", "dk", "dv"), outs[i],
                                    (q_rows, kv_rows, kv_rows), refs):
            assert torch.isfinite(g).all()
            check_grad(f"tile {i} {kv_lists[i]} {name}", to_np(g[rows]), r)
