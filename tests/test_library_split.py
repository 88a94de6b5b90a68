"""The kernels' work list (csrc/plan.h, csrc/split.h) on the CPU: a C++ program
built from the headers prints the order table, the runs and the slot of every
workgroup of a tile, and they are compared with the canonical run lists of the
C ABI: every (item, block) pair once, with its class and mask offset, in
ascending order within a piece, whatever the cut."""

import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2512_20968_amd as ma

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "plan.h"
using namespace mesh_attn;
// argv: head_dim pass (0 forward, 1 dK/dV, 2 dQ) split n P hq hkv causal
//       layout k_q i k_kv j nq q... nkv kv...
int main(int argc, char** argv) {
  std::vector<int> a;
  for (int i = 2; i < argc; ++i) a.push_back(atoi(argv[i]));
  const int d = atoi(argv[1]);
  ma_problem_t p{a[2], a[3], a[4], a[5], d, a[6], a[7], 0.125f};
  const int pass = a[0], kq = a[8], kkv = a[10];
  std::vector<int32_t> q(a.begin() + 13, a.begin() + 13 + a[12]);
  std::vector<int32_t> kv(a.begin() + 14 + a[12], a.end());
  const plan::Slice sq{p.partition_len / kq, a[9] * (p.partition_len / kq)},
      skv{p.partition_len / kkv, a[11] * (p.partition_len / kkv)};
  const split::Pass* ps =
      &(pass == 0 ? fwd_pass(d) : pass == 1 ? dkdv_pass(d) : dq_pass(d));
  const int g = p.num_q_heads / p.num_kv_heads;
  const int nq = static_cast<int>(q.size()), nkv = static_cast<int>(kv.size());
  plan::Side s =
      pass == 1 ? plan::Side{&p, kv.data(), nkv, kBwdBN, skv, q.data(), nq,
                             kBwdBM, sq, false, p.num_kv_heads, 1, g, ps,
                             false}
                : plan::Side{&p, q.data(), nq, pass ? kBwdBM : kFwdBM, sq,
                             kv.data(), nkv, pass ? kBwdBN : kFwdBN, skv, true,
                             p.num_q_heads, g, 1, ps, pass == 0};
  if (!a[1]) s.pass = nullptr;
  const int rows = s.rows(), most = rows + ps->max_parts();
  std::vector<DevRow> table(most);
  std::vector<DevRun> runs(rows * s.nb * 2 + 1);
  std::vector<DevSplit> splits(ps->max_parts());
  std::vector<int32_t> work(rows);
  const plan::Arrays arr{table.data(), most, runs.data(),
                         static_cast<int64_t>(runs.size()), splits.data(),
                         ps->max_parts(), work.data()};
  plan::Built b;
  if (!plan::build(s, arr, &b)) return 1;
  printf("built %d %d %d %d\n", b.m, b.n_splits, b.parts, b.mode);
  // The slots that a workspace reserves: from the sizes, all blocks visible.
  printf("bound %d %lld\n", ps->max_parts(), static_cast<long long>(
         split::parts_bound(int64_t{rows} * s.heads,
                            s.nb * (s.sb.len / s.bm_b) * s.walks, *ps)));
  for (int i = 0; i < b.n_runs; ++i)
    printf("run %d %d %d %d\n", runs[i].blk0, runs[i].nblk, runs[i].cls,
           runs[i].delta);
  for (int i = 0; i < b.n_splits; ++i)
    printf("split %d %d %d\n", splits[i].row, splits[i].part,
           splits[i].nparts);
  for (int slot = 0; slot < b.m * s.heads; ++slot) {
    const SlotPlace at = place_slot(b.mode, slot, b.m, s.heads, s.group);
    const DevRow& c = table[at.probe];
    int e, h;
    place_in_class(b.mode, at, c.before, c.same, s.heads, s.group, &e, &h);
    const DevRow& r = table[e];
    printf("slot %d %d %d %d %d %d %d %d %d\n", h, r.row, r.run, r.off, r.nblk,
           r.part, r.walk, r.run_b, r.run_e);
  }
  // Arrays that are one entry too small are refused, not overrun.
  plan::Arrays small = arr;
  small.cap_rows = b.m - 1;
  plan::Built ignored;
  if (plan::build(s, small, &ignored)) return 2;
  small = arr;
  small.cap_runs = b.n_runs - 1;
  if (b.n_runs > 0 && plan::build(s, small, &ignored)) return 3;
  small = arr;
  small.cap_splits = b.n_splits - 1;
  if (b.n_splits > 0 && plan::build(s, small, &ignored)) return 4;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "main.cpp", d / "main"
    src.write_text(_MAIN)
    subprocess.run(
        [gxx, "-std=c++17", "-Wall", "-fsanitize=undefined,address",
         "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I",
         os.path.join(ROOT, "paper_2512_20968_amd", "csrc"), "-I",
         "/opt/rocm/include", str(src), "-o", str(exe)], check=True)
    return str(exe)


def _tile(n, P, q, kv, hq, hkv, causal=0, layout=0, kq=(1, 0), kkv=(1, 0)):
    return dict(n=n, P=P, q=q, kv=kv, hq=hq, hkv=hkv, causal=causal,
                layout=layout, kq=kq, kkv=kkv)


R = list(range(32))
TILES = [
    # name, tile, forward at head dim 128 split (None: either)
    ("one round, equal", _tile(64, 1024, [0], R[16:32], 4, 1), True),
    ("one round, causal", _tile(8, 1024, [2, 3], R[:4], 8, 2, 1), True),
    ("one head", _tile(9, 1024, [3], [0, 1, 2, 7], 1, 1), True),
    ("short items", _tile(4, 256, [0, 1], [0, 1], 4, 4, 1), False),
    ("unseen keys and rows",
     _tile(16, 256, [0, 9, 3], [4, 0, 11, 2, 1], 4, 4, 1), None),
    ("striped, rotated list",
     _tile(13, 1280, [1, 3, 5, 7, 9], [0, 2, 4, 6, 8, 10], 21, 7, 1, 1), None),
    ("striped, 8 KV heads, any order",
     _tile(7, 512, [3, 0, 6], [6, 1, 3, 0], 16, 8, 1, 1), None),
    ("full rounds", _tile(16, 4096, [4, 5, 6, 7], R[:8], 32, 32, 1), False),
    ("nearly empty last round",
     _tile(40, 256, R[:9], R[9:25], 32, 8), True),
    ("adjacent FULL partitions in reverse",
     _tile(20, 512, [19], R[8:0:-1], 2, 2, 1), None),
    ("chunk, contiguous",
     _tile(8, 1536, [4, 1], [1, 0, 4], 2, 1, 1, 0, (2, 1), (3, 1)), None),
    ("chunk, striped",
     _tile(6, 2048, [5, 0, 2], [1, 3, 0, 2], 8, 8, 1, 1, (4, 3), (2, 0)),
     None),
    ("many heads on one", _tile(4, 512, [3, 0], [1], 11, 1, 1, 1), None),
    ("dQ cut for the places beside dK/dV",
     _tile(8, 2048, [0, 1, 2], [0, 1], 8, 8), None),
]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("pass_", [0, 1, 2])
@pytest.mark.parametrize("may_split", [0, 1])
@pytest.mark.parametrize("name,t,want", TILES, ids=[t[0] for t in TILES])
def test_work_list_covers_the_canonical_one(program, name, t, want, may_split,
                                            pass_, d):
    out = subprocess.run(
        [program, *map(str, (d, pass_, may_split, t["n"], t["P"], t["hq"],
                             t["hkv"], t["causal"], t["layout"], *t["kq"],
                             *t["kkv"], len(t["q"]), *t["q"], len(t["kv"]),
                             *t["kv"]))],
        check=True, capture_output=True, text=True).stdout.split("\n")
    lines = [ln.split() for ln in out if ln]
    m, n_splits, parts, mode = (int(x) for x in lines[0][1:])
    max_parts, bound = (int(x) for x in lines[1][1:])
    runs = [tuple(map(int, ln[1:])) for ln in lines if ln[0] == "run"]
    splits = [tuple(map(int, ln[1:])) for ln in lines if ln[0] == "split"]
    slots = [tuple(map(int, ln[1:])) for ln in lines if ln[0] == "slot"]
    kv_major = pass_ == 1
    heads = t["hkv"] if kv_major else t["hq"]
    walks = t["hq"] // t["hkv"] if kv_major else 1
    if not may_split:
        assert n_splits == 0
    elif want is not None and pass_ == 0 and d == 128:
        assert (n_splits > 0) == want
    assert parts * heads <= bound <= max_parts

    # Element offsets of every visible block pair, from the oracle's positions.
    bm, bn = ma.mesh_attn_block_shape(d, int(pass_ > 0))
    cq, ckv = t["P"] // t["kq"][0], t["P"] // t["kkv"][0]

    def positions(idx, chunk, c):
        rows = np.arange(chunk * c, (chunk + 1) * c)
        return [rows * t["n"] + p if t["layout"] else rows + p * t["P"]
                for p in idx]

    qpos = np.concatenate(positions(t["q"], t["kq"][1], cq))
    kpos = np.concatenate(positions(t["kv"], t["kkv"][1], ckv))
    want_blocks = {}
    for qb in range(len(qpos) // bm):
        qp = qpos[qb * bm:(qb + 1) * bm]
        for kb in range(len(kpos) // bn):
            kp = kpos[kb * bn:(kb + 1) * bn]
            if t["causal"] and kp[0] > qp[-1]:
                continue
            full = not t["causal"] or kp[-1] <= qp[0]
            row, col = (kb, qb) if kv_major else (qb, kb)
            want_blocks.setdefault(row, []).append((col, 2 if full else 1))
    # Every item is covered once by its pieces, in order.
    got = {}
    for h, row, run, off, nblk, part, walk, run_b, run_e in slots:
        seq = []
        while nblk > 0:
            blk0, n, cls, delta = runs[run]
            seq.append((walk, blk0 + off, cls, delta, off))
            nblk -= 1
            off += 1
            if off == n:
                off, run = 0, run + 1
                if run == run_e and kv_major:
                    run, walk = run_b, walk + 1
        got.setdefault((h, row), []).append((part, seq))
    n_rows = (len(kpos) // bn) if kv_major else (len(qpos) // bm)
    assert sorted(got) == [(h, r) for h in range(heads)
                           for r in range(n_rows)]
    seen_parts = []
    split_rows = {row: (part, n) for row, part, n in splits}
    for (h, row), pieces in got.items():
        pieces.sort()
        if row in split_rows:
            part, n = split_rows[row]
            assert [p for p, _ in pieces] == list(range(part, part + n))
            seen_parts += [h * parts + p for p, _ in pieces]
        else:
            assert len(pieces) == 1 and pieces[0][0] == -1
        blocks = [b for _, seq in pieces for b in seq]
        # A split dK/dV item may start a piece at the end of a walk.
        assert [(w, b, c) for w, b, c, _, _ in blocks] == \
            [(w, b, c) for w in range(walks)
             for b, c in want_blocks.get(row, [])]
        for _, blk, cls, delta, off in blocks:
            if cls != 1:
                continue
            qb, kb = (blk, row) if kv_major else (row, blk)
            qp = qpos[qb * bm:(qb + 1) * bm]
            kp = kpos[kb * bn:(kb + 1) * bn]
            # hidden iff key j - query i > delta, counted from the run start
            lim = delta + off * bm if kv_major else delta - off * bn
            i, j = np.meshgrid(np.arange(bm), np.arange(bn), indexing="ij")
            np.testing.assert_array_equal(j - i > lim,
                                          kp[None, :] > qp[:, None])
    assert sorted(seen_parts) == list(range(parts * heads))

