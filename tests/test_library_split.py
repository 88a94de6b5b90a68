"""The cut of long work items into pieces (csrc/split.h), on the CPU: a C++
program built from the header prints, for a set of tiles, the cut, every
piece and its order slot."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "internal.h"
using namespace mesh_attn;
// argv: pass heads group by_kv w...
int main(int argc, char** argv) {
  const split::Pass pass =
      atoi(argv[1]) == 0 ? kFwdPass : atoi(argv[1]) == 1 ? kDkdvPass : kDqPass;
  const int slots = pass.slots, heads = atoi(argv[2]), group = atoi(argv[3]),
            by_kv = atoi(argv[4]);
  std::vector<int32_t> w;
  int32_t longest = 0;
  for (int i = 5; i < argc; ++i) {
    w.push_back(atoi(argv[i]));
    if (w.back() > longest) longest = w.back();
  }
  const int n = static_cast<int>(w.size());
  const split::Cut c = split::choose(w.data(), n, heads, pass);
  printf("cut %d %d\n", c.c, c.whole);
  printf("bound %d %lld\n", pass.max_parts(), static_cast<long long>(split::parts_bound(
                             int64_t{n} * heads, longest, pass)));
  struct P { int row, idx, len, key; };
  std::vector<P> ps;
  for (int r = 0; r < n; ++r) {
    const int k = split::num_pieces(c, r, w[r]);
    for (int j = 0; j < k; ++j) {
      const int b = split::piece_begin(w[r], k, j),
                e = split::piece_begin(w[r], k, j + 1);
      ps.push_back({r, j, e - b, 0});
      printf("piece %d %d %d %d\n", r, j, b, e);
    }
  }
  const int m = static_cast<int>(ps.size()), total = m * heads;
  for (P& p : ps) p.key = total > slots ? -p.len : p.idx;
  for (int h = 0; h < heads; ++h)
    for (int i = 0; i < m; ++i) {
      int before = 0, same = 0, same_before = 0;
      for (int j = 0; j < m; ++j) {
        before += ps[j].key < ps[i].key;
        same += ps[j].key == ps[i].key;
        same_before += ps[j].key == ps[i].key && j < i;
      }
      printf("slot %d\n", split_slot(total, m, heads, group, by_kv != 0, h,
                                     before, same, same_before, slots));
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("split")
    src, exe = d / "main.cpp", d / "main"
    src.write_text(_MAIN)
    subprocess.run(
        [gxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I",
         os.path.join(ROOT, "paper_2512_20968_amd", "csrc"), "-I",
         "/opt/rocm/include", str(src), "-o", str(exe)], check=True)
    return str(exe)


CASES = [
    # name, pass (0 forward, 1 dK/dV, 2 dQ), heads, group, kv heads, work,
    # split expected
    ("one round, equal items", 0, 4, 4, 1, [1024] * 16, True),
    ("one round, causal", 0, 8, 4, 2, list(range(36, 65, 4)), True),
    ("one item", 0, 1, 1, 1, [64], True),
    ("fewer pieces than lanes", 0, 1, 1, 1, [9], None),
    ("rows without keys", 0, 4, 1, 4, [0, 0, 17, 40], True),
    ("short items stay whole", 0, 4, 1, 4, [8, 8], False),
    ("full rounds stay whole", 0, 32, 1, 32, [512] * 64, False),
    ("past the last round that is split", 0, 32, 1, 32, [512] * 65, False),
    ("nearly empty last round", 0, 32, 4, 8, [64] * 9, True),
    ("nearly empty last round, odd heads", 0, 21, 3, 7, [200] * 25, True),
    ("two workgroups per unit", 2, 12, 3, 4, list(range(4, 40, 3)), None),
    ("dK/dV, one round", 1, 4, 1, 4, [96] * 32, True),
    ("dK/dV, two blocks", 1, 4, 1, 4, [4, 4], False),
    ("longest work", 0, 1, 1, 1, [1 << 24] * 3, True),
]


@pytest.mark.parametrize("name,pass_,heads,group,hkv,work,want", CASES,
                         ids=[c[0] for c in CASES])
def test_pieces_cover_items_and_slots(program, name, pass_, heads, group, hkv,
                                      work, want):
    out = subprocess.run(
        [program, *map(str, (pass_, heads, group, int(hkv % 8 == 0), *work))],
        check=True, capture_output=True, text=True).stdout.split("\n")
    rows = [ln.split() for ln in out if ln]
    cut = tuple(int(x) for x in rows[0][1:])
    if want is not None:
        assert (cut[0] > 0) == want
    pieces, slots_seen = {}, []
    for r in rows[2:]:
        if r[0] == "piece":
            pieces.setdefault(int(r[1]), []).append((int(r[3]), int(r[4])))
        else:
            slots_seen.append(int(r[1]))
    parts = 0
    for row, w in enumerate(work):
        ps = pieces[row]
        # consecutive, from the first block to the last, none empty
        assert ps[0][0] == 0 and ps[-1][1] == w
        assert all(a[1] == b[0] for a, b in zip(ps, ps[1:]))
        if len(ps) > 1:
            parts += len(ps)
            assert all(1 <= e - b <= cut[0] for b, e in ps)
            assert row >= cut[1]
    # never more partial results than the workspace and the slots hold
    assert parts * heads <= int(rows[1][2]) <= int(rows[1][1])
    # every piece of every head has a slot of its own, without gaps
    assert sorted(slots_seen) == list(range(len(slots_seen)))
