"""The planner's launch lists, read from the planner itself (plan.cpp uses no HIP) through a small
driver compiled here: which variant of a kernel a launch takes."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_08881_amd", "csrc")

DRIVER = r"""
#include "plan.hpp"
#include <cstdio>
#include <vector>
using namespace acp;
// input: rank, cap, number of tensors, then per tensor its ndims and dims
int main() {
  int rank, nt;
  long long cap;
  if (scanf("%d %lld %d", &rank, &cap, &nt) != 3) return 1;
  std::vector<int32_t> nd(nt);
  std::vector<int64_t> dims;
  for (int i = 0; i < nt; ++i) {
    if (scanf("%d", &nd[i]) != 1) return 1;
    for (int k = 0; k < nd[i]; ++k) {
      long long d;
      if (scanf("%lld", &d) != 1) return 1;
      dims.push_back(d);
    }
  }
  Plan p;
  const std::string err = build_plan(p, nt, nd.data(), dims.data(), rank, cap, true);
  if (!err.empty()) return fprintf(stderr, "%s\n", err.c_str()), 2;
  // every P-step launch over whole rows: class, ragged form or not, tiles of more than 512 columns, of
  // those the ragged ones
  auto show = [&](const char* what, size_t i, const std::vector<Launch>& L) {
    for (const Launch& l : L) {
      if (l.kernel != K_PFUSED) continue;
      int wide = 0, ragged = 0;
      for (int32_t t = 0; t < l.ntiles; ++t) {
        const Tile& x = p.tiles[l.tile_off + t];
        if (x.kind == T_VEC || p.mats[x.idx].scls == 0) continue;
        ++wide;
        ragged += p.mats[x.idx].m % 4 != 0;
      }
      printf("pstep %s %d %d %d %d %d\n", what, int(i), l.variant & ~kRaggedRows, (l.variant & kRaggedRows) != 0, wide,
             ragged);
    }
  };
  for (size_t b = 0; b < p.buckets.size(); ++b) show("bucket", b, p.buckets[b].compress[1]);
  for (size_t g = 0; g < p.group_compress.size(); ++g) show("group", g, p.group_compress[g][1]);
  return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    """plan(shapes, rank, cap) -> the driver's lines, split into words."""
    d = tmp_path_factory.mktemp("plan")
    (d / "driver.cpp").write_text(DRIVER)
    exe = str(d / "driver")
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{CSRC}", f"-I{ROOT}/include", "-o", exe, str(d / "driver.cpp"),
                    os.path.join(CSRC, "plan.cpp"), os.path.join(CSRC, "rng.cpp")], check=True)

    def run(shapes, rank, cap=25 << 20):
        text = f"{rank} {cap} {len(shapes)} " + " ".join(f"{len(s)} " + " ".join(map(str, s)) for s in shapes)
        out = subprocess.run([exe], input=text, text=True, capture_output=True, check=True).stdout
        return [ln.split() for ln in out.splitlines()]

    return run


# row lengths of every P-step class: narrow, one, three and eight waves, 2 to 5 groups, several blocks
ALIGNED = [(40, 60), (40, 512), (40, 700), (40, 900), (40, 2000), (40, 3000), (40, 3500), (40, 4500), (40, 6000)]


@pytest.mark.parametrize("rank", [1, 2, 4])
def test_aligned_rows_take_the_kernels_without_the_ragged_form(plan, rank):
    """The P-step of 2 to 5 groups per lane that holds the ragged form needs more registers: only
    launches with a ragged row take it, and a ragged matrix does not split a group's launch in two."""
    for shapes in (ALIGNED, ALIGNED + [(40, 61), (40, 511), (7,)]):
        lines = plan(shapes, rank)
        assert {w[3] for w in lines} >= {"1", "33", "66"} and all(w[4] == "0" for w in lines)
    for m in (2001, 3001, 4501):
        lines = plan(ALIGNED + [(40, m)], rank, cap=1)  # a bucket per tensor
        for w in lines:
            if w[3] in "2345" and w[5] != "0":
                assert w[1] == "group" or (w[4] == "1") == (w[6] != "0"), w
        groups = [w for w in lines if w[1] == "group"]
        assert len({w[3] for w in groups}) == len(groups)
        assert [w[4] for w in groups if w[6] != "0"] == ["1"]
