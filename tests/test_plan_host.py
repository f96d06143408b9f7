"""The planner's launch lists, read from the planner itself (plan.cpp uses no HIP) through a small
driver compiled here: which variant of a kernel a launch takes, and what the partial products take."""

import math
import os
import random
import subprocess

import pytest

import synthgrad as sg
from tests.test_gpu_split import sums_shapes

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
  // from rank 8 on: whether a compress list splits its sums into parts (P-step: rows of several parts)
  auto form = [&](const char* what, size_t i, int par, const std::vector<Launch>& L) {
    for (const Launch& l : L) {
      if (l.kernel != K_WPSTEP && l.kernel != K_WQSTEP) continue;
      bool parts = l.kernel == K_WQSTEP && l.variant == kWideFine;
      for (int32_t t = 0; t < l.ntiles && l.kernel == K_WPSTEP; ++t) {
        const Tile& x = p.tiles[l.tile_off + t];
        parts = parts || (x.kind != T_VEC && (x.b >> 8) != 0);
      }
      printf("form %s %d %d %d\n", what, int(i), par, int(parts));
    }
  };
  for (int par = 0; par < 2; ++par) {
    for (size_t b = 0; b < p.buckets.size(); ++b) form("bucket", b, par, p.buckets[b].compress[par]);
    for (size_t g = 0; g < p.group_compress.size(); ++g) form("group", g, par, p.group_compress[g][par]);
  }
  // the region of partial products, the ends of its uses in every compress list, per matrix its slot
  printf("partials %lld\n", (long long)p.qpart_floats);
  auto uses = [&](const std::vector<Launch>& L) {
    for (const Launch& l : L)
      for (int32_t t = 0; t < l.ntiles; ++t) {
        const Tile& x = p.tiles[l.tile_off + t];
        if (x.kind == T_VEC) continue;
        const MatDesc& d = p.mats[x.idx];
        long long rows = 0;  // of rank floats, from the matrix's slot on
        if (l.kernel == K_PWIDE) rows = (srows_block(x.b) + 1ll) * d.n;
        if (l.kernel == K_WPSTEP) rows = (x.b >> 8) * 1ll * d.n;
        if (l.kernel == K_QSTEP || l.kernel == K_WQSTEP) rows = (x.a + 1ll) * ((d.m + d.q_cb - 1) / d.q_cb) * d.q_cb;
        const long long next = x.idx + 1 < (int)p.mats.size() ? p.mats[x.idx + 1].qpart : p.qpart_floats;
        if (d.qpart + rows * rank > next) printf("past %d %d\n", x.idx, l.kernel);
      }
  };
  for (const BucketPlan& b : p.buckets)
    for (int par = 0; par < 2; ++par) uses(b.compress[par]);
  for (const auto& g : p.group_compress)
    for (int par = 0; par < 2; ++par) uses(g[par]);
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
        lines = [w for w in plan(shapes, rank) if w[0] == "pstep"]
        assert {w[3] for w in lines} >= {"1", "33", "66"} and all(w[4] == "0" for w in lines)
    for m in (2001, 3001, 4501):
        lines = [w for w in plan(ALIGNED + [(40, m)], rank, cap=1) if w[0] == "pstep"]  # a bucket per tensor
        for w in lines:
            if w[3] in "2345" and w[5] != "0":
                assert w[1] == "group" or (w[4] == "1") == (w[6] != "0"), w
        groups = [w for w in lines if w[1] == "group"]
        assert len({w[3] for w in groups}) == len(groups)
        assert [w[4] for w in groups if w[6] != "0"] == ["1"]


@pytest.mark.parametrize("rank", [1, 2, 4, 8, 16, 32, 64, 128, 256])
def test_partial_products_stay_in_their_slots(plan, rank):
    """Every compress list, split into parts or not, writes its partials inside its matrix's slot."""
    rng = random.Random(rank)
    for _ in range(12):
        shapes = [tuple(int(2.0 ** rng.uniform(2, 15)) for _ in range(2)) for _ in range(rng.randint(1, 6))]
        lines = plan(shapes + [(1 << 24, 5), (300, 1 << 18)][:rng.randint(0, 2)], rank, rng.choice([1, 1 << 20, 25 << 20]))
        assert not [w for w in lines if w[0] == "past"], shapes


@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128, 256])
def test_whole_sums_and_parts_share_one_region(plan, rank):
    """BERT-large's partial products: from rank 64 on one byte per element at most for the parts, below
    that 4 r bytes per 256 rows, and a few per cent for the columns and rows that fill up a part; a
    region for each form took half as much again at ranks 8 to 64."""
    shapes = [p.shape for p in sg.WORKLOADS["bert_large_r32"].params]
    elements = sum(math.prod(s) for s in shapes if len(s) > 1)
    (floats,) = (int(w[1]) for w in plan(shapes, rank) if w[0] == "partials")
    assert 4 * floats <= 1.05 * min(1, rank / 64) * elements


@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128, 256])
def test_large_calls_take_whole_sums(plan, rank):
    """The shapes of test_split_sums_agree_between_calls compare what it says they compare: buckets
    that split their sums with a group that does not."""
    forms = {}
    for w in plan(sums_shapes(rank), rank):
        if w[0] == "form":
            forms.setdefault((w[1], int(w[3])), set()).add(int(w[4]))
    # at rank 256 every list takes a tile per part, below 64 every P-step one per 1024 columns
    assert forms["bucket", 0] == ({0} if rank == 256 else {1}) and forms["group", 0] == {0}
    if 64 <= rank < 256:
        assert forms["bucket", 1] == {1} and forms["group", 1] == {0}
