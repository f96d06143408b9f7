// Host planner: reshape and eligibility, tensor-fusion buckets, factor-buffer offsets, state
// regions and the launch tables of every bucket and phase.
//
// Layout rules (arXiv 2306.08881):
//  * Section IV-C: vector-shaped gradients are not compressed, other gradients are reshaped
//    into matrices; the matrix is n = dim 0 by m = product of the other dims.  A matrix with
//    r >= min(n, m) gains nothing from a rank-r factorisation and is passed through too.
//  * Section IV-B, "Buffer Size": buckets of a fixed byte size (25 MB in PyTorch-DDP, read as
//    MiB), filled with whole tensors in backward order (reverse registration order); a bucket
//    is closed once it reaches the cap.
//  * Section IV-B / IV-C: each bucket's factor buffer holds the compressed factors (P: n x r on
//    P-steps, Q: m x r on Q-steps) and the raw vectors, packed in bucket order.
#include "plan.hpp"

#include <algorithm>
#include <array>
#include <climits>
#include <cmath>
#include <map>

namespace acp {

namespace {

constexpr int64_t kTileElems = 16384;   // gradient elements per streaming tile (unit)
constexpr int64_t kTargetTiles = 1024;     // workgroups a launch class aims for (4 per CU)
constexpr int64_t kMinTileElems = 2048;    // smallest tile of a class that has few elements
constexpr int64_t kPGroup = 8;            // P-step tiles whose rows interleave (r <= 4)
constexpr int64_t kMergeElems = int64_t(16) << 20;  // P-step classes below this share a launch
constexpr int64_t kPMinRows = 8;          // fewest rows of a P-step tile (r <= 4)
constexpr int64_t kPwRows = 64;           // most rows of a K_PWIDE tile
constexpr int64_t kQGroup = 8;            // Q-step row chunks whose rows interleave (r <= 4)
constexpr int64_t kMaxExtent = int64_t(1) << 30;  // bytes of a tile from its first element
constexpr int64_t kVecChunk = 4096;     // raw-vector elements per copy tile
constexpr int64_t kApplyRows = 256;     // factor rows per orthogonalisation tile
constexpr int64_t kSlotAlign = 64;      // floats (256 bytes)

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t align_up(int64_t x, int64_t a) { return cdiv(x, a) * a; }

bool rank_supported(int32_t r) {
  return r == 1 || r == 2 || r == 4 || r == 8 || r == 16 || r == 32 || r == 64 || r == 128 || r == 256;
}

struct TileSink {
  std::vector<Tile>& tiles;
  Launch begin(int32_t kernel, int32_t variant) {
    Launch l{};
    l.kernel = kernel;
    l.variant = variant;
    l.tile_off = static_cast<int64_t>(tiles.size());
    return l;
  }
  void end(Launch& l, std::vector<Launch>& list) {
    l.ntiles = static_cast<int32_t>(static_cast<int64_t>(tiles.size()) - l.tile_off);
    if (l.ntiles > 0) list.push_back(l);
  }
};

}  // namespace

std::string build_plan(Plan& plan, int32_t num_tensors, const int32_t* ndims, const int64_t* dims,
                       int32_t rank, int64_t cap_bytes, bool ef, bool reuse, bool psgd) {
  if (num_tensors <= 0) return "num_tensors must be positive";
  if (!ndims || !dims) return "ndims and dims must not be NULL";
  if (!rank_supported(rank)) return "rank must be one of 1, 2, 4, 8, 16, 32, 64, 128, 256";
  if (cap_bytes <= 0) return "bucket_cap_bytes must be positive";
  if (psgd && !reuse) return "Power-SGD reuses Q";
  plan = Plan{};
  plan.rank = rank;
  plan.cap_bytes = cap_bytes;
  plan.ef = ef;
  plan.reuse = reuse;
  plan.psgd = psgd;
  const int64_t r = rank;

  // ---- tensors: reshape and eligibility
  int64_t di = 0;
  plan.tensors.resize(num_tensors);
  for (int32_t i = 0; i < num_tensors; ++i) {
    const int32_t nd = ndims[i];
    if (nd < 1 || nd > 8) return "tensor " + std::to_string(i) + ": ndims must be in 1..8";
    TensorPlan& t = plan.tensors[i];
    int64_t numel = 1;
    for (int32_t k = 0; k < nd; ++k) {
      const int64_t d = dims[di + k];
      if (d <= 0 || d > (int64_t(1) << 31)) return "tensor " + std::to_string(i) + ": bad dim";
      numel *= d;
      if (numel > (int64_t(1) << 40)) return "tensor " + std::to_string(i) + ": too large";
      t.shape.push_back(d);
    }
    di += nd;
    t.numel = numel;
    if (nd >= 2) {
      const int64_t n = t.shape[0], m = numel / n;
      if (r < std::min(n, m)) {
        // the kernels address a factor of m rows of r floats with 32-bit byte offsets
        if (m > std::min<int64_t>(kMaxCols, ((int64_t(1) << 32) - 1) / (4 * r)))
          return "tensor " + std::to_string(i) +
                 ": compressed matrices may have at most min(2^24, (2^32 - 1) / (4 r)) columns";
        t.compressed = true;
        t.n = n;
        t.m = m;
      }
    }
    if (!t.compressed) {
      // a raw tensor's element offsets travel as 32-bit tile fields
      if (numel > INT32_MAX) return "tensor " + std::to_string(i) + ": raw tensors may have at most 2^31 - 1 elements";
      t.n = numel;
      t.m = 1;
    } else if (t.n > INT32_MAX) {
      return "tensor " + std::to_string(i) + ": compressed matrices may have at most 2^31 - 1 rows";
    }
  }

  // ---- buckets: backward order, close once the byte size reaches the cap
  {
    BucketPlan cur;
    int64_t cur_bytes = 0;
    for (int32_t i = num_tensors - 1; i >= 0; --i) {
      TensorPlan& t = plan.tensors[i];
      cur.tids.push_back(i);
      cur.grad_off.push_back(cur.grad_elems);
      cur.fac_off_p.push_back(cur.fac_elems_p);
      cur.fac_off_q.push_back(cur.fac_elems_q);
      cur.grad_elems += t.numel;
      cur.fac_elems_p += t.compressed ? t.n * r : t.numel;
      cur.fac_elems_q += t.compressed ? t.m * r : t.numel;
      cur_bytes += t.numel * 4;
      if (cur_bytes >= cap_bytes) {
        plan.buckets.push_back(std::move(cur));
        cur = BucketPlan{};
        cur_bytes = 0;
      }
    }
    if (!cur.tids.empty()) plan.buckets.push_back(std::move(cur));
  }

  // ---- launch classes of the kernels up to rank 4 and their total elements: a class with few
  // elements gets smaller tiles, so that its (grouped) launch still has about kTargetTiles
  // workgroups instead of a few long serial ones
  const bool wide = r >= kWideRank;
  std::map<int64_t, int64_t> class_elems;
  auto class_key = [](int32_t kernel, int32_t variant) { return int64_t(kernel) * 65536 + variant; };
  // (P-step kernel, variant), (Q-step kernel, variant), (decompress kernel, variant) of a matrix
  // of m columns
  auto low_classes = [&](int64_t m) {
    std::array<std::pair<int32_t, int32_t>, 3> c{};
    const int64_t m4 = cdiv(m, 4);
    if (m4 <= 128) {
      const int32_t v = narrow_variant(static_cast<int32_t>(m4));
      c = {{{K_PNARROW, v}, {K_QNARROW, v}, {K_RNARROW, v}}};
    } else if (m4 <= 192) {  // three waves cover a row of the P-step
      c = {{{K_PFUSED, 1 | kThreeWaves}, {K_QSTEP, 0}, {K_RECON4, 0}}};
    } else if (m4 > 768 && m4 <= 1024) {  // eight waves of two groups cover a row
      c = {{{K_PFUSED, 2 | kEightWaves}, {K_QSTEP, 0}, {K_RECON4, 0}}};
    } else if (m <= kFusedCols) {
      c = {{{K_PFUSED, static_cast<int32_t>(cdiv(m4, 256))}, {K_QSTEP, 0}, {K_RECON4, 0}}};
    } else {
      c = {{{K_PWIDE, 0}, {K_QSTEP, 1}, {K_RECON4, 0}}};
    }
    return c;
  };
  for (const BucketPlan& bk : plan.buckets)
    for (size_t k = 0; k < bk.tids.size(); ++k) {
      const TensorPlan& t = plan.tensors[bk.tids[k]];
      if (!t.compressed || wide) continue;
      for (const auto& kv : low_classes(t.m)) class_elems[class_key(kv.first, kv.second)] += t.n * t.m;
    }
  // elements per tile of a class: its total over kTargetTiles, between kMinTileElems and `base`
  auto class_tile = [&](int32_t kernel, int32_t variant, int64_t base) {
    const auto it = class_elems.find(class_key(kernel, variant));
    const int64_t tot = it == class_elems.end() ? 0 : it->second;
    return std::max<int64_t>(kMinTileElems, std::min<int64_t>(base, tot / kTargetTiles));
  };

  // P-step launch classes: a class S >= 2 with fewer than kMergeElems elements in all runs in
  // one launch with the other such classes, as the largest of them (pmerge; 0: none)
  int32_t pmerge = 0;
  for (int32_t S = 2; S <= 5; ++S) {
    const auto it = class_elems.find(class_key(K_PFUSED, S));
    if (it != class_elems.end() && it->second > 0 && it->second < kMergeElems) pmerge = S;
  }
  auto class_of_p = [&](int32_t S) -> int32_t {
    if (S < 2 || pmerge == 0) return S;
    const auto it = class_elems.find(class_key(K_PFUSED, S));
    const int64_t tot = it == class_elems.end() ? 0 : it->second;
    return tot < kMergeElems ? pmerge : S;
  };

  // ---- what acp_compress_noalloc's limit is held against: part of that call's interface, stated
  // there, and independent of the chunks that the kernels take.  A matrix counts
  // ceil(n / rows) ceil(m / cols) cols r floats.
  auto whole_words = [&](int64_t m, int64_t off, int64_t offp, int64_t offq) {
    return r == 4 && m <= 5120 && (m | off | offp | offq) % 4 == 0;
  };
  auto row_class = [](int64_t m) { return m <= 64 ? 0 : m <= 128 ? 1 : m <= 256 ? 2 : m <= 512 ? 3 : 4; };
  int64_t word_elems[5] = {0, 0, 0, 0, 0};  // elements of such matrices of the model, by row_class
  for (const BucketPlan& bk : plan.buckets)
    for (size_t k = 0; k < bk.tids.size(); ++k) {
      const TensorPlan& t = plan.tensors[bk.tids[k]];
      if (t.compressed && whole_words(t.m, bk.grad_off[k], bk.fac_off_p[k], bk.fac_off_q[k]))
        word_elems[row_class(t.m)] += t.n * t.m;
    }
  auto limit_floats = [&](int64_t n, int64_t m, int64_t off, int64_t offp, int64_t offq) {
    const int64_t most = std::max<int64_t>(1, (int64_t(1) << 28) / m);
    int64_t rows = std::min<int64_t>(most, r >= 128 ? 2048 : r >= 8 ? 512 : 256), cols = 32;
    if (r < 8) {
      cols = (m | off) % 4 == 0 ? 1024 : 256;
      int64_t c = cdiv(n, 4);
      if (whole_words(m, off, offp, offq)) {
        const int64_t w = std::min<int64_t>(m, 1024);
        c = std::max<int64_t>(2048, word_elems[row_class(m)] / 1024) / w / 16 * 16;
      }
      rows = std::min(rows, std::max<int64_t>(16, c));
    }
    return align_up(cdiv(n, rows) * cdiv(m, cols) * cols * r, kSlotAlign);
  };

  // ---- per-tensor device descriptors and state regions
  int64_t e_floats = 0, fac_floats = 0, gpart = 0;
  for (int32_t b = 0; b < static_cast<int32_t>(plan.buckets.size()); ++b) {
    BucketPlan& bk = plan.buckets[b];
    bk.e_base = e_floats;
    if (ef) e_floats += align_up(bk.grad_elems, kSlotAlign);
    for (int32_t k = 0; k < static_cast<int32_t>(bk.tids.size()); ++k) {
      TensorPlan& t = plan.tensors[bk.tids[k]];
      t.bucket = b;
      t.pos = k;
      if (!t.compressed) {
        VecDesc v{};
        v.grad_off = bk.grad_off[k];
        v.fac_off_p = bk.fac_off_p[k];
        v.fac_off_q = bk.fac_off_q[k];
        v.numel = t.numel;
        v.e_off = bk.e_base + bk.grad_off[k];
        v.bucket = b;
        t.vec = static_cast<int32_t>(plan.vecs.size());
        bk.vecs.push_back(t.vec);
        plan.vecs.push_back(v);
        continue;
      }
      MatDesc d{};
      d.n = static_cast<int32_t>(t.n);
      d.m = static_cast<int32_t>(t.m);
      d.grad_off = bk.grad_off[k];
      d.e_off = bk.e_base + bk.grad_off[k];
      d.fac_off_p = bk.fac_off_p[k];
      d.fac_off_q = bk.fac_off_q[k];
      d.tid = bk.tids[k];
      const int64_t np = align_up(t.n * r, kSlotAlign), mp = align_up(t.m * r, kSlotAlign);
      d.p_slot = fac_floats;
      d.ph_slot = fac_floats + np;
      d.pl_slot = fac_floats + 2 * np;
      d.q_slot = fac_floats + 3 * np;
      d.qh_slot = d.q_slot + mp;
      d.ql_slot = d.q_slot + 2 * mp;
      fac_floats += 3 * np + 3 * mp;
      d.q_cb = wide ? kWideQCols : 1024;
      d.xhold = wide || t.m > kFusedCols ? 1 : 0;
      if (d.xhold) bk.xhold = true;
      // rows per chunk: kQRows (kWideQRows), fewer when a chunk's byte extent would pass 2^30
      // (the kernels address a tile with 32-bit offsets from the tile's first element)
      d.q_rows = static_cast<int32_t>(std::max<int64_t>(
          1, std::min<int64_t>(wide ? (!split_nested(static_cast<int>(r)) ? split_part(static_cast<int>(r)) : r >= kBlockedRank ? 4 * kWideQRows : kWideQRows) : kQRows,
                               (int64_t(1) << 30) / (t.m * 4))));
      if (!wide) {
        // chunk rows of a multiple of 16 holding about the class's elements per tile
        const auto qc = low_classes(t.m)[1];
        const int64_t cols = std::min<int64_t>(t.m, d.q_cb);
        const int64_t want = class_tile(qc.first, qc.second, int64_t(kQRows) * cols) / cols;
        d.q_rows = std::min<int32_t>(d.q_rows, static_cast<int32_t>(std::max<int64_t>(16, want / 16 * 16)));
      }
      // up to rank 4 the Q-step interleaves the rows of kQGroup chunks, unless their byte extent
      // would pass kMaxExtent
      d.q_grp = !wide && t.m > 512 && kQGroup * d.q_rows * t.m * 4 <= kMaxExtent ? static_cast<int32_t>(kQGroup) : 1;
      d.q_chunks = static_cast<int32_t>(cdiv(t.n, d.q_rows));
      bk.limit_floats += limit_floats(t.n, t.m, d.grad_off, d.fac_off_p, d.fac_off_q);
      d.bucket = b;
      // factor rows per Gram slice: at r <= 8 up to 5120 (one slice, and no K_CHOL, for
      // factors of at most that many rows; where nothing runs beside it, as in Power-SGD's second
      // half, one workgroup takes 12 us for 4096 rows, 19 for 8192); at r >= 16 at least 256 and at most 32 slices per factor
      // (K_CHOL adds a factor's slice partials in one workgroup); from kBlockedRank on at least
      // 1024, since every slice adds an r x r partial for K_GSUM to read (1024 measured faster
      // than 256, 512, 2048 and 4096), and again at most 32, so that no slice is much longer
      d.fact_rows = r <= 8 ? 5120
                    : r >= kBlockedRank
                        ? static_cast<int32_t>(std::max<int64_t>(1024, align_up(cdiv(std::max(t.n, t.m), 32), 64)))
                        : static_cast<int32_t>(std::max<int64_t>(256, align_up(cdiv(std::max(t.n, t.m), 32), 64)));
      d.fact_slices_p = static_cast<int32_t>(cdiv(t.n, d.fact_rows));
      d.fact_slices_q = static_cast<int32_t>(cdiv(t.m, d.fact_rows));
      d.gpart = gpart;
      {
        const int64_t nsl = std::max(d.fact_slices_p, d.fact_slices_q);
        if (nsl > 1 || r >= kBlockedRank) gpart += nsl * r * r;
      }
      d.w_slot = static_cast<int64_t>(plan.mats.size()) * r * r;
      t.mat = static_cast<int32_t>(plan.mats.size());
      bk.mats.push_back(t.mat);
      plan.mats.push_back(d);
    }
  }

  // ---- launch tables
  // columns of a Q-step tile from kWideRank on: kWideQWaves column blocks below kSplitRank
  const int64_t q_tile_cols = r < kSplitRank ? kWideQCols * kWideQWaves : split_fix(static_cast<int>(r));
  TileSink sink{plan.tiles};
  auto vec_tiles = [&](const BucketPlan& bk) {
    for (int32_t v : bk.vecs) {
      const int64_t n = plan.vecs[v].numel;
      for (int64_t s = 0; s < n; s += kVecChunk)
        plan.tiles.push_back(Tile{T_VEC, v, static_cast<int32_t>(s),
                                  static_cast<int32_t>(std::min(kVecChunk, n - s))});
    }
  };
  // orthogonalisation tiles of kApplyRows factor rows; from kApplyMfmaRank on one per column
  // block of Xh as well (b = rows | block << 16)
  auto apply_tiles = [&](const std::vector<int32_t>& mats, bool q) {
    const int32_t ncb = r >= kApplyMfmaRank ? apply_blocks(static_cast<int32_t>(r)) : 1;
    for (int32_t mi : mats) {
      const int64_t rows = q ? plan.mats[mi].m : plan.mats[mi].n;
      for (int64_t s = 0; s < rows; s += kApplyRows)
        for (int32_t cb = 0; cb < ncb; ++cb)
          plan.tiles.push_back(Tile{T_ROWS, mi, static_cast<int32_t>(s),
                                    static_cast<int32_t>(std::min(kApplyRows, rows - s)) | (cb << 16)});
    }
  };
  // factor tiles: one per slice of fact_rows factor rows
  auto fact_tiles = [&](int32_t mi, bool q) {
    const MatDesc& d = plan.mats[mi];
    const int32_t nsl = q ? d.fact_slices_q : d.fact_slices_p;
    const int32_t nq = gram_parts(static_cast<int32_t>(r));
    for (int32_t s = 0; s < nsl; ++s)
      for (int32_t q4 = 0; q4 < nq; ++q4) plan.tiles.push_back(Tile{T_FACT, mi, s + 65536 * q4, nsl});
  };
  // Gram finish of the factors of more than one slice
  auto chol_tiles = [&](int32_t mi, bool q) {
    const MatDesc& d = plan.mats[mi];
    const int32_t nsl = q ? d.fact_slices_q : d.fact_slices_p;
    if (nsl > 1 || r >= kBlockedRank) plan.tiles.push_back(Tile{T_FACT, mi, 0, nsl});
  };
  // from kBlockedRank on: the partials' sum, kGsumEntries Gram entries per tile
  auto gsum_tiles = [&](int32_t mi, bool q) {
    const MatDesc& d = plan.mats[mi];
    const int32_t nsl = q ? d.fact_slices_q : d.fact_slices_p;
    for (int32_t e = 0; e < static_cast<int32_t>(r * r / kGsumEntries); ++e)
      plan.tiles.push_back(Tile{T_FACT, mi, e, nsl});
  };
  // the Gram finish after the factor tiles: K_GSUM from kBlockedRank on, then K_CHOL
  auto chol_launches = [&](const std::vector<int32_t>& mats, bool q, std::vector<Launch>& L) {
    if (r >= kBlockedRank) {
      Launch l = sink.begin(K_GSUM, 0);
      for (int32_t mi : mats) gsum_tiles(mi, q);
      sink.end(l, L);
    }
    Launch l = sink.begin(K_CHOL, 0);
    for (int32_t mi : mats) chol_tiles(mi, q);
    sink.end(l, L);
  };
  auto row_tiles = [&](int32_t mi, int64_t rows_per_tile) {
    const MatDesc& d = plan.mats[mi];
    for (int64_t s = 0; s < d.n; s += rows_per_tile)
      plan.tiles.push_back(Tile{T_ROWS, mi, static_cast<int32_t>(s),
                                static_cast<int32_t>(std::min<int64_t>(rows_per_tile, d.n - s))});
  };
  // decompress tiles up to rank 4: 1024-column blocks of kReconRows rows.  Rows go in groups of
  // gr * kReconRows (gr = 8 / column blocks, at least 1); the tiles of a group take rows
  // x, x + gr, x + 2 gr, ... (x < gr) and are ordered (x, block), so that tiles that run together
  // write whole adjacent rows.
  auto recon4_tiles = [&](int32_t mi) {
    const MatDesc& d = plan.mats[mi];
    const int64_t nb = cdiv(d.m, 1024);
    const int64_t gr = std::max<int64_t>(1, 8 / nb);
    for (int64_t g0 = 0; g0 < d.n; g0 += gr * kReconRows) {
      const int64_t end = std::min<int64_t>(d.n, g0 + gr * kReconRows);
      for (int64_t x = 0; x < gr && g0 + x < end; ++x) {
        const int64_t cnt = cdiv(end - g0 - x, gr);
        for (int64_t cb = 0; cb < nb; ++cb)
          plan.tiles.push_back(Tile{T_SROWS, mi, static_cast<int32_t>(g0 + x), srows_pack(cb, gr, cnt)});
      }
    }
  };
  // P-step tiles (r <= 4) of rows_per_tile rows: groups of kPGroup tiles share kPGroup *
  // rows_per_tile rows, tile x of a group taking rows x, x + g, x + 2g, ... of it (g tiles in the
  // group, kPGroup except in the last one)
  auto pstep_tiles = [&](int32_t mi, int64_t rows_per_tile) {
    const MatDesc& d = plan.mats[mi];
    for (int64_t g0 = 0; g0 < d.n; g0 += kPGroup * rows_per_tile) {
      const int64_t rem = std::min<int64_t>(d.n - g0, kPGroup * rows_per_tile);
      const int64_t g = cdiv(rem, rows_per_tile);
      for (int64_t x = 0; x < g; ++x)
        plan.tiles.push_back(Tile{T_SROWS, mi, static_cast<int32_t>(g0 + x), srows_pack(0, g, cdiv(rem - x, g))});
    }
  };
  // K_PWIDE tiles: rows in groups as in pstep_tiles (of one tile where the extent of kPGroup would
  // pass kMaxExtent), one tile per 1024-column block, a group's blocks of a row set together
  auto pwide_tiles = [&](int32_t mi) {
    const MatDesc& d = plan.mats[mi];
    const int64_t want = class_tile(K_PWIDE, 0, kPwRows * 1024) / 1024;
    int64_t rows = std::max<int64_t>(kPMinRows, std::min<int64_t>(kPwRows, want / 8 * 8));
    rows = std::max<int64_t>(1, std::min<int64_t>(rows, kMaxExtent / (int64_t(d.m) * 4)));
    const int64_t grp = kPGroup * rows * d.m * 4 <= kMaxExtent ? kPGroup : 1;
    const int64_t nb = cdiv(d.m, 1024);
    for (int64_t g0 = 0; g0 < d.n; g0 += grp * rows) {
      const int64_t rem = std::min<int64_t>(d.n - g0, grp * rows);
      const int64_t g = cdiv(rem, rows);
      for (int64_t x = 0; x < g; ++x)
        for (int64_t cb = 0; cb < nb; ++cb)
          plan.tiles.push_back(Tile{T_SROWS, mi, static_cast<int32_t>(g0 + x), srows_pack(cb, g, cdiv(rem - x, g))});
    }
  };
  // rows per P-step tile up to rank 4: a multiple of the rows handled per round
  auto rows_for = [&](int32_t mi, int64_t elems) {
    const MatDesc& d = plan.mats[mi];
    const int64_t rb = pstep_rows(static_cast<int>(r), d.scls);
    const int64_t rows = rb * std::max<int64_t>(1, elems / (int64_t(d.m) * rb));
    return std::min<int64_t>(rows, kMaxTileRows);
  };

  // Q-step finish tiles: entry blocks of each matrix's column blocks
  auto qfin_launch = [&](const BucketPlan& bk, std::vector<Launch>& L, bool with_vecs, int32_t variant) {
    Launch l = sink.begin(K_QFIN, variant);
    for (int32_t mi : bk.mats) {
      const MatDesc& d = plan.mats[mi];
      const int64_t nblk = cdiv(int64_t(d.m) * r, qfin_entries(d.q_chunks));
      for (int64_t eb = 0; eb < nblk; ++eb)
        plan.tiles.push_back(Tile{T_QTILE, mi, static_cast<int32_t>(eb), 0});
    }
    if (with_vecs) vec_tiles(bk);
    sink.end(l, L);
  };
  auto emat_launch = [&](BucketPlan& bk) {
    Launch l = sink.begin(K_EMAT, 1);
    for (int32_t mi : bk.mats) row_tiles(mi, std::max<int64_t>(1, kTileElems / plan.mats[mi].m));
    sink.end(l, bk.emat);
  };
  // matrix tiles of a compress list's main launch (ranks 8 and up), and how many fill the GPU
  const int64_t full_tiles = r < kSplitRank ? kWideFullTiles : split_full_tiles(static_cast<int>(r));
  auto main_tiles = [&](const std::vector<Launch>& L) {
    int64_t n = 0;
    for (const Launch& l : L)
      if (l.kernel == K_WPSTEP || l.kernel == K_WQSTEP)
        for (int32_t i = 0; i < l.ntiles; ++i) n += plan.tiles[l.tile_off + i].kind != T_VEC;
    return n;
  };
  // whether the sums of a parity's compress step have parts that tiles can take one by one (at rank 256
  // every list does)
  auto has_parts = [&](int32_t par) { return (par == 0 || r >= kSplitRank) && split_nested(static_cast<int>(r)); };
  // tiles that share a row in a P-step
  auto p_parts = [&](int64_t m, bool fine) -> int64_t {
    const int rk = static_cast<int>(r);
    return r < kSplitRank ? wide_chunks(m) : fine || !split_nested(rk) ? cdiv(m, split_part(rk)) : 1;
  };
  // floats of partial products per matrix: the most that a list in use writes
  std::vector<int64_t> need(plan.mats.size(), 0);
  auto uses_form = [&](const BucketPlan& bk, int32_t par, bool fine) {
    const int64_t pr = part_rows(static_cast<int>(r));
    for (int32_t mi : bk.mats) {
      const MatDesc& d = plan.mats[mi];
      int64_t rows;  // of r floats
      if (par == 1) {
        const int64_t nc = p_parts(d.m, fine);
        rows = nc > 1 ? nc * d.n : 0;
      } else {
        const int64_t last = d.n - int64_t(d.q_chunks - 1) * d.q_rows;  // rows of the last chunk
        const bool parts = fine && has_parts(par);
        rows = (parts ? (d.q_chunks - 1) * cdiv(d.q_rows, pr) + cdiv(last, pr) : d.q_chunks) * align_up(d.m, d.q_cb);
      }
      need[mi] = std::max(need[mi], rows * r);
    }
  };
  auto recon_tiles = [&](const BucketPlan& bk) {  // decompress tiles of kWideRCols columns
    int64_t n = 0;
    for (const Launch& l : bk.recon[0][0])
      if (l.kernel == K_WRECON) n += l.ntiles;
    return n;
  };
  // ranks 8..256: every matrix of the bucket takes the MFMA kernels
  auto wide_lists = [&](BucketPlan& bk) {
    // The compress kernels take matrix tiles, and the raw vectors ride along in the P-step and
    // Q-finish launches; factor tiles go to launches of their own.
    // -- P-step (odd t): Qh = Q W, then row tiles (below kSplitRank one per kWideChunk columns, from
    // there on, fine, one per part), then the sum of a row's chunks or parts
    const int32_t rk = static_cast<int32_t>(r);
    auto p_list = [&](std::vector<Launch>& L, bool fine) {
      Launch l = sink.begin(K_APPLY, 1);
      apply_tiles(bk.mats, true);
      sink.end(l, L);
      const int64_t rows = r < kSplitRank ? 32 : split_fix(rk);
      l = sink.begin(K_WPSTEP, 0);
      for (int32_t mi : bk.mats) {
        const MatDesc& d = plan.mats[mi];
        const int64_t nc = p_parts(d.m, fine);
        for (int64_t s = 0; s < d.n; s += rows)
          for (int64_t c = 0; c < nc; ++c)
            plan.tiles.push_back(Tile{T_ROWS, mi, static_cast<int32_t>(s),
                                      static_cast<int32_t>(std::min(rows, d.n - s) | (nc > 1 ? (c + 1) << 8 : 0))});
      }
      vec_tiles(bk);  // packed by the P-step launch's workgroups
      sink.end(l, L);
      l = sink.begin(K_WPFIN, 0);
      for (int32_t mi : bk.mats)
        if (p_parts(plan.mats[mi].m, fine) > 1) row_tiles(mi, 4 * kBlock / r);
      sink.end(l, L);
    };
    // -- Q-step (even t): Ph = P W, (row chunk, column block) tiles (fine: of the chunks' parts),
    // vectors, finish
    auto q_list = [&](std::vector<Launch>& L, bool fine) {
      Launch l = sink.begin(K_APPLY, 0);
      apply_tiles(bk.mats, false);
      sink.end(l, L);
      const int64_t pr = part_rows(rk);
      l = sink.begin(K_WQSTEP, fine ? kWideFine : 0);
      for (int32_t mi : bk.mats) {
        const MatDesc& d = plan.mats[mi];
        const int32_t ncb = static_cast<int32_t>(cdiv(d.m, q_tile_cols));
        const int32_t parts = fine ? static_cast<int32_t>(cdiv(d.q_rows, pr)) : 1;
        for (int32_t c = 0; c < d.q_chunks * parts; ++c) {
          if (int64_t(c / parts) * d.q_rows + (c % parts) * pr >= d.n) continue;  // no rows
          for (int32_t cb = 0; cb < ncb; ++cb) plan.tiles.push_back(Tile{T_QTILE, mi, c, cb});
        }
      }
      sink.end(l, L);
      qfin_launch(bk, L, true, fine ? kWideFine : 0);  // the vectors packed by the finish launch's workgroups
    };
    for (int32_t par = 0; par < 2; ++par) {
      auto list = [&](std::vector<Launch>& L, bool fine) { par == 1 ? p_list(L, fine) : q_list(L, fine); };
      list(bk.coarse[par], false);
      if (has_parts(par))
        list(bk.fine[par], true);
      else
        bk.fine[par] = bk.coarse[par];
      const bool fine = main_tiles(bk.coarse[par]) < full_tiles;
      bk.compress[par] = (fine ? bk.fine : bk.coarse)[par];
      uses_form(bk, par, fine);
    }
    // -- decompress: factor tiles and vectors, the Gram partials' sum, (row block, 1024-column group)
    // tiles, and beside those the Cholesky
    const int64_t recon_rows = r < kSplitRank ? 32 : kSplitRecon;
    for (int32_t par = 0; par < 2; ++par) {
      std::vector<Launch>& L = bk.recon[0][par];
      const bool q = par == 0;
      Launch l = sink.begin(K_WFACT, 0);
      for (int32_t mi : bk.mats) fact_tiles(mi, q);
      vec_tiles(bk);
      sink.end(l, L);
      if (r >= kBlockedRank) {
        l = sink.begin(K_GSUM, 0);
        for (int32_t mi : bk.mats) gsum_tiles(mi, q);
        sink.end(l, L);
      }
      auto recon_list = [&](std::vector<Launch>& R, int32_t width) {
        Launch w = sink.begin(K_WRECON, width);
        for (int32_t mi : bk.mats) {
          const MatDesc& d = plan.mats[mi];
          const int32_t nrb = static_cast<int32_t>(cdiv(d.n, recon_rows));
          const int32_t ncg = static_cast<int32_t>(cdiv(d.m, width));
          for (int32_t rb = 0; rb < nrb; ++rb)
            for (int32_t cg = 0; cg < ncg; ++cg) plan.tiles.push_back(Tile{T_QTILE, mi, rb, cg});
        }
        sink.end(w, R);
      };
      recon_list(L, kWideRCols);
      l = sink.begin(K_CHOL, 0);
      for (int32_t mi : bk.mats) chol_tiles(mi, q);
      sink.end(l, L);
      // the same with narrower decompress tiles
      std::vector<Launch> narrow;
      recon_list(narrow, kWideRNarrow);
      bk.recon[1][par] = L;
      for (Launch& x : bk.recon[1][par])
        if (x.kernel == K_WRECON) x = narrow[0];
      bk.decompress[par] = bk.recon[recon_tiles(bk) < kWideRFull ? 1 : 0][par];
    }
    emat_launch(bk);
  };

  for (BucketPlan& bk : plan.buckets) {
    if (wide) {
      wide_lists(bk);
      continue;
    }
    // narrow: rows of at most 512 columns (scls 0); three: 513-768 columns (three-wave P-step
    // launch); eight: 3073-4096 columns (eight-wave P-step launch); fast: the others up to
    // kFusedCols; xwide: longer rows
    std::vector<int32_t> fast, narrow, three, eight, xwide;
    for (int32_t mi : bk.mats) {
      MatDesc& d = plan.mats[mi];
      const int64_t m4 = cdiv(d.m, 4);
      d.scls = m4 <= 128 ? 0 : static_cast<int32_t>(std::min<int64_t>(6, cdiv(m4, 256)));
      (m4 <= 128 ? narrow : m4 <= 192 ? three : m4 > 768 && m4 <= 1024 ? eight : d.m <= kFusedCols ? fast : xwide).push_back(mi);
    }
    auto of_narrow = [&](int32_t v) {
      std::vector<int32_t> out;
      for (int32_t mi : narrow)
        if (narrow_variant((plan.mats[mi].m + 3) / 4) == v) out.push_back(mi);
      return out;
    };
    // rows per narrow tile: whole workgroup rounds (256 / L rows), about `elems` elements
    auto narrow_rows = [&](int32_t mi, int64_t elems) {
      const int64_t rw = kBlock / (narrow_variant((plan.mats[mi].m + 3) / 4) >> 4);
      return std::min<int64_t>(rw * std::max<int64_t>(1, elems / (int64_t(plan.mats[mi].m) * rw)),
                               kMaxTileRows);  // the decompress stages the tile's A rows in LDS
    };
    const int32_t narrow_vars[4] = {narrow_variant(16), narrow_variant(32), narrow_variant(64),
                                    narrow_variant(128)};
    auto of_class = [&](int32_t S) {
      std::vector<int32_t> v;
      for (int32_t mi : fast)
        if (plan.mats[mi].scls == S) v.push_back(mi);
      return v;
    };
    // -- P-step (odd t)
    {
      std::vector<Launch>& L = bk.compress[1];
      bool vec_done = bk.vecs.empty();
      Launch l{};
      // the classes S >= 2 with few elements in all (launch variant pmerge) share one launch
      auto pfused_tiles = [&](int32_t S) {
        // rows of 4 KB: 32K elements per tile; rows of 12 KB and more: 64K
        const int64_t base = (S >= 4 ? 4 : 2) * kTileElems;
        for (int32_t mi : of_class(S)) {
          pstep_tiles(mi, rows_for(mi, std::max<int64_t>(kPMinRows * plan.mats[mi].m,
                                                          class_tile(K_PFUSED, S, base))));
          if (S >= 2 && plan.mats[mi].m % 4) l.variant |= kRaggedRows;
        }
      };
      for (int32_t S = 1; S <= 5; ++S) {
        const bool merged = S >= 2 && class_of_p(S) != S;
        if (merged || (S == pmerge && S >= 2)) continue;  // the merged launch follows
        if (of_class(S).empty() && (S > 1 || narrow.empty())) continue;
        l = sink.begin(K_PFUSED, S);
        if (S == 1) {  // the narrow-row matrices' tiles ride in the S = 1 launch
          for (int32_t v : narrow_vars)
            for (int32_t mi : of_narrow(v)) row_tiles(mi, narrow_rows(mi, class_tile(K_PNARROW, v, 2 * kTileElems)));
        }
        pfused_tiles(S);
        if (!vec_done) vec_tiles(bk), vec_done = true;
        sink.end(l, L);
      }
      if (!three.empty()) {
        l = sink.begin(K_PFUSED, 1 | kThreeWaves);
        for (int32_t mi : three)
          pstep_tiles(mi, rows_for(mi, std::max<int64_t>(kPMinRows * plan.mats[mi].m,
                                                          class_tile(K_PFUSED, 1 | kThreeWaves, 2 * kTileElems))));
        if (!vec_done) vec_tiles(bk), vec_done = true;
        sink.end(l, L);
      }
      if (!eight.empty()) {
        l = sink.begin(K_PFUSED, 2 | kEightWaves);
        for (int32_t mi : eight)
          pstep_tiles(mi, rows_for(mi, std::max<int64_t>(kPMinRows * plan.mats[mi].m,
                                                          class_tile(K_PFUSED, 2 | kEightWaves, 4 * kTileElems))));
        if (!vec_done) vec_tiles(bk), vec_done = true;
        sink.end(l, L);
      }
      if (pmerge >= 2) {
        bool any = false;
        for (int32_t S = 2; S <= 5; ++S)
          if (class_of_p(S) == pmerge && !of_class(S).empty()) any = true;
        if (any) {
          l = sink.begin(K_PFUSED, pmerge);
          for (int32_t S = 2; S <= 5; ++S)
            if (class_of_p(S) == pmerge) pfused_tiles(S);
          if (!vec_done) vec_tiles(bk), vec_done = true;
          sink.end(l, L);
        }
      }
      if (!xwide.empty()) {
        l = sink.begin(K_PWIDE, 0);
        for (int32_t mi : xwide) pwide_tiles(mi);
        sink.end(l, L);
        l = sink.begin(K_PFIN, 0);
        for (int32_t mi : xwide) row_tiles(mi, kBlock);
        sink.end(l, L);
      }
      if (!vec_done) {
        l = sink.begin(K_VEC, 1);
        vec_tiles(bk);
        sink.end(l, L);
      }
    }
    // -- Q-step (even t)
    {
      std::vector<Launch>& L = bk.compress[0];
      bool vec_done = bk.vecs.empty();
      Launch l = sink.begin(K_QSTEP, 0);
      auto qtiles = [&](int32_t mi) {
        const MatDesc& d = plan.mats[mi];
        const int32_t ncb = static_cast<int32_t>(cdiv(d.m, d.q_cb));
        for (int32_t c = 0; c < d.q_chunks; ++c)
          for (int32_t cb = 0; cb < ncb; ++cb) plan.tiles.push_back(Tile{T_QTILE, mi, c, cb});
      };
      for (const auto* set : {&narrow, &three, &eight, &fast})
        for (int32_t mi : *set) qtiles(mi);
      if (static_cast<int64_t>(plan.tiles.size()) > l.tile_off && !vec_done) vec_tiles(bk), vec_done = true;
      sink.end(l, L);
      l = sink.begin(K_QSTEP, 1);  // the rows K_PWIDE takes
      for (int32_t mi : xwide) qtiles(mi);
      if (static_cast<int64_t>(plan.tiles.size()) > l.tile_off && !vec_done) vec_tiles(bk), vec_done = true;
      sink.end(l, L);
      qfin_launch(bk, L, false, 0);
      if (!vec_done) {
        l = sink.begin(K_VEC, 0);
        vec_tiles(bk);
        sink.end(l, L);
      }
    }
    // -- decompress (both parities): factor tiles first, then rows, then vectors
    for (int32_t par = 0; par < 2; ++par) {
      std::vector<Launch>& L = bk.decompress[par];
      const bool q = par == 0;
      Launch l = sink.begin(K_RECON4, 0);
      for (int32_t mi : bk.mats) fact_tiles(mi, q);
      vec_tiles(bk);
      for (int32_t v : narrow_vars)
        for (int32_t mi : of_narrow(v)) row_tiles(mi, narrow_rows(mi, class_tile(K_RNARROW, v, kTileElems)));
      for (const auto* set : {&fast, &three, &eight, &xwide})
        for (int32_t mi : *set) recon4_tiles(mi);
      sink.end(l, L);
      l = sink.begin(K_CHOL, 0);
      for (int32_t mi : bk.mats) chol_tiles(mi, q);
      sink.end(l, L);
    }
    emat_launch(bk);
  }
  // ---- no reuse: before each compress the reused factor is drawn anew (K_DRAW) and its W formed
  // (factor tiles from its slot, then the Gram finish); [1]: P-steps draw Q, [0]: Q-steps draw P
  for (BucketPlan& bk : plan.buckets) {
    if (reuse) break;
    for (int32_t par = 0; par < 2; ++par) {
      const bool q = par == 1;
      std::vector<Launch>& L = bk.draw[par];
      Launch l = sink.begin(K_DRAW, q ? 1 : 0);
      for (int32_t mi : bk.mats) {
        const int64_t rows = q ? plan.mats[mi].m : plan.mats[mi].n;
        for (int64_t s0 = 0; s0 < rows; s0 += kDrawRows)
          plan.tiles.push_back(Tile{T_ROWS, mi, static_cast<int32_t>(s0),
                                    static_cast<int32_t>(std::min<int64_t>(kDrawRows, rows - s0))});
      }
      sink.end(l, L);
      l = sink.begin(K_FACT, q ? 1 : 0);
      for (int32_t mi : bk.mats) fact_tiles(mi, q);
      sink.end(l, L);
      chol_launches(bk.mats, q, L);
    }
  }
  // ---- Power-SGD: the first half is the P-step lists with Q as it is, leaving M' in the E arena;
  // the second half copies the all-reduced P into its slot and forms its W, then runs the Q-step
  // lists on M'; decompress is the Q-step decompress
  for (BucketPlan& bk : plan.buckets) {
    if (!psgd) break;
    Launch l = sink.begin(K_FACT, kFactFromBuffer);
    for (int32_t mi : bk.mats) fact_tiles(mi, false);
    sink.end(l, bk.psgd_fact);
    chol_launches(bk.mats, false, bk.psgd_fact);
  }
  {
    Launch l = sink.begin(K_FACT, 1);
    for (int32_t mi = 0; mi < static_cast<int32_t>(plan.mats.size()); ++mi) fact_tiles(mi, true);
    sink.end(l, plan.gram_init);
    std::vector<int32_t> all(plan.mats.size());
    for (int32_t mi = 0; mi < static_cast<int32_t>(plan.mats.size()); ++mi) all[mi] = mi;
    chol_launches(all, true, plan.gram_init);
  }

  // ---- launch families and algorithmic bytes (host-side profiling)
  auto tile_bytes = [&](const Launch& l, const Tile& t, bool odd) -> double {
    // M read, E read, E written per compress element (Power-SGD's second half reads M' only)
    const double eb = ef && (odd || !psgd) ? 12.0 : 4.0;
    if (t.kind == T_VEC) return 8.0 * t.b;
    const MatDesc& d = plan.mats[t.idx];
    const double n = d.n, m = d.m, rr = double(r);
    switch (l.kernel) {
      case K_PFUSED: {  // strided tiles, or a narrow-row matrix's block of rows
        const double rows = t.kind == T_SROWS ? double(srows_count(t.b)) : double(t.b);
        return rows * m * eb + rows * rr * 8.0 + (t.a == 0 ? m * rr * 12.0 : 0.0);
      }
      case K_PWIDE: {  // a column block of its rows and its shares of P
        const double rows = srows_count(t.b), cols = std::min<double>(1024.0, m - 1024.0 * srows_block(t.b));
        return rows * cols * eb + rows * rr * 4.0 + (t.a == 0 ? cols * rr * 12.0 : 0.0);
      }
      case K_PFIN:
        return t.b * rr * 4.0 * (std::ceil(m / 1024.0) + 2.0);
      case K_QSTEP: {
        const double rows = q_chunk_rows(d, t.a).rows;
        const double cols = std::min<double>(d.q_cb, m - double(t.b) * d.q_cb);
        return rows * cols * eb + (t.b == 0 ? rows * rr * 8.0 : 0.0);
      }
      case K_QFIN: {
        const double ne = qfin_entries(d.q_chunks), e0 = double(t.a) * ne;
        return 8.0 * std::max(0.0, std::min<double>(ne, m * rr - e0));
      }
      case K_RECON4:
        if (t.kind == T_FACT) {
          const double rows = odd ? n : m;
          return std::min<double>(d.fact_rows, rows - double(t.a) * d.fact_rows) * rr * 8.0;
        }
        if (t.kind == T_SROWS) {
          const double rows = srows_count(t.b), cols = std::min<double>(1024.0, m - 1024.0 * srows_block(t.b));
          return rows * cols * 4.0 + rows * rr * 4.0 + (t.a == 0 ? cols * rr * 4.0 : 0.0);
        }
        return t.b * m * 4.0 + t.b * rr * 4.0 + (t.a == 0 ? m * rr * 4.0 : 0.0);
      case K_WPSTEP: {
        const double rows = t.b & 0xff, c = (t.b >> 8) - 1;
        const double cw = r < kSplitRank ? kWideChunk : split_part(static_cast<int>(r));
        const bool last = r < kSplitRank && c + 1 == wide_chunks(d.m);
        const double cols = c < 0 ? m : last ? m - c * cw : std::min<double>(cw, m - c * cw);
        return rows * cols * eb + rows * rr * 8.0 + (t.a == 0 ? cols * rr * 8.0 : 0.0);
      }
      case K_WPFIN:
        return t.b * rr * 4.0 * (double(p_parts(d.m, true)) + 2.0);
      case K_WQSTEP: {
        const int32_t pr = part_rows(static_cast<int>(r));
        const int32_t parts = l.variant == kWideFine ? static_cast<int32_t>(cdiv(d.q_rows, pr)) : 1;
        const double r0 = double(t.a / parts) * d.q_rows + double(t.a % parts) * pr;
        const double rows = std::min<double>(parts > 1 ? pr : d.q_rows, n - r0);
        const double cw = double(q_tile_cols);  // a tile's columns
        const double cols = std::min<double>(cw, m - double(t.b) * cw);
        return rows * cols * eb + (t.b == 0 ? rows * rr * 8.0 : 0.0);
      }
      case K_WFACT: {  // from kBlockedRank on a slice's rows are read and copied once, counted on its first part
        const double rows = odd ? n : m;
        if (t.a >> 16) return 0.0;
        return std::min<double>(d.fact_rows, rows - double(t.a & 0xffff) * d.fact_rows) * rr * 8.0;
      }
      case K_WRECON: {
        const double rb = r < kSplitRank ? 32.0 : kSplitRecon;
        const double rows = std::min<double>(rb, n - rb * t.a);
        const double cols = std::min<double>(l.variant, m - double(l.variant) * t.b);
        return rows * cols * 4.0 + (t.b == 0 ? rows * rr * 4.0 : 0.0) + (t.a == 0 ? cols * rr * 4.0 : 0.0);
      }
      case K_APPLY:  // from kApplyMfmaRank on a tile covers one of apply_blocks(r) column blocks
        return (t.b & 0xffff) * rr * 8.0 / apply_blocks(static_cast<int32_t>(r));
      case K_FACT:
        if (t.a >> 16) return 0.0;
        return std::min<double>(d.fact_rows, (l.variant & 1 ? m : n) - double(t.a & 0xffff) * d.fact_rows) * rr *
               (l.variant & kFactFromBuffer ? 8.0 : 4.0);
      case K_EMAT:
        return t.b * m * 8.0;
      case K_GSUM:  // the slices' partials read, the sum written
        return (t.b + 1.0) * kGsumEntries * 8.0;
      case K_DRAW:
        return t.b * rr * 4.0;
      default:
        return 0.0;
    }
  };
  auto family_of = [](int32_t kernel) -> int32_t {
    switch (kernel) {
      case K_PFUSED: case K_PWIDE: case K_PFIN: case K_WPSTEP: case K_WPFIN:
        return 1;  // ACP_KERNEL_P_STEP
      case K_QSTEP: case K_WQSTEP:
        return 2;  // ACP_KERNEL_Q_STEP
      case K_QFIN: return 3;  // ACP_KERNEL_Q_FINISH
      case K_RECON4: case K_WRECON:
        return 4;  // ACP_KERNEL_RECONSTRUCT
      case K_WFACT: return 5;                                              // ACP_KERNEL_ORTH
      case K_APPLY: case K_FACT: case K_CHOL: case K_GSUM: case K_DRAW: return 5;  // ACP_KERNEL_ORTH
      default: return 0;  // K_VEC (raw-vector launches of their own) and K_EMAT: no family
    }
  };
  auto annotate = [&](std::vector<Launch>& list, bool odd) {
    for (Launch& l : list) {
      l.family = family_of(l.kernel);
      l.alg_bytes = 0.0;
      for (int32_t i = 0; i < l.ntiles; ++i) l.alg_bytes += tile_bytes(l, plan.tiles[l.tile_off + i], odd);
    }
  };
  for (BucketPlan& bk : plan.buckets) {
    annotate(bk.compress[0], false);
    for (auto* lists : {bk.coarse, bk.fine}) {
      annotate(lists[0], false);
      annotate(lists[1], true);
    }
    for (auto& lists : bk.recon) {
      annotate(lists[0], false);
      annotate(lists[1], true);
    }
    annotate(bk.compress[1], true);
    annotate(bk.decompress[0], false);
    annotate(bk.decompress[1], true);
    annotate(bk.emat, false);
    annotate(bk.draw[0], false);
    annotate(bk.draw[1], true);
    annotate(bk.psgd_fact, false);
  }
  annotate(plan.gram_init, false);

  // ---- launches over whole groups of buckets: every bucket's launches of one kind merged into
  // one, in the dependency order the per-bucket lists already follow
  auto order_of = [](const Launch& l) -> int32_t {
    switch (l.kernel) {
      case K_DRAW: return -3;
      case K_FACT: return -2;
      case K_APPLY: return 0;
      case K_PFUSED: return (l.variant & kEightWaves) ? 8 : (l.variant & kThreeWaves) ? 7 : 1 + (l.variant & ~kRaggedRows);  // 2..8
      case K_PWIDE: return 10;
      case K_PFIN: return 11;
      case K_WPSTEP: return 12;
      case K_WPFIN: return 13;
      case K_WQSTEP: return 22;
      case K_WFACT: return 40;
      case K_QSTEP: return 20;
      case K_QFIN: return 23;
      case K_RECON4: return 31;
      case K_GSUM: return 41;
      case K_WRECON: return 42;
      case K_CHOL: return 43;
      case K_VEC: return 50;
      default: return 60;
    }
  };
  auto merge = [&](int32_t b0, int32_t b1, auto get, bool odd) {
    std::vector<Launch> all;
    for (int32_t b = b0; b < b1; ++b)
      for (const Launch& l : get(plan.buckets[b])) all.push_back(l);
    // a launch with some ragged rows takes the group's others of its class along: one launch per class
    for (const Launch& x : all)
      for (Launch& y : all)
        if (x.kernel == K_PFUSED && y.kernel == K_PFUSED && y.variant == (x.variant & ~kRaggedRows)) y.variant = x.variant;
    // sorted by kind, then variant: every (kernel, variant) of the group becomes one launch
    std::stable_sort(all.begin(), all.end(), [&](const Launch& x, const Launch& y) {
      return order_of(x) != order_of(y) ? order_of(x) < order_of(y) : x.variant < y.variant;
    });
    std::vector<Launch> out;
    for (size_t i = 0; i < all.size();) {
      size_t j = i;
      Launch m = all[i];
      m.tile_off = static_cast<int64_t>(plan.tiles.size());
      m.ntiles = 0;
      m.alg_bytes = 0.0;
      // the launch's tiles, longest first so that no long tile starts last; factor tiles
      // (short in bytes but a serial Gram / Cholesky) lead
      std::vector<std::pair<double, Tile>> ts;
      while (j < all.size() && all[j].kernel == all[i].kernel && all[j].variant == all[i].variant) {
        for (int32_t k = 0; k < all[j].ntiles; ++k) {
          const Tile tc = plan.tiles[all[j].tile_off + k];
          const double w = tc.kind == T_FACT ? 1e30 : tile_bytes(all[j], tc, odd);
          ts.emplace_back(w, tc);
        }
        m.ntiles += all[j].ntiles;
        m.alg_bytes += all[j].alg_bytes;
        ++j;
      }
      std::stable_sort(ts.begin(), ts.end(),
                       [](const std::pair<double, Tile>& x, const std::pair<double, Tile>& y) {
                         return x.first > y.first;
                       });
      for (const auto& p : ts) plan.tiles.push_back(p.second);
      out.push_back(m);
      i = j;
    }
    return out;
  };
  {
    const int32_t nb = static_cast<int32_t>(plan.buckets.size());
    for (int32_t b0 = 0; b0 < nb; b0 += kMaxGroup) {
      const int32_t b1 = std::min(nb, b0 + kMaxGroup);
      std::array<std::vector<Launch>, 2> gc, gd;
      for (int32_t par = 0; par < 2; ++par) {
        // ranks 8 and up: the whole group's tiles decide whether its sums are split into parts and
        // how many columns its decompress tiles take
        int64_t nt = 0, nr = 0;
        for (int32_t b = b0; b < b1; ++b) nt += main_tiles(plan.buckets[b].coarse[par]), nr += recon_tiles(plan.buckets[b]);
        const bool fine = nt < full_tiles;
        if (wide)
          for (int32_t b = b0; b < b1; ++b) uses_form(plan.buckets[b], par, fine);
        const int32_t rw = nr < kWideRFull ? 1 : 0;
        gc[par] = merge(b0, b1, [par, wide, fine](const BucketPlan& bk) -> const std::vector<Launch>& {
          return !wide ? bk.compress[par] : fine ? bk.fine[par] : bk.coarse[par];
        }, par == 1);
        gd[par] = merge(b0, b1, [par, wide, rw](const BucketPlan& bk) -> const std::vector<Launch>& {
          return !wide ? bk.decompress[par] : bk.recon[rw][par];
        }, par == 1);
      }
      plan.group_compress.push_back(gc);
      plan.group_decompress.push_back(gd);
      std::array<std::vector<Launch>, 2> gw;
      for (int32_t par = 0; par < 2; ++par)
        gw[par] = merge(b0, b1, [par](const BucketPlan& bk) -> const std::vector<Launch>& { return bk.draw[par]; }, par == 1);
      plan.group_draw.push_back(gw);
      plan.group_psgd_fact.push_back(
          merge(b0, b1, [](const BucketPlan& bk) -> const std::vector<Launch>& { return bk.psgd_fact; }, false));
    }
  }

  // ---- partial products: every compress list of a matrix, of its bucket's calls and of the group's,
  // uses the same place
  int64_t qpart = 0;
  for (BucketPlan& bk : plan.buckets) {
    bk.qpart_base = qpart;
    for (int32_t mi : bk.mats) {
      MatDesc& d = plan.mats[mi];
      d.qpart = qpart;
      // up to rank 4 a wide row's shares of P take less than its Q-step partials
      const int64_t floats = wide ? need[mi] : int64_t(d.q_chunks) * align_up(d.m, d.q_cb) * r;
      qpart += align_up(floats, kSlotAlign);
    }
    bk.qpart_floats = qpart - bk.qpart_base;
  }

  // ---- region offsets (bytes)
  auto a256 = [](int64_t x) { return align_up(x, 256); };
  plan.e_floats = e_floats;
  plan.fac_floats = fac_floats;
  plan.w_doubles = static_cast<int64_t>(plan.mats.size()) * r * r;
  plan.gpart_doubles = gpart;
  plan.qpart_floats = qpart;
  int64_t off = 0;
  plan.off_e = off;     off = a256(off + e_floats * 4);
  plan.off_fac = off;   off = a256(off + fac_floats * 4);
  plan.off_w = off;     off = a256(off + plan.w_doubles * 8);
  plan.off_gpart = off; off = a256(off + gpart * 8);
  plan.off_qpart = off; off = a256(off + qpart * 4);
  plan.off_mats = off;  off = a256(off + static_cast<int64_t>(plan.mats.size() * sizeof(MatDesc)));
  plan.off_vecs = off;  off = a256(off + static_cast<int64_t>(plan.vecs.size() * sizeof(VecDesc)));
  plan.off_tiles = off; off = a256(off + static_cast<int64_t>(plan.tiles.size() * sizeof(Tile)));
  plan.total_bytes = std::max<int64_t>(off, 256);
  return "";
}

}  // namespace acp
