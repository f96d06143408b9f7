// Internal descriptors shared by the host planner (HIP-free) and the gfx950 kernels.
//
// Device state block (one per context, allocated by the caller), regions in order, each
// 256-byte aligned:
//   E arena   fp32, one slot per gradient-bucket element (vector slots unused); the E of a
//             matrix sits at its bucket's E base + its offset in the gradient bucket.  After
//             a Q-step it holds F = M' and E = F - P_hat Q_loc^T is implied (deferred).  After
//             a P-step of rank >= 8, or of rows longer than kFusedCols, it holds X = M' and
//             E = X - P_loc Q_hat^T is implied (P-deferred); after another P-step it holds E
//             itself.
//   factors   fp32 per compressed matrix: P (n x r), Ph (n x r), Pl (n x r), Q (m x r),
//             Qh (m x r), Ql (m x r), all row-major.  P / Q hold the aggregated factor of
//             the last step that produced it, Ph / Qh the orthogonalised factors, Pl / Ql the
//             local factor of the last P- / Q-step.
//   W         fp64 r x r per matrix: the upper-triangular map with orth(X) = X W for the
//             factor that the next step orthogonalises.
//   gpart     fp64 Gram partial sums, r x r per slice of factor rows (factors of more than one
//             slice only).
//   qpart     fp32 partial products of a compress call, dead after it: of a Q-step, per row chunk
//             (or, in lists that split the chunks, per part) m_pad x r; of a P-step that splits
//             rows, per column block, chunk or part n x r.
//   tables    MatDesc[], VecDesc[], Tile[] for every launch.
// No kernel communicates across workgroups: every reduction that spans workgroups is
// finished by a later kernel in the same stream.
#pragma once

#include <cstdint>

namespace acp {

constexpr int kBlock = 256;       // threads per workgroup (4 waves of 64)
constexpr int kWave = 64;
constexpr double kTau = 1e-4;     // rank-deficiency threshold of orth()
constexpr int kMaxTileRows = 256; // rows per tile of the low-rank row kernels (factor rows in LDS)
// K_QFIN entries (e = column * r + rank, over the whole matrix) per tile: one thread per entry
// for up to 8 row chunks, 4 threads for up to 32, 8 for up to 64 (so that no thread adds more
// than 8 chunks, all requested at once), 16 threads beyond
constexpr int qfin_entries(int32_t q_chunks) {
  return q_chunks <= 8 ? 1024 : (q_chunks <= 32 ? 64 : (q_chunks <= 64 ? 32 : 16));
}
constexpr int64_t kMaxCols = int64_t(1) << 24;  // columns of a compressed matrix, at most
constexpr int kFusedCols = 5120; // longest row of the one-pass P-step up to rank 4 (k_pfused)
constexpr int kReconRows = 4;   // rows per tile of the decompress up to rank 4
// rows a P-step workgroup of column class S handles at a time, up to rank 4: as many as the
// registers hold beside the class's factor rows (4 S r floats each of Qh and Q_loc)
constexpr int pstep_rows(int r, int S) { return S == 1 ? 8 : S == 2 && r <= 2 ? 4 : S <= 4 ? 2 : r <= 2 ? 2 : 1; }
constexpr int kQRows = 256;       // rows per Q-step row chunk (at most; the chunk's Ph rows sit in LDS)
// Size of the static device array that holds one bucket's Q-step partials for the compress entry
// point that allocates nothing (acp_compress_noalloc); a bucket that needs more is refused.
constexpr int64_t kScratchBytes = int64_t(32) << 20;

struct MatDesc {
  int64_t grad_off;   // offset of the matrix in its gradient bucket (floats)
  int64_t e_off;      // offset of its E slot in the E arena (floats)
  int64_t fac_off_p;  // offset in the P-step factor buffer
  int64_t fac_off_q;  // offset in the Q-step factor buffer
  int64_t p_slot, q_slot, ph_slot, qh_slot, ql_slot, pl_slot;  // float offsets in the factor region
  int64_t w_slot;     // double offset in the W region
  int64_t gpart;      // double offset in the Gram-partial region
  int64_t qpart;      // float offset in the partial-product region
  int32_t n, m;
  int32_t q_rows;     // rows per Q-step row chunk
  int32_t q_chunks;   // number of Q-step row chunks
  int32_t q_cb;       // Q-step column-block width
  int32_t fact_rows;  // factor rows per Gram slice
  int32_t scls;       // column class S up to rank 4 (64 S float4 groups per wave; 0: narrow rows)
  int32_t bucket;     // bucket index
  int32_t fact_slices_p, fact_slices_q;  // Gram slices of the P / Q factor rows
  int32_t q_grp;      // Q-step row chunks whose rows interleave (see q_chunk_rows)
  int32_t tid;        // registration index of the tensor (keys the no-reuse draws)
  int32_t xhold;      // a P-step leaves X in the arena (rank >= 8, rows longer than kFusedCols)
};

// the planner (host compiler) and the kernels (hipcc) share the chunk geometry below
#ifdef __HIPCC__
#define ACP_HOST_DEVICE __host__ __device__
#else
#define ACP_HOST_DEVICE
#endif

// Rows of Q-step row chunk c: chunks go in groups of q_grp that share q_grp * q_rows rows (the
// last group: its rows over q_rows, rounded up), chunk x of a group of g taking rows
// x, x + g, x + 2g, ... of it.  q_grp = 1: chunk c is rows [c q_rows, (c + 1) q_rows).
struct ChunkRows {
  int64_t first;
  int32_t stride, rows;
};
ACP_HOST_DEVICE inline ChunkRows q_chunk_rows(const MatDesc& d, int64_t c) {
  const int64_t gi = c / d.q_grp;
  const int64_t span = int64_t(d.q_grp) * d.q_rows;
  const int64_t base = gi * span;
  const int64_t rem = (d.n - base) < span ? (d.n - base) : span;
  const int64_t g = (rem + d.q_rows - 1) / d.q_rows;
  const int64_t x = c - gi * d.q_grp;
  return ChunkRows{base + x, static_cast<int32_t>(g), static_cast<int32_t>((rem - x + g - 1) / g)};
}

struct VecDesc {
  int64_t grad_off, fac_off_p, fac_off_q, numel;
  int64_t e_off;      // its slot in the E arena (Power-SGD's image of M' holds the raw vector there)
  int32_t bucket, pad;
};

enum TileKind : int32_t { T_ROWS = 0, T_FACT = 1, T_VEC = 2, T_QTILE = 3, T_SROWS = 4 };

// kind T_ROWS : idx = matrix, a = first row, b = row count (K_APPLY from kApplyMfmaRank on: + 65536 x
//               the 64-column block of Xh)
// kind T_SROWS: idx = matrix, a = first row, b = srows_pack(cb, stride, count): columns
//               [1024 cb, 1024 cb + 1024) of rows a + k stride, k < count (k_pfused: all columns)
// kind T_FACT : idx = matrix, a = slice (+ 65536 x part of the Gram blocks from kBlockedRank
//               on: gram_parts(r) parts), b = slice count; K_GSUM: a = entry block of
//               kGsumEntries, b = slice count
// kind T_VEC  : idx = vector, a = first element, b = element count
// kind T_QTILE: idx = matrix, a = row chunk (K_QSTEP) or entry block (K_QFIN), b = column block;
// K_DRAW      : T_ROWS, idx = matrix, a = first factor row, b = row count
struct Tile {
  int32_t kind, idx, a, b;
};

// T_SROWS: 15 bits of column block (kMaxCols / 1024 = 2^14 of them), 4 of stride (at most 8), 9 of
// row count (at most kMaxTileRows)
constexpr int32_t srows_pack(int64_t cb, int64_t stride, int64_t count) {
  return static_cast<int32_t>(cb | (stride << 15) | (count << 19));
}
constexpr int32_t srows_block(int32_t b) { return b & 0x7fff; }
constexpr int32_t srows_stride(int32_t b) { return (b >> 15) & 0xf; }
constexpr int32_t srows_count(int32_t b) { return b >> 19; }

enum KernelId : int32_t {
  K_APPLY = 0,   // Xh = X W (orthogonalise the reused factor), ranks >= 8
  K_PFUSED,      // P-step, r <= 4, one pass: Qh = Q W, P = M' Qh, E = M' - P Qh^T, vectors packed
  K_PWIDE,       // P-step, r <= 4, rows longer than kFusedCols: X = M' written, shares of P
  K_PFIN,        // P-step, r <= 4: P = sum of K_PWIDE's shares -> factor buffer and Pl
  K_QSTEP,       // Q-step, r <= 4: F = M' written back, per-chunk partials of M'^T Ph, vectors packed
                 // (variant 1: the rows K_PWIDE takes)
  K_QFIN,        // Q-step: Q_loc = sum of the chunk partials -> factor buffer and Ql
  K_RECON4,      // decompress, r <= 4: M_hat = P Q^T / p; factor tiles; vectors / p
  K_FACT,        // factor tiles alone: Gram -> W (after bind / restore)
  K_CHOL,        // sum of a factor's Gram partials (more than one slice) -> W
  K_EMAT,        // materialise E into a bucket-shaped buffer
  K_VEC,         // pack raw vectors only
  K_WPSTEP,      // P-step, ranks >= 8 (MFMA): X = M' written, P_loc = X Qh per row tile
  K_WQSTEP,      // Q-step, ranks >= 8 (MFMA): F = M' written, per-chunk (or per-part) partials of F^T Ph
  K_WPFIN,       // P-step, ranks >= 8: P_loc = sum of K_WPSTEP's column chunks (from kSplitRank on:
                 // parts) -> factor buffer and Pl
  K_WRECON,      // decompress, ranks >= 8 (MFMA): M_hat = A B^T / p
  K_WFACT,       // decompress, ranks >= 8: factor tiles and vectors / p
  // tile-size classes of the narrow-row tiles up to rank 4 (rows of at most 512 columns: several
  // rows per wave); they run inside the K_PFUSED (S = 1), K_QSTEP and K_RECON4 launches
  K_PNARROW,
  K_QNARROW,
  K_RNARROW,
  K_GSUM,        // from kBlockedRank on: a factor's Gram partials summed (and mirrored) into the first
  K_DRAW,        // no reuse: a fresh standard normal factor into the P (variant 0) or Q (1) slot
};

// Narrow rows (r <= 4, m4 = ceil(m / 4) <= 128 float4 groups): L lanes per row (16, 32 or 64), G
// float4 groups per lane (1 or 2); the variant is (L << 4) | G.
constexpr int32_t narrow_variant(int32_t m4) {
  return m4 <= 16 ? (16 << 4) | 1 : m4 <= 32 ? (32 << 4) | 1 : m4 <= 64 ? (64 << 4) | 1 : (64 << 4) | 2;
}

constexpr int32_t kWideRank = 8;   // ranks at or above this take the K_W* kernels
constexpr int32_t kBlockedRank = 128;  // ranks whose W K_CHOL forms from Gram partials in global memory
// ranks whose products run on the bf16 matrix cores with split operands (split.hip), and whose W is
// factored in 2 x 2 blocks of 128 (kCholBlockRank)
constexpr int32_t kSplitRank = 64;
constexpr int32_t kCholBlockRank = 256;
// rows (P-step) or columns (Q-step) of a tile from kSplitRank on, and rows of a decompress tile
constexpr int split_fix(int r) { return r >= 256 ? 64 : 128; }
constexpr int kSplitRecon = 128;
// From kSplitRank on both steps' sums are those of parts of split_part(r) columns (P-step) or rows
// (Q-step): a part's partial sum then costs 4 r / split_part(r) = 1 byte per element.  Lists with
// fewer tiles than split_full_tiles (twice the workgroups that 256 CUs hold) take one tile per part.
// At rank 256 the sum of the earlier parts would not fit the registers (P-step of BERT-base 0.96 ms
// without it, 1.23 with): there every list takes one tile per part, and a Q-step chunk is one part
constexpr int split_part(int r) { return 4 * r; }
constexpr bool split_nested(int r) { return r < 256; }
constexpr int64_t split_full_tiles(int r) { return r >= 128 ? 512 : 1024; }
constexpr int part_rows(int r) { return r >= kSplitRank ? split_part(r) : 256; }  // of a Q-step part
constexpr int max_parts(int r) { return r == 128 ? 4 : 2; }  // parts of a Q-step chunk, at most (rank 256: one)
// ranks whose orthogonal factor X W is formed on the fp64 matrix cores (one block of
// min(r, 64) columns per tile; below kBlockedRank a factor has one such block)
constexpr int32_t kApplyMfmaRank = 32;
constexpr int32_t apply_blocks(int32_t r) { return r >= 64 ? r / 64 : 1; }  // column blocks of X W
// tiles that share one slice's Gram from kBlockedRank on: the (r / 64)(r / 64 + 1) / 2 blocks of
// 64 x 64 on and above the diagonal, one per wave of a four-wave tile
constexpr int32_t gram_parts(int32_t r) {
  return r >= kBlockedRank ? ((r / 64) * (r / 64 + 1) / 2 + 3) / 4 : 1;
}
constexpr int32_t kGsumEntries = 4096;  // Gram entries per K_GSUM tile
constexpr int kWideBlock = 64;     // threads per wave of K_WPSTEP and K_WQSTEP, ranks 8..32
constexpr int kWideQCols = 32;     // K_WQSTEP column block (one MFMA block)
constexpr int kWidePWaves = 4;     // ranks 8..32: waves of a K_WPSTEP workgroup (adjacent column blocks)
constexpr int kWideQWaves = 4;     // ranks 8..32: waves of a K_WQSTEP workgroup (adjacent column blocks)
constexpr int kWideQRows = 512;    // K_WQSTEP rows per chunk (at most)
// K_WRECON columns per tile (its variant): a list with fewer than kWideRFull tiles of the wider one
// takes the narrower
constexpr int kWideRCols = 1024, kWideRNarrow = 256;
constexpr int64_t kWideRFull = 128;
// K_WPSTEP, ranks 8..32: a row goes in chunks of kWideChunk columns, a tile each, whose sums K_WPFIN
// adds.  A rest of less than half a chunk goes with the chunk before it, and a row of up to one and a
// half chunks is one: the rest's short tile takes a slot for a fraction of a chunk's work, and one
// chunk needs no K_WPFIN (hidden size 1088 at rank 32 bucket by bucket 1911 us per two steps with the
// rest apart, 1764 this way; 1536, 3470 and 3378; two and a half chunks are better cut in three:
// 2560 columns 1555 us, in two 1578)
constexpr int kWideChunk = 1024;
constexpr int32_t wide_chunks(int64_t m) {
  return m <= kWideChunk * 3 / 2 ? 1 : static_cast<int32_t>((m + kWideChunk / 2) / kWideChunk);
}
// Ranks 8..32: a Q-step chunk's sum is that of its parts of kWideSubRows rows, in order; a list with
// fewer than kWideFullTiles tiles (the workgroups that 256 CUs hold, three each, and a third more)
// takes one tile per part (variant kWideFine of K_WQSTEP and K_QFIN)
constexpr int kWideSubRows = part_rows(32);
constexpr int32_t kWideFine = 1;
constexpr int64_t kWideFullTiles = 1024;
constexpr int kDrawRows = 256;     // K_DRAW factor rows per tile
// K_PFUSED variant bits: S = 1 on three waves, for rows of 516 to 768 columns; S = 2 on eight
// waves, for rows of 3076 to 4096 columns
constexpr int32_t kThreeWaves = 32;
constexpr int32_t kEightWaves = 64;
// ... and on four waves with S = 2 to 5: some row length of the launch is not a multiple of four
constexpr int32_t kRaggedRows = 128;
// K_FACT variants: bit 0 = Q (else P); bit 1 (kFactFromBuffer): the factor is read from the
// aggregated factor buffer (src) and copied into its slot, else read from its slot
constexpr int32_t kFactFromBuffer = 2;

struct Launch {
  int32_t kernel;
  int32_t variant;   // kernel-specific: column class S (K_PFUSED), rows of K_PWIDE (K_QSTEP),
                     // factor P=0 / Q=1 (K_APPLY, K_FACT)
  int64_t tile_off;  // first tile in the tile table
  int32_t ntiles;
  int32_t family;    // ACP_KERNEL_* family (host-side profiling)
  double alg_bytes;  // algorithmic bytes of the launch (host-side profiling)
};


// Buckets per launch: a launch covers the buckets [base, base + kMaxGroup) at most; their
// buffer addresses travel in the kernel arguments.
constexpr int kMaxGroup = 64;

// Kernel arguments (passed by value).
struct KArgs {
  const float* src[kMaxGroup];  // per bucket: gradient bucket (compress) or aggregated factor
                                // buffer (decompress)
  float* dst[kMaxGroup];        // per bucket: factor buffer (compress), output bucket
                                // (decompress, E export)
  float* e;             // E arena
  float* fac;           // factor region
  double* w;            // W region
  double* gpart;        // Gram partials
  float* qpart;         // partial products
  const MatDesc* mats;
  const VecDesc* vecs;
  const Tile* tiles;    // this launch's tiles
  uint64_t deferred;    // bit i: the E arena of bucket base + i holds F (E implied)
  uint64_t deferred_p;  // bit i: the E arena of bucket base + i holds X (E implied)
  int32_t base;         // bucket of src[0] / dst[0]
  int32_t ntiles;
  int32_t variant;
  int32_t ef;           // error feedback on
  float inv_p;          // 1 / world size
  int32_t parity;       // 1 on odd (P-) steps, 0 on even (Q-) steps
  int32_t copy_only;    // factor tiles copy the aggregated factor but build no W (Power-SGD)
  int32_t image;        // P-step of Power-SGD: P = M' Q with Q as it is, M' left in the E arena
  uint64_t seed;        // K_DRAW: the context's seed
  int64_t step;         // K_DRAW: the step whose factors are drawn
};

}  // namespace acp
