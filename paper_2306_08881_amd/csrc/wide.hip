// gfx950 MFMA kernels of the ACP-SGD compressor for ranks 8 to 32 (arXiv 2306.08881,
// Algorithm 2).  At these ranks a step costs 2r multiply-adds per gradient element against
// 12 bytes of HBM traffic, more than the fp32 vector units sustain at full bandwidth, so the
// rank-r contractions run on v_mfma_f32_32x32x2f32.
//
// Both compress steps apply the error-feedback residual of the previous step in deferred
// form and write M' back, so neither waits for its own reduction before writing:
//   P-step:  X = M + E_arena (- Ph Ql^T when the arena holds F), X written to the arena,
//            P_loc = X Qh;  afterwards E = X - P_loc Qh^T is implied (the first half of a
//            Power-SGD step takes Q itself for Qh and keeps X as the second half's source).
//   Q-step:  F = M + E_arena (- Pl Qh^T when the arena holds X), F written to the arena,
//            Q_loc = F^T Ph; afterwards E = F - Ph Q_loc^T is implied.
// Each is one rank-r correction and one rank-r product per element.  From rank 64 on the kernels of
// split.hip take the steps.
//
// MFMA layout (one wave): D (32 x 32) += A (32 x 2) B (2 x 32).  Lane l supplies
// A[l % 32][l / 32] and B[l / 32][l % 32]; register v of lane l holds D[drow(v, l / 32)][l % 32].
// The K index of a step may map to any pair of rank (or row, column) indices as long as A and
// B use the same pair; the kernels use rank (r / 2) h + s on half h at step s, and the row or
// column drow(v, h) at step v, which lets the output of one MFMA feed the next directly.
#include "device.hpp"

#include <type_traits>

namespace acp {

hipError_t launch_split(const Launch& l, int32_t rank, const KArgs& args, hipStream_t s);

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

__device__ inline v16f mfma(float a, float b, const v16f& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ inline int drow(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }
__device__ inline v16f zero16() {
  v16f z;
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = 0.f;
  return z;
}
__device__ inline uint32_t u32(int64_t x) { return static_cast<uint32_t>(x); }

// KH consecutive floats of a factor row starting at byte offset off (kOut: zeros).
template <int KH>
__device__ inline void load_run(Rsrc r, uint32_t off, float* out) {
#pragma unroll
  for (int i = 0; i < KH / 4; ++i) {
    const float4 f = bld4(r, off == kOut ? kOut : off + 16u * i);
    out[4 * i + 0] = f.x;
    out[4 * i + 1] = f.y;
    out[4 * i + 2] = f.z;
    out[4 * i + 3] = f.w;
  }
}

// P-step over a tile of at most 32 rows and all m columns on four waves: wave w walks the
// 32-column blocks w, w + 4, ... in step with the others, so that the workgroup reads 512
// contiguous bytes of each of its rows at a time.  Per step of 128 columns, wave w loads M and E
// for rows 8 w ... 8 w + 7 as 16-byte vectors (lane l: row 8 w + 2 i + l / 32, columns
// 4 (l % 32) ... + 3; one instruction reads 512 contiguous bytes of two rows), puts M + E in a
// 32 x 128 LDS tile, and after a barrier takes its own block back with lane l holding column
// c0 + l % 32 of rows drow(v, l / 32).  It applies the correction (F form) as an MFMA with D
// indexed (row, column).  The product P += X Qh reduces over columns, so it needs the row on the
// lane: X goes through the wave's padded 32 x 33 LDS tile (two of them, alternating) and comes
// back with lane l holding row l % 32 and columns drow(v, l / 32), the A operand; the
// accumulator lane l holds the wave's share of P[r0 + drow(v, l / 32)][l % 32].  After the
// barrier that publishes those tiles, every wave also reads its rows of X in the load layout
// from the four waves' tiles and stores them as 16-byte vectors.  The four shares of P are added
// in wave order through LDS at the end.  The next step's M and E are requested before the
// current block's MFMAs, its factor rows after them.
// A longer row is cut into chunks of kWideChunk columns (wide_chunks; t.b >> 8 is the chunk + 1),
// whose sums of P go to the partial region for k_wpfin: a row walked whole is a serial chain of
// steps of 2.2 us of latency each, and a bucket of 25 MiB at rank 32 has about 200 row tiles for
// the GPU's 768 workgroup slots (BERT-base, rows of 3072 columns: 55 us a bucket, 30 by chunks).
template <int RK>
__global__ __launch_bounds__(kWideBlock * kWidePWaves, 2) void k_wpstep(KArgs a) {
  constexpr int KH = RK / 2;
  constexpr int LD = 33;  // padded LDS row: the transposed reads hit 32 different banks
  constexpr int CS = 32 * kWidePWaves;  // columns per step of the workgroup
  const Tile t = a.tiles[blockIdx.x];
  if (t.kind == T_VEC) {  // a raw vector packed into the factor buffer
    vec_tile(a, t, true);
    return;
  }
  const MatDesc d = a.mats[t.idx];
  const int wave = __builtin_amdgcn_readfirstlane(tid() >> 6);
  const int lane = tid() & 63, h = lane >> 5, li = lane & 31;
  const int64_t m = d.m, r0 = t.a;
  const int rows = t.b & 0xff, chunk = (t.b >> 8) - 1;  // chunk -1: all columns
  const int64_t cbeg = chunk > 0 ? static_cast<int64_t>(chunk) * kWideChunk : 0;
  const int64_t cend = chunk >= 0 && chunk + 1 < wide_chunks(m) ? cbeg + kWideChunk : m;
  const bool fform = deferred_of(a, d.bucket);
  const uint32_t row_bytes = u32(m) * 4u;
  const uint32_t ext = u32(rows) * row_bytes;
  const Rsrc G = tile_rsrc(src_of(a, d.bucket) + d.grad_off + r0 * m, ext);
  const Rsrc E = tile_rsrc(a.e + d.e_off + r0 * m, a.ef ? ext : 0u);
  const Rsrc Phr = tile_rsrc(a.fac + d.ph_slot + r0 * RK, fform ? u32(rows) * RK * 4u : 0u);
  const Rsrc Qlr = tile_rsrc(a.fac + d.ql_slot, fform ? u32(m) * RK * 4u : 0u);
  const Rsrc Qhr = tile_rsrc(a.fac + (a.image ? d.q_slot : d.qh_slot), u32(m) * RK * 4u);
  static_assert(RK < kSplitRank, "from kSplitRank on the rank-split kernel takes the P-step");
  float pa[KH];  // correction A operand: -Ph[r0 + l % 32][KH h + s]
  load_run<KH>(Phr, u32(li * RK + KH * h) * 4u, pa);
#pragma unroll
  for (int s = 0; s < KH; ++s) pa[s] = -pa[s];

  // M and E of the step from column cs: the lane's four rows 8 w + 2 i + h, columns cs + 4 li ...
  // (past cend: zeros); as 16-byte vectors, which need 4-byte alignment only, except where the
  // last of them would reach into the next row: that step moves float by float
  const bool m4 = (m & 3) == 0;
  auto whole = [&](int64_t cs) { return m4 || cs + CS <= m; };
  const int vr = 8 * wave + h, vc = 4 * li;
  auto load_block = [&](int64_t cs, float4* g, float4* e) {
    const int64_t col = cs < cend ? cs + vc : m;
    const bool vec = whole(cs);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t o = u32(vr + 2 * i) * row_bytes + u32(col) * 4u;
      if (vec) {
        g[i] = bld4_nt(G, col < m ? o : kOut);
        e[i] = bld4_nt(E, col < m ? o : kOut);
      } else {
        g[i] = make_float4(bld1_nt(G, col < m ? o : kOut), bld1_nt(G, col + 1 < m ? o + 4u : kOut),
                           bld1_nt(G, col + 2 < m ? o + 8u : kOut), bld1_nt(G, col + 3 < m ? o + 12u : kOut));
        e[i] = make_float4(bld1_nt(E, col < m ? o : kOut), bld1_nt(E, col + 1 < m ? o + 4u : kOut),
                           bld1_nt(E, col + 2 < m ? o + 8u : kOut), bld1_nt(E, col + 3 < m ? o + 12u : kOut));
      }
    }
  };
  // the block's factor operands: Ql rows (correction B) and Qh rows (product B)
  auto load_ops = [&](int64_t c0, float* qa, float* qb) {
    const int64_t qcol = c0 + li;
    if (fform) load_run<KH>(Qlr, qcol < m ? u32(qcol * RK + KH * h) * 4u : kOut, qa);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t col = c0 + drow(v, h);
      qb[v] = bld1(Qhr, (col < m && li < RK) ? u32(col * RK + li) * 4u : kOut);
    }
  };
  // the waves' transposing tiles, two each; a wave's pair starts one float past the previous
  // wave's, so that the row reads of the X stores (four waves' tiles at once) spread over the banks
  constexpr int XW = 2 * 32 * LD + 1;
  __shared__ float xt[kWidePWaves * XW];
  auto xtile = [&](int w, int b) { return xt + w * XW + b * 32 * LD; };
  constexpr int SP = 32 * kWidePWaves + 4;  // staging tile row pitch (floats, 16-byte aligned rows)
  __shared__ __attribute__((aligned(16))) float st[32 * SP];
  float4 g[4], e[4];
  float qa[KH], qb[16];
  load_block(cbeg, g, e);
  load_ops(cbeg + 32 * wave, qa, qb);

  v16f p = zero16();
  int buf = 0;
  // every wave takes the same number of steps (blocks past m: zero loads, dropped stores)
  for (int64_t cs = cbeg; cs < cend; cs += CS, buf ^= 1) {
    const int64_t c0 = cs + 32 * wave;
    // M + E to the staging tile (the previous step's readers have passed its second barrier)
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<float4*>(st + (vr + 2 * i) * SP + vc) = g[i] + e[i];
    load_block(cs + CS, g, e);  // next step (past m: zeros, no traffic)
    __syncthreads();
    v16f x;
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = st[drow(v, h) * SP + 32 * wave + li];
    if (fform) {  // X -= Ph Ql^T: A = -Ph (row, rank), B = Ql^T (rank, column)
#pragma unroll
      for (int s = 0; s < KH; ++s) x = mfma(pa[s], qa[s], x);
    }
    float* tl = xtile(wave, buf);
#pragma unroll
    for (int v = 0; v < 16; ++v) tl[drow(v, h) * LD + li] = x[v];
    __syncthreads();
    // X to the arena in the load layout: the lane's rows 8 w + 2 i + h, columns cs + 4 li ...,
    // from the transposing tile of the wave that formed them (as 16-byte vectors when aligned)
    {
      const float* xs = xtile(li >> 3, buf) + (vc & 31);
      const int64_t col = cs + vc;
      const bool vec = whole(cs);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = vr + 2 * i;
        const float4 xv = make_float4(xs[row * LD], xs[row * LD + 1], xs[row * LD + 2], xs[row * LD + 3]);
        const uint32_t o = u32(row) * row_bytes + u32(col) * 4u;
        if (vec) {
          bst4_nt(E, col < m ? o : kOut, xv);
        } else {
          bst1_nt(E, col < m ? o : kOut, xv.x);
          bst1_nt(E, col + 1 < m ? o + 4u : kOut, xv.y);
          bst1_nt(E, col + 2 < m ? o + 8u : kOut, xv.z);
          bst1_nt(E, col + 3 < m ? o + 12u : kOut, xv.w);
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {  // P += X Qh: A = X (row, column), B = Qh (column, rank)
      p = mfma(tl[li * LD + drow(v, h)], qb[v], p);
    }
    load_ops(c0 + CS, qa, qb);
  }

  // the waves' shares of P, added in wave order: entry (v, lane)
  float* red = xt;  // kWidePWaves x 1024 floats (the transposing tiles are free)
  float* P = chunk < 0 ? dst_of(a, d.bucket) + d.fac_off_p : a.qpart + d.qpart + static_cast<int64_t>(chunk) * d.n * RK;
  float* Pl = a.fac + d.pl_slot;
  __syncthreads();  // the last products have read the tiles
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave * 1024 + v * 64 + lane] = p[v];
  __syncthreads();
  for (int en = tid(); en < 1024; en += kWideBlock * kWidePWaves) {
    float sum = red[en];
#pragma unroll
    for (int q = 1; q < kWidePWaves; ++q) sum += red[q * 1024 + en];
    const int v = en >> 6, ln = en & 63;
    const int row = drow(v, ln >> 5), rank = ln & 31;
    if (rank < RK && row < rows) {
      P[(r0 + row) * RK + rank] = sum;
      if (chunk < 0) Pl[(r0 + row) * RK + rank] = sum;
    }
  }
}

// P of the rows whose P-step ran by column chunks (from kSplitRank on: parts): their sums added in order, to the factor
// buffer and the P_loc slot.  Tile: rows [t.a, t.a + t.b), one thread per four ranks of a row.
template <int RK>
__global__ __launch_bounds__(kBlock) void k_wpfin(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  if (tid() >= t.b * (RK / 4)) return;
  const int64_t e = static_cast<int64_t>(t.a) * RK + tid() * 4;
  const int nc = RK < kSplitRank ? wide_chunks(d.m) : (d.m + split_part(RK) - 1) / split_part(RK);
  const int64_t stride = static_cast<int64_t>(d.n) * RK;  // one chunk's sums
  const float* part = a.qpart + d.qpart + e;
  constexpr int U = 4;  // sums requested at a time
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int c = 0; c < nc; c += U) {
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const float4*>(part + (c + u < nc ? c + u : nc - 1) * stride);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u < nc) s = s + v[u];
  }
  float* P = dst_of(a, d.bucket) + d.fac_off_p + e;
  P[0] = s.x;
  P[1] = s.y;
  P[2] = s.z;
  P[3] = s.w;
  *reinterpret_cast<float4*>(a.fac + d.pl_slot + e) = s;
}

// Q-step over a tile (row chunk t.a of q_rows rows, column blocks 4 t.b ... 4 t.b + 3 of 32
// columns), four waves per workgroup: wave w takes column block 4 t.b + w (columns c0 ...
// c0 + 31) and the waves walk the chunk's 32-row blocks in step, so that the workgroup reads 512
// contiguous bytes of each row at a time.  Per 32-row block, wave w loads M and E for rows
// 8 w ... 8 w + 7 of the workgroup's 128 columns as 16-byte vectors (as the P-step does), puts
// M + E in a 32 x 128 LDS tile and after a barrier takes its own block back with lane l holding
// column c0 + l % 32 of rows drow(v, l / 32).  The block's Pl and Ph rows are loaded once for
// the workgroup into a factor tile beside it.  The correction (X form) is an MFMA with D indexed
// (row, column); F then is the A operand of Q += F^T Ph with the rows as K, and goes back into
// the wave's block of the tile, from which every wave stores its rows of F as 16-byte vectors
// after the block's last barrier.  Lane l's partial Q of column c0 + drow(v, l / 32), rank
// l % 32, goes to the chunk's partial block for K_QFIN.  A chunk's sum is that of its parts of
// kWideSubRows rows, in order; a launch with too few tiles (kWideFine, as in the P-step) takes one
// tile per part (t.a = chunk * parts + part) and leaves their addition to K_QFIN.
template <int RK>
__global__ __launch_bounds__(kWideBlock * kWideQWaves, 2) void k_wqstep(KArgs a) {
  constexpr int KH = RK / 2;
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  const int wave = __builtin_amdgcn_readfirstlane(tid() >> 6);
  const int lane = tid() & 63, h = lane >> 5, li = lane & 31;
  const int64_t n = d.n, m = d.m;
  const bool fine = a.variant == kWideFine;
  const int parts = (d.q_rows + kWideSubRows - 1) / kWideSubRows;
  const int64_t r0 = fine ? static_cast<int64_t>(t.a / parts) * d.q_rows + t.a % parts * kWideSubRows
                          : static_cast<int64_t>(t.a) * d.q_rows;
  const int64_t cap = fine ? (t.a % parts + 1 < parts ? kWideSubRows : d.q_rows - (parts - 1) * kWideSubRows) : d.q_rows;
  const int rows = static_cast<int>((r0 + cap < n) ? cap : n - r0);
  const int64_t c0 = (static_cast<int64_t>(t.b) * kWideQWaves + wave) * d.q_cb;
  // valid columns of the wave's block: none for a block past m (its wave loads zeros, stores
  // nothing and keeps the others' barriers)
  const int64_t w = (m - c0) < 32 ? ((m - c0) > 0 ? (m - c0) : 0) : 32;
  const bool xform = deferred_p_of(a, d);
  const uint32_t row_bytes = u32(m) * 4u;
  // the workgroup's columns ct ... ct + wt - 1
  const int64_t ct = static_cast<int64_t>(t.b) * kWideQWaves * d.q_cb;
  const int64_t wt = (m - ct) < 32 * kWideQWaves ? m - ct : 32 * kWideQWaves;
  const uint32_t extw = u32(rows - 1) * row_bytes + u32(wt) * 4u;
  const float* gbase = src_of(a, d.bucket) + d.grad_off + r0 * m + ct;
  const float* ebase = a.e + d.e_off + r0 * m + ct;
  const Rsrc Gw = tile_rsrc(gbase, extw);
  const Rsrc Ew = tile_rsrc(ebase, a.ef ? extw : 0u);
  const bool vec = (m & 3) == 0 || wt == 32 * kWideQWaves;  // no 16-byte word reaches into the next row
  const Rsrc Qhr = tile_rsrc(a.fac + d.qh_slot + c0 * RK, xform ? u32(w) * RK * 4u : 0u);
  const Rsrc Plr = tile_rsrc(a.fac + d.pl_slot + r0 * RK, xform ? u32(rows) * RK * 4u : 0u);
  const Rsrc Phr = tile_rsrc(a.fac + d.ph_slot + r0 * RK, u32(rows) * RK * 4u);
  static_assert(RK < kSplitRank, "from kSplitRank on the rank-split kernel takes the Q-step");
  float qv[KH];  // correction B operand: Qh[c0 + l % 32][KH h + s]
#pragma unroll
  for (int s = 0; s < KH; ++s) qv[s] = bld1(Qhr, u32(li * RK + KH * h + s) * 4u);

  // M and E of the 32-row block from row rb: the lane's rows rb + 8 w + 2 i + h, columns
  // 4 li ... 4 li + 3 of the workgroup's (past wt or the chunk: zeros); 16-byte vectors (4-byte
  // alignment is enough), except in a last column block of a row length that is not a multiple of
  // four, which moves float by float
  const int vr = 8 * wave + h, vc = 4 * li;
  auto load_block = [&](int rb, float4* g, float4* e) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t o = u32(rb + vr + 2 * i) * row_bytes + u32(vc) * 4u;
      if (vec) {
        g[i] = bld4_nt(Gw, vc < wt ? o : kOut);
        e[i] = bld4_nt(Ew, vc < wt ? o : kOut);
      } else {
        g[i] = make_float4(bld1_nt(Gw, vc < wt ? o : kOut), bld1_nt(Gw, vc + 1 < wt ? o + 4u : kOut),
                           bld1_nt(Gw, vc + 2 < wt ? o + 8u : kOut), bld1_nt(Gw, vc + 3 < wt ? o + 12u : kOut));
        e[i] = make_float4(bld1_nt(Ew, vc < wt ? o : kOut), bld1_nt(Ew, vc + 1 < wt ? o + 4u : kOut),
                           bld1_nt(Ew, vc + 2 < wt ? o + 8u : kOut), bld1_nt(Ew, vc + 3 < wt ? o + 12u : kOut));
      }
    }
  };
  // the block's factor rows, Pl (correction A) and Ph (product B): 32 x RK contiguous floats each
  // (factor slots are 256-byte aligned), loaded once for the workgroup, one 16-byte word per
  // thread, into a factor tile beside the staging tile, from which every wave takes its operands
  constexpr int FP = RK + 4;        // factor tile row pitch (floats, 16-byte aligned rows)
  constexpr int FV = 32 * RK / 4;   // 16-byte words per block and factor
  const bool fw = tid() < FV;       // the thread has a word of the block
  const int frow = tid() * 4 / RK, fcol = tid() * 4 % RK;
  auto load_fac = [&](int rb, float4& l, float4& p) {
    const uint32_t o = u32(rb * RK + tid() * 4) * 4u;
    l = bld4(Plr, fw ? o : kOut);  // zeros past the chunk, and without the X form
    p = bld4(Phr, fw ? o : kOut);
  };
  // two staging tiles in turn: block k's F goes back into tile k % 2 and is stored from there
  // after the block's last barrier, while block k + 1 fills the other
  constexpr int SP = 32 * kWideQWaves + 4;  // staging tile row pitch (floats, 16-byte aligned rows)
  __shared__ __attribute__((aligned(16))) float st[2][32 * SP];
  __shared__ __attribute__((aligned(16))) float ft[2][2][32 * FP];  // [tile][Pl, Ph]
  float4 g[4], e[4], fl, fh;
  load_block(0, g, e);
  load_fac(0, fl, fh);
  v16f q = zero16(), tot = zero16();  // the sum of the current part, of the parts before it
  int buf = 0;
  for (int rb = 0; rb < rows; rb += 32, buf ^= 1) {
    float* sb = st[buf];
    float* fpl = ft[buf][0];
    float* fph = ft[buf][1];
    // M + E and the factor rows to the tiles (their readers of two blocks ago have passed the
    // last barrier)
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<float4*>(sb + (vr + 2 * i) * SP + vc) = g[i] + e[i];
    if (fw) {
      *reinterpret_cast<float4*>(fpl + frow * FP + fcol) = fl;
      *reinterpret_cast<float4*>(fph + frow * FP + fcol) = fh;
    }
    load_block(rb + 32, g, e);  // next block (past the chunk: zeros, no traffic)
    load_fac(rb + 32, fl, fh);
    __syncthreads();
    v16f x;
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = sb[drow(v, h) * SP + 32 * wave + li];
    if (xform) {  // F -= Pl Qh^T: A = -Pl (row, rank), B = Qh^T (rank, column)
      float pa[KH];  // Pl[rb + l % 32][KH h + s]
#pragma unroll
      for (int s = 0; s < KH; ++s) pa[s] = fpl[li * FP + KH * h + s];
#pragma unroll
      for (int s = 0; s < KH; ++s) x = mfma(-pa[s], qv[s], x);
    }
    // F back into the wave's own block of the tile (only this wave has read it)
#pragma unroll
    for (int v = 0; v < 16; ++v) sb[drow(v, h) * SP + 32 * wave + li] = x[v];
    {  // Q += F^T Ph: A = F^T, B = Ph (lane l: rank l % 32 of rows drow(v, l / 32); zero past r)
      const int rk = li < RK ? li : RK - 1;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float pb = fph[drow(v, h) * FP + rk];
        q = mfma(x[v], li < RK ? pb : 0.f, q);
      }
    }
    __syncthreads();  // the waves stay on the same rows; every block's F is in the tile
    // F to the arena in the load layout, as 16-byte vectors when aligned
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 f = *reinterpret_cast<const float4*>(sb + (vr + 2 * i) * SP + vc);
      const uint32_t o = u32(rb + vr + 2 * i) * row_bytes + u32(vc) * 4u;
      if (vec) {
        bst4_nt(Ew, vc < wt ? o : kOut, f);
      } else {
        bst1_nt(Ew, vc < wt ? o : kOut, f.x);
        bst1_nt(Ew, vc + 1 < wt ? o + 4u : kOut, f.y);
        bst1_nt(Ew, vc + 2 < wt ? o + 8u : kOut, f.z);
        bst1_nt(Ew, vc + 3 < wt ? o + 12u : kOut, f.w);
      }
    }
    if ((rb + 32) % kWideSubRows == 0 && rb + 32 < rows) {  // the part ends and another follows
      tot += q;
      q = zero16();
    }
  }
  if (w == 0) return;  // a block past m has no partials
  q = tot + q;
  const int64_t ncb = (m + d.q_cb - 1) / d.q_cb;
  const int64_t stride = ncb * d.q_cb * RK;  // one row chunk of partials
  float* part = a.qpart + d.qpart + static_cast<int64_t>(t.a) * stride + c0 * RK;
  if (li < RK)
#pragma unroll
    for (int v = 0; v < 16; ++v) part[drow(v, h) * RK + li] = q[v];
}

// Decompress up to rank 32 with four waves per tile (32-row block t.a, group t.b of WC columns):
// at step k the waves compute the 32 x 32 blocks 4k ... 4k + 3 (wave w block 4k + w) and put them
// in an LDS tile of 32 rows x 128 columns; then all 256 threads store that tile with 16-byte
// nontemporal stores, thread t taking the four columns 4 (t % 32) ... of rows t / 32 + 8 i, so
// one store instruction writes 512 contiguous bytes of each of two rows.  Two LDS
// tiles alternate, one barrier per step.  Rows past the tile fall outside the output resource;
// columns past m are masked (the last step of a row length that is not a multiple of four stores
// float by float: its last 16-byte word would reach into the next row).
template <int RK, int WC>
__global__ __launch_bounds__(kBlock) void k_wrecon4w(KArgs a) {
  constexpr int KH = RK / 2;
  constexpr int LP = 132;  // LDS row pitch (floats): rows stay 16-byte aligned for the reads
  const Tile t = a.tiles[blockIdx.x];
  const bool odd = a.parity != 0;
  const MatDesc d = a.mats[t.idx];
  const int wave = __builtin_amdgcn_readfirstlane(tid() >> 6);
  const int lane = tid() & 63, h = lane >> 5, li = lane & 31;
  const int64_t n = d.n, m = d.m;
  const int64_t r0 = static_cast<int64_t>(t.a) * 32;
  const int rows = static_cast<int>((r0 + 32 < n) ? 32 : n - r0);
  const float* agg = src_of(a, d.bucket);
  const float* A = odd ? agg + d.fac_off_p : a.fac + d.ph_slot;
  const float* B = odd ? a.fac + d.qh_slot : agg + d.fac_off_q;
  const Rsrc Ar = tile_rsrc(A + r0 * RK, u32(rows) * RK * 4u);
  const Rsrc Br = tile_rsrc(B, u32(m) * RK * 4u);
  float av[KH];  // A operand: A[r0 + l % 32][KH h + s] / p
  load_run<KH>(Ar, u32(li * RK + KH * h) * 4u, av);
#pragma unroll
  for (int s = 0; s < KH; ++s) av[s] *= a.inv_p;
  float* O = dst_of(a, d.bucket) + d.grad_off + r0 * m;
  const uint32_t row_bytes = u32(m) * 4u;
  const Rsrc Or = tile_rsrc(O, u32(rows) * row_bytes);
  const bool m4 = (m & 3) == 0;
  const int64_t c0 = static_cast<int64_t>(t.b) * WC;
  constexpr int NS = WC / 128;  // steps of four blocks
  auto bcol = [&](int k) { return c0 + k * 128 + wave * 32; };  // the wave's block at step k
  auto boff = [&](int k) { return bcol(k) + li < m ? u32((bcol(k) + li) * RK + KH * h) * 4u : kOut; };
  __shared__ __attribute__((aligned(16))) float tile[2][32 * LP];
  float bv[2][KH];
  load_run<KH>(Br, boff(0), bv[0]);
  const int sc = tid() & 31, sr = tid() >> 5;  // store side: float4 column sc of rows sr + 8 i
  for (int k = 0; k < NS; ++k) {
    const int64_t cs = c0 + k * 128;  // the step's first column
    if (cs >= m) break;
    if (k + 1 < NS) load_run<KH>(Br, boff(k + 1), bv[(k + 1) & 1]);
    v16f o = zero16();
#pragma unroll
    for (int s = 0; s < KH; ++s) o = mfma(av[s], bv[k & 1][s], o);
    float* tl = tile[k & 1];
#pragma unroll
    for (int v = 0; v < 16; ++v) tl[drow(v, h) * LP + wave * 32 + li] = o[v];
    __syncthreads();
    const int64_t col = cs + 4 * sc;
    const bool vec = m4 || cs + 128 <= m;  // no 16-byte word reaches into the next row
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = sr + 8 * i;
      const float4 q = *reinterpret_cast<const float4*>(tl + r * LP + 4 * sc);
      const uint32_t off = u32(r) * row_bytes + u32(col) * 4u;
      if (vec) {
        bst4_nt(Or, col < m ? off : kOut, q);
      } else {
        bst1_nt(Or, col < m ? off : kOut, q.x);
        bst1_nt(Or, col + 1 < m ? off + 4u : kOut, q.y);
        bst1_nt(Or, col + 2 < m ? off + 8u : kOut, q.z);
        bst1_nt(Or, col + 3 < m ? off + 12u : kOut, q.w);
      }
    }
  }
}

// Decompress companions of K_WRECON (whole workgroups): factor tiles keep the aggregated
// factor as the next step's reused factor and build its W; vector tiles unpack sum / p.
template <int RK>
__global__ __launch_bounds__(kBlock) void k_wfact(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const bool odd = a.parity != 0;
  if (t.kind == T_VEC) {
    vec_tile(a, t, false);
    return;
  }
  const MatDesc d = a.mats[t.idx];
  const float* src = src_of(a, d.bucket) + (odd ? d.fac_off_p : d.fac_off_q);
  float* dst = a.fac + (odd ? d.p_slot : d.q_slot);
  fact_tile<RK>(a, t, src, dst, odd ? d.n : d.m);
}

template <int RK>
hipError_t launch_wide_rank(const Launch& l, const KArgs& args, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(l.ntiles));
  if (l.kernel == K_WFACT) {
    hipLaunchKernelGGL(k_wfact<RK>, grid, dim3(kBlock), 0, s, args);
  } else if (l.kernel == K_WPFIN) {
    hipLaunchKernelGGL(k_wpfin<RK>, grid, dim3(kBlock), 0, s, args);
  } else if constexpr (RK < kSplitRank) {
    switch (l.kernel) {
      case K_WPSTEP: hipLaunchKernelGGL(k_wpstep<RK>, grid, dim3(kWideBlock * kWidePWaves), 0, s, args); break;
      case K_WQSTEP: hipLaunchKernelGGL(k_wqstep<RK>, grid, dim3(kWideBlock * kWideQWaves), 0, s, args); break;
      case K_WRECON:
        if (l.variant == kWideRNarrow)
          hipLaunchKernelGGL((k_wrecon4w<RK, kWideRNarrow>), grid, dim3(kBlock), 0, s, args);
        else
          hipLaunchKernelGGL((k_wrecon4w<RK, kWideRCols>), grid, dim3(kBlock), 0, s, args);
        break;
      default: return hipErrorInvalidValue;
    }
  } else {
    return launch_split(l, RK, args, s);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_wide(const Launch& l, int32_t rank, const KArgs& args, hipStream_t s) {
  if (l.ntiles <= 0) return hipSuccess;
  switch (rank) {
    case 8: return launch_wide_rank<8>(l, args, s);
    case 16: return launch_wide_rank<16>(l, args, s);
    case 32: return launch_wide_rank<32>(l, args, s);
    case 64: return launch_wide_rank<64>(l, args, s);
    case 128: return launch_wide_rank<128>(l, args, s);
    case 256: return launch_wide_rank<256>(l, args, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace acp
