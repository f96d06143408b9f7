// gfx950 streaming kernels of the ACP-SGD compressor for ranks 1, 2 and 4 (arXiv 2306.08881,
// Algorithms 1 and 2): P-step, Q-step and decompress over any row length and alignment.
//
// At these ranks a step costs at most 4 multiply-adds per byte moved, so every kernel is bound by
// HBM: a P-step reads M and E and writes E once, a Q-step reads M and E and writes F = M + E once,
// a decompress writes M_hat once, each row in 16-byte accesses, with the factor rows of a lane's
// columns in registers for the whole tile.
//
// Rows need 4-byte alignment only: a 16-byte buffer access may start on any dword, and its four
// dwords are checked against the resource's extent one by one (a load past it returns zero, a
// store past it is dropped).  So a row whose length is not a multiple of four is cut by a
// resource of its own that ends with the row; where the rows of several lanes' groups share one
// instruction (narrow rows) the last group's loads are masked and its floats stored one by one.
// Before, such matrices and all of rank 1 and 2 went through general kernels that read M and E
// twice in a P-step (P first, then E), four bytes per lane, with an integer division per element:
// ResNet-152 at rank 2 took 894 us per two steps.
//
// Classes of row length: at most 512 columns, several rows per wave (pnarrow_tile, qnarrow_tile,
// rnarrow_tile); up to 5120, one workgroup per row at a time (k_pfused); beyond, the P-step splits
// a row over column blocks (k_pwide, k_pfin), see there.
#include "device.hpp"

namespace acp {

namespace {

// ---------------------------------------------------------------------------------------
// Narrow rows (at most 512 columns): L lanes per row (16, 32 or 64), G float4 groups per lane (1
// or 2).  A wave holds 64 / L whole rows at a time and the workgroup 256 / L; lane l of row slot
// l / L owns groups (l % L) + L g, whose factor rows stay in registers.  Row sums stay inside the
// wave, so these kernels wait at no barrier per row.  RAG: the row length is not a multiple of four.
template <int L, int G, bool RAG>
struct Narrow {
  static constexpr int SL = 64 / L;   // rows per wave at a time
  static constexpr int RW = 4 * SL;   // rows per workgroup round
  int wave, slot, cl;
  int c4[G];
  int nv[G];        // valid columns of the group
  uint32_t coff[G];  // byte offset of the group in its row
  __device__ explicit Narrow(int m) {
    wave = __builtin_amdgcn_readfirstlane(tid() >> 6);
    const int lane = tid() & 63;
    slot = lane / L;
    cl = lane % L;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      c4[g] = cl + L * g;
      const int left = m - 4 * c4[g];
      nv[g] = left < 0 ? 0 : (left < 4 ? left : 4);
      coff[g] = nv[g] > 0 ? static_cast<uint32_t>(c4[g]) * 16u : kOut;
    }
  }
  __device__ int row(int k) const { return k * RW + wave * SL + slot; }  // tile-relative row of round k
  __device__ uint32_t off(uint32_t roff, int g) const { return coff[g] == kOut ? kOut : roff + coff[g]; }
  // the group's floats past the row's end as zero (they belong to the next row)
  __device__ float4 cut(float4 v, int g) const {
    if constexpr (RAG) {
      v.y = nv[g] > 1 ? v.y : 0.f;
      v.z = nv[g] > 2 ? v.z : 0.f;
      v.w = nv[g] > 3 ? v.w : 0.f;
    }
    return v;
  }
  __device__ void store(Rsrc r, uint32_t roff, int g, const float4& v) const {
    const uint32_t o = off(roff, g);
    if constexpr (RAG) {
      bst4_nt(r, nv[g] == 4 ? o : kOut, v);
      const bool part = nv[g] > 0 && nv[g] < 4;
      bst1_nt(r, part ? o : kOut, v.x);
      bst1_nt(r, part && nv[g] > 1 ? o + 4u : kOut, v.y);
      bst1_nt(r, part && nv[g] > 2 ? o + 8u : kOut, v.z);
    } else {
      bst4_nt(r, o, v);
    }
  }
};

// Sum over the L lanes of a row slot; every lane of the slot gets the same bits.  DPP quad
// butterflies and mirrors give 16-lane sums, a swizzle (xor 16) pairs them for L = 32, and for
// L = 64 the four 16-lane sums are read out and added in order.
template <int L>
__device__ inline float row_sum(float v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  v += dpp<0x140>(v);
  if constexpr (L == 32)
    v += __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));
  if constexpr (L == 64) {
    const int b = __builtin_bit_cast(int, v);
    v = ((__builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0)) +
          __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16))) +
         __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32))) +
        __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
  }
  return v;
}

// (v.x, v.y, v.z, v.w) minus the rank-RK products of f with the four column rows q
template <int RK>
__device__ inline float4 minus_dots(float4 v, const Fr<RK>& f, const Fr<RK> (&q)[4]) {
  v.x -= dot_fr(f, q[0]);
  v.y -= dot_fr(f, q[1]);
  v.z -= dot_fr(f, q[2]);
  v.w -= dot_fr(f, q[3]);
  return v;
}
template <int RK>
__device__ inline void fma_dots(const float4& v, const Fr<RK> (&q)[4], Fr<RK>& acc) {
  fma_fr(v.x, q[0], acc);
  fma_fr(v.y, q[1], acc);
  fma_fr(v.z, q[2], acc);
  fma_fr(v.w, q[3], acc);
}

// The rows of Qh = Q W (of Q itself in Power-SGD's first half) and of Q_loc of the four columns from 4 c4 on, of which nv are in the row
// (the others and, unless E is deferred, Q_loc's are zero); stored to the Qh slot when store_qh.
template <int RK>
__device__ inline void column_factors(const KArgs& a, const MatDesc& d, const double* Wsh, int c4, int nv,
                                      bool store_qh, bool deferred, Fr<RK> (&qh)[4], Fr<RK> (&ql)[4]) {
  const Fr<RK>* Q = reinterpret_cast<const Fr<RK>*>(a.fac + d.q_slot);
  const Fr<RK>* Ql = reinterpret_cast<const Fr<RK>*>(a.fac + d.ql_slot);
  Fr<RK>* Qh = reinterpret_cast<Fr<RK>*>(a.fac + d.qh_slot);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const bool ok = c < nv;
    const int j = ok ? 4 * c4 + c : 0;  // in-range row for columns past m
    const Fr<RK> q0 = Q[j], qw = apply_w(q0, Wsh);
    const Fr<RK> q = a.image ? q0 : qw;
    const Fr<RK> l = Ql[j];
    qh[c] = ok ? q : zero_fr<RK>();
    ql[c] = ok && deferred ? l : zero_fr<RK>();
    if (store_qh && ok) Qh[j] = q;
  }
}

// The row of P whose term E leaves out: in Power-SGD's first half none (M' itself stays in the arena).
template <int RK>
__device__ inline Fr<RK> residual_row(const KArgs& a, const Fr<RK>& P) {
  Fr<RK> f;
#pragma unroll
  for (int k = 0; k < RK; ++k) f.v[k] = a.image ? 0.f : P.v[k];
  return f;
}

// W of a matrix into shared memory (RK x RK doubles); the caller synchronises.
template <int RK>
__device__ inline void stage_w(const KArgs& a, const MatDesc& d, double* Wsh) {
  if (tid() < RK * RK) Wsh[tid()] = a.w[d.w_slot + tid()];
}

// P-step, narrow rows: per row M' = M + E (or M + F - Ph_row Q_loc^T), P = M' Qh (row sum),
// E = M' - P Qh^T (with Power-SGD's first half M' itself), P to the factor buffer.  U rounds of rows are in flight per lane.  Wsh: RK x RK
// doubles of shared memory.
template <int RK, int L, int G, bool RAG>
__device__ void pnarrow_tile(const KArgs& a, const Tile& t, const MatDesc& d, double* Wsh) {
  using NM = Narrow<L, G, RAG>;
  constexpr int U = 2;
  const NM nm(d.m);
  const bool deferred = deferred_of(a, d.bucket);
  const uint32_t row_bytes = static_cast<uint32_t>(d.m) * 4u;
  const uint32_t tile_bytes = static_cast<uint32_t>(t.b) * row_bytes;
  const int64_t first = static_cast<int64_t>(t.a) * d.m;
  const Rsrc Gr = tile_rsrc(src_of(a, d.bucket) + d.grad_off + first, tile_bytes);
  const Rsrc Er = tile_rsrc(a.e + d.e_off + first, a.ef ? tile_bytes : 0u);
  const Rsrc Pr = tile_rsrc(dst_of(a, d.bucket) + d.fac_off_p + static_cast<int64_t>(t.a) * RK,
                            static_cast<uint32_t>(t.b) * 4u * RK);
  const Rsrc Phr = tile_rsrc(a.fac + d.ph_slot + static_cast<int64_t>(t.a) * RK,
                             deferred ? static_cast<uint32_t>(t.b) * 4u * RK : 0u);

  float4 gv[U][G], ev[U][G];
  Fr<RK> ph[U];
  auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t row = static_cast<uint32_t>(nm.row(k0 + u));  // past the tile: zeros
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const uint32_t o = nm.off(row * row_bytes, g);
        gv[u][g] = bld4_nt(Gr, o);
        ev[u][g] = bld4_nt(Er, o);
      }
      ph[u] = bld_fr<RK>(Phr, row * 4u * RK);
    }
  };
  load(0);
  stage_w<RK>(a, d, Wsh);
  __syncthreads();
  Fr<RK> qh[G][4], ql[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g)
    column_factors<RK>(a, d, Wsh, nm.c4[g], nm.nv[g], t.a == 0 && nm.wave == 0 && nm.slot == 0, deferred, qh[g], ql[g]);

  for (int k = 0; k * NM::RW < t.b; k += U) {
    float4 mp[U][G];
    Fr<RK> acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u] = zero_fr<RK>();
#pragma unroll
      for (int g = 0; g < G; ++g) {
        mp[u][g] = minus_dots(nm.cut(gv[u][g] + ev[u][g], g), ph[u], ql[g]);
        fma_dots(mp[u][g], qh[g], acc[u]);
      }
    }
    load(k + U);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Fr<RK> P;
#pragma unroll
      for (int i = 0; i < RK; ++i) P.v[i] = row_sum<L>(acc[u].v[i]);
      const uint32_t row = static_cast<uint32_t>(nm.row(k + u));
#pragma unroll
      for (int g = 0; g < G; ++g) nm.store(Er, row * row_bytes, g, minus_dots(mp[u][g], residual_row(a, P), qh[g]));
      bst_fr(Pr, nm.cl == 0 ? row * 4u * RK : kOut, P);
    }
  }
}

// The Ph rows of a Q-step row chunk, formed in LDS as P W: rows first + i stride, i < rows (zero
// from there to kQRows), stored to the Ph slot when `store`.  Wsh as staged by stage_w; both
// barriers inside.
template <int RK>
__device__ inline void stage_ph(const KArgs& a, const MatDesc& d, int64_t first, int stride, int rows, bool store,
                                double* Wsh, Fr<RK>* phs) {
  static_assert(kQRows <= kBlock, "one thread per staged Ph row");
  stage_w<RK>(a, d, Wsh);
  __syncthreads();
  if (tid() < kQRows) {
    Fr<RK> y = zero_fr<RK>();
    if (tid() < rows) {
      const int64_t row = first + static_cast<int64_t>(tid()) * stride;
      y = apply_w(reinterpret_cast<const Fr<RK>*>(a.fac + d.p_slot)[row], Wsh);
      if (store) reinterpret_cast<Fr<RK>*>(a.fac + d.ph_slot)[row] = y;
    }
    phs[tid()] = y;
  }
  __syncthreads();
}

// Q-step, narrow rows: tile = row chunk t.a.  Per row F = M + E is written back and each lane adds
// F^T Ph over its rows and columns.  The 256 / L row slots' sums are added in slot order through
// LDS and stored as the chunk's partials for K_QFIN.  Shared memory: Wsh (RK x RK doubles), phs
// (kQRows factor rows), red (kNarrowRed factor rows).
constexpr int kNarrowRed = 2048;  // row slots x L G 4 at most (4 x 64 x 2 x 4)
template <int RK, int L, int G, bool RAG>
__device__ void qnarrow_tile(const KArgs& a, const Tile& t, const MatDesc& d, double* Wsh, Fr<RK>* phs,
                             Fr<RK>* red) {
  using NM = Narrow<L, G, RAG>;
  constexpr int U = 2;
  constexpr int NS = 4 * NM::SL;  // row slots of the workgroup
  static_assert(NS * L * G * 4 <= kNarrowRed, "slot sums exceed the shared buffer");
  const NM nm(d.m);
  const int64_t r0 = static_cast<int64_t>(t.a) * d.q_rows;
  const int rows = static_cast<int>((r0 + d.q_rows < d.n) ? d.q_rows : d.n - r0);
  const uint32_t row_bytes = static_cast<uint32_t>(d.m) * 4u;
  const uint32_t ext = static_cast<uint32_t>(rows) * row_bytes;
  const int64_t first = r0 * d.m;
  const Rsrc Gr = tile_rsrc(src_of(a, d.bucket) + d.grad_off + first, ext);
  const Rsrc Er = tile_rsrc(a.e + d.e_off + first, a.ef ? ext : 0u);

  float4 gv[U][G], ev[U][G];
  auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t roff = static_cast<uint32_t>(nm.row(k0 + u)) * row_bytes;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const uint32_t o = nm.off(roff, g);
        gv[u][g] = bld4_nt(Gr, o);
        ev[u][g] = bld4_nt(Er, o);
      }
    }
  };
  load(0);
  stage_ph<RK>(a, d, r0, 1, rows, true, Wsh, phs);

  Fr<RK> acc[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[g][c] = zero_fr<RK>();
  for (int k = 0; k * NM::RW < rows; k += U) {
    float4 f[U][G];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int g = 0; g < G; ++g) f[u][g] = nm.cut(gv[u][g] + ev[u][g], g);
    load(k + U);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = nm.row(k + u);  // < kQRows: rows <= kQRows and 2 RW divides kQRows
      const uint32_t roff = static_cast<uint32_t>(row) * row_bytes;
      const Fr<RK> ph = phs[row & (kQRows - 1)];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        nm.store(Er, roff, g, f[u][g]);
        fma_fr(f[u][g].x, ph, acc[g][0]);
        fma_fr(f[u][g].y, ph, acc[g][1]);
        fma_fr(f[u][g].z, ph, acc[g][2]);
        fma_fr(f[u][g].w, ph, acc[g][3]);
      }
    }
  }
  const int sidx = nm.wave * NM::SL + nm.slot;
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int c = 0; c < 4; ++c) red[sidx * (L * G * 4) + (nm.cl * G + g) * 4 + c] = acc[g][c];
  __syncthreads();
  const int64_t ncb = (d.m + d.q_cb - 1) / d.q_cb;
  Fr<RK>* part = reinterpret_cast<Fr<RK>*>(a.qpart + d.qpart + static_cast<int64_t>(t.a) * ncb * d.q_cb * RK);
  for (int e = tid(); e < L * G * 4; e += kBlock) {
    const int cl = e / (G * 4), g = (e / 4) % G, c = e % 4;
    const int col = 4 * (cl + L * g) + c;
    if (col >= d.m) continue;
    Fr<RK> sum = red[e];
    for (int sl = 1; sl < NS; ++sl) add_fr(sum, red[sl * (L * G * 4) + e]);
    part[col] = sum;
  }
}

// Decompress, narrow rows: M_hat rows from the tile's A rows (staged in LDS, scaled by 1 / p)
// and the lane's B rows in registers.  as: kMaxTileRows factor rows of shared memory.
template <int RK, int L, int G, bool RAG>
__device__ void rnarrow_tile(const KArgs& a, const Tile& t, const MatDesc& d, Fr<RK>* as) {
  using NM = Narrow<L, G, RAG>;
  const bool odd = a.parity != 0;
  const NM nm(d.m);
  const float* agg = src_of(a, d.bucket);
  const float* A = odd ? agg + d.fac_off_p : a.fac + d.ph_slot;
  const float* B = odd ? a.fac + d.qh_slot : agg + d.fac_off_q;
  if (tid() < t.b) as[tid()] = scale_fr(ld_fr<RK>(A + (static_cast<int64_t>(t.a) + tid()) * RK), a.inv_p);
  Fr<RK> b[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int c = 0; c < 4; ++c)
      b[g][c] = c < nm.nv[g] ? ld_fr<RK>(B + static_cast<int64_t>(4 * nm.c4[g] + c) * RK) : zero_fr<RK>();
  __syncthreads();
  __builtin_amdgcn_s_waitcnt(0);
  const uint32_t row_bytes = static_cast<uint32_t>(d.m) * 4u;
  const Rsrc O = tile_rsrc(dst_of(a, d.bucket) + d.grad_off + static_cast<int64_t>(t.a) * d.m,
                           static_cast<uint32_t>(t.b) * row_bytes);
  for (int k = 0; k * NM::RW < t.b; ++k) {
    const int row = nm.row(k);  // past the tile: an unset LDS entry, its stores are dropped
    const Fr<RK> ar = as[row & (kMaxTileRows - 1)];
#pragma unroll
    for (int g = 0; g < G; ++g)
      nm.store(O, static_cast<uint32_t>(row) * row_bytes, g,
               make_float4(dot_fr(ar, b[g][0]), dot_fr(ar, b[g][1]), dot_fr(ar, b[g][2]), dot_fr(ar, b[g][3])));
  }
}

// Narrow-row tiles of a matrix (at most 128 float4 groups per row) inside the P-step, Q-step and
// decompress launches: the variant follows from the row length.
template <typename F>
__device__ inline void narrow_dispatch(int m, F f) {
  auto pick = [&](auto rag) {
    constexpr bool R = decltype(rag)::value;
    switch (narrow_variant((m + 3) >> 2)) {
      case (16 << 4) | 1: f(std::integral_constant<int, 16>{}, std::integral_constant<int, 1>{}, std::bool_constant<R>{}); break;
      case (32 << 4) | 1: f(std::integral_constant<int, 32>{}, std::integral_constant<int, 1>{}, std::bool_constant<R>{}); break;
      case (64 << 4) | 1: f(std::integral_constant<int, 64>{}, std::integral_constant<int, 1>{}, std::bool_constant<R>{}); break;
      default: f(std::integral_constant<int, 64>{}, std::integral_constant<int, 2>{}, std::bool_constant<R>{}); break;
    }
  };
  if (m & 3)
    pick(std::true_type{});
  else
    pick(std::false_type{});
}

// The resource of tile-relative row r of a tile of `rows` rows, `step` bytes apart, of which the
// tile takes `width` bytes each.  RAG (a row length that is not a multiple of four): it ends with
// the row, and is empty past the tile.  Else one resource serves the whole tile (the 3 % that
// a resource per row costs the aligned rows: BERT-large rank 4, 1.80 against 1.75 ms per two steps).
template <bool RAG>
struct RowRsrc {
  const float* base;
  uint32_t step, width;
  int rows;
  bool on;  // false: empty
  Rsrc tile;
  __device__ RowRsrc(const float* b, int rows_, uint32_t step_, uint32_t width_, bool on_ = true)
      : base(b), step(step_), width(width_), rows(rows_), on(on_),
        tile(tile_rsrc(b, on_ ? static_cast<uint32_t>(rows_ - 1) * step_ + width_ : 0u)) {}
  __device__ Rsrc operator()(int r) const {
    if constexpr (!RAG) return tile;
    return tile_rsrc(base, on && r < rows ? static_cast<uint32_t>(r) * step + width : 0u);
  }
};
// f(RAG) for the row length m of a matrix of a launch that takes any (ANY) or only multiples of four.
// A kernel that holds both forms has the registers of the ragged one, which cost the P-step of 4100
// to 5120 columns at rank 4 (and 2) one of its two waves per SIMD (252 VGPRs to 264), that of two
// groups per lane at rank 1 and of three at rank 2 one of three.  So k_pfused of 2 to 5 groups is
// built both ways and a launch without a ragged row takes the second: ResNet-50 rank 4 223.9 to
// 215 us per two steps, ResNet-152 rank 2 411 to 402, rank 4 426 to 418.  The other kernels gain
// nothing from their third wave: with the Q-step split the same way (170 to 148 VGPRs at rank 4)
// BERT-large rank 4 took 1760 us instead of 1755, and with the P-step of one group per lane and
// that of eight waves BERT-large rank 2 1754 instead of 1748.
template <bool ANY, typename F>
__device__ inline void by_raggedness(int m, F f) {
  if constexpr (ANY) {
    if (m & 3) {
      f(std::true_type{});
      return;
    }
  }
  f(std::false_type{});
}

// ---------------------------------------------------------------------------------------
// Column mapping of the one-row-at-a-time kernels.  The W waves of a workgroup (four; three for
// rows of at most 768 columns; eight for rows of 3073 to 4096) split a row of ceil(m / 4) float4
// groups into W segments of 64 Se groups, Se = ceil(groups / 64 W) <= S (a launch of class S also
// carries rows of smaller classes); lane `lane` of wave w owns groups w * 64 Se + s * 64 + lane,
// s < Se, for every row of the tile, so the factor rows of those columns are loaded once per
// workgroup and kept in registers.  The waves work on the same RB rows at a time.
template <int RK, int S, int W = 4>
struct Cols {
  static constexpr int RB = pstep_rows(RK, S);
  int wave, lane;
  int c4[S];
  int nv[S];  // valid columns of the group
  __device__ explicit Cols(int m) {
    wave = tid() >> 6;
    lane = tid() & 63;
    const int m4 = (m + 3) >> 2;
    const int se = (m4 + 64 * W - 1) / (64 * W);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      c4[s] = wave * 64 * se + s * 64 + lane;
      const int left = m - 4 * c4[s];
      nv[s] = s >= se || left < 0 ? 0 : (left < 4 ? left : 4);
    }
  }
};

// P-step, fused single pass (rows of up to 5120 columns).  Each lane keeps, for its columns, the
// rows of Qh = Q W (computed here from the reused factor; the tile holding row 0 also stores Qh)
// and of Q_loc in registers for the whole tile (Q_loc and the tile's Ph rows are zero unless E is
// deferred).  Per row: M' = M + E (or M + F - Ph_row Q_loc^T), P = M' Qh summed over the row (DPP
// wave sums, then the waves' sums in wave order), E = M' - P Qh^T written back, P written to the
// factor buffer.  The next rows' M and E are requested before the reduction.
template <int RK, int S, bool ANY, int W = 4>
__global__ __launch_bounds__(64 * W) void k_pfused(KArgs a) {
  constexpr int RB = Cols<RK, S, W>::RB;
  const Tile t = a.tiles[blockIdx.x];
  if (t.kind == T_VEC) {
    vec_tile(a, t, true);
    return;
  }
  const MatDesc d = a.mats[t.idx];
  __shared__ double Wsh[RK * RK];
  if constexpr (S == 1 && W == 4) {
    if (t.kind == T_ROWS) {  // a narrow-row matrix's tile (the S = 1 launch carries them)
      narrow_dispatch(d.m, [&](auto l, auto g, auto rag) {
        pnarrow_tile<RK, decltype(l)::value, decltype(g)::value, decltype(rag)::value>(a, t, d, Wsh);
      });
      return;
    }
  }
  __shared__ Fr<RK> red[2][W][RB];
  __shared__ Fr<RK> phs[kMaxTileRows];  // the tile's rows of Ph (zero unless E is deferred)
  by_raggedness<ANY>(d.m, [&](auto rag) {
    constexpr bool RAG = decltype(rag)::value;
    const Cols<RK, S, W> cl(d.m);
    const bool deferred = deferred_of(a, d.bucket);
    // tile rows t.a + k * stride, k < rows (T_SROWS)
    const int stride = srows_stride(t.b), rows = srows_count(t.b);
    const uint32_t row_bytes = static_cast<uint32_t>(d.m) * 4u;
    const uint32_t step_bytes = static_cast<uint32_t>(stride) * row_bytes;
    const int64_t first = static_cast<int64_t>(t.a) * d.m;
    const RowRsrc<RAG> G(src_of(a, d.bucket) + d.grad_off + first, rows, step_bytes, row_bytes);
    const RowRsrc<RAG> E(a.e + d.e_off + first, rows, step_bytes, row_bytes, a.ef != 0);
    const Rsrc P = tile_rsrc(dst_of(a, d.bucket) + d.fac_off_p + static_cast<int64_t>(t.a) * RK,
                             static_cast<uint32_t>((rows - 1) * stride + 1) * 4u * RK);
    uint32_t coff[S];
#pragma unroll
    for (int s = 0; s < S; ++s) coff[s] = cl.nv[s] > 0 ? static_cast<uint32_t>(cl.c4[s]) * 16u : kOut;

    // the first rows' M and E are requested before the factor setup
    float4 g[RB][S], e[RB][S];
    auto load_rows = [&](int r0) {  // tile-relative first row
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const Rsrc Gr = G(r0 + rb), Er = E(r0 + rb);
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const uint32_t o = static_cast<uint32_t>(r0 + rb) * step_bytes + coff[s];
          g[rb][s] = bld4_nt(Gr, o);
          e[rb][s] = bld4_nt(Er, o);
        }
      }
    };
    load_rows(0);

    stage_w<RK>(a, d, Wsh);
    for (int i = tid(); i < rows; i += 64 * W)
      phs[i] = deferred ? reinterpret_cast<const Fr<RK>*>(a.fac + d.ph_slot)[t.a + static_cast<int64_t>(i) * stride]
                        : zero_fr<RK>();
    __syncthreads();
    Fr<RK> qh[S][4], ql[S][4];
#pragma unroll
    for (int s = 0; s < S; ++s)
      column_factors<RK>(a, d, Wsh, cl.c4[s], cl.nv[s], t.a == 0, deferred, qh[s], ql[s]);

    int buf = 0;
    for (int r0 = 0; r0 < rows; r0 += RB, buf ^= 1) {
      float4 mp[RB][S];
      Fr<RK> acc[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        // rows past the tile read phs entries that are never used: their stores are dropped
        const Fr<RK> ph = phs[(r0 + rb) & (kMaxTileRows - 1)];
        acc[rb] = zero_fr<RK>();
#pragma unroll
        for (int s = 0; s < S; ++s) {
          mp[rb][s] = minus_dots(g[rb][s] + e[rb][s], ph, ql[s]);
          fma_dots(mp[rb][s], qh[s], acc[rb]);
        }
      }
      load_rows(r0 + RB);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        acc[rb] = wave_sum_dpp(acc[rb]);
        if (cl.lane == 0) red[buf][cl.wave][rb] = acc[rb];
      }
      __syncthreads();
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const uint32_t roff = static_cast<uint32_t>(r0 + rb) * step_bytes;
        const Rsrc Er = E(r0 + rb);
        Fr<RK> Pr = red[buf][0][rb];  // the waves' sums in wave order
#pragma unroll
        for (int w = 1; w < W; ++w) add_fr(Pr, red[buf][w][rb]);
#pragma unroll
        for (int s = 0; s < S; ++s) bst4_nt(Er, roff + coff[s], minus_dots(mp[rb][s], residual_row(a, Pr), qh[s]));
        bst_fr(P, tid() == 0 ? static_cast<uint32_t>((r0 + rb) * stride) * 4u * RK : kOut, Pr);
      }
    }
  });
}

// P-step of rows longer than 5120 columns, whose factor rows no longer fit one workgroup's
// registers: a tile takes the 1024-column block cb of its rows (256 lanes, four columns each) and
// cannot know a row's P, so it leaves X = M' in the arena (E = X - P_loc Qh^T is implied, and the
// next Q-step subtracts that term) and stores the block's share of P, which k_pfin adds over the
// blocks in order.  Reads M and E and writes X once: 12 bytes per element, as k_pfused; the shares
// add 8 RK bytes per 1024 elements.  (Splitting the row over 16 waves instead holds the
// residual's registers and reaches 8192 columns only.)
constexpr int kPwRows = 8;  // rows at a time
template <int RK>
__global__ __launch_bounds__(kBlock) void k_pwide(KArgs a) {
  constexpr int RB = kPwRows;
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  __shared__ double Wsh[RK * RK];
  __shared__ Fr<RK> red[2][4][RB];
  __shared__ Fr<RK> phs[kMaxTileRows];
  by_raggedness<true>(d.m, [&](auto rag) {
    constexpr bool RAG = decltype(rag)::value;
    const int wave = tid() >> 6, lane = tid() & 63;
    const bool deferred = deferred_of(a, d.bucket);
    const int cb = srows_block(t.b), stride = srows_stride(t.b), rows = srows_count(t.b);
    const int c4 = cb * 256 + tid();
    const int left = d.m - 4 * c4;
    const int nv = left < 0 ? 0 : (left < 4 ? left : 4);
    const uint32_t row_bytes = static_cast<uint32_t>(d.m) * 4u;
    const uint32_t step_bytes = static_cast<uint32_t>(stride) * row_bytes;
    const uint32_t width = static_cast<uint32_t>(d.m - cb * 1024 < 1024 ? d.m - cb * 1024 : 1024) * 4u;
    const int64_t first = static_cast<int64_t>(t.a) * d.m + static_cast<int64_t>(cb) * 1024;
    const RowRsrc<RAG> G(src_of(a, d.bucket) + d.grad_off + first, rows, step_bytes, width);
    const RowRsrc<RAG> E(a.e + d.e_off + first, rows, step_bytes, width, a.ef != 0);
    const uint32_t coff = nv > 0 ? static_cast<uint32_t>(tid()) * 16u : kOut;

    float4 g[RB], e[RB];
    auto load_rows = [&](int r0) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const uint32_t o = static_cast<uint32_t>(r0 + rb) * step_bytes + coff;
        g[rb] = bld4_nt(G(r0 + rb), o);
        e[rb] = bld4_nt(E(r0 + rb), o);
      }
    };
    load_rows(0);
    stage_w<RK>(a, d, Wsh);
    for (int i = tid(); i < rows; i += kBlock)
      phs[i] = deferred ? reinterpret_cast<const Fr<RK>*>(a.fac + d.ph_slot)[t.a + static_cast<int64_t>(i) * stride]
                        : zero_fr<RK>();
    __syncthreads();
    Fr<RK> qh[4], ql[4];
    column_factors<RK>(a, d, Wsh, c4, nv, t.a == 0, deferred, qh, ql);
    Fr<RK>* part = reinterpret_cast<Fr<RK>*>(a.qpart + d.qpart) + static_cast<int64_t>(cb) * d.n;

    int buf = 0;
    for (int r0 = 0; r0 < rows; r0 += RB, buf ^= 1) {
      float4 mp[RB];
      Fr<RK> acc[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const Fr<RK> ph = phs[(r0 + rb) & (kMaxTileRows - 1)];
        mp[rb] = minus_dots(g[rb] + e[rb], ph, ql);
        acc[rb] = zero_fr<RK>();
        fma_dots(mp[rb], qh, acc[rb]);
      }
      load_rows(r0 + RB);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        bst4_nt(E(r0 + rb), static_cast<uint32_t>(r0 + rb) * step_bytes + coff, mp[rb]);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        acc[rb] = wave_sum_dpp(acc[rb]);
        if (lane == 0) red[buf][wave][rb] = acc[rb];
      }
      __syncthreads();
      if (tid() < RB && r0 + tid() < rows) {  // the waves' sums in wave order
        Fr<RK> s = red[buf][0][tid()];
#pragma unroll
        for (int w = 1; w < 4; ++w) add_fr(s, red[buf][w][tid()]);
        part[t.a + static_cast<int64_t>(r0 + tid()) * stride] = s;
      }
    }
  });
}

// P of the rows k_pwide took: the column blocks' shares added in block order, to the factor buffer
// and the P_loc slot.  Tile: rows [t.a, t.a + t.b) of the matrix, one thread per row.
template <int RK>
__global__ __launch_bounds__(kBlock) void k_pfin(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  if (tid() >= t.b) return;
  const int64_t row = static_cast<int64_t>(t.a) + tid();
  const int ncb = (d.m + 1023) / 1024;
  const Fr<RK>* part = reinterpret_cast<const Fr<RK>*>(a.qpart + d.qpart) + row;
  constexpr int U = 8;  // shares requested at a time
  Fr<RK> s = zero_fr<RK>();
  for (int cb = 0; cb < ncb; cb += U) {
    Fr<RK> v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = cb + u < ncb ? part[static_cast<int64_t>(cb + u) * d.n] : zero_fr<RK>();
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (cb + u < ncb) add_fr(s, v[u]);
  }
  float* P = dst_of(a, d.bucket) + d.fac_off_p + row * RK;
#pragma unroll
  for (int k = 0; k < RK; ++k) P[k] = s.v[k];
  reinterpret_cast<Fr<RK>*>(a.fac + d.pl_slot)[row] = s;
}

// ---------------------------------------------------------------------------------------
// Q-step: tile = (row chunk of at most kQRows rows, block of 1024 columns).  Lane l of wave w owns
// the four columns 4 (64 w + l) ... of the block in every row of the chunk, so each row's 4 KB
// segment is read by one workgroup.  The chunk's Ph rows are formed in LDS first, as P W, and
// stored by the tiles of column block 0.  Per row: F = M' = M + E written back (deferred E),
// partial Q += M'^T Ph over the lane's columns.  Rows go in groups of U whose loads are issued
// before the previous group's F stores, so stores never hold up the next loads.  Each lane stores
// its partial sums for K_QFIN (columns past m store zeros into the padded partial block).  XF: the
// rows k_pwide takes, whose arena may hold X: F = M + X - P_loc Qh^T (a launch of their own: the
// column rows of Qh take 20, 56 and 60 more registers at ranks 1, 2 and 4, and of rank 2 a wave per SIMD).
template <int RK, bool XF>
__global__ __launch_bounds__(kBlock) void k_qstep(KArgs a) {
  constexpr int U = 8;  // rows per group
  const Tile t = a.tiles[blockIdx.x];
  if (t.kind == T_VEC) {
    vec_tile(a, t, true);
    return;
  }
  const MatDesc d = a.mats[t.idx];
  __shared__ double Wsh[RK * RK];
  __shared__ Fr<RK> phs[kQRows];
  if constexpr (!XF) {
    if (d.scls == 0) {  // a narrow-row matrix's chunk
      __shared__ Fr<RK> red[kNarrowRed];
      narrow_dispatch(d.m, [&](auto l, auto g, auto rag) {
        qnarrow_tile<RK, decltype(l)::value, decltype(g)::value, decltype(rag)::value>(a, t, d, Wsh, phs, red);
      });
      return;
    }
  }
  __shared__ Fr<RK> pls[XF ? kQRows : 1];
  by_raggedness<true>(d.m, [&](auto rag) {
    constexpr bool RAG = decltype(rag)::value;
    const int64_t m = d.m;
    const ChunkRows ch = q_chunk_rows(d, t.a);  // rows ch.first + k * ch.stride, k < ch.rows
    const int64_t r0 = ch.first;
    const int rows = ch.rows;
    const int64_t cb0 = static_cast<int64_t>(t.b) * d.q_cb;
    const int lcol = tid() * 4;  // column within the block
    const int bcols = static_cast<int>((m - cb0) < d.q_cb ? (m - cb0) : d.q_cb);
    const uint32_t step_bytes = static_cast<uint32_t>(ch.stride) * static_cast<uint32_t>(m) * 4u;
    const uint32_t width = static_cast<uint32_t>(bcols) * 4u;
    const int64_t first = r0 * m + cb0;
    const RowRsrc<RAG> G(src_of(a, d.bucket) + d.grad_off + first, rows, step_bytes, width);
    const RowRsrc<RAG> E(a.e + d.e_off + first, rows, step_bytes, width, a.ef != 0);
    const uint32_t coff = lcol < bcols ? static_cast<uint32_t>(lcol) * 4u : kOut;

    float4 g[U], e[U];
    auto load_group = [&](int rr, float4* gg, float4* ee) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t o = static_cast<uint32_t>(rr + u) * step_bytes + coff;
        gg[u] = bld4_nt(G(rr + u), o);
        ee[u] = bld4_nt(E(rr + u), o);
      }
    };
    load_group(0, g, e);

    // the chunk's Ph rows; the rows after them are zero (groups may run past the chunk)
    static_assert(kQRows % U == 0, "whole groups of staged rows");
    Fr<RK> qh[4];
    if constexpr (XF) {
      const bool xform = deferred_p_of(a, d);
      if (tid() < kQRows)
        pls[tid()] = xform && tid() < rows
                         ? reinterpret_cast<const Fr<RK>*>(a.fac + d.pl_slot)[r0 + static_cast<int64_t>(tid()) * ch.stride]
                         : zero_fr<RK>();
#pragma unroll
      for (int c = 0; c < 4; ++c)
        qh[c] = xform && lcol + c < bcols ? reinterpret_cast<const Fr<RK>*>(a.fac + d.qh_slot)[cb0 + lcol + c] : zero_fr<RK>();
    }
    stage_ph<RK>(a, d, r0, ch.stride, rows, t.b == 0, Wsh, phs);

    Fr<RK> acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = zero_fr<RK>();

    for (int rr = 0; rr < rows; rr += U) {
      float4 gn[U], en[U];
      load_group(rr + U, gn, en);
      float4 f[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        f[u] = g[u] + e[u];
        if constexpr (XF) f[u] = minus_dots(f[u], pls[rr + u], qh);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        bst4_nt(E(rr + u), static_cast<uint32_t>(rr + u) * step_bytes + coff, f[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const Fr<RK> ph = phs[rr + u];  // rr + u < kQRows: kQRows is a multiple of U
        fma_fr(f[u].x, ph, acc[0]);
        fma_fr(f[u].y, ph, acc[1]);
        fma_fr(f[u].z, ph, acc[2]);
        fma_fr(f[u].w, ph, acc[3]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        g[u] = gn[u];
        e[u] = en[u];
      }
    }
    const int64_t ncb = (m + d.q_cb - 1) / d.q_cb;
    const int64_t stride = ncb * d.q_cb * RK;  // one row chunk of partials
    Fr<RK>* part = reinterpret_cast<Fr<RK>*>(a.qpart + d.qpart + static_cast<int64_t>(t.a) * stride + (cb0 + lcol) * RK);
#pragma unroll
    for (int c = 0; c < 4; ++c) part[c] = acc[c];
  });
}

// ---------------------------------------------------------------------------------------
// Decompress, M_hat = A B^T / p (odd step: A = P_agg, B = Qh; even step: A = Ph, B = Q_agg): a row
// tile covers one block of 1024 columns (256 float4 groups, one per lane) of kReconRows rows taken
// with a stride (T_SROWS).  The planner orders the tiles so that workgroups launched together
// write adjacent whole rows: a small write footprint per workgroup with a dense band of rows
// across the running ones streams faster than long per-workgroup row blocks.  Each lane keeps the
// rows of B for its columns in registers; stores are nontemporal: plain stores leave M_hat's lines
// dirty in the caches and the next step's kernels pay for writing them back.  Factor tiles keep
// the aggregated factor as the next step's reused factor and build its W.
template <int RK>
__global__ __launch_bounds__(kBlock) void k_recon4(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const bool odd = a.parity != 0;
  if (t.kind == T_VEC) {
    vec_tile(a, t, false);
    return;
  }
  const MatDesc d = a.mats[t.idx];
  if (t.kind == T_FACT) {
    const float* src = src_of(a, d.bucket) + (odd ? d.fac_off_p : d.fac_off_q);
    float* dst = a.fac + (odd ? d.p_slot : d.q_slot);
    fact_tile<RK>(a, t, src, dst, odd ? d.n : d.m);
    return;
  }
  if (t.kind == T_ROWS) {  // a narrow-row matrix's tile
    __shared__ Fr<RK> asn[kMaxTileRows];
    narrow_dispatch(d.m, [&](auto l, auto g, auto rag) {
      rnarrow_tile<RK, decltype(l)::value, decltype(g)::value, decltype(rag)::value>(a, t, d, asn);
    });
    return;
  }
  const int cb = srows_block(t.b), stride = srows_stride(t.b), rows = srows_count(t.b);
  const int cols = (d.m - cb * 1024) < 1024 ? (d.m - cb * 1024) : 1024;
  const int lcol = tid() * 4;
  const float* agg = src_of(a, d.bucket);
  const float* A = odd ? agg + d.fac_off_p : a.fac + d.ph_slot;
  const float* B = odd ? a.fac + d.qh_slot : agg + d.fac_off_q;
  __shared__ Fr<RK> as[kReconRows];  // the tile's rows of A, scaled by 1 / p
  if (tid() < rows) as[tid()] = scale_fr(ld_fr<RK>(A + (t.a + static_cast<int64_t>(tid()) * stride) * RK), a.inv_p);
  Fr<RK> b[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
    b[c] = lcol + c < cols ? ld_fr<RK>(B + (static_cast<int64_t>(cb) * 1024 + lcol + c) * RK) : zero_fr<RK>();
  __syncthreads();
  // the B rows are in registers before the stores, so no wait for them lands between them
  __builtin_amdgcn_s_waitcnt(0);
  const uint32_t step_bytes = static_cast<uint32_t>(stride) * static_cast<uint32_t>(d.m) * 4u;  // between tile rows
  const float* Ob = dst_of(a, d.bucket) + d.grad_off + static_cast<int64_t>(t.a) * d.m + static_cast<int64_t>(cb) * 1024;
  const uint32_t width = static_cast<uint32_t>(cols) * 4u;
  const uint32_t coff = lcol < cols ? static_cast<uint32_t>(lcol) * 4u : kOut;
  // rows past the tile's count read unset LDS entries; their stores fall outside the resource
  by_raggedness<true>(d.m, [&](auto rag) {
    const RowRsrc<decltype(rag)::value> O(Ob, rows, step_bytes, width);
#pragma unroll
    for (int k = 0; k < kReconRows; ++k) {
      const Fr<RK> ar = as[k];
      const float4 o = make_float4(dot_fr(ar, b[0]), dot_fr(ar, b[1]), dot_fr(ar, b[2]), dot_fr(ar, b[3]));
      bst4_nt(O(k), static_cast<uint32_t>(k) * step_bytes + coff, o);
    }
  });
}

template <int RK>
hipError_t launch_low_rank(const Launch& l, const KArgs& args, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(l.ntiles)), block(kBlock);
  switch (l.kernel) {
    case K_PFUSED:
      switch (l.variant) {
        case 1: hipLaunchKernelGGL((k_pfused<RK, 1, true>), grid, block, 0, s, args); break;
        case 1 | kThreeWaves: hipLaunchKernelGGL((k_pfused<RK, 1, true, 3>), grid, dim3(3 * kWave), 0, s, args); break;
        case 2 | kEightWaves: hipLaunchKernelGGL((k_pfused<RK, 2, true, 8>), grid, dim3(8 * kWave), 0, s, args); break;
        case 2: hipLaunchKernelGGL((k_pfused<RK, 2, false>), grid, block, 0, s, args); break;
        case 3: hipLaunchKernelGGL((k_pfused<RK, 3, false>), grid, block, 0, s, args); break;
        case 4: hipLaunchKernelGGL((k_pfused<RK, 4, false>), grid, block, 0, s, args); break;
        case 5: hipLaunchKernelGGL((k_pfused<RK, 5, false>), grid, block, 0, s, args); break;
        case 2 | kRaggedRows: hipLaunchKernelGGL((k_pfused<RK, 2, true>), grid, block, 0, s, args); break;
        case 3 | kRaggedRows: hipLaunchKernelGGL((k_pfused<RK, 3, true>), grid, block, 0, s, args); break;
        case 4 | kRaggedRows: hipLaunchKernelGGL((k_pfused<RK, 4, true>), grid, block, 0, s, args); break;
        case 5 | kRaggedRows: hipLaunchKernelGGL((k_pfused<RK, 5, true>), grid, block, 0, s, args); break;
        default: return hipErrorInvalidValue;
      }
      break;
    case K_PWIDE: hipLaunchKernelGGL(k_pwide<RK>, grid, block, 0, s, args); break;
    case K_PFIN: hipLaunchKernelGGL(k_pfin<RK>, grid, block, 0, s, args); break;
    case K_QSTEP:
      if (l.variant == 0)
        hipLaunchKernelGGL((k_qstep<RK, false>), grid, block, 0, s, args);
      else
        hipLaunchKernelGGL((k_qstep<RK, true>), grid, block, 0, s, args);
      break;
    case K_RECON4: hipLaunchKernelGGL(k_recon4<RK>, grid, block, 0, s, args); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_low(const Launch& l, int32_t rank, const KArgs& args, hipStream_t s) {
  switch (rank) {
    case 1: return launch_low_rank<1>(l, args, s);
    case 2: return launch_low_rank<2>(l, args, s);
    case 4: return launch_low_rank<4>(l, args, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace acp
