// gfx950 MFMA kernels of the ACP-SGD compressor for ranks 64, 128 and 256 (arXiv 2306.08881,
// Algorithm 2).  A compress step costs 4 r flop per gradient element against 12 bytes, a
// decompress 2 r against 4: from rank 64 on that is more than v_mfma_f32_32x32x2f32 does in the
// time the bytes take (157 TFLOP/s against 6.5 TB/s: 24 flop per byte).  The rank-r products
// therefore run on the bf16 matrix cores (16 times that rate) with fp32 operands split into three
// bf16 parts, x = hi + mid + lo: hi is x cut off after eight bits (rounding it would take values past
// the largest bf16 to infinity), mid the nearest bf16 of what that leaves and lo all of the rest, so
// that the sum is x exactly down to 2^-109 in magnitude (below, what the bf16 subnormals hold: within
// 2^-134).  The six products hi hi, hi mid, mid hi, mid mid, hi lo, lo hi are summed in fp32
// accumulators; the three left out are below 2^-22 of the product, 2^-26 on average and of either
// sign.  Against 64 bits the results' error is that of the fp32 matrix cores or less (see the
// measurements at the kernels).  A value that is not finite gives results that are not finite, as in
// fp32, but NaN where fp32 may give an infinity (infinity minus its own part).
//
// Both compress steps are one kernel (k_bstep).  A workgroup keeps 128 (rank 256: 64) "fixed"
// indices i (P-step: rows, Q-step: columns), 32 per wave, one per lane, and walks the other index
// j (P-step: columns, Q-step: rows) in blocks of 32:
//   D[j][i]      = sum_k S1[j][k] R[i][k]       the previous step's rank-r term, if implied
//   X[j][i]      = M + E - D, written back
//   Acc[k][i]   += sum_j S2[j][k] X[j][i]       the step's product
// with (S1, R, S2) = (Q_loc, Ph, Qh) in a P-step and (P_loc, Qh, Ph) in a Q-step.  R is split once
// and stays in registers; a block's S1 and S2 rows are split once for the workgroup into LDS.
// With the lane on i in both products, the first one's output registers are the second one's
// operand: no transpose of X.  From rank 128 on R and Acc of all ranks would not leave registers
// for two waves per SIMD, so KH waves share a block of 32 i: each takes RK / KH of the ranks in
// both products, and they exchange their shares of D through LDS, added in order by each.
//
// MFMA layout (v_mfma_f32_32x32x16_bf16, one wave): D (32 x 32) += A (32 x 16) B (16 x 32).  Lane l
// supplies A[l % 32][8 (l / 32) + e] and B[8 (l / 32) + e][l % 32], e < 8; register v of lane l holds
// D[8 (v / 4) + 4 (l / 32) + v % 4][l % 32].  The K index of a step may map to any 16 indices as long
// as A and B agree: the second product takes j = jrow(s, h, e) on half h at step s, which is where
// the first one's registers 8 s + e hold it.
#include "device.hpp"

namespace acp {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

__device__ inline uint32_t u32(int64_t x) { return static_cast<uint32_t>(x); }
__device__ inline v16f zero16() {
  v16f z;
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = 0.f;
  return z;
}
__device__ inline v16f mfma(const v8bf& a, const v8bf& b, const v16f& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// the j of K element e on half h at step s of the second product
__device__ inline int jrow(int s, int h, int e) { return 16 * s + 4 * h + (e & 3) + 8 * (e >> 2); }

// Eight floats as three bf16 parts.
struct Split {
  v8bf p[3];  // hi, mid, lo
};
__device__ inline Split split8(const float (&x)[8]) {
  Split s;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    // (the residual from the packed parts: from x itself, masked, the rank-256 decompress took 652 us
    // instead of 613)
    const uint32_t x0 = __builtin_bit_cast(uint32_t, x[e]), x1 = __builtin_bit_cast(uint32_t, x[e + 1]);
    const v2bf hi = __builtin_bit_cast(v2bf, __builtin_amdgcn_perm(x1, x0, 0x07060302u));
    const uint32_t wh = __builtin_bit_cast(uint32_t, hi);
    v2f r = {x[e] - __builtin_bit_cast(float, wh << 16), x[e + 1] - __builtin_bit_cast(float, wh & 0xffff0000u)};
    const v2bf mid = __builtin_convertvector(r, v2bf);
    const uint32_t w = __builtin_bit_cast(uint32_t, mid);
    r[0] -= __builtin_bit_cast(float, w << 16);
    r[1] -= __builtin_bit_cast(float, w & 0xffff0000u);
    const v2bf lo = __builtin_convertvector(r, v2bf);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      s.p[0][e + k] = hi[k];
      s.p[1][e + k] = mid[k];
      s.p[2][e + k] = lo[k];
    }
  }
  return s;
}
// D += A B with split operands, the small products first; mfma5 without the high product.
__device__ inline v16f mfma5(const Split& a, const Split& b, v16f d) {
  d = mfma(a.p[2], b.p[0], d);
  d = mfma(a.p[0], b.p[2], d);
  d = mfma(a.p[1], b.p[1], d);
  d = mfma(a.p[1], b.p[0], d);
  return mfma(a.p[0], b.p[1], d);
}
__device__ inline v16f mfma6(const Split& a, const Split& b, const v16f& d) {
  return mfma(a.p[0], b.p[0], mfma5(a, b, d));
}

constexpr int kWalk = 32;   // walked indices per block
constexpr int kPitchM = 36;  // floats per row of a staging tile: 16-byte words of 16 lanes on all banks

// LDS tile of split factor rows [32][RK] for an operand whose lane holds row l % 32 and eight
// consecutive ranks; rows padded by 16 bytes (16 lanes' words then fall on all 64 banks).
template <int RK>
struct RowTile {
  static constexpr int LD = RK + 8;
  __bf16 p[3][32 * LD];
  __device__ void put(int row, int k, const Split& s) {
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<v8bf*>(&p[q][row * LD + k]) = s.p[q];
  }
  __device__ Split get(int row, int k) const {
    Split s;
#pragma unroll
    for (int q = 0; q < 3; ++q) s.p[q] = *reinterpret_cast<const v8bf*>(&p[q][row * LD + k]);
    return s;
  }
  __device__ v8bf high(int row, int k) const { return *reinterpret_cast<const v8bf*>(&p[0][row * LD + k]); }
};
// The transposed form [RK][32] for an operand whose lane holds rank l % 32 of a 32-rank block and
// eight of the 32 rows, rows in the order of jrow: (s, h, e) at 16 s + 8 h + e.
template <int RK>
struct RankTile {
  static constexpr int LD = 32 + 8;
  __bf16 p[3][RK * LD];
  __device__ void put(int rank, int sh, const Split& s) {
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<v8bf*>(&p[q][rank * LD + 8 * sh]) = s.p[q];
  }
  __device__ Split get(int rank, int sh) const {
    Split s;
#pragma unroll
    for (int q = 0; q < 3; ++q) s.p[q] = *reinterpret_cast<const v8bf*>(&p[q][rank * LD + 8 * sh]);
    return s;
  }
};

// The resource of the 32 rows from row j of a factor of `rows` rows (zeros past them).
template <int RK>
__device__ inline Rsrc block_rsrc(const float* f, int64_t j, int64_t rows) {
  const int64_t left = rows - j;
  return tile_rsrc(f + (left > 0 ? j : 0) * RK, left > 0 ? u32(left < kWalk ? left : kWalk) * RK * 4u : 0u);
}

// A block's rows of a factor (32 x RK floats, block_rsrc) on their way into a tile: IT items of
// eight floats per thread, requested one block ahead.
template <int RK, int NT>
struct RowFetch {
  static constexpr int IT = 4 * RK / NT;  // items: eight consecutive ranks of a row
  static_assert(IT * NT == 4 * RK, "whole items per thread");
  float x[IT][8];
  __device__ void load(Rsrc r) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int it = tid() + i * NT, c = it % (RK / 8), j = it / (RK / 8);
      const uint32_t o = u32(j * RK + 8 * c) * 4u;
      const float4 a = bld4(r, o), b = bld4(r, o + 16u);
      x[i][0] = a.x; x[i][1] = a.y; x[i][2] = a.z; x[i][3] = a.w;
      x[i][4] = b.x; x[i][5] = b.y; x[i][6] = b.z; x[i][7] = b.w;
    }
  }
  __device__ void put(RowTile<RK>& t) const {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int it = tid() + i * NT;
      t.put(it / (RK / 8), 8 * (it % (RK / 8)), split8(x[i]));
    }
  }
};
template <int RK, int NT>
struct RankFetch {
  static constexpr int IT = 4 * RK / NT;  // items: eight rows (jrow order) of a rank
  float x[IT][8];
  __device__ void load(Rsrc r) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int it = tid() + i * NT, rank = it % RK, sh = it / RK;
#pragma unroll
      for (int e = 0; e < 8; ++e) x[i][e] = bld1(r, u32(jrow(sh >> 1, sh & 1, e) * RK + rank) * 4u);
    }
  }
  __device__ void put(RankTile<RK>& t) const {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int it = tid() + i * NT;
      t.put(it % RK, it / RK, split8(x[i]));
    }
  }
};

// A 32 x 32 block of M and E (or of X, M_hat on the way out) moves as 16-byte words, eight
// lanes per row of 128 bytes: word u of lane l is row l / 8 + 8 u, columns 4 (l % 8) ... + 3.  The
// block starts at byte `at` of the resource; rows from `rows` on are left out, and `cols` columns
// are in the matrix (a block with fewer than 32 moves float by float when the row length is not a
// multiple of four: its last word would reach into the next row; one with none moves nothing).
template <int NU>
struct BlockMove {
  uint32_t off[NU];  // byte offset of the lane's words u0 ... u0 + NU - 1
  int c, w;          // first column of the words, LDS index of the first
  __device__ BlockMove(int lane, int u0, uint32_t row_bytes, int rows) : c(4 * (lane & 7)) {
    w = ((lane >> 3) + 8 * u0) * kPitchM + c;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int row = (lane >> 3) + 8 * (u0 + u);
      off[u] = row < rows ? u32(row) * row_bytes + u32(c) * 4u : kOut;
    }
  }
  __device__ float4* word(float* tile, int u) const { return reinterpret_cast<float4*>(tile + w + 8 * u * kPitchM); }
  __device__ static float4 load1(Rsrc r, uint32_t o, int left) {  // left: columns in the matrix from here
    return make_float4(bld1_nt(r, left > 0 ? o : kOut), bld1_nt(r, left > 1 ? o + 4u : kOut),
                       bld1_nt(r, left > 2 ? o + 8u : kOut), bld1_nt(r, left > 3 ? o + 12u : kOut));
  }
  // m4: the row length is a multiple of four
  __device__ float4 load(Rsrc r, uint32_t at, int u, int64_t cols, bool m4) const {
    const int left = cols < 32 ? static_cast<int>(cols) - c : 4;
    const uint32_t o = at + off[u];
    return cols >= 32 || m4 ? bld4_nt(r, left > 0 ? o : kOut) : load1(r, o, left);
  }
  __device__ void store(Rsrc r, uint32_t at, int u, int64_t cols, bool m4, const float4& v) const {
    const int left = cols < 32 ? static_cast<int>(cols) - c : 4;
    const uint32_t o = at + off[u];
    if (cols >= 32 || m4) {
      bst4_nt(r, left > 0 ? o : kOut, v);
    } else {
      bst1_nt(r, left > 0 ? o : kOut, v.x);
      bst1_nt(r, left > 1 ? o + 4u : kOut, v.y);
      bst1_nt(r, left > 2 ? o + 8u : kOut, v.z);
      bst1_nt(r, left > 3 ? o + 12u : kOut, v.w);
    }
  }
};

// Waves that share a block of 32 fixed indices, and blocks per workgroup.
constexpr int rank_waves(int rk) { return rk >= 256 ? 4 : rk >= 128 ? 2 : 1; }
constexpr int fix_blocks(int rk) { return split_fix(rk) / 32; }

// Compress step (see above).  PS: P-step over rows [t.a, t.a + t.b) (t.b <= split_fix) and all
// columns, P_loc to the factor buffer and its slot.  Else Q-step over row chunk t.a and column
// block t.b of split_fix columns, the product to the chunk's partials for K_QFIN.
// The product's sum is that of its parts of split_part(r) walked indices, in order; a list with too
// few tiles to fill the GPU (split_full_tiles) takes one tile per part (P-step: t.b >> 8 is the part
// + 1; Q-step: variant kWideFine, t.a = chunk * parts + part), whose sums go to the fine partials
// and are added by k_wpfin or K_QFIN in the same order: the same bits either way.  (One 186 x 5166
// matrix at rank 64 is two tiles of 162 blocks: 774 us per two steps whole, 332 by parts.)  The sums
// by parts are also closer to 64 bits (BERT-large rank 64, worst output 1.6e-6 to 0.7e-6).
// Per block of 32 walked indices: the next block's M, E and factor rows are requested before this
// block's products; a 32 x 32 block of M + E goes through an LDS tile (read with the lane on i) and
// X back, so that memory sees 16-byte words; the factor tiles are shared, with a barrier before
// and after their use.
template <int RK, bool PS>
__global__ __launch_bounds__(64 * fix_blocks(RK) * rank_waves(RK), 2) void k_bstep(KArgs a) {
  constexpr int KH = rank_waves(RK), IB = fix_blocks(RK), NT = 64 * KH * IB, FIX = 32 * IB;
  constexpr int RS = RK / KH, NK = RS / 16, NR = RS / 32;  // the wave's ranks
  constexpr int NU = 4 / KH;                               // its words of the block
  const Tile t = a.tiles[blockIdx.x];
  if (t.kind == T_VEC) {  // a raw vector packed into the factor buffer
    vec_tile(a, t, true);
    return;
  }
  const MatDesc d = a.mats[t.idx];
  const int wave = __builtin_amdgcn_readfirstlane(tid() >> 6);
  const int ib = wave / KH, kh = wave % KH;
  const int lane = tid() & 63, h = lane >> 5, li = lane & 31;
  const int64_t n = d.n, m = d.m;
  const bool m4 = (m & 3) == 0;
  // the tile's rows and first column; walked indices
  constexpr int PART = split_part(RK);
  constexpr bool NEST = split_nested(RK);
  const int parts = (d.q_rows + PART - 1) / PART;  // of a Q-step chunk
  const int part = PS ? (t.b >> 8) - 1 : NEST && a.variant == kWideFine ? t.a % parts : -1;  // -1: all of them
  const int chunk = PS || part < 0 ? t.a : t.a / parts;
  const int64_t r0 = PS ? t.a : static_cast<int64_t>(chunk) * d.q_rows + (part > 0 ? part * PART : 0);
  const int64_t c0 = PS ? (part > 0 ? static_cast<int64_t>(part) * PART : 0) : static_cast<int64_t>(t.b) * FIX;
  const int64_t rend = part >= 0 && part + 1 < parts ? r0 + PART : static_cast<int64_t>(chunk + 1) * d.q_rows;
  const int rows = PS ? t.b & 0xff : static_cast<int>((rend < n ? rend : n) - r0);
  const int64_t walk = !PS ? rows : part >= 0 && m - c0 > PART ? PART : m - c0;
  const uint32_t row_bytes = u32(m) * 4u;
  // the wave's part of the tile: its rows (P-step) or columns (Q-step) and resources, at most 2^31
  // bytes (a row is at most 2^26, a Q-step chunk 2^30)
  const int wrows = PS ? (rows - 32 * ib < 32 ? rows - 32 * ib : 32) : rows;
  const int64_t wm = PS ? m - c0 : m - c0 - 32 * ib;
  const bool on = wrows > 0 && wm > 0;
  const int64_t first = on ? (PS ? (r0 + 32 * ib) * m + c0 : r0 * m + c0 + 32 * ib) : 0;
  const uint32_t ext = on ? u32(wrows - 1) * row_bytes + u32(wm) * 4u : 0u;
  const Rsrc G = tile_rsrc(src_of(a, d.bucket) + d.grad_off + first, ext);
  const Rsrc E = tile_rsrc(a.e + d.e_off + first, a.ef ? ext : 0u);
  const bool term = PS ? deferred_of(a, d.bucket) : deferred_p_of(a, d);
  const int64_t f0 = PS ? r0 : c0;                              // first fixed index
  const int64_t fix = PS ? rows : (m - c0 < FIX ? m - c0 : FIX);  // fixed indices of the tile
  const int64_t w0 = PS ? c0 : r0;                              // first walked index
  const Rsrc R = tile_rsrc(a.fac + (PS ? d.ph_slot : d.qh_slot) + f0 * RK, term ? u32(fix) * RK * 4u : 0u);
  const float* S1 = a.fac + (PS ? d.ql_slot : d.pl_slot) + w0 * RK;
  const float* S2 = a.fac + (PS ? (a.image ? d.q_slot : d.qh_slot) : d.ph_slot) + w0 * RK;

  __shared__ __attribute__((aligned(16))) RowTile<RK> s1;
  __shared__ __attribute__((aligned(16))) RankTile<RK> s2;
  __shared__ __attribute__((aligned(16))) float stage[IB][32 * kPitchM];
  __shared__ float4 share[KH > 1 ? IB * KH : 1][4][64];  // the waves' shares of D
  float* st = stage[ib];
  // the block at walked index j: byte offset of its first element and its columns (none past the
  // walk); the wave moves words kh NU ... of it
  const BlockMove<NU> mv(lane, kh * NU, row_bytes, PS ? wrows : 32);
  auto at = [&](int64_t j) { return PS ? u32(j) * 4u : u32(j) * row_bytes; };
  auto cols = [&](int64_t j) { return j >= walk ? 0 : PS ? wm - j : wm; };
  // a left-out row's kOut plus a P-step's offset in the row (a Q-step leaves out none) does not wrap
  static_assert(uint64_t{kOut} + 4 * uint64_t(kMaxCols + kWalk) < uint64_t{1} << 32, "kOut stays past the tile");

  float4 g[NU], e[NU];
  RowFetch<RK, NT> x1;
  RankFetch<RK, NT> x2;
  auto fetch = [&](int64_t j) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      g[u] = mv.load(G, at(j), u, cols(j), m4);
      e[u] = mv.load(E, at(j), u, cols(j), m4);
    }
    if (term) x1.load(block_rsrc<RK>(S1, j, walk));
    x2.load(block_rsrc<RK>(S2, j, walk));
  };
  fetch(0);
  // the lane's row of R: ranks RS kh + 16 s + 8 h + e
  Split rs[NK];
  if (term)
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      const uint32_t o = u32((32 * ib + li) * RK + RS * kh + 16 * s + 8 * h) * 4u;
      const float4 p = bld4(R, o), q = bld4(R, o + 16u);
      const float x[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
      rs[s] = split8(x);
    }
  v16f acc[NR], tot[NEST ? NR : 1];  // the sum of the current part, of the parts before it
#pragma unroll
  for (int kb = 0; kb < NR; ++kb) {
    acc[kb] = zero16();
    if constexpr (NEST) tot[kb] = zero16();
  }

  for (int64_t j = 0; j < walk; j += kWalk) {
    if (term) x1.put(s1);
    x2.put(s2);
#pragma unroll
    for (int u = 0; u < NU; ++u) *mv.word(st, u) = g[u] + e[u];
    __syncthreads();
    fetch(j + kWalk);  // past the walk: nothing is used, no traffic
    // M + E with the lane on i
    float x[16];
    if constexpr (PS) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(st + li * kPitchM + 8 * q + 4 * h);
        x[4 * q] = v.x; x[4 * q + 1] = v.y; x[4 * q + 2] = v.z; x[4 * q + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) x[v] = st[(8 * (v >> 2) + 4 * h + (v & 3)) * kPitchM + li];
    }
    if (term) {
      v16f dt = zero16();
#pragma unroll
      for (int s = 0; s < NK; ++s) dt = mfma6(s1.get(li, RS * kh + 16 * s + 8 * h), rs[s], dt);
      if constexpr (KH > 1) {
#pragma unroll
        for (int q = 0; q < 4; ++q) share[wave][q][lane] = make_float4(dt[4 * q], dt[4 * q + 1], dt[4 * q + 2], dt[4 * q + 3]);
        __syncthreads();  // every wave of the block has read M + E and written its share
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float4 s = share[ib * KH][q][lane];
#pragma unroll
          for (int w = 1; w < KH; ++w) s = s + share[ib * KH + w][q][lane];
          dt[4 * q] = s.x; dt[4 * q + 1] = s.y; dt[4 * q + 2] = s.z; dt[4 * q + 3] = s.w;
        }
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) x[v] -= dt[v];
      // X back to the LDS tile, a share of it by each of the block's waves
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q / NU != kh) continue;
        if constexpr (PS) {
          *reinterpret_cast<float4*>(st + li * kPitchM + 8 * q + 4 * h) =
              make_float4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
        } else {
#pragma unroll
          for (int v = 4 * q; v < 4 * q + 4; ++v) st[(8 * q + 4 * h + (v & 3)) * kPitchM + li] = x[v];
        }
      }
    }
    // the product
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const float xe[8] = {x[8 * s], x[8 * s + 1], x[8 * s + 2], x[8 * s + 3],
                           x[8 * s + 4], x[8 * s + 5], x[8 * s + 6], x[8 * s + 7]};
      const Split xs = split8(xe);
#pragma unroll
      for (int kb = 0; kb < NR; ++kb) acc[kb] = mfma6(s2.get(RS * kh + 32 * kb + li, 2 * s + h), xs, acc[kb]);
    }
    __syncthreads();  // every wave has read the factor tiles and written its share of X
#pragma unroll
    for (int u = 0; u < NU; ++u) mv.store(E, at(j), u, cols(j), m4, *mv.word(st, u));
    if (NEST && (j + kWalk) % PART == 0 && j + kWalk < walk) {  // the part ends and another follows
#pragma unroll
      for (int kb = 0; kb < NR; ++kb) {
        tot[kb] += acc[kb];
        acc[kb] = zero16();
      }
    }
  }
#pragma unroll
  for (int kb = 0; kb < NR; ++kb)
    if constexpr (NEST) acc[kb] = tot[kb] + acc[kb];

  // lane l: fixed index 32 ib + l % 32, ranks RS kh + 32 kb + 8 q + 4 h ... + 3
  const int64_t i = 32 * ib + li;
  if (i >= fix) return;
  float *o1, *o2 = nullptr;
  if constexpr (PS) {
    if (part >= 0) {
      o1 = a.qpart + d.qpart + (static_cast<int64_t>(part) * n + r0 + i) * RK;
    } else {
      o1 = dst_of(a, d.bucket) + d.fac_off_p + (r0 + i) * RK;
      o2 = a.fac + d.pl_slot + (r0 + i) * RK;
    }
  } else {
    const int64_t ncb = (m + d.q_cb - 1) / d.q_cb;
    o1 = a.qpart + d.qpart + static_cast<int64_t>(t.a) * ncb * d.q_cb * RK + (c0 + i) * RK;
  }
  typedef float v4u_f __attribute__((ext_vector_type(4), aligned(4)));  // the factor buffer is 4-byte aligned
#pragma unroll
  for (int kb = 0; kb < NR; ++kb)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const v4u_f v = {acc[kb][4 * q], acc[kb][4 * q + 1], acc[kb][4 * q + 2], acc[kb][4 * q + 3]};
      const int k = RS * kh + 32 * kb + 8 * q + 4 * h;
      *reinterpret_cast<v4u_f*>(o1 + k) = v;
      if (PS && part < 0) *reinterpret_cast<v4u_f*>(o2 + k) = v;
    }
}

// Decompress, M_hat = A B^T / p, over 128 rows and a.variant columns (tile t.a, t.b): wave w keeps rows
// 32 w ... of A / p split in registers, the workgroup walks the columns in blocks of 32 whose rows
// of B are split once into LDS (two tiles in turn, one barrier per block), and the lane on the row
// holds four adjacent columns per register group: the wave's block goes through its staging tile
// and out as 16-byte words.
template <int RK>
__global__ __launch_bounds__(kBlock, RK == 64 ? 2 : 1) void k_brecon(KArgs a) {
  constexpr int NK = RK / 16;
  const Tile t = a.tiles[blockIdx.x];
  const bool odd = a.parity != 0;
  const MatDesc d = a.mats[t.idx];
  const int wave = __builtin_amdgcn_readfirstlane(tid() >> 6);
  const int lane = tid() & 63, h = lane >> 5, li = lane & 31;
  const int64_t n = d.n, m = d.m;
  const bool m4 = (m & 3) == 0;
  const int64_t r0 = static_cast<int64_t>(t.a) * kSplitRecon, c0 = static_cast<int64_t>(t.b) * a.variant;
  const int rows = static_cast<int>((r0 + kSplitRecon < n) ? kSplitRecon : n - r0);
  const int64_t wcols = m - c0 < a.variant ? m - c0 : a.variant;
  const float* agg = src_of(a, d.bucket);
  const Rsrc A = tile_rsrc((odd ? agg + d.fac_off_p : a.fac + d.ph_slot) + r0 * RK, u32(rows) * RK * 4u);
  const float* B = (odd ? a.fac + d.qh_slot : agg + d.fac_off_q) + c0 * RK;
  const uint32_t row_bytes = u32(m) * 4u;
  const int wrows = rows - 32 * wave < 32 ? rows - 32 * wave : 32;  // the wave's rows
  const float* Ob = dst_of(a, d.bucket) + d.grad_off + (wrows > 0 ? (r0 + 32 * wave) * m + c0 : 0);
  const Rsrc O = tile_rsrc(Ob, wrows > 0 ? u32(wrows - 1) * row_bytes + u32(wcols) * 4u : 0u);
  __shared__ __attribute__((aligned(16))) RowTile<RK> bt[2];
  __shared__ __attribute__((aligned(16))) float stage[4][32 * kPitchM];
  float* st = stage[wave];
  const BlockMove<4> mv(lane, 0, row_bytes, wrows);
  RowFetch<RK, kBlock> xb;
  xb.load(block_rsrc<RK>(B, 0, wcols));
  Split as[NK];
#pragma unroll
  for (int s = 0; s < NK; ++s) {
    const uint32_t o = u32((32 * wave + li) * RK + 16 * s + 8 * h) * 4u;
    const float4 p = bld4(A, o), q = bld4(A, o + 16u);
    float x[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] *= a.inv_p;
    as[s] = split8(x);
  }
  int buf = 0;
  for (int64_t j = 0; j < wcols; j += kWalk, buf ^= 1) {
    xb.put(bt[buf]);
    __syncthreads();
    xb.load(block_rsrc<RK>(B, j + kWalk, wcols));
    // all small products before the high ones, whose large sum is then rounded RK / 16 times, not
    // 6 RK / 16 (rank 256: error of M_hat 2.4e-7 one rank block after the other, 0.9e-7 this way;
    // the fp32 matrix cores' was 1.5e-7)
    v16f o = zero16();
#pragma unroll
    for (int s = 0; s < NK; ++s) o = mfma5(bt[buf].get(li, 16 * s + 8 * h), as[s], o);
    // at rank 256 the high parts of B are read again, not held (BERT-base 3770 us per two steps, held
    // 3900); at 128 holding them is faster by 0.3 % (BERT-large)
    if constexpr (RK >= 256) wave_lds_fence();
#pragma unroll
    for (int s = 0; s < NK; ++s) o = mfma(bt[buf].high(li, 16 * s + 8 * h), as[s].p[0], o);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(st + li * kPitchM + 8 * q + 4 * h) =
          make_float4(o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]);
    wave_lds_fence();  // other lanes' rows are read back (the next block's barrier follows these reads)
#pragma unroll
    for (int u = 0; u < 4; ++u) mv.store(O, u32(j) * 4u, u, m - c0 - j, m4, *mv.word(st, u));
  }
}

template <int RK>
hipError_t launch_split_rank(const Launch& l, const KArgs& args, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(l.ntiles)), block(64 * fix_blocks(RK) * rank_waves(RK));
  switch (l.kernel) {
    case K_WPSTEP: hipLaunchKernelGGL((k_bstep<RK, true>), grid, block, 0, s, args); break;
    case K_WQSTEP: hipLaunchKernelGGL((k_bstep<RK, false>), grid, block, 0, s, args); break;
    case K_WRECON: hipLaunchKernelGGL(k_brecon<RK>, grid, dim3(kBlock), 0, s, args); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_split(const Launch& l, int32_t rank, const KArgs& args, hipStream_t s) {
  switch (rank) {
    case 64: return launch_split_rank<64>(l, args, s);
    case 128: return launch_split_rank<128>(l, args, s);
    case 256: return launch_split_rank<256>(l, args, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace acp
