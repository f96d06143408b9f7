// gfx950 kernels of the ACP-SGD compressor (arXiv 2306.08881, Algorithms 1 and 2) that every rank
// shares: the orthogonalisation of ranks 8 and up, the Q-step finish, the factor tiles, the draws
// and exports, and the launch dispatch.  The streaming kernels of ranks 1, 2 and 4 are in
// lowrank.hip, the MFMA kernels of ranks 8 to 32 in wide.hip, those of ranks 64 to 256 in split.hip.
//
// Every kernel runs 256-thread workgroups (4 waves of 64) over a table of tiles; one
// workgroup per tile.  Workgroups never wait for each other: a reduction that spans
// workgroups writes per-tile partial sums and a later kernel of the same stream adds them in
// tile order.  Together with fixed-order wave butterflies and fixed-order sums across waves
// this makes every result bitwise reproducible, which a data-parallel job needs so that all
// ranks keep the same orthogonalised factor.
//
// The error-feedback residual of a Q-step (E_t = M' - P_hat Q_t^T) is kept in deferred form:
// the Q-step writes F = M' into the E arena and the next P-step subtracts the rank-r term
// P_hat Q_loc^T while it streams F, so each step reads M and E once and writes E once.
#include "device.hpp"

#include <mutex>
#include <vector>

namespace acp {

hipError_t launch_wide(const Launch& l, int32_t rank, const KArgs& args, hipStream_t s);
hipError_t launch_low(const Launch& l, int32_t rank, const KArgs& args, hipStream_t s);

namespace {

// Factor tiles alone: W of the P (variant bit 0 clear) or Q factor of a matrix, read from its slot,
// or with kFactFromBuffer from the aggregated factor buffer and copied into the slot.
template <int RK>
__global__ __launch_bounds__(kBlock) void k_fact(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  const bool q = (a.variant & 1) != 0;
  float* slot = a.fac + (q ? d.q_slot : d.p_slot);
  if (a.variant & kFactFromBuffer)
    fact_tile<RK>(a, t, src_of(a, d.bucket) + (q ? d.fac_off_q : d.fac_off_p), slot, q ? d.m : d.n);
  else
    fact_tile<RK>(a, t, slot, nullptr, q ? d.m : d.n);
}

// No reuse (the ablation of Section V-B): the factor a step would have reused is drawn anew, i.i.d.
// standard normal, from the initial factors' counter-based generator with the step in the high
// half of the key: element i (row-major) of factor f (0: P, 1: Q) of tensor k at step t takes the
// SplitMix64 outputs x = mix(s + (2i + 1) g), y = mix(s + (2i + 2) g) of the stream
// s = mix(seed ^ mix(t 2^32 + 2k + f)) and becomes sqrt(-2 ln u1) cos(2 pi u2) in fp64 with
// u1 = ((x >> 11) + 1) 2^-53, u2 = (y >> 11) 2^-53, rounded to fp32.  Tile: factor rows
// [t.a, t.a + t.b) of the P (variant 0) or Q (variant 1) slot.
__device__ inline uint64_t splitmix_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

template <int RK>
__global__ __launch_bounds__(kBlock) void k_draw(KArgs a) {
  constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
  constexpr double kTwoPi = 2.0 * 3.14159265358979323846;
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  const uint64_t f = static_cast<uint64_t>(a.variant & 1);
  float* slot = a.fac + (f ? d.q_slot : d.p_slot);
  const uint64_t key = (static_cast<uint64_t>(a.step) << 32) + 2ull * static_cast<uint64_t>(d.tid) + f;
  const uint64_t s = splitmix_mix(a.seed ^ splitmix_mix(key));
  const int64_t e0 = static_cast<int64_t>(t.a) * RK, ne = static_cast<int64_t>(t.b) * RK;
  for (int64_t k = tid(); k < ne; k += kBlock) {
    const uint64_t i = static_cast<uint64_t>(e0 + k);
    const uint64_t x = splitmix_mix(s + (2ull * i + 1ull) * kGamma);
    const uint64_t y = splitmix_mix(s + (2ull * i + 2ull) * kGamma);
    const double u1 = static_cast<double>((x >> 11) + 1ull) * 0x1.0p-53;
    const double u2 = static_cast<double>(y >> 11) * 0x1.0p-53;
    const double rad = sqrt(-2.0 * log(u1));
    const double ang = cos(kTwoPi * u2);
    slot[e0 + k] = static_cast<float>(rad * ang);
  }
}

// C = C0 + sg A B for 128 x 128 fp64 blocks in global or shared memory (sg = +1 or -1; C0 = 0
// when c0 is null, else C0[i][j] = c0[i * ldc + j]), by the whole workgroup on the fp64 matrix
// cores: wave w forms the 64 x 64 quadrant at rows 64 (w / 2), columns 64 (w % 2) as 4 x 4
// products of 16 x 16 (v_mfma_f64_16x16x4f64; operand entry [i][k] on lane i + 16 k, result
// entry [4 v + l / 16][l % 16] in item v of lane l), each entry C0 plus a sum over k < 128 in
// increasing groups of four, with A[i][k] = A[i * ai + k * ak] and B[k][j] = B[k * bk + j];
// store(i, j, value) takes the entries.  The next group's operands are requested before the
// current group's products.
template <typename Store>
__device__ void mm128(const double* A, int ai, int ak, const double* B, int bk, const double* c0, int ldc,
                      double sg, Store store) {
  static_assert(kBlock == 4 * kWave, "one 64 x 64 quadrant per wave");
  const int lane = tid() % kWave, i = lane % 16, k = lane / 16;
  const int i0 = 64 * (tid() / kWave / 2), j0 = 64 * (tid() / kWave % 2);
  v4d acc[4][4];
#pragma unroll
  for (int ra = 0; ra < 4; ++ra)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        acc[ra][cb][v] = c0 ? c0[(i0 + 16 * ra + 4 * v + k) * ldc + j0 + 16 * cb + i] : 0.0;
  struct Ops {
    double a[4], b[4];
  };
  auto fetch = [&](int k0, Ops& o) {
#pragma unroll
    for (int ra = 0; ra < 4; ++ra) o.a[ra] = A[(i0 + 16 * ra + i) * ai + (k0 + k) * ak];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) o.b[cb] = B[(k0 + k) * bk + j0 + 16 * cb + i];
  };
  auto step = [&](const Ops& o) {
#pragma unroll
    for (int ra = 0; ra < 4; ++ra)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        acc[ra][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(sg * o.a[ra], o.b[cb], acc[ra][cb], 0, 0, 0);
  };
  // 32 groups of four, taken in pairs; past the last pair the request repeats the last group
  Ops o0, o1;
  fetch(0, o0);
  for (int k0 = 0; k0 < 128; k0 += 8) {
    fetch(k0 + 4, o1);
    __builtin_amdgcn_sched_barrier(0);  // requests ahead of the products that do not need them
    step(o0);
    __builtin_amdgcn_sched_barrier(0);
    fetch(k0 + 8 < 128 ? k0 + 8 : 124, o0);
    __builtin_amdgcn_sched_barrier(0);
    step(o1);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int ra = 0; ra < 4; ++ra)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) store(i0 + 16 * ra + 4 * v + k, j0 + 16 * cb + i, acc[ra][cb][v]);
}

// Dst[e] = Src[(e / C) * lds + e % C] for e < R * C (R x C doubles from global memory into shared
// memory), by the whole workgroup; each thread requests 16 entries before it stores them (one
// request in flight at a time costs a memory latency per entry).
template <int R, int C>
__device__ void rows_to_lds(double* Dst, const double* Src, int lds) {
  constexpr int PT = R * C / kBlock, U = 16;
  static_assert(PT % U == 0, "whole batches");
#pragma unroll 1
  for (int c = 0; c < PT; c += U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = tid() + (c + u) * kBlock;
      v[u] = Src[(e / C) * lds + e % C];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) Dst[tid() + (c + u) * kBlock] = v[u];
  }
}

// W = R^-1 of a 256 x 256 Gram matrix G (global memory: the matrix's first Gram partial, which
// holds the slices' sum) in 2 x 2 blocks of 128, from the factorisation
//   G11 = R11^T R11,  R12 = R11^-T G12,  G22 - R12^T R12 = R22^T R22,
//   W11 = R11^-1,  W22 = R22^-1,  W12 = -W11 R12 W22,  W21 = 0,
// the same pivots in the same order as the unblocked form.  With dropped pivots R11^-T G12 is
// W11^T G12 (W11's zero columns give R12's zero rows) and the pivots of the second block are
// tested against G's own diagonal.  R12 (called Y) is kept in G's lower left block, which the
// upper triangle makes redundant; the shared block S holds G11, then G22 - Y^T Y, then Y W22.
__device__ void chol_split(double* G, double* W, double* S) {
  constexpr int N = 256, H = 128;
  rows_to_lds<H, H>(S, G, N);
  __syncthreads();
  cholesky_w_blocked<H>(S, W, N);  // W11
  __syncthreads();
  double* Y = G + H * N;  // Y[i][j] at Y[i * N + j]
  // Y = W11^T G12
  mm128(W, 1, N, G + H, N, nullptr, 0, 1.0, [&](int i, int j, double v) { Y[i * N + j] = v; });
  __syncthreads();
  // S = G22 - Y^T Y
  mm128(Y, 1, N, Y, N, G + H * N + H, N, -1.0, [&](int i, int j, double v) { S[i * H + j] = v; });
  __syncthreads();
  cholesky_w_blocked<H>(S, W + H * N + H, N, G + H * N + H, N + 1);  // W22
  __syncthreads();
  // S = Y W22
  mm128(Y, N, 1, W + H * N + H, N, nullptr, 0, 1.0, [&](int i, int j, double v) { S[i * H + j] = v; });
  __syncthreads();
  // W12 = -W11 (Y W22)
  mm128(W, N, 1, S, H, nullptr, 0, -1.0, [&](int i, int j, double v) { W[i * N + H + j] = v; });
  for (int e = tid(); e < H * H; e += kBlock) W[(H + e / H) * N + e % H] = 0.0;
}

// From kBlockedRank on: entries [t.a kGsumEntries, ...) of a matrix's Gram, the sum of its t.b
// slices' partials in slice order, into the first partial.  The partials hold the 4 x 4 blocks
// on and above the diagonal; the thread of an entry of a block above the diagonal also writes
// its mirror, so every entry is read and written by one thread only.
template <int RK>
__global__ __launch_bounds__(kBlock) void k_gsum(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  double* gp = a.gpart + d.gpart;
  constexpr int EPT = kGsumEntries / kBlock;  // entries per thread, 256 apart
  static_assert(kGsumEntries % kBlock == 0 && (RK * RK) % kGsumEntries == 0, "whole tiles");
  int64_t e[EPT];
  bool up[EPT];
  double s[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    e[k] = static_cast<int64_t>(t.a) * kGsumEntries + tid() + k * kBlock;
    up[k] = (e[k] / RK) / 4 <= (e[k] % RK) / 4;
    s[k] = 0.0;
  }
  for (int sl = 0; sl < t.b; ++sl) {
    double v[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) v[k] = up[k] ? gp[static_cast<int64_t>(sl) * RK * RK + e[k]] : 0.0;
#pragma unroll
    for (int k = 0; k < EPT; ++k) s[k] += v[k];
  }
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    if (!up[k]) continue;
    const int i = static_cast<int>(e[k] / RK), j = static_cast<int>(e[k] % RK);
    gp[e[k]] = s[k];
    if (i / 4 < j / 4) gp[j * RK + i] = s[k];
  }
}

// W from the Gram partials of a matrix's t.b slices, added in slice order (from kBlockedRank on
// K_GSUM has added them into the first).
template <int RK>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(RK <= 32 ? 2 : 1))) void k_chol(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  constexpr bool SPLIT = RK >= kCholBlockRank;
  __shared__ double Gs[SPLIT ? 128 * 128 : RK >= kBlockedRank ? RK * RK : RK * gram_ld(RK)];
  double* gp = a.gpart + d.gpart;
  if constexpr (RK >= kBlockedRank) {
    if constexpr (SPLIT) {
      static_assert(RK == 256, "2 x 2 blocks of 128");
      chol_split(gp, a.w + d.w_slot, Gs);
    } else {
      rows_to_lds<RK, RK>(Gs, gp, RK);
      __syncthreads();
      cholesky_w_blocked<RK>(Gs, a.w + d.w_slot);
    }
  } else {
    // each entry added in slice order; per round, eight slices of all the thread's entries are
    // requested together (one round trip per eight slices)
    constexpr int EPT = (RK * RK + kBlock - 1) / kBlock;  // entries per thread
    double acc[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) acc[q] = 0.0;
    for (int sl = 0; sl < t.b; sl += 8) {
      double v[EPT][8];
#pragma unroll
      for (int q = 0; q < EPT; ++q) {
        const int e = tid() + q * kBlock;
#pragma unroll
        for (int w = 0; w < 8; ++w)
          v[q][w] = (e < RK * RK && sl + w < t.b) ? gp[static_cast<int64_t>(sl + w) * RK * RK + e] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < EPT; ++q)
#pragma unroll
        for (int w = 0; w < 8; ++w)
          if (sl + w < t.b) acc[q] += v[q][w];
    }
#pragma unroll
    for (int q = 0; q < EPT; ++q)
    {
      const int e = tid() + q * kBlock;
      if (e < RK * RK) Gs[e / RK * gram_ld(RK) + e % RK] = acc[q];
    }
    __syncthreads();
    cholesky_w<RK>(Gs, a.w + d.w_slot);
  }
}

// Xh = X W from kApplyMfmaRank on, for rows [t.a, t.a + rows) and the BW = min(r, 64) columns
// c0 = BW cb ... of Xh (t.b = rows | cb << 16), on the fp64 matrix cores: wave w forms rows
// 64 w ... + 63 as 4 x BW / 16 products of 16 x 16 (v_mfma_f64_16x16x4f64; operand entry
// [i][k] on lane i + 16 k, result entry [4 v + l / 16][l % 16] in item v of lane l), over the
// ranks 0 ... c0 + BW - 1 in steps of 16.  W is upper triangular: later ranks add zero, and so do the ranks from c0 + 16 (b + 1) on
// for the columns c0 + 16 b ... + 15, whose products are skipped.  Within a step, lane i + 16 k
// holds the four ranks 4 k ... + 3 of its row as one 16-byte word, and product s of the step
// takes rank 4 k + s from lane i + 16 k in both operands, so every rank enters once.  The next
// step's rows of X are requested before the current step's products.
template <int RK>
__device__ void apply_mfma(const KArgs& a, const Tile& t, const MatDesc& d) {
  constexpr int CB = RK >= 64 ? 4 : RK / 16;  // 16-column groups of the block
  static_assert(CB % 2 == 0, "the 16-rank steps are taken in pairs");
  const int rows = t.b & 0xffff, c0 = 16 * CB * (t.b >> 16);
  const int lane = tid() % kWave, i = lane % 16, k = lane / 16;
  const int rb = 64 * (tid() / kWave);
  if (rb >= rows) return;
  const bool q = a.variant == 1;
  const float* X = a.fac + (q ? d.q_slot : d.p_slot);
  float* Y = a.fac + (q ? d.qh_slot : d.ph_slot);
  const double* W = a.w + d.w_slot;
  // rows past the tile read its last row (no branch around the loads); they are not stored
  const float* xr[4];
#pragma unroll
  for (int ra = 0; ra < 4; ++ra) {
    const int r = rb + 16 * ra + i;
    xr[ra] = X + (static_cast<int64_t>(t.a) + (r < rows ? r : rows - 1)) * RK + 4 * k;
  }
  const double* wr = W + static_cast<int64_t>(4 * k) * RK + c0 + i;
  v4d acc[4][CB];
#pragma unroll
  for (int ra = 0; ra < 4; ++ra)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[ra][cb] = v4d{0.0, 0.0, 0.0, 0.0};
  // per step the W rows (from L2, where every tile of the matrix reads them) are requested
  // first, then the next step's X rows (from HBM), so that the wait for the former leaves the
  // latter in flight
  typedef float4 XBuf[4];
  auto fetch_x = [&](int k0, XBuf& b) {
#pragma unroll
    for (int ra = 0; ra < 4; ++ra) b[ra] = *reinterpret_cast<const float4*>(xr[ra] + k0);
  };
  auto step = [&](int k0, XBuf& b, int k1, XBuf& nb) {
    // column group cb of the block takes ranks up to c0 + 16 cb + 15 only (W is upper triangular)
    const int kz = k0 - c0;
    double w[4][CB];  // [s][cb]
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) w[s][cb] = wr[static_cast<int64_t>(k0 + s) * RK + 16 * cb];
    __builtin_amdgcn_sched_barrier(0);  // in this order
    fetch_x(k1, nb);
    __builtin_amdgcn_sched_barrier(0);
    // the conversions stay behind those requests
#pragma unroll
    for (int ra = 0; ra < 4; ++ra)
      asm volatile("" : "+v"(b[ra].x), "+v"(b[ra].y), "+v"(b[ra].z), "+v"(b[ra].w));
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double xa[4];
#pragma unroll
      for (int ra = 0; ra < 4; ++ra) {
        const float4 v = b[ra];
        xa[ra] = static_cast<double>(s == 0 ? v.x : s == 1 ? v.y : s == 2 ? v.z : v.w);
      }
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        if (kz <= 16 * cb)
#pragma unroll
          for (int ra = 0; ra < 4; ++ra)
            acc[ra][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[ra], w[s][cb], acc[ra][cb], 0, 0, 0);
    }
  };
  // c0 + BW ranks: an even number of 16-rank steps, taken in pairs; past the last pair the X
  // request repeats the last step's ranks, unused (no branch around it)
  const int kend = c0 + 16 * CB;
  XBuf x0, x1;
  fetch_x(0, x0);
  for (int k0 = 0; k0 < kend; k0 += 32) {
    step(k0, x0, k0 + 16, x1);
    step(k0 + 16, x1, min(k0 + 32, kend - 16), x0);
  }
#pragma unroll
  for (int ra = 0; ra < 4; ++ra)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = rb + 16 * ra + 4 * v + k;
      if (r < rows)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          Y[(static_cast<int64_t>(t.a) + r) * RK + c0 + 16 * cb + i] = static_cast<float>(acc[ra][cb][v]);
    }
}

template <int RK>
__global__ __launch_bounds__(kBlock, RK >= kApplyMfmaRank ? 2 : 1) void k_apply(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  if constexpr (RK >= kApplyMfmaRank) {
    apply_mfma<RK>(a, t, d);
  } else {
    // W (upper triangular) is read at wave-uniform addresses, through the scalar cache into
    // SGPRs: every product takes its W entry from there rather than from an LDS broadcast
    const double* __restrict__ W = a.w + d.w_slot;
    {
      const int64_t row = static_cast<int64_t>(t.a) + tid();
      if (tid() >= t.b) return;
      const bool q = a.variant == 1;
      const float* X = a.fac + (q ? d.q_slot : d.p_slot) + row * RK;
      float* Y = a.fac + (q ? d.qh_slot : d.ph_slot) + row * RK;
      double x[RK];
      float y[RK];
#pragma unroll
      for (int l = 0; l < RK; l += 4) {  // factor slots are 256-byte aligned: rows are 16-byte aligned
        const float4 v = *reinterpret_cast<const float4*>(X + l);
        x[l] = v.x;
        x[l + 1] = v.y;
        x[l + 2] = v.z;
        x[l + 3] = v.w;
      }
      // y[k] = sum over l <= k of x[l] W[l][k], added in increasing l; by rows of W, each
      // row's entries loaded together
      double acc[RK];
#pragma unroll
      for (int k = 0; k < RK; ++k) acc[k] = 0.0;
#pragma unroll
      for (int l = 0; l < RK; ++l)
#pragma unroll
        for (int k = l; k < RK; ++k) acc[k] = fma(x[l], W[l * RK + k], acc[k]);
#pragma unroll
      for (int k = 0; k < RK; ++k) y[k] = static_cast<float>(acc[k]);
#pragma unroll
      for (int k = 0; k < RK; k += 4)
        *reinterpret_cast<float4*>(Y + k) = make_float4(y[k], y[k + 1], y[k + 2], y[k + 3]);
    }
  }
}

// Write E of a tile of rows into a bucket-shaped output: the arena itself, F - Ph Q_loc^T
// (after a Q-step) or X - P_loc Qh^T (after a P-step that leaves X).
template <int RK>
__global__ __launch_bounds__(kBlock) void k_emat(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const MatDesc d = a.mats[t.idx];
  const int64_t m = d.m;
  const bool fform = deferred_of(a, d.bucket), xform = deferred_p_of(a, d);
  const float* L = a.fac + (xform ? d.qh_slot : d.ql_slot);  // column factor of the term
  const float* R = a.fac + (xform ? d.pl_slot : d.ph_slot);  // row factor of the term
  float* out = dst_of(a, d.bucket);
  const int64_t total = static_cast<int64_t>(t.b) * m;
  for (int64_t e = tid(); e < total; e += kBlock) {
    const int64_t row = t.a + e / m, j = e % m;
    const int64_t idx = row * m + j;
    float v = a.e[d.e_off + idx];
    if (fform || xform)
#pragma unroll
      for (int k = 0; k < RK; ++k) v -= R[row * RK + k] * L[j * RK + k];
    out[d.grad_off + idx] = v;
  }
}

// Q-step finish: Q_loc = sum over the row chunks' partials.  A tile covers the NE entries
// [t.a * NE, t.a * NE + NE) of the matrix (entry e = column * r + rank, NE = qfin_entries):
// with NE > 256 each thread takes NE / 256 entries 256 apart, otherwise 256 / NE threads share
// an entry.  FINE: the partials are those of the chunks' parts (part_rows(r) rows), added first.  Each thread adds a contiguous share of the chunks in chunk order, eight chunks
// requested at a time, and the shares are added in thread order.  The result goes to the factor
// buffer and to the Ql slot.
template <int RK, bool FINE>
__global__ __launch_bounds__(kBlock) void k_qfin(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  if (t.kind == T_VEC) {  // from kWideRank on the finish launch packs the raw vectors too
    vec_tile(a, t, true);
    return;
  }
  const MatDesc d = a.mats[t.idx];
  const int64_t m = d.m;
  const int64_t ncb = (m + d.q_cb - 1) / d.q_cb;
  const int64_t stride = ncb * d.q_cb * RK;  // one row chunk of partials
  const int ne = qfin_entries(d.q_chunks);   // entries per tile
  const float* part = a.qpart + d.qpart;
  constexpr int PR = part_rows(RK), MP = max_parts(RK);
  const int parts = FINE ? (d.q_rows + PR - 1) / PR : 1;  // at most MP
  // chunk c's sum at entry offset o
  auto chunk = [&](int64_t c, int64_t o) {
    if constexpr (!FINE) return part[c * stride + o];
    const float* p = part + c * parts * stride + o;
    float s = p[0];
#pragma unroll
    for (int k = 1; k < MP; ++k) {
      // a part past the chunk or the matrix has no rows: the first one is read again, without a
      // branch, so that all parts of all the thread's entries are requested together
      const bool has = k < parts && c * d.q_rows + k * PR < d.n;
      const float v = p[has ? k * stride : 0];
      s = has ? s + v : s;
    }
    return s;
  };
  float* out = dst_of(a, d.bucket) + d.fac_off_q;
  float* ql = a.fac + d.ql_slot;
  constexpr int U = 8;
  if (ne > kBlock) {  // at most 8 chunks: one thread per entry
    constexpr int EPT = 4;  // entries per thread (ne = 1024)
    float s[EPT];
    int64_t e[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      e[k] = static_cast<int64_t>(t.a) * ne + tid() + k * kBlock;
      s[k] = 0.f;
    }
    {
      // all (at most 8) chunks of the thread's entries requested together, added in chunk order
      float v[EPT][8];
#pragma unroll
      for (int k = 0; k < EPT; ++k)
#pragma unroll
        for (int u = 0; u < 8; ++u)
          v[k][u] = chunk(u < d.q_chunks ? u : 0, e[k] < m * RK ? e[k] : 0);  // no branch around the requests
#pragma unroll
      for (int k = 0; k < EPT; ++k)
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (u < d.q_chunks) s[k] += v[k][u];
    }
#pragma unroll
    for (int k = 0; k < EPT; ++k)
      if (e[k] < m * RK) {
        out[e[k]] = s[k];
        ql[e[k]] = s[k];
      }
    return;
  }
  const int ng = kBlock / ne;                // threads per entry
  const int gq = tid() / ne, el = tid() % ne;
  const int64_t e = static_cast<int64_t>(t.a) * ne + el;
  const bool on = e < m * RK;
  const int per = (d.q_chunks + ng - 1) / ng;
  const int ch0 = gq * per, ch1 = (ch0 + per < d.q_chunks) ? ch0 + per : d.q_chunks;
  float s = 0.f;
  if (on) {
    int ch = ch0;
    for (; ch + U <= ch1; ch += U) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = chunk(ch + u, e);
#pragma unroll
      for (int u = 0; u < U; ++u) s += v[u];
    }
    if (ch < ch1) {  // the rest (fewer than U chunks) requested together too, added in order
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = chunk(ch + u < ch1 ? ch + u : ch, e);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (ch + u < ch1) s += v[u];
    }
  }
  __shared__ float red[kBlock];
  red[tid()] = s;
  __syncthreads();
  if (gq == 0 && on) {
    float tot = red[el];
    for (int g = 1; g < ng; ++g) tot += red[g * ne + el];
    out[e] = tot;
    ql[e] = tot;
  }
}

__global__ __launch_bounds__(kBlock) void k_vec(KArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  vec_tile(a, t, true);
}


template <int RK>
hipError_t launch_rank(const Launch& l, const KArgs& args, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(l.ntiles)), block(kBlock);
  switch (l.kernel) {  // only the kernels the rank's launch lists use
    case K_APPLY:
      if constexpr (RK >= kWideRank) {
        hipLaunchKernelGGL(k_apply<RK>, grid, block, 0, s, args);
        break;
      } else {
        return hipErrorInvalidValue;
      }
    case K_GSUM:
      if constexpr (RK >= kBlockedRank) {
        hipLaunchKernelGGL(k_gsum<RK>, grid, block, 0, s, args);
        break;
      } else {
        return hipErrorInvalidValue;
      }
    case K_EMAT: hipLaunchKernelGGL(k_emat<RK>, grid, block, 0, s, args); break;
    case K_FACT: hipLaunchKernelGGL(k_fact<RK>, grid, block, 0, s, args); break;
    case K_CHOL: hipLaunchKernelGGL(k_chol<RK>, grid, block, 0, s, args); break;
    case K_QFIN:
      if constexpr (RK >= kWideRank && split_nested(RK)) {
        if (l.variant == kWideFine) {
          hipLaunchKernelGGL((k_qfin<RK, true>), grid, block, 0, s, args);
          break;
        }
      }
      hipLaunchKernelGGL((k_qfin<RK, false>), grid, block, 0, s, args);
      break;
    case K_VEC: hipLaunchKernelGGL(k_vec, grid, block, 0, s, args); break;
    case K_DRAW: hipLaunchKernelGGL(k_draw<RK>, grid, block, 0, s, args); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch(const Launch& l, int32_t rank, const KArgs& args, hipStream_t s) {
  if (l.ntiles <= 0) return hipSuccess;
  if (l.kernel == K_WPSTEP || l.kernel == K_WPFIN || l.kernel == K_WQSTEP || l.kernel == K_WRECON || l.kernel == K_WFACT)
    return launch_wide(l, rank, args, s);
  if (l.kernel == K_PFUSED || l.kernel == K_PWIDE || l.kernel == K_PFIN || l.kernel == K_QSTEP || l.kernel == K_RECON4)
    return launch_low(l, rank, args, s);
  switch (rank) {
    case 1: return launch_rank<1>(l, args, s);
    case 2: return launch_rank<2>(l, args, s);
    case 4: return launch_rank<4>(l, args, s);
    case 8: return launch_rank<8>(l, args, s);
    case 16: return launch_rank<16>(l, args, s);
    case 32: return launch_rank<32>(l, args, s);
    case 64: return launch_rank<64>(l, args, s);
    case 128: return launch_rank<128>(l, args, s);
    case 256: return launch_rank<256>(l, args, s);
    default: return hipErrorInvalidValue;
  }
}

// Q-step partials of acp_compress_noalloc: a file-scope device array, one copy on every GPU the
// library runs on, kept until the process ends.  In host code its name is only a symbol, not a
// device address: scratch_address() looks up the current device's copy once with
// hipGetSymbolAddress and keeps that address per device; every launch takes the address.
static __device__ __align__(256) float scratch[kScratchBytes / 4];

hipError_t scratch_address(int device, float** out) {
  static std::mutex mu;
  static std::vector<float*> addr;  // per device; null until looked up
  std::lock_guard<std::mutex> lock(mu);
  if (device < 0) return hipErrorInvalidDevice;
  if (addr.size() <= static_cast<size_t>(device)) addr.resize(static_cast<size_t>(device) + 1, nullptr);
  if (!addr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[device] = static_cast<float*>(p);
  }
  *out = addr[device];
  return hipSuccess;
}

}  // namespace acp
