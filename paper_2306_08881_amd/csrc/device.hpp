// Device helpers shared by the gfx950 kernel files: lane and buffer primitives, DPP wave
// sums, bucket buffers of a launch, raw-vector tiles and the Gram/Cholesky orthogonalisation
// tiles (arXiv 2306.08881, Algorithm 2: the orthogonalisation of the reused factor).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "acp_internal.hpp"

namespace acp {
namespace {

__device__ inline int tid() { return static_cast<int>(threadIdx.x); }

// Between a wave's writes to shared memory and its reads of what other lanes wrote: the wave's LDS
// accesses take effect in program order, so it is enough that the compiler keeps that order.
__device__ inline void wave_lds_fence() { asm volatile("" ::: "memory"); }

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ inline float4 operator+(const float4& a, const float4& b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

typedef float v4f __attribute__((ext_vector_type(4)));

// Tile-relative buffer accesses.  A buffer resource spans one tile from its first element;
// a load past num_records returns zero and a store past it is dropped, so lanes and rows that
// fall outside the tile need no branch: they take the offset kOut (or any offset past the
// extent).  Branch-free loads and stores let the compiler count outstanding memory operations
// exactly, so stores stay in flight while the next rows' loads are waited for.  Every extent
// and in-tile offset is below 2^30, so kOut plus an offset does not wrap.
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr uint32_t kOut = 0x80000000u;
constexpr int kAuxNT = 2;  // cache policy: nontemporal (streamed once)

__device__ inline Rsrc tile_rsrc(const float* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, static_cast<int>(bytes),
                                           0x00020000);
}
// The buffer builtins move raw 32-bit words (unsigned int); values cross them bit-cast.
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
__device__ inline float4 bld4_nt(Rsrc r, uint32_t off) {
  const v4f v = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kAuxNT));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline float bld1_nt(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kAuxNT));
}
__device__ inline void bst4_nt(Rsrc r, uint32_t off, const float4& v) {
  const v4f w = {v.x, v.y, v.z, v.w};
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, w), r, off, 0, kAuxNT);
}
__device__ inline void bst4(Rsrc r, uint32_t off, const float4& v) {
  const v4f w = {v.x, v.y, v.z, v.w};
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, w), r, off, 0, 0);
}
__device__ inline float4 bld4(Rsrc r, uint32_t off) {
  const v4f v = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline float bld1(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ inline void bst1(Rsrc r, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, 0, 0);
}
__device__ inline void bst1_nt(Rsrc r, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, 0, kAuxNT);
}

// Sum over the 64 lanes with DPP: quad butterflies, half-row and row mirrors give every lane
// its 16-lane row sum; the four row sums are then read out and added in row order.  Every lane
// gets the same bits.
template <int CTRL>
__device__ inline float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                               0xF, 0xF, false));
}
__device__ inline float wave_sum_dpp(float v) {
  v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp<0x141>(v);  // row_half_mirror
  v += dpp<0x140>(v);  // row_mirror
  const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
  const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16));
  const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
  const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 48));
  return ((r0 + r1) + r2) + r3;
}
// One row of a rank-RK factor (RK <= 4): the register and LDS form of the low-rank kernels.
template <int RK>
struct alignas(4 * RK) Fr {
  float v[RK];
};
// RK contiguous floats that need only 4-byte alignment (rows in the caller's factor buffers).
template <int RK>
__device__ inline Fr<RK> ld_fr(const float* p) {
  Fr<RK> f;
  if constexpr (RK == 4) {
    typedef float vu __attribute__((ext_vector_type(4), aligned(4)));
    const vu x = *reinterpret_cast<const vu*>(p);
#pragma unroll
    for (int k = 0; k < 4; ++k) f.v[k] = x[k];
  } else if constexpr (RK == 2) {
    typedef float vu __attribute__((ext_vector_type(2), aligned(4)));
    const vu x = *reinterpret_cast<const vu*>(p);
    f.v[0] = x[0];
    f.v[1] = x[1];
  } else {
    f.v[0] = p[0];
  }
  return f;
}
template <int RK>
__device__ inline Fr<RK> zero_fr() {
  Fr<RK> f;
#pragma unroll
  for (int k = 0; k < RK; ++k) f.v[k] = 0.f;
  return f;
}
template <int RK>
__device__ inline Fr<RK> scale_fr(Fr<RK> a, float s) {
#pragma unroll
  for (int k = 0; k < RK; ++k) a.v[k] *= s;
  return a;
}
template <int RK>
__device__ inline float dot_fr(const Fr<RK>& a, const Fr<RK>& b) {
  float s = a.v[0] * b.v[0];
#pragma unroll
  for (int k = 1; k < RK; ++k) s += a.v[k] * b.v[k];
  return s;
}
template <int RK>
__device__ inline void fma_fr(float s, const Fr<RK>& v, Fr<RK>& acc) {
#pragma unroll
  for (int k = 0; k < RK; ++k) acc.v[k] = fmaf(s, v.v[k], acc.v[k]);
}
template <int RK>
__device__ inline void add_fr(Fr<RK>& a, const Fr<RK>& b) {
#pragma unroll
  for (int k = 0; k < RK; ++k) a.v[k] += b.v[k];
}
template <int RK>
__device__ inline Fr<RK> bld_fr(Rsrc r, uint32_t off) {
  Fr<RK> f;
  if constexpr (RK == 4) {
    const float4 x = bld4(r, off);
    f.v[0] = x.x;
    f.v[1] = x.y;
    f.v[2] = x.z;
    f.v[3] = x.w;
  } else {
#pragma unroll
    for (int k = 0; k < RK; ++k) f.v[k] = bld1(r, off + 4u * k);
  }
  return f;
}
template <int RK>
__device__ inline void bst_fr(Rsrc r, uint32_t off, const Fr<RK>& f) {
  if constexpr (RK == 4) {
    bst4(r, off, make_float4(f.v[0], f.v[1], f.v[2], f.v[3]));
  } else {
#pragma unroll
    for (int k = 0; k < RK; ++k) bst1(r, off + 4u * k, f.v[k]);
  }
}
template <int RK>
__device__ inline Fr<RK> wave_sum_dpp(Fr<RK> f) {
#pragma unroll
  for (int k = 0; k < RK; ++k) f.v[k] = wave_sum_dpp(f.v[k]);
  return f;
}

// x W for one row of a rank-RK factor (W upper triangular, fp64, row-major), rounded to fp32.
template <int RK>
__device__ inline Fr<RK> apply_w(const Fr<RK>& x, const double* W) {
  Fr<RK> y;
#pragma unroll
  for (int k = 0; k < RK; ++k) {
    double s = static_cast<double>(x.v[k]) * W[k * RK + k];
#pragma unroll
    for (int l = k - 1; l >= 0; --l) s = fma(static_cast<double>(x.v[l]), W[l * RK + k], s);
    y.v[k] = static_cast<float>(s);
  }
  return y;
}

// Buffers of a bucket in this launch's group.
__device__ inline const float* src_of(const KArgs& a, int32_t b) { return a.src[b - a.base]; }
__device__ inline float* dst_of(const KArgs& a, int32_t b) { return a.dst[b - a.base]; }
__device__ inline bool deferred_of(const KArgs& a, int32_t b) {
  return ((a.deferred >> (b - a.base)) & 1ull) != 0;
}
// the arena holds X for this matrix (up to rank 4 only the wide rows' P-step leaves it)
__device__ inline bool deferred_p_of(const KArgs& a, const MatDesc& d) {
  return d.xhold != 0 && ((a.deferred_p >> (d.bucket - a.base)) & 1ull) != 0;
}

// Raw vectors: pack the gradient into the factor buffer (compress; the first half of a Power-SGD
// step with error feedback also keeps them in the E arena, the second half's source) or unpack the
// aggregated sum / p into the output bucket (decompress).
__device__ void vec_tile(const KArgs& a, const Tile& t, bool compress) {
  const VecDesc v = a.vecs[t.idx];
  const int64_t foff = a.parity ? v.fac_off_p : v.fac_off_q;
  const float* src = src_of(a, v.bucket);
  float* dst = dst_of(a, v.bucket);
  for (int i = tid(); i < t.b; i += static_cast<int>(blockDim.x)) {  // launches of 3 or 4 waves
    const int64_t k = static_cast<int64_t>(t.a) + i;
    if (compress) {
      const float x = src[v.grad_off + k];
      dst[foff + k] = x;
      if (a.image && a.ef) a.e[v.e_off + k] = x;
    } else {
      dst[v.grad_off + k] = src[foff + k] * a.inv_p;
    }
  }
}

// ---------------------------------------------------------------------------------------
// Orthogonalisation, Gram/Cholesky form.  For a factor X (k x r) the Gram-Schmidt factor is
// orth(X) = X W with W = R^-1 and G = X^T X = R^T R (R upper triangular, positive diagonal):
// the same columns as Gram-Schmidt in exact arithmetic.  G is accumulated in fp64 from fp32
// products (exact) and factored in fp64.  A column j is dropped (its column of W is zero) when
// G_jj = 0 or its residual d_j = G_jj - sum_{i<j} R_ij^2 is at most tau^2 G_jj, i.e. when the
// residual norm is at most tau times the column norm.

typedef double v4d __attribute__((ext_vector_type(4)));

// The lane's double from lane `src` of the wave (src uniform).
__device__ inline double readlane_d(double v, int src) {
  const int2 h = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(h.x, src),
                                              __builtin_amdgcn_readlane(h.y, src)));
}

// 1 / sqrt(x) for x > 0: the hardware estimate, then two Newton steps y += y (1 - x y^2) / 2, each
// of which squares the relative error.
__device__ inline double rsqrt_newton(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return y;
}

// Cholesky G = R^T R with L^-1 = R^-T beside it, by the first wave, in place in A (shared memory, B
// rows of 2 B: [G | I] on entry, [R | L^-1] on return; the caller synchronises before and after).
// At pivot p the updated diagonal decides the drop (against ref(p)), row p is scaled by 1 / sqrt of
// it and subtracted from the rows after it, in both halves:
//   row p *= rinv;  row i -= R[p][i] row p  (i > p).
// L^-1 = W^T, and its entries are those of the back substitution W[a][c] = (delta_ac - sum over
// i < c of R[i][c] W[a][i]) / R[c][c] in the same order.  A dropped pivot's row is zero in both.
// Lane j holds column j of A, rows p ... in g[0] ...: each pivot's
// update also shifts the rows down one register, so that the pivots are one rolled loop.  The
// chain is bound by latency, and before that by fetching instructions: unrolled over the pivots
// the code ran once through tens of KB that no cache held (this form unrolled took 53 us a launch
// at rank 32).  Launch at rank 32 with a second, unrolled pass of dependent divisions for W 22 us,
// this way 17.7; rank 256, whose eight diagonal blocks come here, 432 and 351 us.
template <int B, typename Ref>
__device__ inline void chol_inverse(double* A, Ref ref) {
  constexpr int LD = 2 * B;
  static_assert(LD <= kWave, "one column per lane");
  if (tid() >= kWave) return;
  const int j = tid();
  const bool on = j < LD;
  double g[B < 2 ? 2 : B];
  g[1] = 0.0;
#pragma unroll
  for (int a = 0; a < B; ++a) g[a] = A[a * LD + (on ? j : 0)];
  const double refl = ref(j < B ? j : 0);
  // 1 / sqrt of pivot p's diagonal dk, zero when it is dropped
  auto pivot = [&](double dk, int p) {
    const double rf = readlane_d(refl, p);
    const double y = rsqrt_newton(dk);
    return rf > 0.0 && dk > kTau * kTau * rf ? y : 0.0;
  };
  double rinv = pivot(readlane_d(g[0], 0), 0);
#pragma unroll 1
  for (int p = 0; p < B; ++p) {
    double* row = A + p * LD;
    // G's columns left of the pivot hold nothing of R's row; nor does a dropped pivot's, whatever g is
    const double y = rinv > 0.0 && j >= p ? g[0] * rinv : 0.0;
    if (on) row[j] = y;
    wave_lds_fence();
    // all of the row is requested at once (three entries at a time, as the compiler had it, were
    // 640 of a pivot's 760 cycles); past R's row: rows that do not exist
    double r[B < 3 ? 1 : B - 2];
#pragma unroll
    for (int a = 1; a < B - 1; ++a) r[a - 1] = row[p + 1 + a];
    __builtin_amdgcn_sched_barrier(0);
    // the next pivot's row and its root meanwhile
    const double n0 = fma(-readlane_d(y, p + 1), y, g[1]);
    rinv = pivot(readlane_d(n0, p + 1), p + 1 < B ? p + 1 : p);
#pragma unroll
    for (int a = 1; a < B - 1; ++a) g[a] = fma(-r[a - 1], y, g[a + 1]);
    g[0] = n0;
    wave_lds_fence();
  }
}

// A = [G | I] for chol_inverse, G in its left half already; by the whole workgroup.
template <int B>
__device__ inline void beside_identity(double* A) {
  for (int e = tid(); e < B * B; e += kBlock) A[e / B * 2 * B + B + e % B] = e / B == e % B ? 1.0 : 0.0;
}

// Cholesky G = R^T R and W = R^-1 of a Gram matrix in shared memory (RK = 64 or 128, row-major; only
// the upper triangle is read) for ranks from 64 on, by the whole workgroup, in blocks
// of 32.  For each diagonal block K in order:
//   (i)   one wave factors the block and forms W_KK = R_KK^-1 beside it (chol_inverse);
//   (ii)  the block row right of it: R_KJ = W_KK^T G_KJ (with dropped pivots W_KK's zero columns
//         give R's zero rows, as forward substitution over the kept pivots would);
//   (iii) the trailing upper triangle: G_IJ -= R_KI^T R_KJ.
// These are the pivots of the unblocked right-looking form, in the same order.  Then block column
// J of W (J = 1, 2, 3) from the earlier ones: W_IJ = -(sum_{I <= L < J} W_IL R_LJ) W_JJ.  W[i][c]
// (i < c) is kept in the strictly lower triangle at G[RK-1-i][RK-1-c] and its diagonal apart.
// Dropped pivots give zero rows and columns of R and W.  G[] is overwritten.  The drop test
// compares with the diagonal gref[i * gstride] (G's own unless given: a trailing block of a
// larger Gram matrix is tested against that matrix's diagonal); W goes to w_out with rows ldw
// apart.
template <int RK>
__device__ __attribute__((always_inline)) void cholesky_w_blocked(double* G, double* w_out, int ldw = RK,
                                                                const double* gref = nullptr, int gstride = 0) {
  static_assert((RK == 64 || RK == 128) && kBlock == 256, "blocks of 32 on 256 threads");
  constexpr int B = 32, NBK = RK / B;
  __shared__ double g0[RK], wdiag[RK];
  // a diagonal block beside the identity, then one block column's W[0:k0][.] R[.][block] products
  __shared__ double T[(RK - B) * B > 2 * B * B ? (RK - B) * B : 2 * B * B];
  auto wl = [&](int i, int c) -> double& { return G[(RK - 1 - i) * RK + (RK - 1 - c)]; };  // W[i][c], i < c
  for (int i = tid(); i < RK; i += kBlock) g0[i] = gref ? gref[i * gstride] : G[i * RK + i];
  __syncthreads();
  const int lane = tid() & 63;
  for (int K = 0; K < NBK; ++K) {
    const int k0 = K * B, nc = RK - k0 - B;  // columns right of the block
    // (i) the diagonal block and W_KK (chol_inverse in T, which is free here)
    for (int e = tid(); e < B * B; e += kBlock) {
      const int a = e / B, c = e % B;
      T[a * 2 * B + c] = G[(k0 + (a < c ? a : c)) * RK + k0 + (a < c ? c : a)];
    }
    beside_identity<B>(T);
    __syncthreads();
    chol_inverse<B>(T, [&](int p) { return g0[k0 + p]; });
    __syncthreads();
    for (int e = tid(); e < B * B; e += kBlock) {
      const int a = e / B, c = e % B;
      if (a <= c) G[(k0 + a) * RK + k0 + c] = T[a * 2 * B + c];
      if (a < c) wl(k0 + a, k0 + c) = T[c * 2 * B + B + a];
      if (a == c) wdiag[k0 + a] = T[a * 2 * B + B + a];
    }
    __syncthreads();
    if (nc == 0) break;
    // (ii) R_KJ = W_KK^T G_KJ on the fp64 matrix cores in 16 x 16 tiles (row block t % 2, column
    // block t / 2, tile t on wave t % 4; one v_mfma_f64_16x16x4f64 per four ranks b, W_KK's operand
    // zero past its column a >= b); every tile is formed before any is written
    {
      constexpr int QN = (2 * (RK - B) / 16 + 3) / 4;  // tiles per wave, at most
      const int nt = 2 * (nc / 16), w = tid() / kWave, li = lane % 16, lk = lane / 16, c0 = k0 + B;
      v4d acc[QN];
#pragma unroll
      for (int q = 0; q < QN; ++q) {
        acc[q] = v4d{0.0, 0.0, 0.0, 0.0};
        const int t = w + 4 * q, a = 16 * (t % 2) + li;
        if (t < nt)
#pragma unroll
          for (int s4 = 0; s4 < B / 4; ++s4) {
            const int b = 4 * s4 + lk;
            const double wv = b < a ? wl(k0 + b, k0 + a) : (b == a ? wdiag[k0 + a] : 0.0);
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv, G[(k0 + b) * RK + c0 + 16 * (t / 2) + li], acc[q], 0, 0, 0);
          }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < QN; ++q) {
        const int t = w + 4 * q;
        if (t < nt)
#pragma unroll
          for (int v = 0; v < 4; ++v) G[(k0 + 16 * (t % 2) + 4 * v + lk) * RK + c0 + 16 * (t / 2) + li] = acc[q][v];
      }
      __syncthreads();
    }
    // (iii) the trailing upper triangle: G[i][j] -= sum_a R[k0 + a][i] R[k0 + a][j], i <= j, on
    // the fp64 matrix cores in 16 x 16 tiles (tiles ti <= tj, tile t on wave t % 4; one
    // v_mfma_f64_16x16x4f64 per four rows a); entries below the diagonal of a diagonal tile are
    // not written (that triangle keeps W)
    {
      const int nt = nc / 16, w = tid() / kWave, li = lane % 16, lk = lane / 16, c0 = k0 + B;
      int t = 0;
      for (int ti = 0; ti < nt; ++ti)
        for (int tj = ti; tj < nt; ++tj, ++t) {
          if (t % (kBlock / kWave) != w) continue;
          v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int s4 = 0; s4 < B / 4; ++s4) {
            const double* r = G + (k0 + 4 * s4 + lk) * RK + c0 + li;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(r[16 * ti], r[16 * tj], acc, 0, 0, 0);
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int i = c0 + 16 * ti + 4 * v + lk, j = c0 + 16 * tj + li;
            if (i <= j) G[i * RK + j] -= acc[v];
          }
        }
    }
    __syncthreads();
  }
  // block columns of W: T = W[0:k0][0:k0] R[0:k0][block], then W[0:k0][block] = -T W_JJ, both
  // on the fp64 matrix cores in 16 x 16 tiles (tile t of the k0 / 16 x 2 on wave t % 4; one
  // v_mfma_f64_16x16x4f64 per four ranks, the operands of W taken from its triangle: zero below
  // the diagonal, wdiag on it)
  {
    const int w = tid() / kWave, li = lane % 16, lk = lane / 16;
    auto wv = [&](int r, int c) { return c > r ? wl(r, c) : (c == r ? wdiag[r] : 0.0); };  // W[r][c]
    for (int J = 1; J < NBK; ++J) {
      const int k0 = J * B, nt = 2 * (k0 / 16);
      for (int t = w; t < nt; t += kBlock / kWave) {
        const int i0 = 16 * (t / 2), c0 = 16 * (t % 2);
        v4d acc = {0.0, 0.0, 0.0, 0.0};
        for (int l0 = i0; l0 < k0; l0 += 4)  // W[i][l] is zero for l < i
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(wv(i0 + li, l0 + lk), G[(l0 + lk) * RK + k0 + c0 + li],
                                                     acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) T[(i0 + 4 * v + lk) * B + c0 + li] = acc[v];
      }
      __syncthreads();
      for (int t = w; t < nt; t += kBlock / kWave) {
        const int i0 = 16 * (t / 2), c0 = 16 * (t % 2);
        v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q0 = 0; q0 < B; q0 += 4)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(T[(i0 + li) * B + q0 + lk], wv(k0 + q0 + lk, k0 + c0 + li),
                                                     acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) wl(i0 + 4 * v + lk, k0 + c0 + li) = -acc[v];
      }
      __syncthreads();
    }
  }
  for (int e = tid(); e < RK * RK; e += kBlock) {
    const int i = e / RK, c = e % RK;
    w_out[i * ldw + c] = i < c ? wl(i, c) : (i == c ? wdiag[c] : 0.0);
  }
}

// Floats between the rows of a Gram matrix in shared memory up to rank 64: the left half of [G | I]
// where chol_inverse takes the whole matrix.  Rank 64 goes in two blocks of 32: in one, 126
// multiply-adds a pivot on two columns per lane made the launch 89 us.
constexpr int gram_ld(int rk) { return rk <= 32 ? 2 * rk : rk; }

// W = R^-1 of the Gram matrix in A (shared memory, RK rows of gram_ld) into w_out, by the whole
// workgroup; every entry of A is in place on entry.
template <int RK>
__device__ inline void cholesky_w(double* A, double* w_out) {
  if constexpr (RK > 32) {
    cholesky_w_blocked<RK>(A, w_out);
  } else {
    __shared__ double diag[RK];
    beside_identity<RK>(A);
    if (tid() < RK) diag[tid()] = A[tid() * (2 * RK + 1)];
    __syncthreads();
    chol_inverse<RK>(A, [&](int p) { return diag[p]; });
    __syncthreads();
    for (int e = tid(); e < RK * RK; e += kBlock) w_out[e] = A[e % RK * 2 * RK + RK + e / RK];
  }
}

template <int RK, bool DIAG, int NB = 4>
__device__ void gram_band(const float* X, int64_t r0, int64_t r1, float* copy, int I, int J, int nw, int w,
                          v4d (&acc)[NB][NB]);

// Gram of rows [r0, r1) of X (row-major, RK columns) into shared G (RK rows of gram_ld),
// by the whole workgroup, in a fixed order; the rows are also copied to `copy` when it is set.
template <int RK>
__device__ void gram_rows(const float* X, int64_t r0, int64_t r1, double* G, float* copy) {
  static_assert(RK <= 8 || RK == 16 || RK == 32 || RK == 64, "from kBlockedRank on gram_blocked forms the Gram");
  if constexpr (RK <= 8) {
    constexpr int NT = RK * (RK + 1) / 2;
    constexpr int PER = 8;  // rows per thread per pass, loaded together
    double g[NT];
#pragma unroll
    for (int e = 0; e < NT; ++e) g[e] = 0.0;
    for (int64_t base = r0; base < r1; base += int64_t(kBlock) * PER) {
      float x[PER][RK];
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int64_t row = base + u * kBlock + tid();
#pragma unroll
        for (int k = 0; k < RK; ++k) x[u][k] = row < r1 ? X[row * RK + k] : 0.f;
      }
      if (copy) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const int64_t row = base + u * kBlock + tid();
          if (row < r1)
#pragma unroll
            for (int k = 0; k < RK; ++k) copy[row * RK + k] = x[u][k];
        }
      }
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        int e = 0;
#pragma unroll
        for (int i = 0; i < RK; ++i)
#pragma unroll
          for (int j = i; j < RK; ++j, ++e)
            g[e] = fma(static_cast<double>(x[u][i]), static_cast<double>(x[u][j]), g[e]);
      }
    }
    __shared__ double red[4][NT];
#pragma unroll
    for (int e = 0; e < NT; ++e) g[e] = wave_sum(g[e]);
    if ((tid() & 63) == 0)
#pragma unroll
      for (int e = 0; e < NT; ++e) red[tid() >> 6][e] = g[e];
    __syncthreads();
    if (tid() < NT) {
      const int e = tid();
      int i = 0, rem = e;
      while (rem >= RK - i) rem -= RK - i, ++i;
      const int j = i + rem;
      const double s = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
      G[i * gram_ld(RK) + j] = s;
      G[j * gram_ld(RK) + i] = s;
    }
    __syncthreads();
  } else if constexpr (RK == 16 || RK == 32 || RK == 64) {
    // on the fp64 matrix cores (gram_band, one band of all RK columns): the four waves take
    // interleaved steps of 16 rows, each forming the products a <= b of the band's 16-column
    // blocks; their sums are added into G in wave order, then the blocks a > b mirrored
    constexpr int NB = RK / 16;
    const int w = tid() / kWave, lane = tid() % kWave, i = lane % 16, k = lane / 16;
    v4d acc[NB][NB];
    gram_band<RK, true, NB>(X, r0, r1, copy, 0, 0, kBlock / kWave, w, acc);
    for (int q = 0; q < kBlock / kWave; ++q) {
      if (w == q)
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
          for (int b = a; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              double& g = G[(16 * a + 4 * v + k) * gram_ld(RK) + 16 * b + i];
              g = q == 0 ? acc[a][b][v] : g + acc[a][b][v];
            }
      __syncthreads();
    }
    for (int e = tid(); e < RK * RK; e += kBlock) {
      const int r = e / RK, c = e % RK;
      if (r / 16 > c / 16) G[r * gram_ld(RK) + c] = G[c * gram_ld(RK) + r];
    }
    __syncthreads();
  }
}

// Band block X_I^T X_J of rows [r0, r1) of X (row-major, RK columns; 64-column bands I <= J)
// into acc, on the fp64 matrix cores: 4 x 4 products of 16 x 16 (v_mfma_f64_16x16x4f64, four rows
// of X each; operand entry [i][k] on lane i + 16 k, result entry [4 v + l / 16][l % 16] in item v
// of lane l), product (a, b) for the columns 16 a ... and 16 b ... of the two bands; a diagonal
// block (DIAG) skips its products a > b, whose entries lie below the diagonal.  The rows go in
// steps of 16, of which the wave takes steps w, w + nw, ...; each product adds them in increasing
// groups of four, and the wave's next step is requested before the current one's products.  A
// diagonal block also copies its steps' rows of the band to `copy` when set.
template <int RK, bool DIAG, int NB>
__device__ void gram_band(const float* X, int64_t r0, int64_t r1, float* copy, int I, int J, int nw, int w,
                          v4d (&acc)[NB][NB]) {
  constexpr int G = 4;  // groups of four rows per step
  constexpr int BW = 16 * NB;  // band width (columns)
  const int lane = tid() % kWave, i = lane % 16, k = lane / 16;
  const float* xa = X + BW * I + i;
  const float* xb = X + BW * J + i;
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = v4d{0.0, 0.0, 0.0, 0.0};
  // rows past the slice read its last row (no branch around the loads, so the wait for a step's
  // rows leaves the next step's requests in flight); the A operand of those rows is zeroed
  auto row_of = [&](int64_t g0, int s) {
    const int64_t row = g0 + 4 * s + k;
    return row < r1 ? row : r1 - 1;
  };
  // two register buffers of G groups, filled and consumed in turn
  typedef float Buf[G][NB];
  auto fetch = [&](int64_t g0, Buf& ba, Buf& bb) {
#pragma unroll
    for (int s = 0; s < G; ++s) {
      const float* pa = xa + row_of(g0, s) * RK;
      const float* pb = xb + row_of(g0, s) * RK;
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        ba[s][a] = pa[16 * a];
        if (!DIAG) bb[s][a] = pb[16 * a];
      }
    }
  };
  auto step = [&](int64_t g0, Buf& ba, Buf& bb) {
    // the conversions stay behind the other buffer's requests, issued just before
#pragma unroll
    for (int s = 0; s < G; ++s)
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        asm volatile("" : "+v"(ba[s][a]));
        if (!DIAG) asm volatile("" : "+v"(bb[s][a]));
      }
    // a row past the slice stores its clamped row's own values again
    if (DIAG && copy)
#pragma unroll
      for (int s = 0; s < G; ++s)
#pragma unroll
        for (int a = 0; a < NB; ++a) copy[row_of(g0, s) * RK + BW * I + 16 * a + i] = ba[s][a];
#pragma unroll
    for (int s = 0; s < G; ++s) {
      const bool in = g0 + 4 * s + k < r1;
      double xa4[NB], xb4[NB];
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        xa4[a] = in ? static_cast<double>(ba[s][a]) : 0.0;
        xb4[a] = static_cast<double>(DIAG ? ba[s][a] : bb[s][a]);
      }
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (!DIAG || a <= b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa4[a], xb4[b], acc[a][b], 0, 0, 0);
    }
  };
  // steps of 4 G rows: this wave takes steps w, w + nw, ... of the slice
  const int64_t sd = 4 * G * nw;
  Buf a0, b0, a1, b1;
  fetch(r0 + 4 * G * w, a0, b0);
  for (int64_t g0 = r0 + 4 * G * w; g0 < r1; g0 += 2 * sd) {  // a second step past the slice adds zeros
    fetch(g0 + sd, a1, b1);
    step(g0, a0, b0);
    fetch(g0 + 2 * sd, a0, b0);
    step(g0 + sd, a1, b1);
  }
}

// Part `part` of the Gram of rows [r0, r1) of X (RK >= kBlockedRank columns) into `out` (RK x RK
// doubles, global memory): G is symmetric, so only its band blocks with I <= J are formed
// (gram_band), numbered row by row; wave w of part p takes block 4 p + w over all the rows.
// K_GSUM mirrors the entries of the 4 x 4 blocks above the diagonal.
template <int RK>
__device__ void gram_blocked(const float* X, int64_t r0, int64_t r1, double* out, float* copy, int part) {
  constexpr int NB = RK / 64, NP = NB * (NB + 1) / 2;
  static_assert(gram_parts(RK) * (kBlock / kWave) >= NP, "every band block needs a wave");
  const int pr = part * (kBlock / kWave) + tid() / kWave;
  if (pr >= NP) return;
  int I = 0, rem = pr;
  while (rem >= NB - I) rem -= NB - I, ++I;
  const int J = I + rem, lane = tid() % kWave, i = lane % 16, k = lane / 16;
  v4d acc[4][4];
  if (rem == 0)
    gram_band<RK, true>(X, r0, r1, copy, I, I, 1, 0, acc);
  else
    gram_band<RK, false>(X, r0, r1, copy, I, J, 1, 0, acc);
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if (rem != 0 || a <= b)
#pragma unroll
        for (int v = 0; v < 4; ++v) out[(64 * I + 16 * a + 4 * v + k) * RK + 64 * J + 16 * b + i] = acc[a][b][v];
}

// Factor tile: slice t.a of the t.b slices of fact_rows rows of the factor `src` (rows x RK).
// When `dst` is set the slice is also copied there (the aggregated factor becomes the next
// step's reused factor).  A factor of one slice finishes W here; otherwise the slice's Gram is
// stored as a partial and K_CHOL adds the partials and finishes W.  From kBlockedRank on the
// Gram always goes to a partial (its blocks on and above the diagonal), K_GSUM adds and mirrors
// the partials and K_CHOL finishes W.
template <int RK>
__device__ void fact_tile(const KArgs& a, const Tile& t, const float* src, float* dst, int64_t rows) {
  const MatDesc d = a.mats[t.idx];
  if (a.copy_only) {  // Power-SGD keeps the aggregated Q as it is: copied, no W
    const int sl = RK >= kBlockedRank ? (t.a & 0xffff) : t.a;
    if (!dst || (RK >= kBlockedRank && (t.a >> 16) != 0)) return;
    const int64_t r0 = static_cast<int64_t>(sl) * d.fact_rows;
    const int64_t r1 = r0 + d.fact_rows < rows ? r0 + d.fact_rows : rows;
    for (int64_t e = r0 * RK + tid(); e < r1 * RK; e += static_cast<int64_t>(blockDim.x)) dst[e] = src[e];
    return;
  }
  if constexpr (RK >= kBlockedRank) {  // always a partial: K_CHOL forms W
    const int sl = t.a & 0xffff, part = t.a >> 16;
    const int64_t r0 = static_cast<int64_t>(sl) * d.fact_rows;
    const int64_t r1 = r0 + d.fact_rows < rows ? r0 + d.fact_rows : rows;
    gram_blocked<RK>(src, r0, r1, a.gpart + d.gpart + static_cast<int64_t>(sl) * RK * RK, dst, part);
  } else {
    const int64_t r0 = static_cast<int64_t>(t.a) * d.fact_rows;
    const int64_t r1 = r0 + d.fact_rows < rows ? r0 + d.fact_rows : rows;
    __shared__ double G[RK * gram_ld(RK)];
    gram_rows<RK>(src, r0, r1, G, dst);
    if (t.b == 1) {
      cholesky_w<RK>(G, a.w + d.w_slot);
    } else {
      double* part = a.gpart + d.gpart + static_cast<int64_t>(t.a) * RK * RK;
      for (int e = tid(); e < RK * RK; e += kBlock) part[e] = G[e / RK * gram_ld(RK) + e % RK];
    }
  }
}

}  // namespace
}  // namespace acp
