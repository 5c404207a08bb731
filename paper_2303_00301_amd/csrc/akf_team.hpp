// akf_team.hpp -- device-side dense FP64 linear algebra for one workgroup
// ("team") working on D x D matrices, D in {16, 32, 64}, on gfx950.
//
// Layout conventions
//  * A team is 1 wavefront (D <= 32) or 4 wavefronts (D = 64).  Each wave owns
//    a QD x QD quadrant (QD = min(D, 32)) made of 16 x 16 tiles.
//  * Register matrices (RM) hold the quadrant in the accumulator layout of
//    v_mfma_f64_16x16x4f64: in tile q, lane l, register r holds element
//    (row0 + 4*r + l/16, col0 + l%16) (measured on gfx950).  Every RM in a team uses the same
//    ownership map, so element-wise arithmetic needs no data movement.
//  * LDS matrices are row-major with leading dimension LD = D + 1 doubles (the
//    odd stride spreads column accesses over the banks).
//  * Runtime size d <= D: padded rows/columns are zero in every matrix
//    (factors and inverses included).
//
// GEMMs run on the f64 matrix cores.  Inverses and Cholesky factors of SPD
// matrices go by 2 x 2 blocks, two levels deep at D = 64: each 16 x 16 pivot
// tile is swept inside one wave (lane broadcasts, no LDS), and every product is
// an MFMA chain on tiles.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

namespace akf {

typedef double dbl4 __attribute__((ext_vector_type(4)));

template <int D_>
struct Cfg {
  static constexpr int D = D_;
  static constexpr int QD = D < 32 ? D : 32;
  static constexpr int NW = (D / QD) * (D / QD);
  static constexpr int NT = 64 * NW;
  static constexpr int TS = QD / 16;
  static constexpr int TPW = TS * TS;
  static constexpr int NB = D / 16;
  static constexpr int LD = D + 1;
  static constexpr int MAT = D * LD;  // entries of an LDS matrix
};

__device__ __forceinline__ double lane_bcast(double v, int src) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, src);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), src);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Orders this wave's LDS accesses (LDS operations of one wave complete in
// issue order; this keeps the compiler from moving them across the point).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Team barrier that orders LDS only: threads of a team exchange data through
// LDS, never through global memory within one launch, so the barrier waits
// for the team's LDS operations but not for its outstanding global loads and
// stores (a per-step store of a result need not finish before the next step).
__device__ __forceinline__ void team_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// s plus the value of the lane 16 (32) on in the wave's exchange order: a half
// exchange in the vector unit (a lane permute through LDS takes 83 cycles)
__device__ __forceinline__ double half_sum(uint32_t lo0, uint32_t hi0, uint32_t lo1, uint32_t hi1) {
  return __builtin_bit_cast(double, ((uint64_t)hi0 << 32) | lo0) +
         __builtin_bit_cast(double, ((uint64_t)hi1 << 32) | lo1);
}
__device__ __forceinline__ double sum_x16(double s) {
  const uint64_t u = __builtin_bit_cast(uint64_t, s);
  const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return half_sum(a[0], b[0], a[1], b[1]);
}
__device__ __forceinline__ double sum_x32(double s) {
  const uint64_t u = __builtin_bit_cast(uint64_t, s);
  const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return half_sum(a[0], b[0], a[1], b[1]);
}
// sum over the lanes with the same l%16
__device__ __forceinline__ double sum_groups(double s) { return sum_x32(sum_x16(s)); }

// lane (l + N) of the row of 16
template <int N>
__device__ __forceinline__ double row_ror(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x120 + N, 0xF, 0xF, true);
  const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x120 + N, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// sum over the wave, to every lane
__device__ __forceinline__ double wave_total(double v) {
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  v += row_ror<1>(v);
  return sum_groups(v);
}

template <int D>
struct RM {
  dbl4 t[Cfg<D>::TPW];
};

template <int D>
__device__ __forceinline__ int rm_row(int q, int r) {
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int r0 = (D == 64) ? 32 * (w >> 1) : 0;
  return r0 + 16 * (q / Cfg<D>::TS) + 4 * r + (l >> 4);
}

template <int D>
__device__ __forceinline__ int rm_col(int q) {
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int c0 = (D == 64) ? 32 * (w & 1) : 0;
  return c0 + 16 * (q % Cfg<D>::TS) + (l & 15);
}

#define AKF_RM_FOR(D, q, r, i, j)                                   \
  _Pragma("unroll") for (int q = 0; q < Cfg<D>::TPW; ++q)           \
    _Pragma("unroll") for (int r = 0; r < 4; ++r)                   \
      if (const int i = rm_row<D>(q, r), j = rm_col<D>(q); true)

template <int D>
__device__ __forceinline__ void rm_zero(RM<D>& a) {
#pragma unroll
  for (int q = 0; q < Cfg<D>::TPW; ++q) a.t[q] = dbl4{0.0, 0.0, 0.0, 0.0};
}

// identity on the leading d x d block
template <int D>
__device__ __forceinline__ void rm_eye(RM<D>& a, int d) {
  AKF_RM_FOR(D, q, r, i, j) a.t[q][r] = (i == j && i < d) ? 1.0 : 0.0;
}

// a = G[i*ld + j] on the leading d x d block, zero elsewhere (global memory)
template <int D>
__device__ __forceinline__ void rm_load(RM<D>& a, const double* __restrict__ g, int ld, int d) {
  AKF_RM_FOR(D, q, r, i, j) a.t[q][r] = (i < d && j < d) ? g[(size_t)i * ld + j] : 0.0;
}

template <int D>
__device__ __forceinline__ void rm_add_load(RM<D>& a, const double* __restrict__ g, int ld, int d) {
  AKF_RM_FOR(D, q, r, i, j) if (i < d && j < d) a.t[q][r] += g[(size_t)i * ld + j];
}

template <int D>
__device__ __forceinline__ void rm_store(const RM<D>& a, double* __restrict__ g, int ld, int d) {
  AKF_RM_FOR(D, q, r, i, j) if (i < d && j < d) g[(size_t)i * ld + j] = a.t[q][r];
}

// transposed store of the whole D x D tile: G[j*ld + i] = a_ij
template <int D>
__device__ __forceinline__ void rm_store_t(const RM<D>& a, double* __restrict__ g, int ld) {
  AKF_RM_FOR(D, q, r, i, j) g[(size_t)j * ld + i] = a.t[q][r];
}

template <int D>
__device__ __forceinline__ void rm_stage(const RM<D>& a, double* s) {
  AKF_RM_FOR(D, q, r, i, j) s[i * Cfg<D>::LD + j] = a.t[q][r];
}

template <int D>
__device__ __forceinline__ void rm_stage_t(const RM<D>& a, double* s) {
  AKF_RM_FOR(D, q, r, i, j) s[j * Cfg<D>::LD + i] = a.t[q][r];
}

template <int D>
__device__ __forceinline__ void rm_unstage(RM<D>& a, const double* s) {
  AKF_RM_FOR(D, q, r, i, j) a.t[q][r] = s[i * Cfg<D>::LD + j];
}

// store(e, load(e)) for every e < n (n <= CAP) by a team of NT threads, each
// lane issuing G loads before their stores (all of them by default).  A
// lane-strided loop (e = tid; e < n; e += NT) has no trip count the compiler
// can see, stays rolled and waits out one memory latency per iteration (16
// round trips for a 64 x 64 matrix over 256 lanes, about 20k cycles).  Code
// that holds most of the register file passes a small G: each group of G
// loads costs one round trip and 2 G registers.
template <int NT, int CAP, int G = (CAP + NT - 1) / NT, typename L, typename S>
__device__ __forceinline__ void team_move(int n, L load, S store) {
  constexpr int PER = (CAP + NT - 1) / NT;
  const int tid = threadIdx.x;
#pragma unroll
  for (int k0 = 0; k0 < PER; k0 += G) {
    double v[G];
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const int e = tid + (k0 + k) * NT;
      v[k] = (k0 + k < PER && e < n) ? load(e) : 0.0;
    }
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const int e = tid + (k0 + k) * NT;
      if (k0 + k < PER && e < n) store(e, v[k]);
    }
  }
}

// LDS matrix s (leading dimension LD) from element (i, j) = at(i, j) of the
// D x D block, read from global memory by the whole team, G loads per lane
// in flight (see team_move).
template <int D, int G = D * D / Cfg<D>::NT, typename F>
__device__ __forceinline__ void lds_fill(double* s, F at) {
  using C = Cfg<D>;
  team_move<C::NT, D * D, G>(
      D * D, [&](int e) { return at(e / D, e % D); },
      [&](int e, double v) { s[(e / D) * C::LD + (e % D)] = v; });
}

// dst[e] = src[e] for e < n by NT threads, eight loads per lane in flight
// before their stores (same reason as lds_fill).
template <int NT>
__device__ __forceinline__ void team_copy(double* __restrict__ dst,
                                          const double* __restrict__ src, int n) {
  const int tid = threadIdx.x;
  for (int base = 0; base < n; base += 8 * NT) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int e = base + k * NT + tid;
      v[k] = e < n ? src[e] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int e = base + k * NT + tid;
      if (e < n) dst[e] = v[k];
    }
  }
}

// y += alpha * x
template <int D>
__device__ __forceinline__ void rm_axpy(RM<D>& y, double alpha, const RM<D>& x) {
#pragma unroll
  for (int q = 0; q < Cfg<D>::TPW; ++q) y.t[q] += alpha * x.t[q];
}

// y = x - y
template <int D>
__device__ __forceinline__ void rm_rsub(RM<D>& y, const RM<D>& x) {
#pragma unroll
  for (int q = 0; q < Cfg<D>::TPW; ++q) y.t[q] = x.t[q] - y.t[q];
}

// 0.5 (a + a^T) through an LDS scratch matrix (team-wide; starts and ends
// with a barrier, so s may still be in use by a preceding product)
template <int D>
__device__ __forceinline__ void rm_symmetrise(RM<D>& a, double* s) {
  team_sync();
  rm_stage_t<D>(a, s);
  team_sync();
  AKF_RM_FOR(D, q, r, i, j) a.t[q][r] = 0.5 * (a.t[q][r] + s[i * Cfg<D>::LD + j]);
  team_sync();
}

// c = op(A) op(B) (+ c when ACC), A and B D x D in LDS.  U k-steps per
// unrolled iteration: the full D / 4 lets every operand load issue ahead of
// the products that need it (one team at D = 64: 4.4k cycles, against 6.5k
// with U = 4), at the price of registers, so kernels near the register limit
// keep U = 4.
template <int D, bool TA, bool TB, bool ACC, int U = 4>
__device__ __forceinline__ void gemm(RM<D>& c, const double* sA, const double* sB) {
  using C = Cfg<D>;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int r0 = (D == 64) ? 32 * (w >> 1) : 0, c0 = (D == 64) ? 32 * (w & 1) : 0;
  const int li = l & 15, lk = l >> 4;
  if (!ACC) rm_zero<D>(c);
#pragma unroll U
  for (int kb = 0; kb < D / 4; ++kb) {
    const int k = 4 * kb + lk;
    double a[C::TS], b[C::TS];
#pragma unroll
    for (int ti = 0; ti < C::TS; ++ti) {
      const int i = r0 + 16 * ti + li;
      a[ti] = TA ? sA[k * C::LD + i] : sA[i * C::LD + k];
    }
#pragma unroll
    for (int tj = 0; tj < C::TS; ++tj) {
      const int j = c0 + 16 * tj + li;
      b[tj] = TB ? sB[j * C::LD + k] : sB[k * C::LD + j];
    }
#pragma unroll
    for (int ti = 0; ti < C::TS; ++ti)
#pragma unroll
      for (int tj = 0; tj < C::TS; ++tj)
        c.t[ti * C::TS + tj] =
            __builtin_amdgcn_mfma_f64_16x16x4f64(a[ti], b[tj], c.t[ti * C::TS + tj], 0, 0, 0);
  }
}

// c1 = op(A) B1, c2 = op(A) B2 (+ c when ACC): two products that share their
// left operand, interleaved so that each k-step loads A's fragments once and
// issues twice as many independent MFMA chains behind its loads.
template <int D, bool TA, bool ACC, int U = 4>
__device__ __forceinline__ void gemm2(RM<D>& c1, RM<D>& c2, const double* sA, const double* sB1,
                                      const double* sB2) {
  using C = Cfg<D>;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int r0 = (D == 64) ? 32 * (w >> 1) : 0, c0 = (D == 64) ? 32 * (w & 1) : 0;
  const int li = l & 15, lk = l >> 4;
  if (!ACC) {
    rm_zero<D>(c1);
    rm_zero<D>(c2);
  }
#pragma unroll U
  for (int kb = 0; kb < D / 4; ++kb) {
    const int k = 4 * kb + lk;
    double a[C::TS], b1[C::TS], b2[C::TS];
#pragma unroll
    for (int ti = 0; ti < C::TS; ++ti) {
      const int i = r0 + 16 * ti + li;
      a[ti] = TA ? sA[k * C::LD + i] : sA[i * C::LD + k];
    }
#pragma unroll
    for (int tj = 0; tj < C::TS; ++tj) {
      const int j = c0 + 16 * tj + li;
      b1[tj] = sB1[k * C::LD + j];
      b2[tj] = sB2[k * C::LD + j];
    }
#pragma unroll
    for (int ti = 0; ti < C::TS; ++ti)
#pragma unroll
      for (int tj = 0; tj < C::TS; ++tj) {
        c1.t[ti * C::TS + tj] =
            __builtin_amdgcn_mfma_f64_16x16x4f64(a[ti], b1[tj], c1.t[ti * C::TS + tj], 0, 0, 0);
        c2.t[ti * C::TS + tj] =
            __builtin_amdgcn_mfma_f64_16x16x4f64(a[ti], b2[tj], c2.t[ti * C::TS + tj], 0, 0, 0);
      }
  }
}

// 16 x 16 x 16 tile product on one wave: c + A B with the operands given as
// per-k-step fragments: a[s] = A[l%16][4s + l/16], b[s] = B[4s + l/16][l%16].
// In the accumulator layout, register s of a tile M is M[4s + l/16][l%16], so
// the registers of M are its own B fragments and the A fragments of M'.
__device__ __forceinline__ dbl4 mfma16(const double a[4], const double b[4], dbl4 c) {
#pragma unroll
  for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], c, 0, 0, 0);
  return c;
}
__device__ __forceinline__ void tile_regs(const dbl4& t, double x[4]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) x[s] = t[s];
}

// log-determinant accumulator: mantissa product and binary exponent sum
struct LogDet {
  double m = 1.0;
  int e = 0;
  __device__ __forceinline__ void mul(double x, double y = 1.0) {  // 1/2 <= m < 1: m x is in range with x
    int ex;
    m = frexp((m * x) * y, &ex);
    e += ex;
  }
  __device__ __forceinline__ double value() const { return log(m) + e * 0.69314718055994530942; }
};

// f(integral_constant<int, K>) for K = B .. E-1 (compile-time loop)
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Broadcast of lane K of every row of 16 lanes to the whole row (64-bit DPP
// row_newbcast).
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + K, 0xF, 0xF, true);
}

// v from lane src of the wave (ds_bpermute; no LDS memory involved)
__device__ __forceinline__ double lane_fetch(double v, int src) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// 1/q for q > 0: the hardware reciprocal estimate (relative error e about
// 2^-23) refined by one cubic step r <- r + r (e + e^2), e = 1 - q r: three
// dependent operations where two Newton-Raphson steps take four.  For 1/q in the
// normal range (q below 2^1022); an infinite q, where a variance or a product of
// two overflowed, gives NaN, not 0.
__device__ __forceinline__ double recip(double q) {
  const double r = __builtin_amdgcn_rcp(q);
  const double e = fma(-q, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// 1/sqrt(q) for q > 0: hardware estimate refined by two Newton-Raphson steps
// r <- r (3 - q r^2) / 2.
__device__ __forceinline__ double rsqrt_nr(double q) {
  double r = __builtin_amdgcn_rsq(q);
  const double h = 0.5 * q;
  r = r * fma(-h * r, r, 1.5);
  r = r * fma(-h * r, r, 1.5);
  return r;
}

// w[k] = the value of v in lane 16 k + l%16: each group's row to every lane, by
// half exchanges.
__device__ __forceinline__ void group_rows(double v, double w[4]) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  uint32_t h[2][4];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const uint32_t x = (uint32_t)(u >> (32 * s));
    const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const auto c = __builtin_amdgcn_permlane16_swap(a[i], a[i], false, false);
      h[s][2 * i] = c[0];
      h[s][2 * i + 1] = c[1];
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    w[k] = __builtin_bit_cast(double, ((uint64_t)h[1][k] << 32) | h[0][k]);
}

// v[l/16]
__device__ __forceinline__ double group_pick(const double v[4]) {
  const int l = threadIdx.x;
  const double a = (l & 16) ? v[1] : v[0], b = (l & 16) ? v[3] : v[2];
  return (l & 32) ? b : a;
}

// One wave inverts a symmetric positive definite 16 x 16 tile held in the
// accumulator layout (p[r] = P[4r + l/16][l%16]) by four steps of the
// symmetric sweep operator on blocks of four pivots: with W the block's rows
// (4 x 16, one register of the layout) and B their 4 x 4 block,
//   a <- a - W' B^{-1} W,  block columns <- W' B^{-1},  block rows <- B^{-1} W,
//   block <- -B^{-1},
// which leaves -P^{-1}.  With W~ = W, but -I in the block's columns, all of it
// is one MFMA, m a - W' G with G = B^{-1} W~ and m = 0 in the block's columns,
// and the block's rows are G itself.  Every lane factors B = L D L' for itself
// (W's rows reach all lane groups by half exchanges, B's entries by DPP
// broadcasts) and solves for its own column of G.  The pivots are those of the
// LDL' factorisation of the tile; with CHOL the columns of L D are the rows
// L^{-1} W, transposed into place by a second MFMA off the chain, and scaled by
// 1/sqrt(pivot) at the end, one square root for all sixteen.  Bound by the
// issue of about 110 vector instructions a block and the MFMA's latency:
// 2.4k cycles a tile, with CHOL 2.6k; sixteen single pivots, each a lane
// permute (58 cycles), a scaling and an update in a chain, took 3.0k and 3.8k.
// Indices >= nv are padding: they get a unit diagonal.  A non-positive pivot
// clears ok (the results are then unspecified).
template <bool CHOL, int PART = 0>
__device__ __forceinline__ void tile_sweep16(double p[4], int nv, double Lk[4], LogDet& ld,
                                             bool& ok) {
  const int l = threadIdx.x & 63, lg = l >> 4, lc = l & 15;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (4 * r + lg >= nv && 4 * r + lg == lc) p[r] = 1.0;
  dbl4 La = {0.0, 0.0, 0.0, 0.0};
  double qd = 1.0;
  auto step = [&](auto bc) {
    constexpr int b = decltype(bc)::value;
    const double W = p[b];
    double w[4], v[4], g[4];
    group_rows(W, w);
    const double a00 = row_bcast<4 * b>(w[0]), a01 = row_bcast<4 * b + 1>(w[0]),
                 a02 = row_bcast<4 * b + 2>(w[0]), a03 = row_bcast<4 * b + 3>(w[0]);
    const double a11 = row_bcast<4 * b + 1>(w[1]), a12 = row_bcast<4 * b + 2>(w[1]),
                 a13 = row_bcast<4 * b + 3>(w[1]);
    const double a22 = row_bcast<4 * b + 2>(w[2]), a23 = row_bcast<4 * b + 3>(w[2]);
    const double a33 = row_bcast<4 * b + 3>(w[3]);
    // B = L D L': pivots q, their reciprocals i, columns of L
    const double i0 = recip(a00);
    const double l1 = a01 * i0, l2 = a02 * i0, l3 = a03 * i0;
    const double b11 = fma(-l1, a01, a11), b12 = fma(-l1, a02, a12), b13 = fma(-l1, a03, a13);
    const double b22 = fma(-l2, a02, a22), b23 = fma(-l2, a03, a23), b33 = fma(-l3, a03, a33);
    const double i1 = recip(b11);
    const double m2 = b12 * i1, m3 = b13 * i1;
    const double c22 = fma(-m2, b12, b22), c23 = fma(-m2, b13, b23), c33 = fma(-m3, b13, b33);
    const double i2 = recip(c22);
    const double n3 = c23 * i2;
    const double q3 = fma(-n3, c23, c33);
    const double i3 = recip(q3);
    ok = ok && (a00 > 0.0) && (b11 > 0.0) && (c22 > 0.0) && (q3 > 0.0);
    // in pivot order, as single pivots are taken: two large pivots multiplied with
    // each other first would overflow where the four together do not
    ld.mul((a00 * b11) * c22, q3);
    // opaque to the compiler, which would otherwise hold the lane masks in
    // registers across the loops around the sweep (and spill)
    int lcb = lc;
    asm volatile("" : "+v"(lcb));
    const bool blk = (lcb >> 2) == b;
    const double mc = blk ? 0.0 : 1.0;
    auto forward = [&](const double x[4]) {  // L^{-1} x
      v[0] = x[0];
      v[1] = fma(-l1, v[0], x[1]);
      v[2] = fma(-m2, v[1], fma(-l2, v[0], x[2]));
      v[3] = fma(-n3, v[2], fma(-m3, v[1], fma(-l3, v[0], x[3])));
    };
    if constexpr (CHOL) {
      forward(w);
      La = __builtin_amdgcn_mfma_f64_16x16x4f64(group_pick(v), lcb == 4 * b + lg ? 1.0 : 0.0, La, 0,
                                                0, 0);
      const double qk[4] = {a00, b11, c22, q3};
#pragma unroll
      for (int k = 0; k < 4; ++k) qd = lcb == 4 * b + k ? qk[k] : qd;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = blk ? (lcb == 4 * b + k ? -1.0 : 0.0) : w[k];
    forward(w);
    g[3] = v[3] * i3;
    g[2] = fma(-n3, g[3], v[2] * i2);
    g[1] = fma(-m2, g[2], fma(-m3, g[3], v[1] * i1));
    g[0] = fma(-l1, g[1], fma(-l2, g[2], fma(-l3, g[3], v[0] * i0)));
    const double G = group_pick(g);
    const dbl4 a = {p[0] * mc, p[1] * mc, p[2] * mc, p[3] * mc};
    const dbl4 o = __builtin_amdgcn_mfma_f64_16x16x4f64(-W, G, a, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = (r == b) ? G : o[r];
  };
  // one pivot k < 4: a_ij <- a_ij - c_i c_j / q, column and row k as above
  auto single = [&](auto kc) {
    constexpr int k = decltype(kc)::value;
    if (k >= nv) return;
    double ci[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) ci[r] = row_bcast<k>(p[r]);
    const double q = lane_bcast(p[0], 17 * k);
    const double cj = lane_fetch(p[0], 16 * k + lc);
    ok = ok && (q > 0.0);
    const double iq = recip(q);
    ld.mul(q);
    const bool jk = (lc == k);
    const double gj = jk ? iq : -(cj * iq);
    const double mc = jk ? 0.0 : 1.0;
    if constexpr (CHOL) {
#pragma unroll
      for (int r = 0; r < 4; ++r) La[r] = jk ? p[r] : La[r];
      qd = jk ? q : qd;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = fma(ci[r], gj, p[r] * mc);
    p[0] = (lg == k) ? -gj : p[0];
  };
  if (!PART || nv >= 16) {
    static_for<0, 4>(step);
  } else if (PART == 2 && nv < 4) {
    // a block of four costs as much as three and a half single pivots
    static_for<0, 3>(single);
  } else {
    // PART, a tile with padding (a team wider than d): the blocks of padded
    // pivots change no valid entry (their column is zero there), so they are
    // skipped and the padded part is set to what they would have left (unit
    // diagonal).  2: with single pivots, for the 16-wide bodies (in wider ones
    // that path costs registers).
    auto some = [&](auto bc) {
      if (4 * decltype(bc)::value < nv) step(bc);
    };
    static_for<0, 4>(some);
  }
  if constexpr (CHOL) {
    const double isq = rsqrt_nr(qd);
#pragma unroll
    for (int r = 0; r < 4; ++r) Lk[r] = (4 * r + lg >= lc) ? La[r] * isq : 0.0;
  }
  if (PART && nv < 16) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 4 * r + lg;
      if (i >= nv || lc >= nv) {
        p[r] = (i == lc) ? -1.0 : 0.0;  // negated below
        if constexpr (CHOL) Lk[r] = (i == lc) ? 1.0 : 0.0;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) p[r] = -p[r];
}

// G = L^{-T} for a 16 x 16 tile from its Cholesky factor (Lk, acc layout) and
// the inverse of the tile (ainv, symmetric): G0 = A^{-1} L, then one Newton
// step G = G0 + G0 (I - L' G0), with L^{-1} ~ L' A^{-1} as G0' in the
// correction.  Forming L^{-T} through A^{-1} alone loses accuracy with the
// conditioning of the tile; the Newton step restores it.
__device__ __forceinline__ void chol_tile_rinv(const double ainv[4], const double Lk[4],
                                               double G[4]) {
  const int l = threadIdx.x & 63, lg = l >> 4, lc = l & 15;
  const dbl4 z = {0.0, 0.0, 0.0, 0.0};
  double H[4], R[4];
  tile_regs(mfma16(ainv, Lk, z), G);  // A^{-1} L  (acc of L^{-T})
  tile_regs(mfma16(Lk, ainv, z), H);  // L' A^{-1} (acc of L^{-1})
  const dbl4 T = mfma16(Lk, G, z);    // L' G ~ I
#pragma unroll
  for (int r = 0; r < 4; ++r) R[r] = ((4 * r + lg == lc) ? 1.0 : 0.0) - T[r];
  dbl4 g = {G[0], G[1], G[2], G[3]};
  tile_regs(mfma16(H, R, g), G);  // G + G (I - L' G)
}

// One Newton-Schulz step X <- X + X (I - A X) on an approximate inverse X of
// the register matrix A (both zero outside the leading d x d block): squares
// the residual, so an inverse accurate to r relative becomes accurate to
// ~cond(A) r^2 plus rounding.  s1, s2: free LDS matrices.  Team-wide; ends
// synchronised.
template <int D>
__device__ void inv_refine(RM<D>& X, const RM<D>& A, int d, double* s1, double* s2) {
  team_sync();
  rm_stage<D>(X, s1);
  rm_stage<D>(A, s2);
  team_sync();
  RM<D> T;
  gemm<D, false, false, false>(T, s2, s1);  // A X
  AKF_RM_FOR(D, q, r, i, j) T.t[q][r] = ((i == j && i < d) ? 1.0 : 0.0) - T.t[q][r];
  team_sync();
  rm_stage<D>(T, s2);
  team_sync();
  gemm<D, false, false, true>(X, s1, s2);  // X + X (I - A X)
  team_sync();
}

// transpose of a tile through 16 x 17 doubles of LDS
__device__ __forceinline__ dbl4 tile_t(const dbl4& t, double* s) {
  const int l = threadIdx.x & 63, lg = l >> 4, lc = l & 15;
#pragma unroll
  for (int r = 0; r < 4; ++r) s[lc * 17 + 4 * r + lg] = t[r];
  wave_lds_fence();
  dbl4 o;
#pragma unroll
  for (int r = 0; r < 4; ++r) o[r] = s[(4 * r + lg) * 17 + lc];
  wave_lds_fence();
  return o;
}

// c + a' b of one tile
__device__ __forceinline__ dbl4 tile_tn(const dbl4& a, const dbl4& b, dbl4 c) {
#pragma unroll
  for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], c, 0, 0, 0);
  return c;
}

template <int D>
__device__ __forceinline__ void rm_mask(RM<D>& a, int d) {
  AKF_RM_FOR(D, q, r, i, j) if (i >= d || j >= d) a.t[q][r] = 0.0;
}

__device__ __forceinline__ dbl4 tile_of(const double p[4]) { return dbl4{p[0], p[1], p[2], p[3]}; }

// In-place inverse of a symmetric positive definite matrix held by one wave
// (zero outside the leading d x d block) by 2 x 2 blocks of tiles
// [[a, b], [b', c]]: with P = a^{-1}, X = P b and S = c - b' X,
//   inverse = [[P + X S^{-1} X', -X S^{-1}], [-S^{-1} X', S^{-1}]].
// Reads the diagonal and upper tiles; the result's lower tile mirrors its
// upper one.  KT = 1: d <= 16, the first tile alone (the others are not
// touched).  Returns false on a non-positive pivot (the result is then
// unspecified); the pivots go into ld.  scr: one padded tile of LDS (D = 32).
template <int D, int KT = Cfg<D>::TS>
__device__ __forceinline__ bool wave_inv(RM<D>& A, int d, double* scr, LogDet& ld) {
  bool ok = true;
  double p[4], dummy[4];
  tile_regs(A.t[0], p);
  tile_sweep16<false, KT == 1 ? 2 : 0>(p, d, dummy, ld, ok);
  if constexpr (KT == 1) {
    A.t[0] = tile_of(p);
    const int l = threadIdx.x & 63, lg = l >> 4, lc = l & 15;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * r + lg >= d || lc >= d) A.t[0][r] = 0.0;
  } else {
    const dbl4 z = {0.0, 0.0, 0.0, 0.0};
    const dbl4 P = tile_of(p);
    const dbl4 X = tile_tn(P, A.t[1], z);           // P b
    const dbl4 Z = tile_t(X, scr);                  // X'
    const dbl4 S = A.t[3] - tile_tn(A.t[1], X, z);  // c - b' X
    tile_regs(S, p);
    tile_sweep16<false, 1>(p, d - 16, dummy, ld, ok);
    const dbl4 Si = tile_of(p);
    const dbl4 Wt = tile_tn(Si, Z, z);  // S^{-1} X'
    A.t[0] = tile_tn(Z, Wt, P);         // P + X S^{-1} X'
    A.t[2] = -Wt;
    A.t[1] = tile_t(A.t[2], scr);
    A.t[3] = Si;
    rm_mask<D>(A, d);
  }
  return ok;
}

// Lower Cholesky factor of a symmetric positive definite matrix held by one
// wave (diagonal and upper tiles read): the diagonal tiles' factors l0, l1
// (unit diagonal at padded indices) and both orientations of the tile between.
// INV: also the tiles of the factor's inverse transpose, g0 = l0^{-T},
// g1 = l1^{-T}, k01 = -g0 l10' g1.  scr: one padded tile of LDS.
struct Chol32 {
  dbl4 l0, l1, l10, l10t, g0, g1, k01;
};
template <bool INV>
__device__ __forceinline__ bool chol32(const dbl4& a, const dbl4& b, const dbl4& c, int d, double* scr,
                                       Chol32& o) {
  const dbl4 z = {0.0, 0.0, 0.0, 0.0};
  bool ok = true;
  LogDet ld;
  double p[4], Lk[4], G[4];
  tile_regs(a, p);
  tile_sweep16<true, 0>(p, d, Lk, ld, ok);
  o.l0 = tile_of(Lk);
  chol_tile_rinv(p, Lk, G);
  o.g0 = tile_of(G);
  o.l10t = tile_tn(o.g0, b, z);  // (l10)' = l0^{-1} b
  o.l10 = tile_tn(b, o.g0, z);
  const dbl4 S = c - tile_tn(o.l10t, o.l10t, z);
  tile_regs(S, p);
  tile_sweep16<true, INV ? 0 : 1>(p, d - 16, Lk, ld, ok);
  o.l1 = tile_of(Lk);
  if constexpr (INV) {
    chol_tile_rinv(p, Lk, G);
    o.g1 = tile_of(G);
    o.k01 = -tile_tn(tile_t(o.g0, scr), tile_tn(o.l10, o.g1, z), z);
  }
  return ok;
}

// Lower Cholesky factor L of a matrix held by one wave, and its transpose LT.
template <int D>
__device__ __forceinline__ bool wave_chol(const RM<D>& A, RM<D>& L, RM<D>& LT, int d, double* scr) {
  bool ok = true;
  if constexpr (D == 16) {
    LogDet ld;
    double p[4], Lk[4];
    tile_regs(A.t[0], p);
    tile_sweep16<true, 2>(p, d, Lk, ld, ok);
    L.t[0] = tile_of(Lk);
  } else {
    const dbl4 z = {0.0, 0.0, 0.0, 0.0};
    Chol32 c;
    ok = chol32<false>(A.t[0], A.t[1], A.t[3], d, scr, c);
    L.t[0] = c.l0;
    L.t[1] = z;
    L.t[2] = c.l10;
    L.t[3] = c.l1;
    LT.t[1] = c.l10t;
    LT.t[2] = z;
  }
  AKF_RM_FOR(D, q, r, i, j) if (j > i || i >= d) L.t[q][r] = 0.0;
  LT.t[0] = tile_t(L.t[0], scr);
  if constexpr (D == 32) {
    LT.t[3] = tile_t(L.t[3], scr);
    AKF_RM_FOR(D, q, r, i, j) if (i >= d || j >= d) LT.t[q][r] = 0.0;
  }
  return ok;
}

// ---------------------------------------------------------------------------
// Factorisations by a team.  Below D = 64 the team is one wave.  At D = 64 the
// matrix is split into 32 x 32 blocks [[a, b], [b', c]] and the four waves go
// through the formulas of wave_inv / chol32 one level up: the 32 x 32 blocks
// are factored by every wave for itself (from LDS, so nothing is broadcast),
// and each wave forms one tile of every 32 x 32 product: 19.9k cycles for the
// inverse and 23.3k for the factor of a 64 x 64 matrix, four pivot tiles of
// 2.4k (with the factor 2.6k) in each.  Four panels of the whole matrix, each
// with its pivot tile, its block row through LDS and a third of the tiles'
// updates behind uniform branches, took 27.7k and 34.9k with tiles of 3.0k and
// 3.8k.
// ---------------------------------------------------------------------------
// doubles of LDS scratch
template <int D>
constexpr int inv_scratch() {
  return D == 16 ? 0 : (D == 32 ? 16 * 17 : 3 * 32 * 34);
}

// 32 x 32 blocks in LDS; the leading dimension makes one block hold a padded
// tile (16 x 17) for each of the four waves
struct Blk {
  static constexpr int LD = 34, SIZE = 32 * LD;
  // tile (ti, tj) in the accumulator layout, and its transpose
  static __device__ __forceinline__ dbl4 get(const double* s, int ti, int tj) {
    const int l = threadIdx.x & 63, lg = l >> 4, lc = l & 15;
    const double* p = s + (16 * ti + lg) * LD + 16 * tj + lc;
    return dbl4{p[0], p[4 * LD], p[8 * LD], p[12 * LD]};
  }
  static __device__ __forceinline__ dbl4 get_t(const double* s, int ti, int tj) {
    const int l = threadIdx.x & 63, lg = l >> 4, lc = l & 15;
    const double* p = s + (16 * ti + lc) * LD + 16 * tj + lg;
    return dbl4{p[0], p[4], p[8], p[12]};
  }
  static __device__ __forceinline__ void put(double* s, int ti, int tj, const dbl4& t) {
    const int l = threadIdx.x & 63, lg = l >> 4, lc = l & 15;
    double* p = s + (16 * ti + lg) * LD + 16 * tj + lc;
    p[0] = t[0];
    p[4 * LD] = t[1];
    p[8 * LD] = t[2];
    p[12 * LD] = t[3];
  }
};

__device__ __forceinline__ dbl4 pick2(int k, const dbl4& a, const dbl4& b) {
  dbl4 o;
#pragma unroll
  for (int r = 0; r < 4; ++r) o[r] = k ? b[r] : a[r];
  return o;
}

// In-place inverse of a symmetric positive definite matrix held in registers
// (zero outside the leading d x d block).  Returns false on a non-positive
// pivot (the result is then unspecified); *logdet = log det A from the pivots.
// scr: inv_scratch<D>() doubles of LDS, free at entry; the call begins and
// ends with a team barrier.
template <int D>
__device__ bool spd_inv(RM<D>& A, int d, double* scr, double* logdet) {
  static_assert(inv_scratch<D>() <= Cfg<D>::MAT, "scratch must fit one LDS matrix");
  LogDet ld;
  bool ok;
  team_sync();
  if constexpr (D <= 32) {
    ok = wave_inv<D>(A, d, scr, ld);
  } else {
    const int w = threadIdx.x >> 6, R0 = w >> 1, C0 = w & 1;
    double *Ba = scr, *Bb = Ba + Blk::SIZE, *Bc = Bb + Blk::SIZE;
    double* own = w == 0 ? Ba : (w == 1 ? Bb : Bc);
    if (w != 2) {
#pragma unroll
      for (int q = 0; q < 4; ++q) Blk::put(own, q >> 1, q & 1, A.t[q]);
    }
    team_sync();
    RM<32> P, Si;
    P.t[0] = Blk::get(Ba, 0, 0);
    P.t[1] = Blk::get(Ba, 0, 1);
    P.t[3] = Blk::get(Ba, 1, 1);
    team_sync();  // Ba is the waves' tile scratch now, then X
    ok = wave_inv<32>(P, min(d, 32), Ba + w * 16 * 17, ld);  // a^{-1}
    {
      dbl4 x = {0.0, 0.0, 0.0, 0.0};  // X = P b
      x = tile_tn(pick2(R0, P.t[0], P.t[1]), Blk::get(Bb, 0, C0), x);
      x = tile_tn(pick2(R0, P.t[2], P.t[3]), Blk::get(Bb, 1, C0), x);
      team_sync();
      Blk::put(Ba, R0, C0, x);
    }
    team_sync();
    {
      dbl4 x = {0.0, 0.0, 0.0, 0.0};  // S = c - b' X
      x = tile_tn(Blk::get(Bb, 0, R0), Blk::get(Ba, 0, C0), x);
      x = tile_tn(Blk::get(Bb, 1, R0), Blk::get(Ba, 1, C0), x);
      Blk::put(Bc, R0, C0, Blk::get(Bc, R0, C0) - x);
    }
    team_sync();
    Si.t[0] = Blk::get(Bc, 0, 0);
    Si.t[1] = Blk::get(Bc, 0, 1);
    Si.t[3] = Blk::get(Bc, 1, 1);
    team_sync();  // Bc is scratch
    if (d <= 48) {  // S is one tile (filter at d = 33, N = 100: 398 -> 380 us, lone element build 47 -> 45)
      ok = wave_inv<32, 1>(Si, d - 32, nullptr, ld) && ok;
      Si.t[1] = Si.t[2] = Si.t[3] = dbl4{0.0, 0.0, 0.0, 0.0};
    } else {
      ok = wave_inv<32>(Si, d - 32, Bc + w * 16 * 17, ld) && ok;
    }
    {
      dbl4 x = {0.0, 0.0, 0.0, 0.0};  // S^{-1} X', over b
      x = tile_tn(pick2(R0, Si.t[0], Si.t[1]), Blk::get_t(Ba, C0, 0), x);
      x = tile_tn(pick2(R0, Si.t[2], Si.t[3]), Blk::get_t(Ba, C0, 1), x);
      Blk::put(Bb, R0, C0, x);
    }
    team_sync();
    {
      // P + X S^{-1} X', over S
      dbl4 x = pick2(R0, pick2(C0, P.t[0], P.t[1]), pick2(C0, P.t[2], P.t[3]));
      x = tile_tn(Blk::get_t(Ba, R0, 0), Blk::get(Bb, 0, C0), x);
      x = tile_tn(Blk::get_t(Ba, R0, 1), Blk::get(Bb, 1, C0), x);
      Blk::put(Bc, R0, C0, x);
    }
    team_sync();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (w == 0)
        A.t[q] = Blk::get(Bc, q >> 1, q & 1);
      else if (w == 1)
        A.t[q] = -Blk::get_t(Bb, q & 1, q >> 1);
      else if (w == 2)
        A.t[q] = -Blk::get(Bb, q >> 1, q & 1);
      else
        A.t[q] = Si.t[q];
    }
  }
  team_sync();
  *logdet = ld.value();
  return ok;
}

// Lower Cholesky factor (positive diagonal) of a symmetric positive definite
// matrix held in registers (zero outside the leading d x d block), in place;
// the strict upper triangle is zeroed.  Returns false on a non-positive pivot.
// Same scr contract as spd_inv.  At D = 64 with m = (chol a)^{-T}:
// L10' = m' b, then chol(c - L10 L10').
template <int D>
__device__ bool chol_reg(RM<D>& A, int d, double* scr) {
  static_assert(inv_scratch<D>() <= Cfg<D>::MAT, "scratch must fit one LDS matrix");
  const dbl4 z = {0.0, 0.0, 0.0, 0.0};
  bool ok = true;
  team_sync();
  if constexpr (D == 16) {
    LogDet ld;
    double p[4], Lk[4];
    tile_regs(A.t[0], p);
    tile_sweep16<true, 2>(p, d, Lk, ld, ok);
    A.t[0] = tile_of(Lk);
  } else if constexpr (D == 32) {
    Chol32 c;
    ok = chol32<false>(A.t[0], A.t[1], A.t[3], d, scr, c);
    A.t[0] = c.l0;
    A.t[2] = c.l10;
    A.t[3] = c.l1;
  } else {
    const int w = threadIdx.x >> 6, R0 = w >> 1, C0 = w & 1;
    double *Ba = scr, *Bb = Ba + Blk::SIZE, *Bc = Bb + Blk::SIZE;
    double* own = w == 0 ? Ba : (w == 1 ? Bb : Bc);
    if (w != 2) {
#pragma unroll
      for (int q = 0; q < 4; ++q) Blk::put(own, q >> 1, q & 1, A.t[q]);
    }
    team_sync();
    Chol32 c, e;
    {
      const dbl4 a0 = Blk::get(Ba, 0, 0), a1 = Blk::get(Ba, 0, 1), a3 = Blk::get(Ba, 1, 1);
      team_sync();  // Ba is the waves' tile scratch now, then L10'
      ok = chol32<true>(a0, a1, a3, min(d, 32), Ba + w * 16 * 17, c);
    }
    {
      // tile row 0 of m' b takes g0 alone, row 1 takes k01 and g1
      dbl4 x = tile_tn(pick2(R0, c.g0, c.k01), Blk::get(Bb, 0, C0), z);
      if (R0) x = tile_tn(c.g1, Blk::get(Bb, 1, C0), x);
      team_sync();
      Blk::put(Ba, R0, C0, x);
    }
    team_sync();
    {
      dbl4 x = tile_tn(Blk::get(Ba, 0, R0), Blk::get(Ba, 0, C0), z);
      x = tile_tn(Blk::get(Ba, 1, R0), Blk::get(Ba, 1, C0), x);
      Blk::put(Bc, R0, C0, Blk::get(Bc, R0, C0) - x);
    }
    team_sync();
    ok = chol32<false>(Blk::get(Bc, 0, 0), Blk::get(Bc, 0, 1), Blk::get(Bc, 1, 1), d - 32, nullptr, e) &&
         ok;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (w == 2)
        A.t[q] = Blk::get_t(Ba, q & 1, q >> 1);
      else if (w != 1)
        A.t[q] = pick2(w, q == 0 ? c.l0 : (q == 2 ? c.l10 : c.l1),
                       q == 0 ? e.l0 : (q == 2 ? e.l10 : e.l1));
    }
  }
  AKF_RM_FOR(D, q, r, i, j) if (j > i || i >= d) A.t[q][r] = 0.0;
  team_sync();
  return ok;
}

// y[i] = add[i] + sum_j op(A)[i][j] x[j] for i < D (LDS matrix; add may be
// null, may alias y, and may live in global memory; x must not alias y).
// Every wave takes D / NW rows and splits each row over 64 / (D / NW) lanes,
// reduced by half exchanges, so the dependent chain is 8 (D >= 32) or 2 FMAs
// long.  Team-wide; ends with a barrier, after which y is visible to all.
template <int D, bool TA>
__device__ __forceinline__ void matvec(double* y, const double* sA, const double* x,
                                       const double* add = nullptr) {
  using C = Cfg<D>;
  constexpr int R = D / C::NW;  // rows per wave
  constexpr int P = 64 / R;     // lanes per row
  constexpr int JL = D / P;     // columns per lane
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int i = w * R + (l % R), j0 = (l / R) * JL;
  double a[2] = {0.0, 0.0};
#pragma unroll
  for (int jj = 0; jj < JL; ++jj) {
    const int j = j0 + jj;
    a[jj & 1] = fma(TA ? sA[j * C::LD + i] : sA[i * C::LD + j], x[j], a[jj & 1]);
  }
  const double s = R == 16 ? sum_groups(a[0] + a[1]) : sum_x32(a[0] + a[1]);
  if (l < R) y[i] = (add ? add[i] : 0.0) + s;
  team_sync();
}

// team-wide sum of one double per thread (result returned to every thread)
template <int D>
__device__ __forceinline__ double team_sum(double v, double* sRed) {
  using C = Cfg<D>;
  v = wave_total(v);
  const int tid = threadIdx.x;
  if ((tid & 63) == 0) sRed[tid >> 6] = v;
  team_sync();
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < C::NW; ++i) s += sRed[i];
  team_sync();
  return s;
}

}  // namespace akf
