// akf_wave.hpp -- one-wave (D = 16 and 32) bodies of the filter and sampler
// kernels, with every matrix operand in registers.
//
// A lone wave holding whole matrices needs no staging for its products: in the
// accumulator layout (akf_team.hpp) a tile's registers are its own B fragments
// and the A fragments of its transpose, so x' y takes its operands as they
// are.  Every product of the filter and the sampler is written in that form,
// with the constant F kept as F'; the transposes that remain (one tile to
// mirror a symmetric result, the diagonal tiles of a symmetrisation) go
// through a 16 x 17 LDS tile.  Symmetric results form their upper tiles only.
// A wave's LDS operations complete in order, so no barrier is needed; LDS per
// team is a few KB, and the registers alone decide how many waves share a
// SIMD.  With operands staged through LDS instead (a store, a wait and two
// loads around each product) a fold step of a lone wave took 10.8k cycles at
// D = 16 and 38k at D = 32.  Bound by the chain of products (256 cycles a tile)
// and pivot tiles of a lone wave, or by the registers' one or two waves a SIMD:
// fold of d = 8, N = 1024 20 -> 12.6 us; 128 ragged chains of up to 8192 steps,
// D = 32: fold 3.05 -> 1.90 ms, re-scan 2.45 -> 1.21, element build 3.4 -> 2.2.
#pragma once
#include "akf_internal.h"
#include "akf_team.hpp"

namespace akf {

// ---------------------------------------------------------------------------
// tiles and products
// ---------------------------------------------------------------------------
template <int D>
constexpr int wave_scr() {  // doubles of LDS scratch: one padded tile per tile of a matrix
  return Cfg<D>::TPW * 16 * 17;
}

// LDS bytes of every one-wave body: scratch tiles and eight vectors
template <int D>
constexpr size_t wave_lds_bytes() {
  return (size_t)(wave_scr<D>() + 8 * D) * sizeof(double);
}

template <int D>
__device__ __forceinline__ RM<D> rm_t(const RM<D>& a, double* scr) {
  constexpr int TS = Cfg<D>::TS;
  RM<D> o;
#pragma unroll
  for (int ti = 0; ti < TS; ++ti)
#pragma unroll
    for (int tj = 0; tj < TS; ++tj)
      o.t[tj * TS + ti] = tile_t(a.t[ti * TS + tj], scr + (ti * TS + tj) * 16 * 17);
  return o;
}

// c += x' y over the first KT tile rows of x and y, result tile rows < RT and
// columns < CT; UP: only the tiles on and above the diagonal.
template <int D, bool UP = false, int KT = Cfg<D>::TS, int RT = Cfg<D>::TS, int CT = Cfg<D>::TS>
__device__ __forceinline__ void tn(RM<D>& c, const RM<D>& x, const RM<D>& y) {
  constexpr int TS = Cfg<D>::TS;
#pragma unroll
  for (int k = 0; k < KT; ++k)
#pragma unroll
    for (int ti = 0; ti < RT; ++ti)
#pragma unroll
      for (int tj = UP ? ti : 0; tj < CT; ++tj)
        c.t[ti * TS + tj] = tile_tn(x.t[k * TS + ti], y.t[k * TS + tj], c.t[ti * TS + tj]);
}

// c = x' y (same parameters)
template <int D, bool UP = false, int KT = Cfg<D>::TS, int RT = Cfg<D>::TS, int CT = Cfg<D>::TS>
__device__ __forceinline__ RM<D> tn0(const RM<D>& x, const RM<D>& y) {
  RM<D> c;
  rm_zero<D>(c);
  tn<D, UP, KT, RT, CT>(c, x, y);
  return c;
}

// lower tiles from the upper ones
template <int D>
__device__ __forceinline__ void mirror(RM<D>& c, double* scr) {
  if constexpr (D == 32) c.t[2] = tile_t(c.t[1], scr);
}

// the same with the diagonal tiles averaged with their transposes
template <int D>
__device__ __forceinline__ void symm(RM<D>& c, double* scr) {
  constexpr int TS = Cfg<D>::TS;
  dbl4 o[TS];
#pragma unroll
  for (int k = 0; k < TS; ++k) o[k] = tile_t(c.t[k * TS + k], scr + k * 16 * 17);
  if constexpr (D == 32) c.t[2] = tile_t(c.t[1], scr + 2 * 16 * 17);
#pragma unroll
  for (int k = 0; k < TS; ++k) c.t[k * TS + k] = 0.5 * (c.t[k * TS + k] + o[k]);
}

// a_ij = G[i*ld + j] for i < rows, j < cols, zero elsewhere
template <int D>
__device__ __forceinline__ void rm_load_rect(RM<D>& a, const double* __restrict__ g, int ld,
                                             int rows, int cols) {
  AKF_RM_FOR(D, q, r, i, j) a.t[q][r] = (i < rows && j < cols) ? g[(size_t)i * ld + j] : 0.0;
}

// a_ij = G[j*ld + i] for i < rows, j < cols, zero elsewhere
template <int D>
__device__ __forceinline__ void rm_load_t(RM<D>& a, const double* __restrict__ g, int ld, int rows,
                                          int cols) {
  AKF_RM_FOR(D, q, r, i, j) a.t[q][r] = (i < rows && j < cols) ? g[(size_t)j * ld + i] : 0.0;
}

// ---------------------------------------------------------------------------
// vectors: in LDS, and in registers by row (element 16 ti + 4 r + l/16)
// ---------------------------------------------------------------------------
template <int D>
struct RV {
  double v[Cfg<D>::TS][4];
};

template <int D>
__device__ __forceinline__ RV<D> rv(const double* s) {
  const int lg = (threadIdx.x & 63) >> 4;
  RV<D> o;
#pragma unroll
  for (int ti = 0; ti < Cfg<D>::TS; ++ti)
#pragma unroll
    for (int r = 0; r < 4; ++r) o.v[ti][r] = s[16 * ti + 4 * r + lg];
  return o;
}

// lane l < D: (x' v)_l; other lanes: unspecified
template <int D, int KT = Cfg<D>::TS>
__device__ __forceinline__ double mv(const RM<D>& x, const RV<D>& v) {
  constexpr int TS = Cfg<D>::TS;
  double s[TS];
#pragma unroll
  for (int tj = 0; tj < TS; ++tj) {
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int ti = 0; ti < KT; ++ti) {
      a = fma(x.t[ti * TS + tj][0], v.v[ti][0], a);
      b = fma(x.t[ti * TS + tj][1], v.v[ti][1], b);
      a = fma(x.t[ti * TS + tj][2], v.v[ti][2], a);
      b = fma(x.t[ti * TS + tj][3], v.v[ti][3], b);
    }
    s[tj] = sum_groups(a + b);
  }
  if constexpr (TS == 1) return s[0];
  else return (threadIdx.x & 16) ? s[1] : s[0];
}

// the value of lane l < D into s[l]
template <int D>
__device__ __forceinline__ void vec_put(double* s, double v) {
  const int l = threadIdx.x;
  if (l < D) s[l] = v;
  wave_lds_fence();
}

// ---------------------------------------------------------------------------
// factorisations
// ---------------------------------------------------------------------------
// x_ij *= v_i
template <int D>
__device__ __forceinline__ void scale_rows(RM<D>& x, const RV<D>& v) {
  constexpr int TS = Cfg<D>::TS;
#pragma unroll
  for (int q = 0; q < Cfg<D>::TPW; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) x.t[q][r] *= v.v[q / TS][r];
}

template <int D>
__device__ __forceinline__ void add_eye(RM<D>& x, int d) {
  AKF_RM_FOR(D, q, r, i, j) if (i == j && i < d) x.t[q][r] += 1.0;
}

// ---------------------------------------------------------------------------
// Filter, block fold (the recursion above filter_fold_impl)
// ---------------------------------------------------------------------------
// The general-observation update with KT tile rows of observations (dobs <= 16
// needs one): with Mo = H Pp, N = Mo' and Mt = H T, S = H N + R,
//   C = Pp - Mo' S^{-1} Mo, A = T - Mo' S^{-1} Mt, J += Mt' S^{-1} Mt.
template <int D, int KT, bool FIRST>
__device__ __forceinline__ bool wave_update_gh(const FilterArgs& P, int t, const RM<D>& HT,
                                               const RM<D>& Pp, const RM<D>& T, RM<D>& A, RM<D>& Cc,
                                               RM<D>& J, double* vb, double* veta, double* vmu,
                                               double* vs, double* scr, LogDet& ld, double& q_part) {
  constexpr int TS = Cfg<D>::TS;
  const int l = threadIdx.x, m = P.dyo;
  const double y = l < m ? P.yo[(int64_t)t * m + l] : 0.0;
  const RM<D> Mo = tn0<D, false, TS, KT>(HT, Pp);
  RM<D> N;
#pragma unroll
  for (int ti = 0; ti < KT; ++ti)
#pragma unroll
    for (int tj = 0; tj < TS; ++tj)
      N.t[tj * TS + ti] = tile_t(Mo.t[ti * TS + tj], scr + (ti * TS + tj) * 16 * 17);
  RM<D> S;
  rm_load<D>(S, P.Ro, m, m);
  tn<D, true, TS, KT, KT>(S, N, HT);  // Mo H' + R
  const double hm = mv<D>(HT, rv<D>(vmu));  // H mu
  const double vw = l < m ? y - hm : 0.0;
  const bool ok = wave_inv<D, KT>(S, m, scr, ld);
  vec_put<D>(vs, vw);
  const double si = mv<D, KT>(S, rv<D>(vs));  // S^{-1} w
  q_part += l < D ? vw * si : 0.0;
  vec_put<D>(vs, l < m ? si : 0.0);
  const RV<D> rs = rv<D>(vs);
  RM<D> U = tn0<D, false, KT, KT>(S, Mo);
  Cc = tn0<D, true, KT>(Mo, U);
  rm_rsub<D>(Cc, Pp);
  const double b = mv<D, KT>(Mo, rs);
  if constexpr (!FIRST) {
    const RM<D> Mt = tn0<D, false, TS, KT>(HT, T);
    U = tn0<D, false, KT, KT>(S, Mt);
    tn<D, true, KT>(J, Mt, U);
    A = tn0<D, false, KT>(Mo, U);
    rm_rsub<D>(A, T);
    const double e = mv<D, KT>(Mt, rs);
    if (l < D) veta[l] += e;
  }
  if (l < D) vb[l] = vmu[l] + b;
  wave_lds_fence();
  return ok;
}

template <int D, int OBS, bool FIRST>
__device__ __forceinline__ void wave_fold(const KModel& M, const FilterArgs& P, int item) {
  constexpr bool GH = (OBS == OBS_GH);
  extern __shared__ double lds[];
  double* scr = lds;
  double* vb = scr + wave_scr<D>();
  double* veta = vb + D;
  double* vmu = veta + D;
  double* vs = vmu + D;
  double* vom = vs + D;
  const int l = threadIdx.x, d = M.d;
  const int s0 = item * P.B, s1 = min(M.N, s0 + P.B);
  const int dobs = GH ? P.dyo : d;
  RM<D> FT, HT, A, Cc, J;
  if (!P.Ft) rm_load_t<D>(FT, M.F, d, d, d);
  if constexpr (GH) rm_load_t<D>(HT, P.Ho, d, d, P.dyo);
  rm_zero<D>(Cc);
  rm_zero<D>(J);
  rm_zero<D>(A);
  if (l < D) vb[l] = veta[l] = 0.0;
  wave_lds_fence();
  LogDet ld;
  double q_part = 0.0;
  bool ok = true;
  // this step's omega_t and Omega_t, fetched one step ahead
  const bool in = l < d;
  double om_n = 0.0, Om_n = 0.0;
  if (OBS != OBS_GH && in) {
    om_n = P.om[(int64_t)s0 * d + l];
    if (OBS == OBS_DIAG || !P.Omd) Om_n = P.Om[(int64_t)s0 * d + l];
  }
  for (int t = s0; t < s1; ++t) {
    const double om = om_n, Om = Om_n;
    if (OBS != OBS_GH && in && t + 1 < s1) {
      om_n = P.om[(int64_t)(t + 1) * d + l];
      if (OBS == OBS_DIAG || !P.Omd) Om_n = P.Om[(int64_t)(t + 1) * d + l];
    }
    RM<D> Pp, T;
    double mu = 0.0;
    if (t == 0) {
      rm_load<D>(Pp, M.P0, d, d);
      mu = in ? M.m0[l] : 0.0;
    } else {
      rm_load<D>(Pp, M.Q, d, d);
      const double* F = P.Ft ? P.Ft + (int64_t)t * d * d : M.F;
      const double* bt = P.Ft ? P.bt + (int64_t)t * d : M.b;
      mu = (in && bt) ? bt[l] : 0.0;
      if (!FIRST && t == s0) {  // A = I, C = 0, b = 0
        rm_load<D>(T, F, d, d);
      } else {
        if (P.Ft) rm_load_t<D>(FT, F, d, d, d);
        const RM<D> V = tn0<D>(Cc, FT);  // C F'
        if constexpr (!FIRST) T = tn0<D>(FT, A);
        tn<D, true>(Pp, FT, V);  // Q + F C F'
        mirror<D>(Pp, scr);
        mu += mv<D>(FT, rv<D>(vb));
      }
    }
    if constexpr (GH) {
      vec_put<D>(vmu, mu);
      if (D == 16 || P.dyo <= 16)
        ok = wave_update_gh<D, 1, FIRST>(P, t, HT, Pp, T, A, Cc, J, vb, veta, vmu, vs, scr, ld,
                                         q_part) && ok;
      else
        ok = wave_update_gh<D, Cfg<D>::TS, FIRST>(P, t, HT, Pp, T, A, Cc, J, vb, veta, vmu, vs, scr,
                                                  ld, q_part) && ok;
      symm<D>(Cc, scr);
      continue;
    }
    const double w = in ? om - mu : 0.0;
    RM<D> S = Pp;
    const bool diag = OBS == OBS_DIAG || !P.Omd;
    vec_put<D>(vom, Om);
    vec_put<D>(vs, w);
    const RV<D> rom = rv<D>(vom);
    if (diag) {
      constexpr int TS = Cfg<D>::TS;
      AKF_RM_FOR(D, q, r, i, j) if (i == j) S.t[q][r] += rom.v[q / TS][r];
    } else {
      rm_add_load<D>(S, P.Omd, d, d);
    }
    ok = wave_inv<D>(S, d, scr, ld) && ok;  // S^{-1}
    const double si = mv<D>(S, rv<D>(vs));  // S^{-1} w
    q_part += l < D ? w * si : 0.0;
    vec_put<D>(vs, si);
    RM<D> R;
    if constexpr (OBS == OBS_DIAG) {
      // I - Pp S^{-1} = Omega S^{-1}: products only, nothing cancels
      Cc = tn0<D, true>(S, Pp);
      scale_rows<D>(Cc, rom);
      symm<D>(Cc, scr);
      if constexpr (!FIRST) {
        R = tn0<D>(S, T);
        tn<D, true>(J, T, R);
        A = R;
        scale_rows<D>(A, rom);
      }
      vec_put<D>(vb, in ? om - Om * si : 0.0);
    } else {
      R = tn0<D>(S, Pp);
      Cc = tn0<D, true>(Pp, R);
      rm_rsub<D>(Cc, Pp);
      symm<D>(Cc, scr);
      const double b = mv<D>(Pp, rv<D>(vs));
      if constexpr (!FIRST) {
        R = tn0<D>(S, T);
        tn<D, true>(J, T, R);
        A = tn0<D>(Pp, R);
        rm_rsub<D>(A, T);
      }
      vec_put<D>(vb, mu + b);
    }
    if constexpr (!FIRST) {
      const double e = mv<D>(T, rv<D>(vs));
      if (l < D) veta[l] += e;
      wave_lds_fence();
    }
  }
  if (!ok && l == 0) atomicOr(P.status, P.fail_bit);
  symm<D>(J, scr);
  using EL = ElemLayout<D>;
  double* out = P.elem + (int64_t)item * EL::SIZE;
  rm_store<D>(A, out + EL::A, D, D);
  rm_store<D>(Cc, out + EL::C, D, D);
  rm_store<D>(J, out + EL::J, D, D);
  if (l < D) {
    out[EL::b + l] = vb[l];
    out[EL::eta + l] = veta[l];
  }
  const double q = wave_total(q_part);
  if (l == 0)
    out[EL::lc] = -0.5 * ((s1 - s0) * dobs * 1.8378770664093454835606594728112 + ld.value() + q);
}

// ---------------------------------------------------------------------------
// Filter combine (the formulas above filter_combine); SIDE as there
// ---------------------------------------------------------------------------
// M = (I + C J)^{-1} C from L, L' (C = L L') and J; log det (I + C J) into ld
template <int D>
__device__ __forceinline__ bool wave_M(RM<D>& Mm, const RM<D>& L, const RM<D>& LT, const RM<D>& J,
                                       int d, double* scr, LogDet& ld) {
  const RM<D> R = tn0<D>(J, L);      // J L
  RM<D> Wm = tn0<D, true>(L, R);     // L' J L
  add_eye<D>(Wm, d);
  const bool ok = wave_inv<D>(Wm, d, scr, ld);
  const RM<D> K = tn0<D>(Wm, LT);  // W^{-1} L'
  Mm = tn0<D, true>(LT, K);        // L W^{-1} L'
  mirror<D>(Mm, scr);
  return ok;
}

template <int D, int SIDE>
__device__ __forceinline__ void wave_combine(const KModel& M, const double* __restrict__ ei,
                                             const double* __restrict__ ej,
                                             double* __restrict__ out, int* status, int fail_bit) {
  using EL = ElemLayout<D>;
  extern __shared__ double lds[];
  double* scr = lds;
  double* va = scr + wave_scr<D>();
  const int l = threadIdx.x, d = M.d;
  const bool in = l < D;
  RM<D> Ci, Jj, Ai, Ji, AjT, Cj;
  rm_load<D>(Ci, ei + EL::C, D, D);
  rm_load<D>(Jj, ej + EL::J, D, D);
  const double bi = in ? ei[EL::b + l] : 0.0, etaj = in ? ej[EL::eta + l] : 0.0;
  // needed after the factorisations
  if constexpr (SIDE != 2) {
    rm_load<D>(Ai, ei + EL::A, D, D);
    rm_load<D>(Ji, ei + EL::J, D, D);
  }
  rm_load_t<D>(AjT, ej + EL::A, D, D, D);
  if constexpr (SIDE != 1) rm_load<D>(Cj, ej + EL::C, D, D);
  RM<D> L, LT, Mm;
  LogDet ld;
  bool ok = wave_chol<D>(Ci, L, LT, d, scr);
  ok = wave_M<D>(Mm, L, LT, Jj, d, scr, ld) && ok;
  vec_put<D>(va, bi);
  const double c = etaj - mv<D>(Jj, rv<D>(va));  // c = eta_j - J_j b_i
  vec_put<D>(va + D, c);
  const double w = mv<D>(Mm, rv<D>(va + D));  // M c
  vec_put<D>(va + 2 * D, w);
  if constexpr (SIDE != 2) {
    const double k = c - mv<D>(Jj, rv<D>(va + 2 * D));  // c - J_j M c
    vec_put<D>(va, k);
    const RM<D> Pm = tn0<D>(Jj, Ai);  // P = J_j A_i
    RM<D> Z = tn0<D>(Mm, Pm);
    rm_rsub<D>(Z, Ai);  // Z = A_i - M P
    const double e = mv<D>(Ai, rv<D>(va));
    if (in) out[EL::eta + l] = ei[EL::eta + l] + e;
    tn<D, true>(Ji, Z, Pm);  // Z' P + J_i
    symm<D>(Ji, scr);
    rm_store<D>(Ji, out + EL::J, D, D);
    const RM<D> An = tn0<D>(AjT, Z);
    rm_store<D>(An, out + EL::A, D, D);
  }
  if constexpr (SIDE != 1) {
    const RM<D> V = tn0<D>(Mm, AjT);  // M A_j'
    tn<D, true>(Cj, AjT, V);          // A_j M A_j' + C_j
    vec_put<D>(va + 3 * D, w + bi);
    const double b = mv<D>(AjT, rv<D>(va + 3 * D));
    symm<D>(Cj, scr);
    rm_store<D>(Cj, out + EL::C, D, D);
    if (in) out[EL::b + l] = b + ej[EL::b + l];
    const double q = wave_total(in ? bi * (etaj + c) + c * w : 0.0);
    if (l == 0) out[EL::lc] = ei[EL::lc] + ej[EL::lc] - 0.5 * ld.value() + 0.5 * q;
  }
  if (!ok && l == 0) atomicOr(status, fail_bit);
}

// Moment pair (x) element (the formulas above moment_combine)
template <int D>
__device__ __forceinline__ void wave_moment(const KModel& M, const double* Pin, const double* min_,
                                            const double* el, double* Pout, double* mout,
                                            int* status, int fail_bit, const double* lcin,
                                            double* lcout) {
  using EL = ElemLayout<D>;
  extern __shared__ double lds[];
  double* scr = lds;
  double* va = scr + wave_scr<D>();
  const int l = threadIdx.x, d = M.d;
  const bool in = l < D;
  RM<D> Ci, Jj, AT, Ce;
  rm_load<D>(Ci, Pin, D, D);
  rm_load<D>(Jj, el + EL::J, D, D);
  rm_load_t<D>(AT, el + EL::A, D, D, D);
  rm_load<D>(Ce, el + EL::C, D, D);
  const double m = in ? min_[l] : 0.0, eta = in ? el[EL::eta + l] : 0.0;
  const double be = in ? el[EL::b + l] : 0.0;
  RM<D> L, LT, Mm;
  LogDet ld;
  bool ok = wave_chol<D>(Ci, L, LT, d, scr);
  ok = wave_M<D>(Mm, L, LT, Jj, d, scr, ld) && ok;
  vec_put<D>(va, m);
  const double c = eta - mv<D>(Jj, rv<D>(va));
  vec_put<D>(va + D, c);
  const double w = mv<D>(Mm, rv<D>(va + D));
  if (lcout) {
    const double q = wave_total(in ? m * (eta + c) + c * w : 0.0);
    if (l == 0) *lcout = *lcin + el[EL::lc] - 0.5 * ld.value() + 0.5 * q;
  }
  const RM<D> V = tn0<D>(Mm, AT);
  tn<D, true>(Ce, AT, V);
  vec_put<D>(va + 2 * D, w + m);
  const double z = mv<D>(AT, rv<D>(va + 2 * D));
  if (in) mout[l] = z + be;
  symm<D>(Ce, scr);
  rm_store<D>(Ce, Pout, D, D);
  if (!ok && l == 0) atomicOr(status, fail_bit);
}

// ---------------------------------------------------------------------------
// Filter, block re-scan (the recursion above filter_final_body)
// ---------------------------------------------------------------------------
template <int D, int KT>
__device__ __forceinline__ bool wave_final_gh(const FilterArgs& P, int t, const RM<D>& HT,
                                              const RM<D>& Pp, RM<D>& Pm, double* vm, double* vmp,
                                              double* vs, double* scr, LogDet& ld, double& q) {
  constexpr int TS = Cfg<D>::TS;
  const int l = threadIdx.x, m = P.dyo;
  const double y = l < m ? P.yo[(int64_t)t * m + l] : 0.0;
  const RM<D> Mo = tn0<D, false, TS, KT>(HT, Pp);
  RM<D> N;
#pragma unroll
  for (int ti = 0; ti < KT; ++ti)
#pragma unroll
    for (int tj = 0; tj < TS; ++tj)
      N.t[tj * TS + ti] = tile_t(Mo.t[ti * TS + tj], scr + (ti * TS + tj) * 16 * 17);
  RM<D> S;
  rm_load<D>(S, P.Ro, m, m);
  tn<D, true, TS, KT, KT>(S, N, HT);
  const double hm = mv<D>(HT, rv<D>(vmp));  // H m^p
  const double vw = l < m ? y - hm : 0.0;
  const bool ok = wave_inv<D, KT>(S, m, scr, ld);
  vec_put<D>(vs, vw);
  const double si = mv<D, KT>(S, rv<D>(vs));
  q = l < D ? vw * si : 0.0;
  vec_put<D>(vs, l < m ? si : 0.0);
  const RM<D> U = tn0<D, false, KT, KT>(S, Mo);
  Pm = tn0<D, true, KT>(Mo, U);
  rm_rsub<D>(Pm, Pp);
  const double b = mv<D, KT>(Mo, rv<D>(vs));
  vec_put<D>(vm, l < D ? vmp[l] + b : 0.0);
  return ok;
}

template <int D, int OBS>
__device__ __forceinline__ void wave_final(const KModel& M, const FilterArgs& P, int item) {
  constexpr bool GH = (OBS == OBS_GH);
  using EL = ElemLayout<D>;
  using PL = PrefLayout<D>;
  extern __shared__ double lds[];
  double* scr = lds;
  double* vm = scr + wave_scr<D>();
  double* vmp = vm + D;
  double* vs = vmp + D;
  double* vom = vs + D;
  const int l = threadIdx.x, d = M.d;
  const int s0 = item * P.B, s1 = min(M.N, s0 + P.B);
  const int dobs = GH ? P.dyo : d;
  const bool in = l < d;
  RM<D> FT, HT, Pm;
  if (!P.Ft) rm_load_t<D>(FT, M.F, d, d, d);
  if constexpr (GH) rm_load_t<D>(HT, P.Ho, d, d, P.dyo);
  if (s0 > 0) {
    const double* pin = P.pre_elem ? P.pre_elem + (int64_t)(item - 1) * EL::SIZE
                                   : P.pre + (int64_t)item * PL::SIZE;
    rm_load<D>(Pm, pin + (P.pre_elem ? (int)EL::C : (int)PL::P), D, D);
    vec_put<D>(vm, l < D ? pin[(P.pre_elem ? (int)EL::b : (int)PL::m) + l] : 0.0);
  }
  double om_n = 0.0, Om_n = 0.0;
  if (OBS != OBS_GH && in) {
    om_n = P.om[(int64_t)s0 * d + l];
    if (OBS == OBS_DIAG || !P.Omd) Om_n = P.Om[(int64_t)s0 * d + l];
  }
  bool ok = true;
  for (int t = s0; t < s1; ++t) {
    const double om = om_n, Om = Om_n;
    if (OBS != OBS_GH && in && t + 1 < s1) {
      om_n = P.om[(int64_t)(t + 1) * d + l];
      if (OBS == OBS_DIAG || !P.Omd) Om_n = P.Om[(int64_t)(t + 1) * d + l];
    }
    RM<D> Pp;
    double mp = 0.0;
    if (t == 0) {
      rm_load<D>(Pp, M.P0, d, d);
      mp = in ? M.m0[l] : 0.0;
    } else {
      rm_load<D>(Pp, M.Q, d, d);
      const double* bt = P.Ft ? P.bt + (int64_t)t * d : M.b;
      mp = (in && bt) ? bt[l] : 0.0;
      if (P.Ft) rm_load_t<D>(FT, P.Ft + (int64_t)t * d * d, d, d, d);
      const RM<D> V = tn0<D>(Pm, FT);
      tn<D, true>(Pp, FT, V);
      mirror<D>(Pp, scr);
      mp += mv<D>(FT, rv<D>(vm));
    }
    LogDet ld;
    double q;
    if constexpr (GH) {
      vec_put<D>(vmp, mp);
      if (D == 16 || P.dyo <= 16)
        ok = wave_final_gh<D, 1>(P, t, HT, Pp, Pm, vm, vmp, vs, scr, ld, q) && ok;
      else
        ok = wave_final_gh<D, Cfg<D>::TS>(P, t, HT, Pp, Pm, vm, vmp, vs, scr, ld, q) && ok;
    } else {
      const double w = in ? om - mp : 0.0;
      RM<D> S = Pp;
      vec_put<D>(vom, Om);
      vec_put<D>(vs, w);
      const RV<D> rom = rv<D>(vom);
      if (OBS == OBS_DIAG || !P.Omd) {
        constexpr int TS = Cfg<D>::TS;
        AKF_RM_FOR(D, qq, r, i, j) if (i == j) S.t[qq][r] += rom.v[qq / TS][r];
      } else {
        rm_add_load<D>(S, P.Omd, d, d);
      }
      ok = wave_inv<D>(S, d, scr, ld) && ok;
      const double si = mv<D>(S, rv<D>(vs));
      q = l < D ? w * si : 0.0;
      if constexpr (OBS == OBS_DIAG) {
        if (P.Sinv) {  // kept transposed; S^{-1} is symmetric
          rm_store<D>(S, P.Sinv + (int64_t)t * D * D, D, D);
          if (l == 0) P.ldS[t] = ld.value();
        }
        Pm = tn0<D, true>(S, Pp);
        scale_rows<D>(Pm, rom);
        vec_put<D>(vm, in ? om - Om * si : 0.0);
      } else {
        vec_put<D>(vs, si);
        const RM<D> R = tn0<D>(S, Pp);
        Pm = tn0<D, true>(Pp, R);
        rm_rsub<D>(Pm, Pp);
        const double b = mv<D>(Pp, rv<D>(vs));
        vec_put<D>(vm, mp + b);
      }
    }
    q = wave_total(q);
    if (l == 0) P.ell[t] = -0.5 * (dobs * 1.8378770664093454835606594728112 + ld.value() + q);
    symm<D>(Pm, scr);
    if (P.mf) {
      if (in) P.mf[(int64_t)t * P.ldm + l] = vm[l];
      rm_store<D>(Pm, P.Pf + (int64_t)t * P.ldm * P.ldm, P.ldm, d);
    }
  }
  if (!ok && l == 0) atomicOr(P.status, P.fail_bit);
}

// ---------------------------------------------------------------------------
// Sampler, element build (the formulas above samp_build_body)
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void wave_sbuild(const KModel& M, const SampArgs& S, int t) {
  extern __shared__ double lds[];
  double* scr = lds;
  double* va = scr + wave_scr<D>();
  double* vxi = va + D;
  const int l = threadIdx.x, d = M.d;
  const bool in = l < d;
  RM<D> Pf, L, LT;
  rm_load<D>(Pf, S.Pf + (int64_t)t * S.ldm * S.ldm, S.ldm, d);
  const double m = in ? S.mf[(int64_t)t * S.ldm + l] : 0.0;
  vec_put<D>(va, m);
  vec_put<D>(vxi, in ? S.xi_x[(int64_t)t * d + l] : 0.0);
  bool ok = true;
  double g = m;
  if (t == M.N - 1) {
    ok = wave_chol<D>(Pf, L, LT, d, scr);
    RM<D> Z;
    rm_zero<D>(Z);
    rm_store<D>(Z, S.E + (int64_t)t * D * D, D, D);
    if (S.Et) rm_store<D>(Z, S.Et + (int64_t)t * D * D, D, D);
  } else {
    // the transition into step t + 1
    RM<D> FT, Pp, X;
    rm_load_t<D>(FT, S.Ft ? S.Ft + (int64_t)(t + 1) * d * d : M.F, d, d, d);
    rm_load<D>(Pp, M.Q, d, d);
    const double* bt = S.Ft ? S.bt + (int64_t)(t + 1) * d : M.b;
    const double mp = ((in && bt) ? bt[l] : 0.0) + mv<D>(FT, rv<D>(va));
    RM<D> G;
    {
      const RM<D> GT = tn0<D>(Pf, FT);  // P^f F' = G'
      tn<D, true>(Pp, FT, GT);          // Q + F P^f F'
      mirror<D>(Pp, scr);
      G = rm_t<D>(GT, scr);
    }
    X = Pp;
    LogDet ld;
    ok = wave_inv<D>(X, d, scr, ld);
    {  // Newton-Schulz step X + X (I - P^p X): P^p inherits the conditioning of Q
      RM<D> R = tn0<D>(Pp, X);
      AKF_RM_FOR(D, q, r, i, j) R.t[q][r] = ((i == j && i < d) ? 1.0 : 0.0) - R.t[q][r];
      const RM<D> Xo = X;
      tn<D>(X, Xo, R);
    }
    const RM<D> ET = tn0<D>(X, G);  // E' = (P^p)^{-1} G
    {
      const RM<D> E = rm_t<D>(ET, scr);
      rm_store<D>(E, S.E + (int64_t)t * D * D, D, D);
    }
    if (S.Et) rm_store<D>(ET, S.Et + (int64_t)t * D * D, D, D);
    vec_put<D>(va, mp);
    g = m - mv<D>(ET, rv<D>(va));  // m^f - E m^p
    // L_t = P^f - E G, averaged with its transpose: where P^p is ill
    // conditioned one triangle alone is 3x further from the exact L_t
    RM<D> Lm = tn0<D>(G, ET);
    rm_rsub<D>(Lm, Pf);
    if constexpr (D == 32) Lm.t[1] = 0.5 * (Lm.t[1] + tile_t(Lm.t[2], scr));
    symm<D>(Lm, scr);
    ok = wave_chol<D>(Lm, L, LT, d, scr) && ok;
  }
  if (S.Lc) rm_store<D>(LT, S.Lc + (int64_t)t * D * D, D, D);  // chol(L_t), kept transposed
  const double u = g + mv<D>(LT, rv<D>(vxi));
  if (l < D) S.U[(int64_t)t * D + l] = u;
  if (!ok && l == 0) atomicOr(S.status, ST_FWD_NOT_PD);
}

// ---------------------------------------------------------------------------
// Sampler, element build at D = 64 by one wave (the formulas of wave_sbuild).
// A step's factorisations are serial chains that a team's waves repeat or wait
// for, and its products are bound by the matrix cores either way; one step to
// a wave, four to a CU, leaves the chains of four steps to overlap: 163k
// cycles for four steps, 112k of them on the matrix cores, against 170k for
// two by teams of four waves (573 -> 306 us at d = 64, N = 4096).  The 16
// tiles of a 64 x 64 matrix take 128 of the lone wave's 512 registers, so two
// matrices and a symmetric one are held at a time, and F, then G, lives in the
// wave's own LDS (leading dimension 65), read tile by tile transposed in the
// shadow of the products.
// ---------------------------------------------------------------------------
// n doubles read through a buffer resource: an index past them gives zero, so
// padding needs no branch (a select on a loaded value is turned into one, with
// a wait for each load)
struct ZeroPad {
  static constexpr int OUT = 1 << 26;  // n stays below it, and two of them in 32 bits of bytes
  __amdgpu_buffer_rsrc_t rs;
  __device__ __forceinline__ ZeroPad(const double* g, int n)
      : rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(g), 0, 8 * n, 0x00020000)) {}
  __device__ __forceinline__ double get(int i) const {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, 8 * i, 0, 0));
  }
};

struct W64 {
  static constexpr int LD = 65;
  dbl4 t[16];  // tile (ti, tj) at 4 ti + tj

  // doubles of LDS: a matrix, a padded tile, three vectors
  static constexpr int LDS = 64 * LD + 16 * 17 + 3 * 64;

  // the leading d x d entries of g (uniform), zero elsewhere
  __device__ __forceinline__ void load(const double* g, int ld, int d, bool up) {
    const int l = threadIdx.x, lg = l >> 4, lc = l & 15;
    const ZeroPad b(g, d * ld);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      if (up && (q >> 2) > (q & 3)) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * (q >> 2) + 4 * r + lg, j = 16 * (q & 3) + lc;
        t[q][r] = b.get((j < d ? j : ZeroPad::OUT) + (i < d ? i * ld : ZeroPad::OUT));
      }
    }
  }
  // all 64 x 64 entries
  __device__ __forceinline__ void store(double* __restrict__ g) const {
    const int l = threadIdx.x, lg = l >> 4, lc = l & 15;
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        g[(16 * (q >> 2) + 4 * r + lg) * 64 + 16 * (q & 3) + lc] = t[q][r];
  }
  __device__ __forceinline__ void store_t(double* __restrict__ g) const {
    const int l = threadIdx.x, lg = l >> 4, lc = l & 15;
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        g[(16 * (q & 3) + lc) * 64 + 16 * (q >> 2) + 4 * r + lg] = t[q][r];
  }
  __device__ __forceinline__ void mirror(double* tile) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = i + 1; j < 4; ++j) t[4 * j + i] = tile_t(t[4 * i + j], tile);
  }
};

// tile (k, j) of the transpose of the matrix in LDS
__device__ __forceinline__ dbl4 w64_get_t(const double* s, int k, int j) {
  const int l = threadIdx.x, lg = l >> 4, lc = l & 15;
  const double* p = s + (16 * j + lc) * W64::LD + 16 * k + lg;
  return dbl4{p[0], p[4], p[8], p[12]};
}

// lane 16 * tj + lc: (x' v)_j over the first tile rows of column tj (KT(tj) of
// them), v by row in LDS
template <typename F>
__device__ __forceinline__ double w64_mv(const F& tile, const double* v, bool up) {
  const int l = threadIdx.x, lg = l >> 4;
  double s[4];
#pragma unroll
  for (int tj = 0; tj < 4; ++tj) {
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (up && k > tj) continue;
      const dbl4 x = tile(k, tj);
      const double* vk = v + 16 * k + lg;
      a = fma(x[0], vk[0], a);
      b = fma(x[1], vk[4], b);
      a = fma(x[2], vk[8], a);
      b = fma(x[3], vk[12], b);
    }
    s[tj] = sum_groups(a + b);
  }
  const double lo = (l & 16) ? s[1] : s[0], hi = (l & 16) ? s[3] : s[2];
  return (l & 32) ? hi : lo;
}

// the leading, the off-diagonal and the trailing 32 x 32 block's tile (i, j)
#define AKF_W64_A(i, j) t[4 * (i) + (j)]
#define AKF_W64_B(i, j) t[4 * (i) + 2 + (j)]
#define AKF_W64_C(i, j) t[4 * (2 + (i)) + 2 + (j)]

// In-place inverse of a symmetric positive definite matrix (upper tiles read,
// all written) by 2 x 2 blocks of 32, as spd_inv.
__device__ __forceinline__ bool w64_inv(W64& A, int d, double* tile) {
  const dbl4 z = {0.0, 0.0, 0.0, 0.0};
  LogDet ld;
  RM<32> P, S, X, Z;
  P.t[0] = A.AKF_W64_A(0, 0);
  P.t[1] = A.AKF_W64_A(0, 1);
  P.t[3] = A.AKF_W64_A(1, 1);
  bool ok = wave_inv<32>(P, min(d, 32), tile, ld);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)  // X = P b
      X.t[2 * i + j] = tile_tn(P.t[2 + i], A.AKF_W64_B(1, j), tile_tn(P.t[i], A.AKF_W64_B(0, j), z));
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = i; j < 2; ++j)  // S = c - b' X
      S.t[2 * i + j] = A.AKF_W64_C(i, j) - tile_tn(A.AKF_W64_B(1, i), X.t[2 + j],
                                                   tile_tn(A.AKF_W64_B(0, i), X.t[j], z));
  ok = wave_inv<32>(S, d - 32, tile, ld) && ok;
  #pragma unroll
  for (int q = 0; q < 4; ++q) Z.t[2 * (q & 1) + (q >> 1)] = tile_t(X.t[q], tile);
  RM<32> W;  // S^{-1} X'
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      W.t[2 * i + j] = tile_tn(S.t[2 + i], Z.t[2 + j], tile_tn(S.t[i], Z.t[j], z));
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = i; j < 2; ++j)  // P + X S^{-1} X'
      P.t[2 * i + j] = tile_tn(Z.t[2 + i], W.t[2 + j], tile_tn(Z.t[i], W.t[j], P.t[2 * i + j]));
  A.AKF_W64_A(0, 0) = P.t[0];
  A.AKF_W64_A(0, 1) = P.t[1];
  A.AKF_W64_A(1, 0) = tile_t(P.t[1], tile);
  A.AKF_W64_A(1, 1) = P.t[3];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      A.t[4 * (2 + i) + j] = -W.t[2 * i + j];
      A.AKF_W64_B(j, i) = tile_t(-W.t[2 * i + j], tile);
      A.AKF_W64_C(i, j) = S.t[2 * i + j];
    }
  return ok;
}

// L' (upper tiles written) for L the lower Cholesky factor of a matrix (upper
// tiles read), in place, as chol_reg.
__device__ __forceinline__ bool w64_chol_t(W64& A, int d, double* tile) {
  const dbl4 z = {0.0, 0.0, 0.0, 0.0};
  Chol32 c, e;
  bool ok = chol32<true>(A.AKF_W64_A(0, 0), A.AKF_W64_A(0, 1), A.AKF_W64_A(1, 1), min(d, 32), tile, c);
  dbl4 X[4];
#pragma unroll
  for (int j = 0; j < 2; ++j) {  // L10' = m' b
    X[j] = tile_tn(c.g0, A.AKF_W64_B(0, j), z);
    X[2 + j] = tile_tn(c.g1, A.AKF_W64_B(1, j), tile_tn(c.k01, A.AKF_W64_B(0, j), z));
  }
  dbl4 S[3];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = i; j < 2; ++j)
      S[i + j] = A.AKF_W64_C(i, j) - tile_tn(X[2 + i], X[2 + j], tile_tn(X[i], X[j], z));
  ok = chol32<false>(S[0], S[1], S[2], d - 32, tile, e) && ok;
  A.AKF_W64_A(0, 0) = tile_t(c.l0, tile);
  A.AKF_W64_A(0, 1) = c.l10t;
  A.AKF_W64_A(1, 1) = tile_t(c.l1, tile);
#pragma unroll
  for (int q = 0; q < 4; ++q) A.AKF_W64_B(q >> 1, q & 1) = X[q];
  A.AKF_W64_C(0, 0) = tile_t(e.l0, tile);
  A.AKF_W64_C(0, 1) = e.l10t;
  A.AKF_W64_C(1, 1) = tile_t(e.l1, tile);
  const int l = threadIdx.x, lg = l >> 4, lc = l & 15;
#pragma unroll
  for (int q = 0; q < 16; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if ((q >> 2) > (q & 3) || 16 * (q >> 2) + 4 * r + lg > 16 * (q & 3) + lc ||
          16 * (q & 3) + lc >= d)
        A.t[q][r] = 0.0;
  return ok;
}

__device__ __forceinline__ void w64_sbuild(const KModel& M, const SampArgs& S, int t) {
  extern __shared__ double lds[];
  double* sm = lds;  // F, then G' (by rows, so that transposed tiles of it are G's)
  double* tile = sm + 64 * W64::LD;
  double* vm = tile + 16 * 17;
  double* vxi = vm + 64;
  double* vmp = vxi + 64;
  const int l = threadIdx.x, lg = l >> 4, lc = l & 15, d = M.d;
  const bool in = l < d;
  const dbl4 z = {0.0, 0.0, 0.0, 0.0};
  const double* Pfg = S.Pf + (int64_t)t * S.ldm * S.ldm;
  double* Eo = S.E + (int64_t)t * 64 * 64;
  const double m = in ? S.mf[(int64_t)t * S.ldm + l] : 0.0;
  vm[l] = m;
  vxi[l] = in ? S.xi_x[(int64_t)t * d + l] : 0.0;
  bool ok = true;
  double g = m;
  W64 L;
  if (t == M.N - 1) {
    W64 Z;
#pragma unroll
    for (int q = 0; q < 16; ++q) Z.t[q] = z;
    Z.store(Eo);
    if (S.Et) Z.store(S.Et + (int64_t)t * 64 * 64);
    L.load(Pfg, S.ldm, d, true);
  } else {
    // the transition into step t + 1
    const double* F = S.Ft ? S.Ft + (int64_t)(t + 1) * d * d : M.F;
    const double* bt = S.Ft ? S.bt + (int64_t)(t + 1) * d : M.b;
    W64 X, Y;
    X.load(Pfg, S.ldm, d, false);
    const ZeroPad fb(F, d * d);
    const int lo = in ? l : ZeroPad::OUT;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      double v[32];
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = fb.get((32 * h + i) * d + lo);  // rows past d: past the end
#pragma unroll
      for (int i = 0; i < 32; ++i) sm[(32 * h + i) * W64::LD + l] = v[i];
    }
    const double bl = (in && bt) ? bt[l] : 0.0;
    wave_lds_fence();
    W64 Pp;
    Pp.load(M.Q, d, d, true);
#pragma unroll
    for (int q = 0; q < 16; ++q) Y.t[q] = z;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const dbl4 f = w64_get_t(sm, k, j);
#pragma unroll
        for (int i = 0; i < 4; ++i) Y.t[4 * i + j] = tile_tn(X.t[4 * k + i], f, Y.t[4 * i + j]);
      }  // Y = G' = P^f F'
    const double mp = bl + w64_mv([&](int k, int j) { return w64_get_t(sm, k, j); }, vm, false);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const dbl4 f = w64_get_t(sm, k, j);
#pragma unroll
        for (int i = 0; i <= j; ++i) Pp.t[4 * i + j] = tile_tn(Y.t[4 * k + i], f, Pp.t[4 * i + j]);
      }  // Q + F P^f F'
    vmp[l] = mp;
    wave_lds_fence();
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        sm[(16 * (q >> 2) + 4 * r + lg) * W64::LD + 16 * (q & 3) + lc] = Y.t[q][r];
    wave_lds_fence();
    X = Pp;
    ok = w64_inv(X, d, tile);
    Pp.mirror(tile);
    {  // Newton-Schulz step X + X (I - P^p X): P^p inherits the conditioning of Q
      W64 Xn;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        dbl4 R[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          dbl4 c = z;
#pragma unroll
          for (int k = 0; k < 4; ++k) c = tile_tn(Pp.t[4 * k + i], X.t[4 * k + j], c);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            R[i][r] = ((i == j && 4 * r + lg == lc && 16 * j + lc < d) ? 1.0 : 0.0) - c[r];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          dbl4 c = X.t[4 * i + j];
#pragma unroll
          for (int k = 0; k < 4; ++k) c = tile_tn(X.t[4 * k + i], R[k], c);
          Xn.t[4 * i + j] = c;
        }
      }
      X = Xn;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) Y.t[q] = z;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const dbl4 f = w64_get_t(sm, k, j);
#pragma unroll
        for (int i = 0; i < 4; ++i) Y.t[4 * i + j] = tile_tn(X.t[4 * k + i], f, Y.t[4 * i + j]);
      }  // Y = E' = (P^p)^{-1} G
    L.load(Pfg, S.ldm, d, true);  // ahead of the stores, which it would wait for
    Y.store_t(Eo);
    if (S.Et) Y.store(S.Et + (int64_t)t * 64 * 64);
    g = m - w64_mv([&](int k, int j) { return Y.t[4 * k + j]; }, vmp, false);  // m^f - E m^p
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      dbl4 c[4] = {z, z, z, z};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const dbl4 f = w64_get_t(sm, k, i);
#pragma unroll
        for (int j = 0; j < 4; ++j) c[j] = tile_tn(f, Y.t[4 * k + j], c[j]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j >= i) L.t[4 * i + j] -= 0.5 * c[j];
        if (j <= i) L.t[4 * j + i] -= 0.5 * tile_t(c[j], tile);
      }
    }  // L_t = P^f - (E G + (E G)') / 2, as in wave_sbuild
  }
  ok = w64_chol_t(L, d, tile) && ok;
  if (S.Lc) L.store(S.Lc + (int64_t)t * 64 * 64);  // chol(L_t), kept transposed
  S.U[(int64_t)t * 64 + l] = g + w64_mv([&](int k, int j) { return L.t[4 * k + j]; }, vxi, true);
  if (!ok && l == 0) atomicOr(S.status, ST_FWD_NOT_PD);
}

// ---------------------------------------------------------------------------
// Sampler, scan over the block aggregates and final pass.  Only the path is
// wanted, so once every aggregate is a suffix product of its group the state
// entering a block is a short chain of matrix-vector products, formed by the
// block's own wave before its steps.  kPathRadix aggregates are scanned in one
// workgroup, a wave each, in log2 steps through LDS; a tree of pairs took one
// launch per level up and one down (16 launches of 2.3 - 3.4 us at 256 blocks
// of width 16).
// ---------------------------------------------------------------------------
// Eight at D = 32, where 16 waves on four SIMDs would wait for the matrix cores
// (125 blocks: 10.2 us for the scan against 21.7).  A level of at most kPathChain
// nodes is not scanned: the chain goes through its nodes.
template <int D>
constexpr int kPathRadix = D == 16 ? 16 : 8;
constexpr int kPathChain = 16;

template <int D>
constexpr size_t path_scan_lds_bytes() {
  return (size_t)kPathRadix<D> * (Cfg<D>::MAT + D) * sizeof(double);
}

// Node j of the level (an aggregate, str apart) becomes node j o ... o the
// last of its group of kPathRadix, in place.  The group's first node is then
// its total, the group's node one level up (str * kPathRadix).
template <int D>
__device__ __forceinline__ void path_scan(double* agg, int n, int64_t str, int group) {
  using SL = SampLayout<D>;
  extern __shared__ double lds[];
  constexpr int SLOT = Cfg<D>::MAT + D;
  const int l = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cnt = min(kPathRadix<D>, n - group * kPathRadix<D>);
  const bool on = w < cnt;
  double* my = lds + w * SLOT;
  double* el = agg + (int64_t)(group * kPathRadix<D> + w) * str * SL::SIZE;
  RM<D> ET;  // the node's E transposed: x' y of a right neighbour's E with it is (E E_r)'
  double u = 0.0;
  if (on) {
    RM<D> X;
    rm_load<D>(X, el + SL::E, D, D);
    u = el[SL::U + l % D];
    rm_stage<D>(X, my);
    if (l < D) my[Cfg<D>::MAT + l] = u;
    wave_lds_fence();
    AKF_RM_FOR(D, q, r, i, j) ET.t[q][r] = my[j * Cfg<D>::LD + i];
  }
#pragma unroll 1
  for (int s = 1; s < kPathRadix<D>; s <<= 1) {
    __syncthreads();
    const bool go = w + s < cnt;
    RM<D> c;
    double un = 0.0;
    if (go) {
      const double* nb = my + s * SLOT;
      RM<D> X;
      rm_unstage<D>(X, nb);
      un = u + mv<D>(ET, rv<D>(nb + Cfg<D>::MAT));
      c = tn0<D>(X, ET);
    }
    __syncthreads();
    if (go) {
      ET = c;
      u = un;
      rm_stage_t<D>(ET, my);
      if (l < D) my[Cfg<D>::MAT + l] = u;
    }
  }
  if (w + 1 < cnt) {  // the last node of a group is unchanged
    wave_lds_fence();
    RM<D> X;
    rm_unstage<D>(X, my);
    rm_store<D>(X, el + SL::E, D, D);
    if (l < D) el[SL::U + l] = u;
  }
}

// Row l % D of a D x D matrix in global memory, a part of its columns per lane
template <int D>
struct PathRow {
  double e[D * D / 64];
  double u;
};
template <int D>
__device__ __forceinline__ PathRow<D> path_row(const double* __restrict__ E,
                                               const double* __restrict__ U) {
  constexpr int JL = D * D / 64;
  const int l = threadIdx.x & 63;
  PathRow<D> o;
#pragma unroll
  for (int m = 0; m < JL; ++m) o.e[m] = E[(l % D) * D + (l / D) * JL + m];
  o.u = U[l % D];
  return o;
}
// E x + U for the lane's row; x by lane (l % D), exchanged through vx
template <int D>
__device__ __forceinline__ double path_apply(const PathRow<D>& R, double x, double* vx) {
  constexpr int JL = D * D / 64;
  const int l = threadIdx.x & 63;
  vec_put<D>(vx, x);
  double a = 0.0, b = 0.0;
#pragma unroll
  for (int m = 0; m < JL; m += 2) {
    a = fma(R.e[m], vx[(l / D) * JL + m], a);
    b = fma(R.e[m + 1], vx[(l / D) * JL + m + 1], b);
  }
  wave_lds_fence();
  a += b;
  return R.u + (D == 16 ? sum_groups(a) : sum_x32(a));
}

// x* just after block k, from the state `root` after the last block and the n
// scanned aggregates (path_scan on every level of more than kPathChain nodes)
template <int D>
__device__ __forceinline__ double path_entry(const double* agg, int n, const double* root, int k,
                                             double* vx) {
  using SL = SampLayout<D>;
  auto row = [&](int64_t j) {
    const double* el = agg + j * SL::SIZE;
    return path_row<D>(el + SL::E, el + SL::U);
  };
  int64_t str = 1;
  int top = n;
  while (top > kPathChain) {
    top = (top + kPathRadix<D> - 1) / kPathRadix<D>;
    str *= kPathRadix<D>;
  }
  double x = root[threadIdx.x % D];
  const int jt = (int)(k / str);
  if (top - 1 > jt) {
    PathRow<D> nx = row((top - 1) * str);
    for (int j = top - 1; j > jt; --j) {
      const PathRow<D> cur = nx;
      if (j - 1 > jt) nx = row((j - 1) * str);
      x = path_apply<D>(cur, x, vx);
    }
  }
  while (str > 1) {
    str /= kPathRadix<D>;
    const int64_t j = k / str + 1, nl = (n + str - 1) / str;
    if (j % kPathRadix<D> != 0 && j < nl) x = path_apply<D>(row(j * str), x, vx);
  }
  return x;
}

// x*_t = E_t x*_{t+1} + U_t inside block `item`, x = x* just after it
template <int D>
__device__ __forceinline__ void wave_path(const KModel& M, const SampArgs& S, int item, double x,
                                          double* vx) {
  const int l = threadIdx.x & 63, d = M.d;
  const int s0 = item * S.B, s1 = min(M.N, s0 + S.B);
  auto row = [&](int t) {
    return path_row<D>(S.E + (int64_t)t * D * D, S.U + (int64_t)t * D);
  };
  PathRow<D> nx = row(s1 - 1);
  for (int t = s1 - 1; t >= s0; --t) {
    const PathRow<D> cur = nx;
    if (t > s0) nx = row(t - 1);
    x = path_apply<D>(cur, x, vx);
    if (l < d) S.xs[(int64_t)t * d + l] = x;
  }
}

}  // namespace akf
