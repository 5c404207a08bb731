// akf_adjoint.hip -- (E, g, L) suffix scans, the RTS smoother, and the
// reverse-mode adjoint of the Kalman log marginal likelihood.
//
// (E, g, L) scan (eq. EgL_comb): elements e_t = (E_t, g_t, L_t) with the
// operator (earlier i, later j)  (E_i E_j, E_i g_j + g_i, E_i L_j E_i' + L_i).
// The suffix scan e_t o ... o e_{N-1} with a terminal element of E = 0 yields,
// for the RTS smoother elements, the smoothing moments (m^s_t, P^s_t).  Blocked
// like the other scans: fold per block (backwards), tree over block
// aggregates (up: combine; down: propagate the suffix state (g, L) entering
// each node from the right), final per block.
//
// Adjoint.  For the LGSSM x_t = F x_{t-1} + N(0, Q), y_t = H x_t + N(0, R)
// (App. A, eq. lgssm-app) the log-likelihood L = sum_t ell_t of the Kalman
// filter (Alg. "Kalman filter", predictive form) has the reverse-mode adjoint
//   mbar_t = Phi_t' mbar_{t+1} + H' w_t,
//   Pbar_t = Phi_t' Pbar_{t+1} Phi_t + G_t,
//   G_t    = -1/2 H'(S^{-1} - w w')H + sym((mbar_t - H'w_t)(H'w_t)'),
// where mbar_t = dL/dm^p_t, Pbar_t = dL/dP^p_t (symmetric), Phi_t = F (I - K_t H),
// S_t = H P^p_t H' + R, K_t = P^p_t H' S_t^{-1}, w_t = S_t^{-1}(y_t - H m^p_t).
// Both are suffix scans: mbar with path elements (E, U) = (Phi', H'w) and
// Pbar with (E, L) = (Phi', G).  Parameter gradients are sums of local terms:
//   dL/dF = sum_{t<N-1} [mbar_{t+1} m^f_t' + 2 Pbar_{t+1} F P^f_t]
//   dL/dQ = sum_{t>=1} Pbar_t
//   dL/dH = sum_t [w m^p' - Sig H P^p + w (P^f fbar)' - (K' fbar) m^f' - 2 K' Fbar P^f]
//   dL/dR = sum_t [-Sig/2 - sym(K' fbar w') + K' Fbar K]
// with Sig = S^{-1} - w w', fbar = F' mbar_{t+1}, Fbar = F' Pbar_{t+1} F (zero at
// t = N-1).  The forward filtering moments (m^f, P^f) are the checkpoint; every
// other per-step quantity is recomputed from them.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "akf_team.hpp"
#include "akf_internal.h"
#include "akf_wave.hpp"

namespace akf {

__device__ __forceinline__ void flag_status2(int* st, int bit) { atomicOr(st, bit); }

template <int D>
__device__ __forceinline__ void lds_load_pad2(double* s, const double* __restrict__ g) {
  lds_fill<D>(s, [=](int i, int j) { return g[i * D + j]; });
}

template <int D>
__device__ __forceinline__ void lds_load_user(double* s, const double* __restrict__ g, int rows,
                                              int cols) {
  lds_fill<D>(s, [=](int i, int j) { return (i < rows && j < cols) ? g[i * cols + j] : 0.0; });
}

template <int D>
__device__ __forceinline__ void rm_store_t(const RM<D>& a, double* __restrict__ g, int ld, int d) {
  AKF_RM_FOR(D, q, r, i, j) if (i < d && j < d) g[(size_t)j * ld + i] = a.t[q][r];
}

// ---------------------------------------------------------------------------
// (E, g, L) scan
// ---------------------------------------------------------------------------
template <int D>
struct EglLayout {
  static constexpr int E = 0, L = D * D, g = 2 * D * D;
  static constexpr int SIZE = 2 * D * D + D;
};
template <int D>
struct EglState {  // suffix state entering a node from the right
  static constexpr int L = 0, g = D * D;
  static constexpr int SIZE = D * D + D;
};

// One-wave bodies (D <= 32, akf_wave.hpp).  With E' in registers (one transpose
// a step), E L E' = (E')' (L E') and E E~ = (E')' E~ need no staging.
//
// L_t of the scan: the stored matrix, plus sym((mb_t - h_t) h_t') when mb is
// given (the adjoint's G_t from its Cm_t, added as it is read instead of in a
// pass of its own over N D^2 entries).
template <int D>
__device__ __forceinline__ void egl_load_L(RM<D>& L, const EglArgs& A, int t) {
  rm_load<D>(L, A.L + (int64_t)t * D * D, D, D);
  if (A.mb) {
    constexpr int TS = Cfg<D>::TS;
    const double* h = A.h + (int64_t)t * D;
    const double* mb = A.mb + (int64_t)t * D;
    const RV<D> hr = rv<D>(h), mr = rv<D>(mb);
    const int lc = threadIdx.x & 15;
#pragma unroll
    for (int tj = 0; tj < TS; ++tj) {
      const double hc = h[16 * tj + lc], ac = mb[16 * tj + lc] - hc;
#pragma unroll
      for (int ti = 0; ti < TS; ++ti)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          L.t[ti * TS + tj][r] += 0.5 * ((mr.v[ti][r] - hr.v[ti][r]) * hc + ac * hr.v[ti][r]);
    }
  }
}

// L <- E L E' + Ln (upper tiles, mirrored; Ln is consumed)
template <int D>
__device__ __forceinline__ void egl_cov(RM<D>& L, const RM<D>& ET, RM<D>& Ln, double* scr) {
  const RM<D> W = tn0<D>(L, ET);  // L E'
  tn<D, true>(Ln, ET, W);
  symm<D>(Ln, scr);
  L = Ln;
}

template <int D>
__device__ __forceinline__ void wave_egl_fold(const EglArgs& A) {
  using EL = EglLayout<D>;
  extern __shared__ double lds[];
  double* scr = lds;
  double* vg = scr + wave_scr<D>();
  const int blk = blockIdx.x, l = threadIdx.x;
  const int s0 = blk * A.B, s1 = min(A.N, s0 + A.B);
  RM<D> Et, Lt, En, Ln;
  rm_load<D>(Et, A.E + (int64_t)(s1 - 1) * D * D, D, D);
  egl_load_L<D>(Lt, A, s1 - 1);
  double g = (l < D && A.g) ? A.g[(int64_t)(s1 - 1) * D + l] : 0.0, gn = 0.0;
  auto fetch = [&](int t) {  // a step ahead of its use
    rm_load<D>(En, A.E + (int64_t)t * D * D, D, D);
    egl_load_L<D>(Ln, A, t);
    gn = (l < D && A.g) ? A.g[(int64_t)t * D + l] : 0.0;
  };
  if (s1 - 2 >= s0) fetch(s1 - 2);
  for (int t = s1 - 2; t >= s0; --t) {
    const RM<D> ET = rm_t<D>(En, scr);
    RM<D> Lc = Ln;
    const double gc = gn;
    if (t > s0) fetch(t - 1);
    Et = tn0<D>(ET, Et);  // E_t E~
    egl_cov<D>(Lt, ET, Lc, scr);
    if (A.g) {
      vec_put<D>(vg, g);
      g = gc + mv<D>(ET, rv<D>(vg));
    }
  }
  double* out = A.agg + (int64_t)blk * EL::SIZE;
  rm_store<D>(Et, out + EL::E, D, D);
  rm_store<D>(Lt, out + EL::L, D, D);
  if (l < D) out[EL::g + l] = g;
}

template <int D>
__device__ __forceinline__ void wave_egl_up(const EglTree& T) {
  using EL = EglLayout<D>;
  extern __shared__ double lds[];
  double* scr = lds;
  double* vg = scr + wave_scr<D>();
  const int k = blockIdx.x, l = threadIdx.x;
  const double* el = T.src + (int64_t)(2 * k) * EL::SIZE;
  double* out = T.dst + (int64_t)k * EL::SIZE;
  if (2 * k + 1 >= T.n_src) {
    team_copy<64>(out, el, EL::SIZE);
    return;
  }
  const double* er = el + EL::SIZE;
  RM<D> X, Er, Lr, Ll;
  rm_load<D>(X, el + EL::E, D, D);
  rm_load<D>(Er, er + EL::E, D, D);
  rm_load<D>(Lr, er + EL::L, D, D);
  rm_load<D>(Ll, el + EL::L, D, D);
  vec_put<D>(vg, l < D ? er[EL::g + l] : 0.0);
  const double gl = l < D ? el[EL::g + l] : 0.0;
  const RM<D> ET = rm_t<D>(X, scr);
  const RM<D> E = tn0<D>(ET, Er);
  rm_store<D>(E, out + EL::E, D, D);
  const double g = gl + mv<D>(ET, rv<D>(vg));
  if (l < D) out[EL::g + l] = g;
  egl_cov<D>(Lr, ET, Ll, scr);
  rm_store<D>(Lr, out + EL::L, D, D);
}

template <int D>
__device__ __forceinline__ void wave_egl_down(const EglTree& T) {
  using EL = EglLayout<D>;
  using ES = EglState<D>;
  extern __shared__ double lds[];
  double* scr = lds;
  double* vg = scr + wave_scr<D>();
  const int k = blockIdx.x, l = threadIdx.x;
  const double* sin = T.pre_src + (int64_t)k * ES::SIZE;
  double* sl = T.pre_dst + (int64_t)(2 * k) * ES::SIZE;
  RM<D> Ls;
  rm_load<D>(Ls, sin + ES::L, D, D);
  const double gs = l < D ? sin[ES::g + l] : 0.0;
  double* inherits = (2 * k + 1 < T.n_dst) ? sl + ES::SIZE : sl;  // the rightmost child
  rm_store<D>(Ls, inherits + ES::L, D, D);
  if (l < D) inherits[ES::g + l] = gs;
  if (inherits == sl) return;
  const double* er = T.src + (int64_t)(2 * k + 1) * EL::SIZE;
  RM<D> X, Lr;
  rm_load<D>(X, er + EL::E, D, D);
  rm_load<D>(Lr, er + EL::L, D, D);
  const double gr = l < D ? er[EL::g + l] : 0.0;
  const RM<D> ET = rm_t<D>(X, scr);
  vec_put<D>(vg, gs);
  const double g = gr + mv<D>(ET, rv<D>(vg));
  if (l < D) sl[ES::g + l] = g;
  egl_cov<D>(Ls, ET, Lr, scr);
  rm_store<D>(Ls, sl + ES::L, D, D);
}

template <int D>
__device__ __forceinline__ void wave_egl_final(const EglArgs& A) {
  using ES = EglState<D>;
  extern __shared__ double lds[];
  double* scr = lds;
  double* vg = scr + wave_scr<D>();
  const int blk = blockIdx.x, l = threadIdx.x;
  const int s0 = blk * A.B, s1 = min(A.N, s0 + A.B);
  const double* sin = A.state + (int64_t)blk * ES::SIZE;
  RM<D> Lm, En, Ln;
  rm_load<D>(Lm, sin + ES::L, D, D);
  double g = l < D ? sin[ES::g + l] : 0.0, gn = 0.0;
  auto fetch = [&](int t) {
    rm_load<D>(En, A.E + (int64_t)t * D * D, D, D);
    egl_load_L<D>(Ln, A, t);
    gn = (l < D && A.g) ? A.g[(int64_t)t * D + l] : 0.0;
  };
  fetch(s1 - 1);
  for (int t = s1 - 1; t >= s0; --t) {
    const RM<D> ET = rm_t<D>(En, scr);
    RM<D> Lc = Ln;
    const double gc = gn;
    if (t > s0) fetch(t - 1);
    egl_cov<D>(Lm, ET, Lc, scr);
    rm_store<D>(Lm, A.outL + (int64_t)t * A.ldo * A.ldo, A.ldo, A.dout);
    if (A.outg) {
      vec_put<D>(vg, g);
      g = gc + mv<D>(ET, rv<D>(vg));
      if (l < A.dout) A.outg[(int64_t)t * A.ldo + l] = g;
    }
  }
}

// The team kernels' GEMMs are fully unrolled (U = D / 4).
//
// acc <- e_t o acc for t = s1-2 .. s0, starting from acc = e_{s1-1}.
template <int D>
__global__ void __launch_bounds__(Cfg<D>::NT) k_egl_fold(EglArgs A) {
  if constexpr (D <= 32) {
    wave_egl_fold<D>(A);
  } else {
    using C = Cfg<D>;
    using EL = EglLayout<D>;
    extern __shared__ double lds[];
    double* B1 = lds;
    double* B2 = B1 + C::MAT;
    double* B3 = B2 + C::MAT;
    double* vg = B3 + C::MAT;
    double* vn = vg + D;
    const int blk = blockIdx.x, tid = threadIdx.x;
    const int s0 = blk * A.B, s1 = min(A.N, s0 + A.B);
    RM<D> Et, Lt, T;
    rm_load<D>(Et, A.E + (int64_t)(s1 - 1) * D * D, D, D);
    rm_load<D>(Lt, A.L + (int64_t)(s1 - 1) * D * D, D, D);
    if (tid < D) vg[tid] = A.g ? A.g[(int64_t)(s1 - 1) * D + tid] : 0.0;
    for (int t = s1 - 2; t >= s0; --t) {
      lds_load_pad2<D>(B1, A.E + (int64_t)t * D * D);
      rm_stage<D>(Et, B2);
      rm_stage<D>(Lt, B3);
      team_sync();
      gemm<D, false, false, false, D / 4>(Et, B1, B2);  // E_t E~
      gemm<D, false, false, false, D / 4>(T, B1, B3);   // E_t L~
      matvec<D, false>(vn, B1, vg);
      team_sync();
      rm_stage<D>(T, B3);
      if (tid < D) vg[tid] = vn[tid] + (A.g ? A.g[(int64_t)t * D + tid] : 0.0);
      team_sync();
      gemm<D, false, true, false, D / 4>(Lt, B3, B1);  // (E_t L~) E_t'
      rm_add_load<D>(Lt, A.L + (int64_t)t * D * D, D, D);
      rm_symmetrise<D>(Lt, B2);
    }
    double* out = A.agg + (int64_t)blk * EL::SIZE;
    rm_store<D>(Et, out + EL::E, D, D);
    rm_store<D>(Lt, out + EL::L, D, D);
    if (tid < D) out[EL::g + tid] = vg[tid];
  }
}

template <int D>
__global__ void __launch_bounds__(Cfg<D>::NT) k_egl_up(EglTree T) {
  if constexpr (D <= 32) {
    wave_egl_up<D>(T);
  } else {
    using C = Cfg<D>;
    using EL = EglLayout<D>;
    extern __shared__ double lds[];
    double* B1 = lds;
    double* B2 = B1 + C::MAT;
    double* B3 = B2 + C::MAT;
    double* vg = B3 + C::MAT;
    double* vn = vg + D;
    const int k = blockIdx.x, tid = threadIdx.x;
    const double* el = T.src + (int64_t)(2 * k) * EL::SIZE;
    double* out = T.dst + (int64_t)k * EL::SIZE;
    if (2 * k + 1 >= T.n_src) {
      team_copy<C::NT>(out, el, EL::SIZE);
      return;
    }
    const double* er = el + EL::SIZE;
    lds_load_pad2<D>(B1, el + EL::E);
    lds_load_pad2<D>(B2, er + EL::E);
    lds_load_pad2<D>(B3, er + EL::L);
    if (tid < D) vg[tid] = er[EL::g + tid];
    team_sync();
    RM<D> R1, R2;
    gemm<D, false, false, false, D / 4>(R1, B1, B2);  // E_l E_r
    gemm<D, false, false, false, D / 4>(R2, B1, B3);  // E_l L_r
    matvec<D, false>(vn, B1, vg);
    rm_store<D>(R1, out + EL::E, D, D);
    team_sync();
    rm_stage<D>(R2, B3);
    if (tid < D) out[EL::g + tid] = vn[tid] + el[EL::g + tid];
    team_sync();
    gemm<D, false, true, false, D / 4>(R1, B3, B1);  // E_l L_r E_l'
    rm_add_load<D>(R1, el + EL::L, D, D);
    rm_symmetrise<D>(R1, B2);
    rm_store<D>(R1, out + EL::L, D, D);
  }
}

// State entering node k of level l (pre_src) -> its children at level l-1:
// right child inherits; left child gets e_right o state = (E_r g + g_r, E_r L E_r' + L_r).
template <int D>
__global__ void __launch_bounds__(Cfg<D>::NT) k_egl_down(EglTree T) {
  if constexpr (D <= 32) {
    wave_egl_down<D>(T);
  } else {
    using C = Cfg<D>;
    using EL = EglLayout<D>;
    using ES = EglState<D>;
    extern __shared__ double lds[];
    double* B1 = lds;
    double* B2 = B1 + C::MAT;
    double* vg = B2 + C::MAT;
    double* vn = vg + D;
    const int k = blockIdx.x, tid = threadIdx.x;
    const double* sin = T.pre_src + (int64_t)k * ES::SIZE;
    const bool has_right = (2 * k + 1 < T.n_dst);
    double* sl = T.pre_dst + (int64_t)(2 * k) * ES::SIZE;
    if (!has_right) {
      team_copy<C::NT>(sl, sin, ES::SIZE);
      return;
    }
    double* sr = T.pre_dst + (int64_t)(2 * k + 1) * ES::SIZE;
    team_copy<C::NT>(sr, sin, ES::SIZE);
    const double* er = T.src + (int64_t)(2 * k + 1) * EL::SIZE;
    lds_load_pad2<D>(B1, er + EL::E);
    lds_load_pad2<D>(B2, sin + ES::L);
    if (tid < D) vg[tid] = sin[ES::g + tid];
    team_sync();
    RM<D> R1;
    gemm<D, false, false, false, D / 4>(R1, B1, B2);  // E_r L
    matvec<D, false>(vn, B1, vg);
    team_sync();
    rm_stage<D>(R1, B2);
    if (tid < D) sl[ES::g + tid] = vn[tid] + er[EL::g + tid];
    team_sync();
    gemm<D, false, true, false, D / 4>(R1, B2, B1);  // E_r L E_r'
    rm_add_load<D>(R1, er + EL::L, D, D);
    rm_symmetrise<D>(R1, B2);
    rm_store<D>(R1, sl + ES::L, D, D);
  }
}

// Final: state = incoming; for t = s1-1 .. s0: state = e_t o state; write it.
template <int D>
__global__ void __launch_bounds__(Cfg<D>::NT) k_egl_final(EglArgs A) {
  if constexpr (D <= 32) {
    wave_egl_final<D>(A);
  } else {
    using C = Cfg<D>;
    using ES = EglState<D>;
    extern __shared__ double lds[];
    double* B1 = lds;
    double* B2 = B1 + C::MAT;
    double* vg = B2 + C::MAT;
    double* vn = vg + D;
    const int blk = blockIdx.x, tid = threadIdx.x;
    const int s0 = blk * A.B, s1 = min(A.N, s0 + A.B);
    const double* sin = A.state + (int64_t)blk * ES::SIZE;
    RM<D> Lm, T;
    rm_load<D>(Lm, sin + ES::L, D, D);
    if (tid < D) vg[tid] = sin[ES::g + tid];
    for (int t = s1 - 1; t >= s0; --t) {
      lds_load_pad2<D>(B1, A.E + (int64_t)t * D * D);
      rm_stage<D>(Lm, B2);
      team_sync();
      gemm<D, false, false, false, D / 4>(T, B1, B2);
      matvec<D, false>(vn, B1, vg);
      team_sync();
      rm_stage<D>(T, B2);
      if (tid < D) vg[tid] = vn[tid] + (A.g ? A.g[(int64_t)t * D + tid] : 0.0);
      team_sync();
      gemm<D, false, true, false, D / 4>(Lm, B2, B1);
      rm_add_load<D>(Lm, A.L + (int64_t)t * D * D, D, D);
      rm_symmetrise<D>(Lm, B2);
      rm_store<D>(Lm, A.outL + (int64_t)t * A.ldo * A.ldo, A.ldo, A.dout);
      if (A.outg && tid < A.dout) A.outg[(int64_t)t * A.ldo + tid] = vg[tid];
    }
  }
}

// ---------------------------------------------------------------------------
// RTS smoother elements (eq. init-dnc): E_t = P^f_t F' (P^p_{t+1})^{-1},
// g_t = m^f_t - E_t (F m^f_t + b), L_t = P^f_t - E_t F P^f_t; terminal (0, m^f, P^f).
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(Cfg<D>::NT) k_smooth_build(KModel M, SmoothArgs S) {
  using C = Cfg<D>;
  extern __shared__ double lds[];
  double* sF = lds;
  double* B1 = sF + C::MAT;
  double* B2 = B1 + C::MAT;
  double* B3 = B2 + C::MAT;
  double* vm = B3 + C::MAT;
  double* vmp = vm + D;
  double* vg = vmp + D;
  const int t = blockIdx.x, tid = threadIdx.x, d = M.d;
  RM<D> Pf, R1, R2;
  rm_load<D>(Pf, S.Pf + (int64_t)t * S.ldm * S.ldm, S.ldm, d);
  if (tid < D) vm[tid] = (tid < d) ? S.mf[(int64_t)t * S.ldm + tid] : 0.0;
  if (t == M.N - 1) {
    rm_zero<D>(R1);
    rm_store<D>(R1, S.E + (int64_t)t * D * D, D, D);
    rm_store<D>(Pf, S.L + (int64_t)t * D * D, D, D);
    if (tid < D) S.g[(int64_t)t * D + tid] = vm[tid];
    return;
  }
  bool ok = true;
  double ld;
  rm_load<D>(R2, M.Q, d, d);  // issued early: its latency overlaps G = F P^f
  lds_load_user<D>(sF, M.F, d, d);
  rm_stage<D>(Pf, B1);
  team_sync();
  gemm<D, false, false, false, D / 4>(R1, sF, B1);  // G = F P^f
  team_sync();
  rm_stage<D>(R1, B1);
  team_sync();
  gemm<D, false, true, true, D / 4>(R2, B1, sF);  // Q + G F'
  matvec<D, false>(vmp, sF, vm);
  if (tid < d && M.b) vmp[tid] += M.b[tid];
  {
    const RM<D> Pp = R2;
    ok = spd_inv<D>(R2, d, B3, &ld) && ok;  // (P^p)^{-1}
    inv_refine<D>(R2, Pp, d, B2, B3);       // P^p inherits the conditioning of Q
  }
  rm_stage<D>(R2, B2);
  team_sync();
  gemm<D, true, false, false, D / 4>(R1, B1, B2);  // E = G' (P^p)^{-1}
  rm_store<D>(R1, S.E + (int64_t)t * D * D, D, D);
  rm_stage<D>(R1, B3);
  team_sync();
  gemm<D, false, false, false, D / 4>(R2, B3, B1);  // E G
  rm_rsub<D>(R2, Pf);                        // L = P^f - E G
  matvec<D, false>(vg, B3, vmp);
  if (tid < D) S.g[(int64_t)t * D + tid] = vm[tid] - vg[tid];
  rm_symmetrise<D>(R2, B2);
  rm_store<D>(R2, S.L + (int64_t)t * D * D, D, D);
  if (!ok && tid == 0) flag_status2(S.status, ST_FWD_NOT_PD);
}

// ---------------------------------------------------------------------------
// LGSSM helpers
// ---------------------------------------------------------------------------
// Q = diag(exp(logq)), R = diag(exp(logr)) (dense, user dims)
__global__ void k_lgssm_prep(LgArgs G) {
  const int tid = threadIdx.x + blockIdx.x * blockDim.x;
  const int nq = G.dx * G.dx, nr = G.dy * G.dy;
  if (tid < nq) {
    const int i = tid / G.dx, j = tid % G.dx;
    G.Q[tid] = (i == j) ? exp(G.logq[i]) : 0.0;
  } else if (tid < nq + nr) {
    const int e = tid - nq, i = e / G.dy, j = e % G.dy;
    G.R[e] = (i == j) ? exp(G.logr[i]) : 0.0;
  }
}

// sum of ell (fixed-order tree within one team); NaN when the filter that
// wrote ell set a status bit (status may be null)
// (one workgroup of kSumThreads, four loads in flight per thread: with 256
// threads and one the 16384 terms of a long chain took 18 us)
constexpr int kSumThreads = 1024;
__global__ void __launch_bounds__(kSumThreads) k_sum(const double* __restrict__ a, int n, double* out,
                                                     const int* status) {
  __shared__ double red[kSumThreads / 64];
  double s4[4] = {0.0, 0.0, 0.0, 0.0};
  int i = threadIdx.x;
  for (; i + 3 * kSumThreads < n; i += 4 * kSumThreads) {
#pragma unroll
    for (int q = 0; q < 4; ++q) s4[q] += a[i + q * kSumThreads];
  }
  for (; i < n; i += kSumThreads) s4[0] += a[i];
  double s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int k = 0; k < kSumThreads / 64; ++k) t += red[k];
    *out = (status && *status != 0) ? __builtin_nan("") : t;
  }
}

// The filter quantities of step t, recomputed from the checkpoint by one wave
// (D <= 32, KT tile rows of observations): m^p and P^p from the moments of step
// t - 1 (mf1, Pf1; the prior at t = 0), Mo = H P^p, Si = S^{-1} (only its
// KT x KT tiles are set), w = S^{-1} v.  mp and w: value of lane l < D.
template <int D, int KT>
struct AdjStep {
  RM<D> Mo, Si;
  double mp, w;
};
template <int D, int KT>
__device__ __forceinline__ bool adj_step(AdjStep<D, KT>& q, const KModel& M, const LgArgs& G, int t,
                                         const RM<D>& FT, const RM<D>& HT, const RM<D>& Pf1,
                                         double mf1, double* scr, double* va) {
  constexpr int TS = Cfg<D>::TS;
  const int l = threadIdx.x, d = G.dx, p = G.dy;
  const double y = l < p ? G.y[(int64_t)t * p + l] : 0.0;
  RM<D> Pp, N;
  rm_load<D>(q.Si, G.R, p, p);
  if (t == 0) {
    rm_load<D>(Pp, M.P0, d, d);
    q.mp = l < d ? M.m0[l] : 0.0;
  } else {
    rm_load<D>(Pp, G.Q, d, d);
    const RM<D> V = tn0<D>(Pf1, FT);
    tn<D, true>(Pp, FT, V);
    mirror<D>(Pp, scr);
    vec_put<D>(va, mf1);
    q.mp = mv<D>(FT, rv<D>(va));
  }
  q.Mo = tn0<D, false, TS, KT>(HT, Pp);
#pragma unroll
  for (int ti = 0; ti < KT; ++ti)
#pragma unroll
    for (int tj = 0; tj < TS; ++tj)
      N.t[tj * TS + ti] = tile_t(q.Mo.t[ti * TS + tj], scr + (ti * TS + tj) * 16 * 17);
  tn<D, true, TS, KT, KT>(q.Si, N, HT);  // S = H P^p H' + R
  vec_put<D>(va, l < D ? q.mp : 0.0);
  const double hm = mv<D>(HT, rv<D>(va));
  LogDet ld;
  const bool ok = wave_inv<D, KT>(q.Si, p, scr, ld);
  vec_put<D>(va, l < p ? y - hm : 0.0);
  const double w = mv<D, KT>(q.Si, rv<D>(va));
  q.w = l < p ? w : 0.0;
  return ok;
}

// Adjoint elements of step t: E_t = Phi_t' (0 at t = N-1), U_t = h_t = H' w_t,
// Cm_t = -1/2 H' (S^{-1} - w w') H.  One wave per t, D <= 32:
// E = F' - H' (K' F') with K = Mo' S^{-1}.
template <int D, int KT>
__device__ __forceinline__ void adj_build_body(const KModel& M, const LgArgs& G) {
  constexpr int TS = Cfg<D>::TS;
  extern __shared__ double lds[];
  double* scr = lds;
  double* va = scr + wave_scr<D>();
  const int t = blockIdx.x, l = threadIdx.x, d = G.dx, p = G.dy;
  RM<D> FT, HT, Hm, Pf1;
  if (t > 0) rm_load<D>(Pf1, G.Pf + (int64_t)(t - 1) * D * D, D, D);
  const double mf1 = (t > 0 && l < D) ? G.mf[(int64_t)(t - 1) * D + l] : 0.0;
  rm_load_t<D>(FT, M.F, d, d, d);
  rm_load_t<D>(HT, G.H, d, d, p);
  rm_load_rect<D>(Hm, G.H, d, p, d);
  AdjStep<D, KT> q;
  const bool ok = adj_step<D, KT>(q, M, G, t, FT, HT, Pf1, mf1, scr, va);
  vec_put<D>(va, q.w);
  const RV<D> w = rv<D>(va);
  const double h = mv<D, KT>(Hm, w);
  if (l < D) G.U[(int64_t)t * D + l] = h;
  const RM<D> K = tn0<D, false, KT, TS, KT>(q.Mo, q.Si);  // (H P^p)' S^{-1}
  {
    RM<D> Sig = q.Si;
    const int lc = l & 15;
#pragma unroll
    for (int tj = 0; tj < KT; ++tj) {
      const double wc = va[16 * tj + lc];
#pragma unroll
      for (int ti = 0; ti < KT; ++ti)
#pragma unroll
        for (int r = 0; r < 4; ++r) Sig.t[ti * TS + tj][r] -= w.v[ti][r] * wc;
    }
    const RM<D> SH = tn0<D, false, KT, KT>(Sig, Hm);  // Sig H
    RM<D> Cm = tn0<D, true, KT>(Hm, SH);              // H' Sig H
#pragma unroll
    for (int k = 0; k < Cfg<D>::TPW; ++k) Cm.t[k] *= -0.5;
    mirror<D>(Cm, scr);
    rm_store<D>(Cm, G.Cm + (int64_t)t * D * D, D, D);
  }
  RM<D> E;
  if (t == M.N - 1) {
    rm_zero<D>(E);
  } else {
    const RM<D> KF = tn0<D, false, TS, KT>(K, FT);  // K' F'
    E = tn0<D, false, KT>(Hm, KF);                  // H' K' F'
    rm_rsub<D>(E, FT);
  }
  rm_store<D>(E, G.E + (int64_t)t * D * D, D, D);
  if (!ok && l == 0) flag_status2(G.status, ST_FWD_NOT_PD);
}

// Bound by its products' 64-cycle matrix instructions and the one pivot sweep;
// at d = 32, d_y = 16, T = 16384 the form with staged operands took 445 us.
template <int D, int KT>
__global__ void __launch_bounds__(64, 2) k_adj_build(KModel M, LgArgs G) {
  adj_build_body<D, KT>(M, G);
}

// Per-block accumulation of the parameter gradients (one wave per block of
// steps; partial sums [F (D*D) | H (D*D) | q (D) | r (D)] per block).  With
// Y = F' Pbar_{t+1}: Pbar F P^f = Y' P^f and Fbar = F' Y'; with Z = Fbar K:
// K' Fbar P^f = Z' P^f and diag(K' Fbar K) the column sums of Z o K.
template <int D, int KT>
__device__ __forceinline__ void adj_grad_body(const KModel& M, const LgArgs& G) {
  constexpr int TS = Cfg<D>::TS, TPW = Cfg<D>::TPW;
  extern __shared__ double lds[];
  double* scr = lds;
  double* va = scr + wave_scr<D>();
  double* vb = va + D;
  const int blk = blockIdx.x, l = threadIdx.x, lc = l & 15, d = G.dx, p = G.dy, N = M.N;
  const int s0 = blk * G.B, s1 = min(N, s0 + G.B);
  RM<D> FT, Fm, HT, Pf1, Pf, gF, gH, Sacc;
  dbl4 Pacc[TS];  // diagonal tiles of sum Pbar_{t+1}
  rm_load_t<D>(FT, M.F, d, d, d);
  rm_load<D>(Fm, M.F, d, d);
  rm_load_t<D>(HT, G.H, d, d, p);
  rm_zero<D>(gF);
  rm_zero<D>(gH);
  rm_zero<D>(Sacc);
#pragma unroll
  for (int k = 0; k < TS; ++k) Pacc[k] = dbl4{0.0, 0.0, 0.0, 0.0};
  double racc = 0.0, mf1 = 0.0;
  if (s0 > 0) {
    rm_load<D>(Pf1, G.Pf + (int64_t)(s0 - 1) * D * D, D, D);
    mf1 = l < D ? G.mf[(int64_t)(s0 - 1) * D + l] : 0.0;
  }
  bool ok = true;
  for (int t = s0; t < s1; ++t) {
    const bool last = (t == N - 1);
    RM<D> Pb;
    rm_load<D>(Pf, G.Pf + (int64_t)t * D * D, D, D);
    const double mf = l < D ? G.mf[(int64_t)t * D + l] : 0.0;
    double mb = 0.0;
    if (!last) {
      rm_load<D>(Pb, G.Pbar + (int64_t)(t + 1) * D * D, D, D);
      mb = l < D ? G.mbar[(int64_t)(t + 1) * D + l] : 0.0;
    }
    AdjStep<D, KT> q;
    ok = adj_step<D, KT>(q, M, G, t, FT, HT, Pf1, mf1, scr, va) && ok;
    const RM<D> K = tn0<D, false, KT, TS, KT>(q.Mo, q.Si);
    // fbar = F' mbar_{t+1}, K' fbar, P^f fbar, Mo' w
    vec_put<D>(va, mb);
    const RV<D> mbr = rv<D>(va);
    const double fb = mv<D>(Fm, mbr);
    vec_put<D>(vb, l < D ? fb : 0.0);
    const RV<D> fbr = rv<D>(vb);
    const double kf = mv<D>(K, fbr);
    const double vk = l < p ? kf : 0.0;
    const double pf = mv<D>(Pf, fbr);
    vec_put<D>(va, q.w);
    const RV<D> wr = rv<D>(va);
    const double mw = mv<D, KT>(q.Mo, wr);
    vec_put<D>(va, vk);
    const RV<D> vkr = rv<D>(va);
    // dL/dH: w (m^p + Mo' w + P^f fbar)' - (K' fbar) m^f' - S^{-1} Mo - 2 K' Fbar P^f
    vec_put<D>(va, l < D ? q.mp + mw + pf : 0.0);
    vec_put<D>(vb, mf);
#pragma unroll
    for (int tj = 0; tj < TS; ++tj) {
      const double c1 = va[16 * tj + lc], c2 = vb[16 * tj + lc];
#pragma unroll
      for (int ti = 0; ti < KT; ++ti)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          gH.t[ti * TS + tj][r] += wr.v[ti][r] * c1 - vkr.v[ti][r] * c2;
      // half of dL/dF: mbar m^f' / 2 + Pbar F P^f
#pragma unroll
      for (int ti = 0; ti < TS; ++ti)
#pragma unroll
        for (int r = 0; r < 4; ++r) gF.t[ti * TS + tj][r] += 0.5 * mbr.v[ti][r] * c2;
    }
    wave_lds_fence();
    {
      const RM<D> SM = tn0<D, false, KT, KT>(q.Si, q.Mo);
#pragma unroll
      for (int k = 0; k < KT * TS; ++k) gH.t[k] -= SM.t[k];
    }
    // dL/dR_jj: -1/2 (S^{-1}_jj - w_j^2) - (K' fbar)_j w_j + (K' Fbar K)_jj
#pragma unroll
    for (int k = 0; k < KT; ++k) Sacc.t[k * TS + k] += q.Si.t[k * TS + k];
    racc += 0.5 * q.w * q.w - vk * q.w;
    if (!last) {
#pragma unroll
      for (int k = 0; k < TS; ++k) Pacc[k] += Pb.t[k * TS + k];
      const RM<D> Y = tn0<D>(Fm, Pb);  // F' Pbar
      tn<D>(gF, Y, Pf);                // Pbar F P^f
      const RM<D> PF = rm_t<D>(Y, scr);
      RM<D> Fb = tn0<D, true>(Fm, PF);  // F' Pbar F
      mirror<D>(Fb, scr);
      const RM<D> Z = tn0<D, false, TS, TS, KT>(Fb, K);  // Fbar K
      const RM<D> ZP = tn0<D, false, TS, KT>(Z, Pf);     // K' Fbar P^f
#pragma unroll
      for (int k = 0; k < KT * TS; ++k) gH.t[k] -= 2.0 * ZP.t[k];
      double zk[TS];
#pragma unroll
      for (int tj = 0; tj < TS; ++tj) {
        zk[tj] = 0.0;
        if (tj < KT) {
#pragma unroll
          for (int ti = 0; ti < TS; ++ti)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              zk[tj] = fma(Z.t[ti * TS + tj][r], K.t[ti * TS + tj][r], zk[tj]);
          zk[tj] = sum_groups(zk[tj]);
        }
      }
      if constexpr (TS == 1) racc += zk[0];
      else racc += (l & 16) ? zk[1] : zk[0];
    }
    Pf1 = Pf;
    mf1 = mf;
  }
#pragma unroll
  for (int k = 0; k < TPW; ++k) gF.t[k] *= 2.0;
  double* out = G.part + (int64_t)blk * (2 * D * D + 2 * D);
  rm_store<D>(gF, out, D, D);
  rm_store<D>(gH, out + D * D, D, D);
  // the diagonals of sum Pbar_{t+1} (dL/dQ_ii) and of sum S^{-1}
  AKF_RM_FOR(D, k, r, i, j) {
    if (i == j) {
      va[i] = Pacc[k / TS][r];
      vb[i] = Sacc.t[k][r];
    }
  }
  wave_lds_fence();
  if (l < D) {
    out[2 * D * D + l] = va[l];
    out[2 * D * D + D + l] = l < p ? racc - 0.5 * vb[l] : 0.0;
  }
  if (!ok && l == 0) flag_status2(G.status, ST_FWD_NOT_PD);
}

template <int D, int KT>
__global__ void __launch_bounds__(64) k_adj_grad(KModel M, LgArgs G) {
  adj_grad_body<D, KT>(M, G);
}

// Sum the block partials in a fixed order and map to (dF, dlogq, dH, dlogr),
// scaled by the upstream gradient ll_bar.
// thread rows of the reduction: a row's loads are a serial chain of 1024 / 32 at
// 1024 blocks (with eight rows 27 us at d = 32, d_y = 16)
constexpr int kReduceRows = 32;

template <int D>
__global__ void __launch_bounds__(32 * kReduceRows) k_adj_reduce(LgArgs G, int nblk, const double* ll_bar) {
  // 32 parameters per workgroup; thread row r adds blocks r, r + kReduceRows, ...
  // and the rows are added in row order, so the result does not depend on timing
  __shared__ double acc[kReduceRows][33];
  const int px = threadIdx.x & 31, gy = threadIdx.x >> 5;
  const int tid = blockIdx.x * 32 + px;
  const int d = G.dx, p = G.dy;
  const int tot = d * d + d + p * d + p;
  const bool valid = tid < tot;
  int off = 0;
  double* dst = nullptr;
  double mul = 1.0;
  if (!valid) {
  } else if (tid < d * d) {
    const int i = tid / d, j = tid % d;
    off = i * D + j;
    dst = G.dF + tid;
  } else if (tid < d * d + d) {
    const int i = tid - d * d;
    off = 2 * D * D + i;
    dst = G.dlogq + i;
    mul = exp(G.logq[i]);
  } else if (tid < d * d + d + p * d) {
    const int e = tid - d * d - d, k = e / d, j = e % d;
    off = D * D + k * D + j;
    dst = G.dH + e;
  } else {
    const int k = tid - d * d - d - p * d;
    off = 2 * D * D + D + k;
    dst = G.dlogr + k;
    mul = exp(G.logr[k]);
  }
  double s = 0.0;
  if (valid)
    for (int b = gy; b < nblk; b += kReduceRows) s += G.part[(int64_t)b * (2 * D * D + 2 * D) + off];
  acc[gy][px] = s;
  __syncthreads();
  if (gy == 0 && valid) {
    double t = acc[0][px];
#pragma unroll
    for (int r = 1; r < kReduceRows; ++r) t += acc[r][px];
    const double sc = ll_bar ? *ll_bar : 1.0;
    // a failed forward or adjoint pass (any status bit) leaves no gradient
    *dst = (*G.status != 0) ? __builtin_nan("") : sc * mul * t;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int D>
size_t lds_bytes_mats(int nmat, int nvec) {
  return (size_t)(nmat * Cfg<D>::MAT + nvec * D + 16) * sizeof(double);
}

template <int D>
hipError_t launch_egl_scan(EglArgs A, EglTree* up, EglTree* down, int n_levels, hipStream_t st) {
  const int nb = (A.N + A.B - 1) / A.B;
  const size_t lds3 = D <= 32 ? wave_lds_bytes<D>() : lds_bytes_mats<D>(3, 2);
  const size_t lds2 = D <= 32 ? wave_lds_bytes<D>() : lds_bytes_mats<D>(2, 2);
  hipLaunchKernelGGL(k_egl_fold<D>, dim3(nb), dim3(Cfg<D>::NT), lds3, st, A);
  for (int l = 0; l < n_levels; ++l)
    hipLaunchKernelGGL(k_egl_up<D>, dim3(up[l].n_dst), dim3(Cfg<D>::NT), lds3,
                       st, up[l]);
  for (int l = n_levels - 1; l >= 0; --l)
    hipLaunchKernelGGL(k_egl_down<D>, dim3(down[l].n_src), dim3(Cfg<D>::NT),
                       lds2, st, down[l]);
  hipLaunchKernelGGL(k_egl_final<D>, dim3(nb), dim3(Cfg<D>::NT), lds2, st, A);
  return hipGetLastError();
}

hipError_t launch_egl_scan_any(int D, EglArgs A, EglTree* up, EglTree* down, int nl,
                               hipStream_t st) {
  switch (D) {
    case 16: return launch_egl_scan<16>(A, up, down, nl, st);
    case 32: return launch_egl_scan<32>(A, up, down, nl, st);
    case 64: return launch_egl_scan<64>(A, up, down, nl, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_smooth_build_any(int D, const KModel& M, SmoothArgs S, hipStream_t st) {
  switch (D) {
    case 16:
      hipLaunchKernelGGL(k_smooth_build<16>, dim3(M.N), dim3(64), lds_bytes_mats<16>(4, 7), st, M, S);
      break;
    case 32:
      hipLaunchKernelGGL(k_smooth_build<32>, dim3(M.N), dim3(64), lds_bytes_mats<32>(4, 7), st, M, S);
      break;
    case 64:
      hipLaunchKernelGGL(k_smooth_build<64>, dim3(M.N), dim3(256), lds_bytes_mats<64>(4, 7), st, M,
                         S);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_lgssm_prep(LgArgs G, hipStream_t st) {
  const int n = G.dx * G.dx + G.dy * G.dy;
  hipLaunchKernelGGL(k_lgssm_prep, dim3((n + 255) / 256), dim3(256), 0, st, G);
  return hipGetLastError();
}

hipError_t launch_sum(const double* a, int n, double* out, const int* status, hipStream_t st) {
  hipLaunchKernelGGL(k_sum, dim3(1), dim3(kSumThreads), 0, st, a, n, out, status);
  return hipGetLastError();
}

template <int D>
hipError_t launch_adj_build_t(const KModel& M, LgArgs G, hipStream_t st) {
  timing_mark(FAM_ADJ_BUILD, 1, st);
  // one tile row of observations where d_y fits it
  if (D == 16 || G.dy <= 16)
    hipLaunchKernelGGL((k_adj_build<D, 1>), dim3(M.N), dim3(64), wave_lds_bytes<D>(), st, M, G);
  else
    hipLaunchKernelGGL((k_adj_build<D, Cfg<D>::TS>), dim3(M.N), dim3(64), wave_lds_bytes<D>(), st, M,
                       G);
  timing_mark(FAM_ADJ_BUILD, 0, st);
  return hipGetLastError();
}
template <int D>
hipError_t launch_adj_finish_t(const KModel& M, LgArgs G, int nblk, const double* ll_bar,
                               hipStream_t st) {
  timing_mark(FAM_ADJ_GRAD, 1, st);
  if (D == 16 || G.dy <= 16)
    hipLaunchKernelGGL((k_adj_grad<D, 1>), dim3(nblk), dim3(64), wave_lds_bytes<D>(), st, M, G);
  else
    hipLaunchKernelGGL((k_adj_grad<D, Cfg<D>::TS>), dim3(nblk), dim3(64), wave_lds_bytes<D>(), st, M,
                       G);
  timing_mark(FAM_ADJ_GRAD, 0, st);
  const int tot = G.dx * G.dx + G.dx + G.dy * G.dx + G.dy;
  hipLaunchKernelGGL(k_adj_reduce<D>, dim3((tot + 31) / 32), dim3(32 * kReduceRows), 0, st, G,
                     nblk, ll_bar);
  return hipGetLastError();
}
hipError_t launch_adj_build_any(int D, const KModel& M, LgArgs G, hipStream_t st) {
  if (D == 16) return launch_adj_build_t<16>(M, G, st);
  if (D == 32) return launch_adj_build_t<32>(M, G, st);
  return hipErrorInvalidValue;
}
hipError_t launch_adj_finish_any(int D, const KModel& M, LgArgs G, int nblk, const double* ll_bar,
                                 hipStream_t st) {
  if (D == 16) return launch_adj_finish_t<16>(M, G, nblk, ll_bar, st);
  if (D == 32) return launch_adj_finish_t<32>(M, G, nblk, ll_bar, st);
  return hipErrorInvalidValue;
}

}  // namespace akf
