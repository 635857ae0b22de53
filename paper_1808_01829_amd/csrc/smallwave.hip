// The n x n FP64 algebra of one block iteration for n <= 16, with every matrix
// held in the registers of one wave (the recurrences are those of
// smallmat.hip, which keeps n > 16).
//
// Layout: lane (g = lane / 16, c = lane % 16), element e = entry (4e + g, c),
// NE = ceil(n / 4) elements; entries past n are zero. This is the accumulator
// layout of v_mfma_f64_16x16x4, and element s is at the same time the operand
// of contraction step s for the rows of a right factor and for the columns of
// a conjugate-transposed left factor. So L^H B runs from registers to
// registers with no data movement (wm_mulh); a plain left factor is loaded
// conjugate-transposed from memory instead.
//
// What bounds these kernels is latency: a chain of two eliminations and about
// ten dependent products per iteration, with nothing to fill the waits. One
// work-group of four waves per shift keeps that chain short:
//   wave 0  alpha_k = G_k^-1, V^H V from the expansion, its Cholesky factor
//   wave 1  the shift's recurrence, beside wave 0 (below it needs G_k only)
//   all     once rho_k is known, the products with it and the update window
// An elimination step needs one row and one column of the matrix: the column
// entry of each lane's rows comes by a DPP row broadcast, the pivot row by two
// cross-row swaps, so a step has no LDS round trip and no barrier.
//
// The shift recurrence is taken in Hermitian form. With
//   N = 1 - beta^(s), H_k = G_k + dsig + Z, Z = rho_{k-1} G_{k-1} N_{k-1} rho_{k-1}^H
// (dsig = s_s - s_0, G_k = alpha_k^-1) Algorithm 1's
//   beta_k = (1 + dsig alpha_k + alpha_k rho_{k-1} G_{k-1} N_{k-1} rho_{k-1}^H)^-1
// is beta_k = H_k^-1 G_k, hence N_k = H_k^-1 (dsig + Z) with no cancellation,
// and alpha^(s)_k = H_k^-1 rho_{k-1} G_{k-1} alpha^(s)_{k-1}. G N is Hermitian and
// positive semi-definite by induction (G - G H^-1 G with H >= G), so H_k is
// Hermitian positive definite: its inverse needs no pivoting and no alpha_k.
//
// Measured per launch (rocprofv3; the LDS form of smallmat.hip before): n = 1, 8
// shifts 15.4 -> 6.9 us; n = 4, 12 shifts 26.7 -> 7.2; n = 8, 16 shifts 44.7 -> 12.9
// (FP32 blocks 40.3 -> 11.6); n = 12, 15 shifts 58.8 -> 15.7; n = 16, 20 shifts,
// FP32 blocks 79.6 -> 20.4.
#include "blas.h"

namespace {

typedef double dx4 __attribute__((ext_vector_type(4)));

constexpr int WP = 17;  // row pitch of a matrix in LDS
constexpr int WLDS = 16 * WP;

template <int NE>
struct WM {
  double re[NE], im[NE];
};

// ---- moves between lanes ----------------------------------------------------

// lane P of every row of 16 lanes to the whole row
template <int P>
__device__ __forceinline__ double col_bcast(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)u, 0x150 + P, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), 0x150 + P, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
// row GP of 16 lanes to all four rows
template <int GP>
__device__ __forceinline__ int row_bcast(int v) {
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  const int w = (int)h[GP >> 1];
  const auto r = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return (int)r[GP & 1];
}
template <int GP>
__device__ __forceinline__ double row_bcast(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const int lo = row_bcast<GP>((int)u), hi = row_bcast<GP>((int)(u >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// ---- loads and stores ---------------------------------------------------------

// entry (r, c) of row-major m (n x n, row pitch ld)
template <int NE>
__device__ __forceinline__ WM<NE> wm_load(const double2* m, int ld, int n, int g, int c) {
  WM<NE> a;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int r = 4 * e + g;
    const bool ok = r < n && c < n;
    const double2 v = m[ok ? r * ld + c : 0];
    a.re[e] = ok ? v.x : 0.0;
    a.im[e] = ok ? v.y : 0.0;
  }
  return a;
}
// the conjugate transpose of m
template <int NE>
__device__ __forceinline__ WM<NE> wm_loadh(const double2* m, int ld, int n, int g, int c) {
  WM<NE> a;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int r = 4 * e + g;
    const bool ok = r < n && c < n;
    const double2 v = m[ok ? c * ld + r : 0];
    a.re[e] = ok ? v.x : 0.0;
    a.im[e] = ok ? -v.y : 0.0;
  }
  return a;
}
template <int NE, typename C>
__device__ __forceinline__ void wm_store(C* m, int ld, int n, int g, int c, const WM<NE>& a) {
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int r = 4 * e + g;
    if (r < n && c < n) m[r * ld + c] = from_d<C>(make_double2(a.re[e], a.im[e]));
  }
}
// the LDS writes of this wave are complete and visible to its own reads
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// (a + a^H) / 2 through this wave's LDS area
template <int NE>
__device__ __forceinline__ WM<NE> wm_hermitian(double2* lds, int n, int g, int c, WM<NE> a) {
  wm_store(lds, WP, n, g, c, a);
  wave_lds_sync();
  const WM<NE> h = wm_loadh<NE>(lds, WP, n, g, c);
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    a.re[e] = 0.5 * (a.re[e] + h.re[e]);
    a.im[e] = 0.5 * (a.im[e] + h.im[e]);
  }
  return a;
}

// ---- algebra ------------------------------------------------------------------

// L^H B (+ C0)
template <int NE>
__device__ __forceinline__ WM<NE> wm_mulh(const WM<NE>& l, const WM<NE>& b,
                                          const WM<NE>* c0 = nullptr) {
  dx4 r0{0, 0, 0, 0}, r1{0, 0, 0, 0}, i0{0, 0, 0, 0}, i1{0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < NE; ++s) {
    r0 = __builtin_amdgcn_mfma_f64_16x16x4f64(l.re[s], b.re[s], r0, 0, 0, 0);
    i0 = __builtin_amdgcn_mfma_f64_16x16x4f64(l.re[s], b.im[s], i0, 0, 0, 0);
    r1 = __builtin_amdgcn_mfma_f64_16x16x4f64(l.im[s], b.im[s], r1, 0, 0, 0);
    i1 = __builtin_amdgcn_mfma_f64_16x16x4f64(l.im[s], b.re[s], i1, 0, 0, 0);
  }
  WM<NE> d;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    d.re[e] = r0[e] + r1[e];
    d.im[e] = i0[e] - i1[e];
    if (c0) {
      d.re[e] += c0->re[e];
      d.im[e] += c0->im[e];
    }
  }
  return d;
}

// Step P of an elimination of a Hermitian positive definite matrix.
// FWD = false: in-place Gauss-Jordan; after all steps `a` is the inverse.
// FWD = true: rows below P only; after all steps row i holds d_i times row i
// of the unit upper factor U (columns >= i) and row i of L^-1 = U^-H (columns
// < i) of a = U^H diag(d) U, and dr the pivots of this lane's rows.
// st: 0, or the status of the first pivot that is not above `floor`.
template <int P, bool FWD, int NE>
__device__ __forceinline__ void elim_step(WM<NE>& a, int g, int c, double (&dr)[NE], double floor,
                                          int& st) {
  constexpr int EP = P / 4, GP = P % 4;
  const double pr = row_bcast<GP>(a.re[EP]), pi = row_bcast<GP>(a.im[EP]);
  const double d = col_bcast<P>(pr);
  if (st == 0 && !(d > floor)) st = d == d ? BMS_EBREAKDOWN : BMS_ENAN;
  const double inv = 1.0 / d;
  const bool cp = c == P;
  const double sr = cp ? inv : pr * inv, si = cp ? 0.0 : pi * inv;
#pragma unroll
  for (int e = FWD ? EP : 0; e < NE; ++e) {
    const double fr = col_bcast<P>(a.re[e]), fi = col_bcast<P>(a.im[e]);
    double ar = cp ? 0.0 : a.re[e], ai = cp ? 0.0 : a.im[e];
    ar = fma(-fr, sr, ar);
    ar = fma(fi, si, ar);
    ai = fma(-fr, si, ai);
    ai = fma(-fi, sr, ai);
    if (e == EP) {
      const bool own = FWD ? g <= GP : g == GP;
      ar = own ? (FWD ? a.re[e] : sr) : ar;
      ai = own ? (FWD ? a.im[e] : si) : ai;
    }
    a.re[e] = ar;
    a.im[e] = ai;
  }
  if (FWD) dr[EP] = g == GP ? d : dr[EP];
}
template <int P, bool FWD, int NE>
__device__ __forceinline__ void elim_from(WM<NE>& a, int n, int g, int c, double (&dr)[NE],
                                          double floor, int& st) {
  if constexpr (P < 4 * NE) {
    if (P >= n) return;
    elim_step<P, FWD, NE>(a, g, c, dr, floor, st);
    elim_from<P + 1, FWD, NE>(a, n, g, c, dr, floor, st);
  }
}

// a <- a^-1 for Hermitian positive definite a; returns the status
template <int NE>
__device__ __forceinline__ int wm_inverse(WM<NE>& a, int n, int g, int c) {
  double dr[NE];
  int st = 0;
  elim_from<0, false, NE>(a, n, g, c, dr, 0.0, st);
  return __builtin_amdgcn_readfirstlane(st);
}

// Cholesky factor a = R^H R: `r` the upper R, `rih` the lower R^-H, returns
// the status (a pivot not above tol * trace, or not finite)
template <int NE>
__device__ __forceinline__ int wm_cholesky(WM<NE> a, int n, int g, int c, double tol, double trace,
                                           WM<NE>& r, WM<NE>& rih) {
  int st = 0;
  if (!(trace == trace) || !(fabs(trace) < 1e300)) st = BMS_ENAN;
  double dr[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) dr[e] = 1.0;
  elim_from<0, true, NE>(a, n, g, c, dr, tol * trace, st);
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int row = 4 * e + g;
    const double q = sqrt(dr[e]), qi = 1.0 / q;
    const bool up = c > row, dg = c == row;
    r.re[e] = dg ? q : (up ? a.re[e] * qi : 0.0);
    r.im[e] = up ? a.im[e] * qi : 0.0;
    rih.re[e] = dg ? qi : (up ? 0.0 : a.re[e] * qi);
    rih.im[e] = dg || up ? 0.0 : a.im[e] * qi;
  }
  return __builtin_amdgcn_readfirstlane(st);
}

// ---- the iteration ------------------------------------------------------------

// What the four waves exchange once rho_k is known: rho, alpha^(s), for a shift beta^(s)^H,
// for sigma_0 alpha (in bh) and rho^-H (in t).
struct SmallLds {
  double2 rho[WLDS], mx[WLDS], bh[WLDS], t[WLDS];
  int st1, st2, st3;
};

// One block's arrival. kind: 0 its shift is above tol, 1 it met tol (or is frozen), 2 it
// raised an error, 3 it waits for the explicit Gram. The last block ends the solve when
// every shift met tol (or raised an error) and advances the iteration counter, or, if
// blocks wait, pauses the iteration (raises need_explicit; with no fallback kernels
// behind it, stop and halted too). Only the last arrival may write those flags: every block
// has read them by then. Everything it needs is in the counter (arrivals, shifts done,
// errors, waiting blocks in 8 bits each), so no fence orders the blocks' other
// writes; the next kernel sees them all.
__device__ __forceinline__ void arrive(const SmallParams& p, const SmallState& s, SolverFlags* fl,
                                       int kind) {
  const int add = kind == 0 ? 1 : (kind == 1 ? 1 + (1 << 8) : (kind == 2 ? 1 + (1 << 16) : 1 << 24));
  const int v = atomicAdd(s.counter, add) + add;
  const int waiting = v >> 24;
  if ((v & 0xff) + waiting != p.ns) return;
  if (waiting) {
    fl->need_explicit = 1;
    if (!p.inline_explicit) fl->stop = fl->halted = 2;
    atomicSub(s.counter, waiting << 24);
    return;
  }
  if (((v >> 8) & 0xff) == p.ns || ((v >> 16) & 0xff)) fl->stop = 1;
  fl->need_explicit = 0;
  fl->iter = fl->iter + 1;
  atomicExch(s.counter, 0);
}

__device__ __forceinline__ void set_error(SolverFlags* fl, int code) {
  atomicCAS(&fl->error, 0, code);
  fl->stop = 1;
  fl->halted = 1;
}

// Everything that needs rho_k (l.rho), with Mx = alpha^(s)_k in l.mx and, for
// a shift, beta^(s)_k^H in l.bh: Mp, the shift's residual coefficients and
// convergence, and the step into its update window (SmallState::wst; the
// algebra is that of win_step in smallmat.hip). ga: G_k alpha^(s)_k (wave 1 of
// a shift), dl: delta_{k-1} (wave 1 of sigma_0).
template <typename T, int NE>
__device__ __forceinline__ void rho_part_w(const SmallParams& p, const SmallState& s,
                                           SolverFlags* fl, cplx<T>* Mp, cplx<T>* Wm,
                                           const SmallLds& l, const WM<NE>& ga, const WM<NE>& dl,
                                           int q, int cur, int j0, int wave, int lane) {
  using C = cplx<T>;
  const int n = p.n, nn = n * n, g = lane >> 4, c = lane & 15;
  const int ws = cur ^ 1;
  const WM<NE> rh = wm_loadh<NE>(l.rho, WP, n, g, c);  // rho_k^H
  // Mp = beta rho^H, for sigma_0 rho^H
  WM<NE> mp = rh;
  if (q > 0) mp = wm_mulh(wm_load<NE>(l.bh, WP, n, g, c), rh);
  const WM<NE> mx = wm_load<NE>(l.mx, WP, n, g, c);
  const size_t fam = (size_t)BMS_MAX_WIN * nn;
  const double2* ox = s.wst + (size_t)(cur * p.ns + q) * 2 * fam;
  const double2* op = ox + fam;
  double2* nx = s.wst + (size_t)(ws * p.ns + q) * 2 * fam;
  double2* np = nx + fam;
  C* tx = Wm + (size_t)q * 2 * fam;
  C* tp = tx + fam;
  if (wave == 1) {
    // delta^(s)_k = rho_k G_k alpha^(s)_k, for sigma_0 rho_k delta_{k-1}
    const WM<NE> d = wm_mulh(rh, q > 0 ? ga : dl);
    if (q == 0) wm_store(s.delta, n, n, g, c, d);
    // max over the columns of |delta e_i| / |b_i|
    double m = 0;
#pragma unroll
    for (int e = 0; e < NE; ++e) m += d.re[e] * d.re[e] + d.im[e] * d.im[e];
    m += __shfl_xor(m, 16);
    m += __shfl_xor(m, 32);
    double r = c < n ? sqrt(m) / s.norm0[c] : 0.0;
    if (!(r == r)) r = 1e300;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) r = fmax(r, __shfl_xor(r, off));
    if (lane == 0) {
      const bool conv = q > 0 && r < p.freeze_tol;
      fl->res[q] = r;
      if (q > 0) fl->conv[q] = conv;
      if (r >= 1e300) {
        atomicCAS(&fl->error, 0, BMS_ENAN);
        fl->halted = 1;
      }
      fl->win_j[ws][q] = j0 + 1;
      fl->win_flush[ws][q] = (j0 + 1 >= (q == 0 ? 1 : p.win)) || conv;
      arrive(p, s, fl, r >= 1e300 ? 2 : (r < p.tol ? 1 : 0));
    }
  } else if (wave == 2) {
    wm_store(Mp + (size_t)q * nn, n, n, g, c, mp);
    wm_store(np + (size_t)j0 * nn, n, n, g, c, mp);
    wm_store(tp + (size_t)j0 * nn, n, n, g, c, mp);
    if (q == 0) wm_store(s.rhob + (size_t)cur * nn, n, n, g, c, wm_load<NE>(l.rho, WP, n, g, c));
  } else if (wave == 3) {
    if (q == 0) {
      // rho^-1 and -alpha rho^-1 for the update's Q step
      const WM<NE> ri = wm_loadh<NE>(l.t, WP, n, g, c);
      WM<NE> ar = wm_mulh(wm_loadh<NE>(l.bh, WP, n, g, c), ri);
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        ar.re[e] = -ar.re[e];
        ar.im[e] = -ar.im[e];
      }
      wm_store(s.rhoinv, n, n, g, c, ri);
      wm_store(s.arho, n, n, g, c, ar);
    }
    wm_store(nx + (size_t)j0 * nn, n, n, g, c, mx);
    wm_store(tx + (size_t)j0 * nn, n, n, g, c, mx);
  }
  // the window's older matrices, dealt to the waves
  for (int i = wave; i < j0; i += BMS_WG / 64) {
    const WM<NE> ph = wm_loadh<NE>(op + (size_t)i * nn, n, n, g, c);
    const WM<NE> x0 = wm_load<NE>(ox + (size_t)i * nn, n, n, g, c);
    const WM<NE> x1 = wm_mulh(ph, mx, &x0), p1 = wm_mulh(ph, mp);
    wm_store(nx + (size_t)i * nn, n, n, g, c, x1);
    wm_store(tx + (size_t)i * nn, n, n, g, c, x1);
    wm_store(np + (size_t)i * nn, n, n, g, c, p1);
    wm_store(tp + (size_t)i * nn, n, n, g, c, p1);
  }
}

// iterations already gathered in the open window of shift q (0: a fresh one)
__device__ __forceinline__ int window_fill(const SolverFlags* fl, int cur, int q) {
  return fl->win_flush[cur][q] ? 0 : fl->win_j[cur][q];
}

// the diagonal of a matrix staged in LDS, summed in order
__device__ __forceinline__ double lds_trace(const double2* m, int n) {
  double t = 0;
  for (int i = 0; i < n; ++i) t += m[i * WP + i].x;
  return t;
}

// rho_k (for sigma_0 also rho_k^-H and alpha_k) to where the other waves find them
template <int NE>
__device__ __forceinline__ void put_rho(SmallLds& l, int n, int g, int c, int q, const WM<NE>& r,
                                        const WM<NE>& rih, const WM<NE>& alpha) {
  wm_store(l.rho, WP, n, g, c, r);
  if (q > 0) return;
  wm_store(l.t, WP, n, g, c, rih);
  wm_store(l.bh, WP, n, g, c, alpha);
}

// One iteration's n x n work after G4 = [P^H W, Q^H W, W^H W, Q^H Q] (the steps and
// the state are those of k_small_iter). Blocks read the flags of one launch while
// another block may raise an error (stop): the waves of a block can then disagree and
// some leave early, which only leaves values behind that a stopped solve never reads.
// SUM: the Grams come as nparts partials, added here in a fixed order (the same in every
// block).
template <typename T, int NE, bool SUM>
__global__ __launch_bounds__(BMS_WG) void k_small_iter_w(SmallParams p, SmallState s,
                                                         SolverFlags* fl, cplx<T>* Mx,
                                                         cplx<T>* Mp, cplx<T>* Wm,
                                                         const double2* __restrict__ part,
                                                         int nparts) {
  __shared__ SmallLds l;
  __shared__ double2 gs[SUM ? (64 * NE * NE > BMS_WG ? 64 * NE * NE : BMS_WG) : 1];
  const int n = p.n, nn = n * n, q = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int stop = fl->stop;
  if (stop || fl->iter >= p.max_iter) {
    if (q == 0 && threadIdx.x == 0 && stop != 2) {
      fl->stop = 1;
      fl->halted = 1;
    }
    return;
  }
  const int cur = fl->iter & 1, prev = cur ^ 1;
  if (q > 0 && (fl->conv[q] || !fl->active[q])) {
    // frozen: its last window was applied when it converged
    if (threadIdx.x == 0) {
      fl->active[q] = 0;
      fl->win_j[prev][q] = 0;
      fl->win_flush[prev][q] = 1;
      arrive(p, s, fl, 1);
    }
    return;
  }
  const int j0 = q == 0 ? 0 : window_fill(fl, cur, q);
  if constexpr (SUM) {
    const int E = 4 * nn, ng = E < BMS_WG ? BMS_WG / E : 1;
    const int grp = threadIdx.x / E;
    if (grp < ng)
      for (int e = threadIdx.x - grp * E; e < E; e += BMS_WG) {
        double2 a = make_double2(0, 0);
#pragma unroll 8
        for (int b = grp; b < nparts; b += ng) a = cadd(a, part[(size_t)b * E + e]);
        gs[grp * E + e] = a;
      }
    __syncthreads();
    if (ng > 1) {
      double2 a = make_double2(0, 0);
      if ((int)threadIdx.x < E)
        for (int k = 0; k < ng; ++k) a = cadd(a, gs[k * E + threadIdx.x]);
      __syncthreads();
      if ((int)threadIdx.x < E) gs[threadIdx.x] = a;
      __syncthreads();
    }
  }
  const double2* G4 = SUM ? gs : s.G4;
  WM<NE> ga, dl;
  if (wave < 2) {
    // G_k = P^H (A + s0) P, Hermitian up to rounding
    WM<NE> G = wm_load<NE>(G4, n, n, g, c);
    const WM<NE> Gt = wm_loadh<NE>(G4, n, n, g, c);
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      G.re[e] = 0.5 * (G.re[e] + Gt.re[e]);
      G.im[e] = 0.5 * (G.im[e] + Gt.im[e]);
    }
    if (q == 0) dl = wm_load<NE>(s.delta, n, n, g, c);
    if (wave == 0) {
      const WM<NE> qwh = wm_loadh<NE>(G4 + nn, n, n, g, c);    // (Q^H W)^H
      const WM<NE> ww = wm_load<NE>(G4 + 2 * nn, n, n, g, c);  // W^H W
      const WM<NE> qq = wm_load<NE>(G4 + 3 * nn, n, n, g, c);
      if (q == 0) wm_store(s.Gb + (size_t)cur * nn, n, n, g, c, G);
      WM<NE> A = G;
      const int st1 = wm_inverse(A, n, g, c);  // alpha_k
      if (q == 0) {
        wm_store(s.alpha, n, n, g, c, A);
        const WM<NE> m0 = wm_mulh(A, dl);  // alpha^(0)_k = alpha_k delta_{k-1}
        wm_store(s.alpha_s, n, n, g, c, m0);
        wm_store(Mx, n, n, g, c, m0);
        wm_store(l.mx, WP, n, g, c, m0);
      }
      // V^H V = Q^H Q - (Q^H W) A + A^H (W^H W A - W^H Q)
      WM<NE> t = wm_mulh(ww, A);
      const WM<NE> qwa = wm_mulh(qwh, A);
      WM<NE> E;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        t.re[e] -= qwh.re[e];
        t.im[e] -= qwh.im[e];
        E.re[e] = qq.re[e] - qwa.re[e];
        E.im[e] = qq.im[e] - qwa.im[e];
      }
      E = wm_mulh(A, t, &E);
      // traces in diagonal order, and the Hermitian part
      wm_store(l.t, WP, n, g, c, qq);
      wave_lds_sync();
      const double tq = lds_trace(l.t, n);
      wave_lds_sync();
      E = wm_hermitian(l.t, n, g, c, E);
      const double tv = lds_trace(l.t, n);
      // The expansion cancels when V is small next to Q; then the explicit
      // Gram of V is used instead.
      const bool cancel = !(tv >= 1e-4 * tq);
      WM<NE> R, rih;
      int st2 = BMS_EBREAKDOWN;
      if (!cancel) {
        st2 = wm_cholesky(E, n, g, c, p.breakdown_tol, tv, R, rih);
        if (st2 == 0 && st1 == 0) put_rho(l, n, g, c, q, R, rih, A);
      }
      if (lane == 0) {
        l.st1 = st1;
        l.st2 = st2;
      }
    } else if (q > 0) {
      const double dsig = p.sigma[q] - p.sigma[0];
      const WM<NE> rhoh = wm_loadh<NE>(s.rhob + (size_t)prev * nn, n, n, g, c);
      const WM<NE> Gp = wm_load<NE>(s.Gb + (size_t)prev * nn, n, n, g, c);
      const WM<NE> N = wm_load<NE>(s.beta_s + (size_t)q * nn, n, n, g, c);
      const WM<NE> as = wm_load<NE>(s.alpha_s + (size_t)q * nn, n, n, g, c);
      // Z = rho (G N) rho^H (G N Hermitian), K = rho G alpha^(s)
      WM<NE> Z = wm_mulh(rhoh, wm_mulh(wm_mulh(Gp, N), rhoh));
      const WM<NE> K = wm_mulh(rhoh, wm_mulh(Gp, as));
      WM<NE> H;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        if (4 * e + g == c && c < n) Z.re[e] += dsig;
        H.re[e] = G.re[e] + Z.re[e];
        H.im[e] = G.im[e] + Z.im[e];
      }
      const int st = wm_inverse(H, n, g, c);
      if (lane == 0) l.st3 = st == BMS_ENAN ? st : 0;
      const WM<NE> a1 = wm_mulh(H, K);      // alpha^(s)_k
      const WM<NE> N1 = wm_mulh(H, Z);      // 1 - beta^(s)_k
      const WM<NE> bh = wm_mulh(G, H);      // beta^(s)_k^H = G H^-1
      wm_store(l.mx, WP, n, g, c, a1);
      wm_store(l.bh, WP, n, g, c, bh);
      wm_store(s.beta_s + (size_t)q * nn, n, n, g, c, N1);
      wm_store(s.alpha_s + (size_t)q * nn, n, n, g, c, a1);
      wm_store(Mx + (size_t)q * nn, n, n, g, c, a1);
      ga = wm_mulh(G, a1);
    }
  }
  __syncthreads();
  if (l.st1) {
    if (q == 0 && threadIdx.x == 0) set_error(fl, l.st1);
    return;
  }
  if (q > 0 && l.st3) {
    if (threadIdx.x == 0) set_error(fl, l.st3);
    return;
  }
  if (l.st2) {
    if (threadIdx.x == 0) {
      if (l.st2 != BMS_ENAN)
        arrive(p, s, fl, 3);  // the explicit Gram finishes this iteration
      else if (q == 0)
        set_error(fl, BMS_ENAN);
    }
    return;
  }
  rho_part_w<T, NE>(p, s, fl, Mp, Wm, l, ga, dl, q, cur, j0, wave, lane);
}

// Fallback when the expansion lost accuracy: rho_k from the explicit V^H V
// (Gqr), the rest from what k_small_iter_w stored.
template <typename T, int NE>
__global__ __launch_bounds__(BMS_WG) void k_small_rho_explicit_w(SmallParams p, SmallState s,
                                                                 SolverFlags* fl, cplx<T>* Mp,
                                                                 cplx<T>* Wm) {
  __shared__ SmallLds l;
  const int n = p.n, nn = n * n, q = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, c = lane & 15;
  if (fl->stop || !fl->need_explicit) return;
  if (q > 0 && !fl->active[q]) return;  // already counted by k_small_iter_w
  const int cur = fl->iter & 1;
  const int j0 = q == 0 ? 0 : window_fill(fl, cur, q);
  WM<NE> ga, dl;
  if (wave == 0) {
    WM<NE> E = wm_load<NE>(s.Gqr, n, n, g, c), R, rih;
    E = wm_hermitian(l.t, n, g, c, E);
    const int st = wm_cholesky(E, n, g, c, p.breakdown_tol, lds_trace(l.t, n), R, rih);
    if (st == 0) put_rho(l, n, g, c, q, R, rih, wm_load<NE>(s.alpha, n, n, g, c));
    if (lane == 0) l.st2 = st;
  } else if (wave == 1) {
    const WM<NE> a1 = wm_load<NE>(s.alpha_s + (size_t)q * nn, n, n, g, c);
    wm_store(l.mx, WP, n, g, c, a1);
    if (q > 0) {
      const WM<NE> G = wm_load<NE>(s.Gb + (size_t)cur * nn, n, n, g, c);
      WM<NE> bh = wm_loadh<NE>(s.beta_s + (size_t)q * nn, n, n, g, c);
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        bh.re[e] = (4 * e + g == c && c < n ? 1.0 : 0.0) - bh.re[e];
        bh.im[e] = -bh.im[e];
      }
      wm_store(l.bh, WP, n, g, c, bh);
      ga = wm_mulh(G, a1);
    } else {
      dl = wm_load<NE>(s.delta, n, n, g, c);
    }
  }
  __syncthreads();
  if (l.st2) {
    if (q == 0 && threadIdx.x == 0) set_error(fl, l.st2);
    return;
  }
  rho_part_w<T, NE>(p, s, fl, Mp, Wm, l, ga, dl, q, cur, j0, wave, lane);
}

}  // namespace

template <typename T, bool SUM>
static hipError_t small_iter_w(hipStream_t st, const SmallParams& p, SmallState s,
                               SolverFlags* fl, cplx<T>* Mx, cplx<T>* Mp, cplx<T>* Wm,
                               const double2* part, int nparts) {
#define ITER_W(NE) \
  k_small_iter_w<T, NE, SUM><<<p.ns, BMS_WG, 0, st>>>(p, s, fl, Mx, Mp, Wm, part, nparts)
  switch ((p.n + 3) / 4) {
    case 1: ITER_W(1); break;
    case 2: ITER_W(2); break;
    case 3: ITER_W(3); break;
    case 4: ITER_W(4); break;
    default: return hipErrorInvalidValue;
  }
#undef ITER_W
  return hipGetLastError();
}

template <typename T>
hipError_t launch_small_iter_w(hipStream_t st, const SmallParams& p, SmallState s,
                               SolverFlags* fl, cplx<T>* Mx, cplx<T>* Mp, cplx<T>* Wm,
                               const double2* part, int nparts) {
  return nparts ? small_iter_w<T, true>(st, p, s, fl, Mx, Mp, Wm, part, nparts)
                : small_iter_w<T, false>(st, p, s, fl, Mx, Mp, Wm, part, 0);
}

template <typename T>
hipError_t launch_small_rho_explicit_w(hipStream_t st, const SmallParams& p, SmallState s,
                                       SolverFlags* fl, cplx<T>* Mp, cplx<T>* Wm) {
  switch ((p.n + 3) / 4) {
    case 1: k_small_rho_explicit_w<T, 1><<<p.ns, BMS_WG, 0, st>>>(p, s, fl, Mp, Wm); break;
    case 2: k_small_rho_explicit_w<T, 2><<<p.ns, BMS_WG, 0, st>>>(p, s, fl, Mp, Wm); break;
    case 3: k_small_rho_explicit_w<T, 3><<<p.ns, BMS_WG, 0, st>>>(p, s, fl, Mp, Wm); break;
    case 4: k_small_rho_explicit_w<T, 4><<<p.ns, BMS_WG, 0, st>>>(p, s, fl, Mp, Wm); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

#define INST_W(T, C)                                                                        \
  template hipError_t launch_small_iter_w<T>(hipStream_t, const SmallParams&, SmallState,   \
                                             SolverFlags*, C*, C*, C*, const double2*, int); \
  template hipError_t launch_small_rho_explicit_w<T>(hipStream_t, const SmallParams&,       \
                                                     SmallState, SolverFlags*, C*, C*);
INST_W(double, double2)
INST_W(float, float2)
