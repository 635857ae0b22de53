// Fused block update on the matrix cores (v_mfma_f64_16x16x4 in FP64,
// v_mfma_f32_16x16x4 for the shift updates of the mixed solver).
//
// Same arithmetic as the vector update kernels, per iteration k of
// Algorithm 1 (block CG with Cholesky-QR, Sec. III):
//   Q_{k+1} = (Q_k - W alpha_k) rho_k^-1   computed as  Q_k rho^-1 + W (-alpha rho^-1)
//   X^(s)  += P^(s) Mx^(s)                 (Mx = alpha^(s)_k)
//   P^(s)   = Q_{k+1} + P^(s) Mp^(s)       (Mp = beta^(s)_k rho_k^dag)
// for every shift still active. The Q step always runs in FP64 (FP32 blocks
// are widened on load), the shift updates in the block precision.
//
// A complex row of n entries is 2n interleaved reals; a right product with a
// complex n x n matrix M is the real product with the 2n x 2n matrix
//   [ Re M  Im M ]
//   [-Im M  Re M ]   (rows in (re, im) pairs, columns permuted: all real parts
// first, then all imaginary parts). Each wave owns 16-row tiles. The MFMA
// operand layouts (A[i][k] in lane i + 16k, B[k][j] in lane j + 16k; the
// accumulator D[i][j] in lane j + 16(i%4), element i/4 for f64 and in lane
// j + 16(i/4), element i%4 for f32 -- both measured on gfx950) give:
//   A operand: lane (g = lane/16, c = lane%16) holds row c, reals g*KS .. g*KS+KS-1
//              (the contraction order is free, so each lane reads one contiguous run);
//   D: lane (g, c) holds four rows of the tile at real output column nt*16 + c,
//      which for n = 16 is (Re, Im) of complex column c in the two n-tiles: one
//      complex per row, so X and P are read and written as whole complex numbers.
// The coefficients of the Q step (rho^-1 and -alpha rho^-1, both from the small step)
// and of the shifts are kept in LDS as complex n x n matrices, and each lane forms
// its B operands from them one k-step at a time.
#include <algorithm>

#include "blas.h"

namespace {

typedef double dx4 __attribute__((ext_vector_type(4)));
typedef float fx4 __attribute__((ext_vector_type(4)));

constexpr int MF_WAVES = BMS_WG / 64;

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void glob_void;

// Copy `bytes` rounded up to whole KiB (both regions hold that much) from
// global memory into LDS by direct-to-LDS loads (global_load_lds_dwordx4, lane
// l of a wave writing 16 bytes at the wave's destination + 16 l): wave w
// copies the KiB chunks w, w + 4, ... Nothing passes through registers, so
// every load of a shift's coefficients is in flight at once instead of one
// round trip per matrix.
__device__ __forceinline__ void lds_copy(const void* src, void* dst, int bytes, int wave,
                                         int lane) {
  for (int off = wave * 1024; off < bytes; off += MF_WAVES * 1024)
    __builtin_amdgcn_global_load_lds((glob_void*)((const char*)src + off + lane * 16),
                                     (lds_void*)((char*)dst + off), 16, 0, 0);
}

template <typename F>
struct Mf;
template <>
struct Mf<double> {
  using V = dx4;
  __device__ static __forceinline__ V mfma(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // tile row of accumulator element p in lane group g
  __device__ static __forceinline__ int row(int g, int p) { return g + 4 * p; }
};
template <>
struct Mf<float> {
  using V = fx4;
  __device__ static __forceinline__ V mfma(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static __forceinline__ int row(int g, int p) { return 4 * g + p; }
};

// Waves and threads of a work-group of k_update_close.
constexpr int CL_WAVES = 8, CL_THREADS = CL_WAVES * 64;

// N: block width (8 or 16), or the largest width (12, 16, 24 or 32) the form for a width
// known at run time takes. wide: the products of mfma_wide below.
template <int N>
struct MfShape {
  static constexpr bool wide = N > 8;
  static constexpr int KS = N / 2;            // reals of a row per lane group: k-steps of 4
  static constexpr int NT = wide ? 2 : 1;     // 16-column output tiles
  static constexpr int PITCH = NT * 16;       // reals per row of the staged output tiles
};

// The shift coefficients are kept in LDS as the complex n x n matrix, (re,
// im) pairs, half of the expanded form; each lane forms its B-operand
// reals from it: B[2k][j] = Re M[k][j], B[2k][n+j] = Im, B[2k+1][j] = -Im,
// B[2k+1][n+j] = Re, at kk = g*KS + ks, flat = nt*16 + c.
// d += a * B(M), the B operands read from LDS one k-step at a time (few
// registers live: the kernel keeps four waves per SIMD)
template <int N, typename F>
__device__ __forceinline__ void mfma_acc_c(typename Mf<F>::V (&d)[MfShape<N>::NT],
                                           const F (&a)[MfShape<N>::KS], const F* M, int g,
                                           int c) {
  using S = MfShape<N>;
#pragma unroll
  for (int ks = 0; ks < S::KS; ++ks) {
    const int kk = g * S::KS + ks, k = kk >> 1, rim = kk & 1, j = c % N, cim = c / N;
    const F v = M[2 * (k * N + j) + (rim ^ cim)];
    d[0] = Mf<F>::mfma(a[ks], rim && !cim ? -v : v, d[0]);
  }
}

// n > 8: the complex right product. With the A operand of a lane holding complex columns
// KC g .. KC g + KC - 1 of its row (KC = N / 4; the same contiguous run as above), k-step ks
// contracts over complex column kc = KC g + ks, and output column c of every accumulator is
// complex column c, so the results land in the layout of the n-tiles above (tile 0 real
// parts, tile 1 imaginary parts; wide_re, wide_im). M: complex n x n in LDS, (re, im) pairs.
// For n < N the columns past n meet a zero A operand and read row 0 (finite) instead; output
// columns past n are not used.
//
// ACC = 3: Gauss's three real products,
//   d0 = sum Re a Re M,  d1 = sum Im a Im M,  d2 = sum (Re a + Im a)(Re M + Im M),
//   Re(a M) = d0 - d1,  Im(a M) = d2 - d0 - d1,
// 3 N / 4 matrix-core steps per product and 16-row tile. ACC = 2: the four products, N steps,
// with the rounding of plain complex multiply-adds.
//
// The windows take three products up to n = 16, and above in FP64, where they are bound by
// the matrix cores; the Q step of every width but 16, and FP32 windows above 16, take four,
// which costs them little. Against the vector kernels that updated every iteration with plain
// multiply-adds, rms error of X after 12 or 16 iterations (4 x 6 x 4 x 6, five shifts,
// the mean over them): FP64 0.82 at n = 9, 0.84 at 12, 0.78 at 15, 0.99 to 1.02 from 17 to
// 32; FP32 0.97, 0.96, 0.94, and 0.93 falling to 0.87. Four products in all windows: 0.78,
// 0.81, 0.76 and FP32 0.92, 0.91, 0.91, for 10 % of the update's time (n = 12 FP64 81 -> 90
// us at 16^4).
template <typename F, int N, bool RT, int ACC>
__device__ __forceinline__ void mfma_wide(typename Mf<F>::V (&d)[ACC],
                                          const F (&a)[MfShape<N>::KS], const F* M, int nrt, int g,
                                          int c) {
  constexpr int KC = N / 4;
  const int n = RT ? nrt : N;
#pragma unroll
  for (int ks = 0; ks < KC; ++ks) {
    const int kc = KC * g + ks;
    const int e = 2 * ((RT && kc >= n ? 0 : kc) * n + c);
    const F mr = M[e], mi = M[e + 1];
    const F ar = a[2 * ks], ai = a[2 * ks + 1];
    d[0] = Mf<F>::mfma(ar, mr, d[0]);
    if constexpr (ACC == 3) {
      d[1] = Mf<F>::mfma(ai, mi, d[1]);
      d[2] = Mf<F>::mfma(ar + ai, mr + mi, d[2]);
    } else {
      d[1] = Mf<F>::mfma(ar, mi, d[1]);
      d[0] = Mf<F>::mfma(-ai, mi, d[0]);
      d[1] = Mf<F>::mfma(ai, mr, d[1]);
    }
  }
}
template <typename V>
__device__ __forceinline__ V wide_re(const V (&d)[3]) {
  return d[0] - d[1];
}
template <typename V>
__device__ __forceinline__ V wide_im(const V (&d)[3]) {
  return d[2] - d[0] - d[1];
}
template <typename V>
__device__ __forceinline__ V wide_re(const V (&d)[2]) {
  return d[0];
}
template <typename V>
__device__ __forceinline__ V wide_im(const V (&d)[2]) {
  return d[1];
}

// A-operand reals of one tile row (row r, reals g*KS .. g*KS+KS-1) in the
// arithmetic type F. Rows past the end read row 0 (a row only reaches its own results,
// and those are not stored), with no branch around the loads and, at a fixed width, no
// select behind them: a select waits for its load at once, and the loads of the next shift
// would not be in flight while this one is computed. Columns past n are zeroed.
template <int N, bool RT, typename F, typename C>
__device__ __forceinline__ void aload(const C* base, int r, int rows, int nrt, int g,
                                      F (&a)[MfShape<N>::KS]) {
  using S = MfShape<N>;
  constexpr int KC = S::KS / 2;
  const int n = RT ? nrt : N;
  const C* p = base + (size_t)(r < rows ? r : 0) * n + g * KC;
#pragma unroll
  for (int h = 0; h < KC; ++h) {
    const bool okc = !RT || g * KC + h < n;
    C v = p[okc ? h : -g * KC];
    a[2 * h] = okc ? (F)v.x : (F)0;
    a[2 * h + 1] = okc ? (F)v.y : (F)0;
  }
}

// D-layout access: lane (g, c), element p is tile row Mf<F>::row(g, p); widths above 8:
// complex column c (real parts in tile 0, imaginary in tile 1), n = 8: real column c, part
// c / 8 (0 = re, 1 = im) of complex column c % 8.
template <int N, bool RT, typename F, typename C>
__device__ __forceinline__ void dload(const C* base, int r0, int rows, int nrt, int g, int c,
                                      typename Mf<F>::V (&d)[MfShape<N>::NT]) {
  const int n = RT ? nrt : N;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = r0 + Mf<F>::row(g, p);
    const size_t rr = r < rows ? (size_t)r : 0;
    if constexpr (MfShape<N>::wide) {
      C v = base[rr * n + (!RT || c < n ? c : 0)];
      d[0][p] = (F)v.x;
      d[1][p] = (F)v.y;
    } else {
      d[0][p] = (F)((const decltype(C().x)*)base)[rr * 2 * N + 2 * (c % N) + c / N];
    }
  }
}

template <int N, bool RT, typename F, typename C>
__device__ __forceinline__ void dstore(C* base, int r0, int rows, int nrt, int g, int c,
                                       const typename Mf<F>::V (&d)[MfShape<N>::NT]) {
  using R = decltype(C().x);
  const int n = RT ? nrt : N;
  const bool whole = r0 + 16 <= rows;  // the same for the wave: no lane masks
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = r0 + Mf<F>::row(g, p);
    if (!whole && r >= rows) continue;
    if constexpr (MfShape<N>::wide) {
      C v;
      v.x = (R)d[0][p];
      v.y = (R)d[1][p];
      if (!RT || c < n) base[(size_t)r * n + c] = v;
    } else {
      ((R*)base)[(size_t)r * 2 * N + 2 * (c % N) + c / N] = (R)d[0][p];
    }
  }
}

// Longest window of the deferred shift update whose coefficients (2 x window
// complex n x n matrices of one shift) the kernel stages in LDS: 32 KiB at
// n = 16 in either precision.
template <typename F>
struct MfWin {
  static constexpr int MW = sizeof(F) == 8 ? 4 : 8;
};

// The shifts whose window this update applies (by lane, as a mask), and those of them
// that k_update_close takes when it follows: windows of two iterations and more, if there
// are kCloseMin of them at least (it reads Q_k and Q_{k+1} once more than k_update_mfma;
// at 32^4, n = 16, one launch against the two: 2.15 and 1.92 ms in FP64, 1.65 and 1.59 in
// FP32 with three such windows).
constexpr int kCloseMin = 3;
__device__ __forceinline__ unsigned long long windows_due(const SolverFlags* fl, int ns,
                                                          int closing,
                                                          unsigned long long& late) {
  const int lane = threadIdx.x & 63, slot = fl->iter & 1;
  const int j = lane < ns ? fl->win_j[slot][lane] : 0;
  const bool due = j > 0 && (fl->win_flush[slot][lane] || fl->stop);
  late = __ballot(due && closing && j > 1);
  if (__popcll(late) < kCloseMin) late = 0;
  return __ballot(due);
}

// F: block and shift-update arithmetic type (double, or float in the mixed
// solver). NTILE: 16-row tiles per wave (processed one after the other inside
// each shift).
//
// The Q step reads Q_k from ring buffer k % win and writes Q_{k+1} to
// buffer (k+1) % win (in place for win = 1). Then every shift whose update
// window the small step closed (or, when the solve stops here, every open
// one) is applied, with j iterations in its window:
//   X += P Cx + sum_{i < j-1} Q_{k-j+2+i} Ex_i
//   P  = Q_{k+1} + P Cp + sum_{i < j-1} Q_{k-j+2+i} Ep_i     (in place)
// (sigma_0: j = 1 every iteration, the plain X += P Mx, P = Q + P Mp). At the widths known
// at run time the sums run from Q_k down and take P last: a shift far above sigma_0 is nearly
// solved by its first iteration, so P Cx is as large as X and the other terms are small, and
// taken first it had every later term rounded at its size (FP32 blocks, n = 12, a shift of
// 10: error 1.2e-7 updated every iteration, 3.2e-7 so, 1.2e-7 from Q_k down). A
// shift moves 4 block vectors per window instead of 4 per iteration; the
// ring buffers it also reads are the same for every shift, so after the
// first shift of a tile they come from L2.
// One tile per wave: four waves per SIMD in FP32, three in FP64 (the register
// count the compiler picks by itself leaves fewer; in FP64 four waves need
// spills, whose scratch traffic reached HBM).
// RT: the width is a.n (9 .. 15, at most N), else N. Measured at 16^4 with
// 12 shifts, FP64, k_update_close included, against the every-iteration vector kernel, us per
// iteration: n = 9 265 -> 87, n = 12 354 -> 77 to 84, n = 14 501 -> 115.
// gridDim.y: the shifts are dealt to that many groups of work-groups (shift s to
// group s % gridDim.y), which all form Q_{k+1} and of which the first stores
// it; more than one only with a ring (win > 1), where nothing is overwritten.
template <typename F, int N, int NTILE, bool RT>
__global__ __launch_bounds__(BMS_WG)
__attribute__((amdgpu_waves_per_eu(
    NTILE == 1 ? (sizeof(F) == 4 ? 4 : 3) : 1)))
void k_update_mfma(UpdateArgs<F, F> a) {
  using S = MfShape<N>;
  using CF = cplx<F>;
  using VF = typename Mf<F>::V;
  constexpr int MW = MfWin<F>::MW;
  constexpr bool DOWN = RT;  // the order of a window's sums, see above
  // LDS: the Q step's two coefficient matrices (FP64), then (FP32) the
  // per-wave layout change of Q, then one shift's window coefficients (F); each
  // copied region in whole KiB, and a matrix row's worth past the last one
  // (output columns past the width read there)
  constexpr int QREG = (N * N * 16 + 1023) / 1024 * 1024;
  constexpr int SREG = (MW * N * N * (int)sizeof(CF) + 1023) / 1024 * 1024;
  constexpr int TBYTES = MF_WAVES * NTILE * 16 * S::PITCH * 8;
  constexpr int CBYTES = 2 * (QREG > SREG ? QREG : SREG) + 256;
  constexpr int LBYTES = CBYTES > TBYTES ? CBYTES : TBYTES;
  __shared__ __align__(16) unsigned char lds[LBYTES];
  const double* qb0 = (const double*)lds;           // rho^-1
  const double* qb1 = (const double*)(lds + QREG);  // -alpha rho^-1
  SolverFlags* fl = a.flags;
  if (fl->halted) return;
  const int tid = threadIdx.x;
  const int iter = fl->iter;  // k + 1: the small step of iteration k has counted it
  const int stop = fl->stop;
  const int slot = iter & 1;
  const bool lead = blockIdx.y == 0;
  // the next small step and the drain read these (nothing else in this
  // kernel reads them)
  if (lead && blockIdx.x == 0 && tid == 0) {
    fl->upd_done = iter;
    fl->upd_stop = stop;
  }
  if (lead && blockIdx.x == 0 && tid < 64) log_update(fl, a.upd_log, a.max_iter, a.ns);
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int n = RT ? a.n : N, nn = n * n;
  const int rows = a.rows, ns = a.ns, win = a.win;
  const size_t blk = (size_t)rows * n;
  const int k = iter - 1;
  const CF* Qin = a.Qring + (size_t)(k % win) * blk;
  CF* Qout = a.Qring + (size_t)((k + 1) % win) * blk;
  const int tile0 = (blockIdx.x * MF_WAVES + wave) * NTILE;
  unsigned long long late;
  unsigned long long mask = windows_due(fl, ns, a.closing, late);
  mask &= ~late & __ballot(lane % gridDim.y == blockIdx.y);
  if (!lead && !mask) return;

  // coefficients of the Q step
  lds_copy(a.rhoinv, lds, nn * 16, wave, lane);
  lds_copy(a.arho, lds + QREG, nn * 16, wave, lane);
  double av[NTILE][S::KS], wv[NTILE][S::KS];
#pragma unroll
  for (int t = 0; t < NTILE; ++t) {
    const int r0 = (tile0 + t) * 16;
    aload<N, RT>(Qin, r0 + c, rows, n, g, av[t]);
    aload<N, RT>(a.W, r0 + c, rows, n, g, wv[t]);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  dx4 qd[NTILE][S::NT];
#pragma unroll
  for (int t = 0; t < NTILE; ++t) {
    if constexpr (S::wide) {
      constexpr int QACC = RT ? 2 : 3;
      dx4 d[QACC];
#pragma unroll
      for (int i = 0; i < QACC; ++i) d[i] = dx4{0.0, 0.0, 0.0, 0.0};
      mfma_wide<double, N, RT>(d, av[t], qb0, n, g, c);
      mfma_wide<double, N, RT>(d, wv[t], qb1, n, g, c);
      qd[t][0] = wide_re(d);
      qd[t][1] = wide_im(d);
    } else {
      qd[t][0] = dx4{0.0, 0.0, 0.0, 0.0};
      mfma_acc_c<N>(qd[t], av[t], qb0, g, c);
      mfma_acc_c<N>(qd[t], wv[t], qb1, g, c);
    }
  }
  // every lane of the wave has read its Q tiles before any is overwritten
  // (win = 1: Q_{k+1} replaces Q_k in place)
  if (lead) {
#pragma unroll
    for (int t = 0; t < NTILE; ++t)
      dstore<N, RT, double>(Qout, (tile0 + t) * 16, rows, n, g, c, qd[t]);
  }
  __syncthreads();  // the Q-step LDS is reused below
  // Q_{k+1} in the shift-update layout and precision: the same registers in
  // FP64; in FP32 rounded and moved to the f32 row mapping through LDS
  VF qn[NTILE][S::NT];
  if constexpr (sizeof(F) == 8) {
#pragma unroll
    for (int t = 0; t < NTILE; ++t)
#pragma unroll
      for (int nt = 0; nt < S::NT; ++nt) qn[t][nt] = qd[t][nt];
  } else {
    double* tq = (double*)lds + wave * (NTILE * 16 * S::PITCH);
#pragma unroll
    for (int t = 0; t < NTILE; ++t)
#pragma unroll
      for (int nt = 0; nt < S::NT; ++nt)
#pragma unroll
        for (int p = 0; p < 4; ++p)
          tq[(t * 16 + Mf<double>::row(g, p)) * S::PITCH + nt * 16 + c] = qd[t][nt][p];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NTILE; ++t)
#pragma unroll
      for (int nt = 0; nt < S::NT; ++nt)
#pragma unroll
        for (int p = 0; p < 4; ++p)
          qn[t][nt][p] = (F)tq[(t * 16 + Mf<F>::row(g, p)) * S::PITCH + nt * 16 + c];
    __syncthreads();  // the shift coefficients overwrite this LDS
  }

  // the first A operand (P, or from Q_k down that) and X tiles of a shift (the next
  // shift's first operand, and for n = 8 its X, are loaded while the current one finishes;
  // for n > 8 X is loaded after the products, which keeps the three-accumulator form at
  // three waves per SIMD with 20 bytes of spills outside the product loop)
  F pa[NTILE][S::KS];
  VF xa[NTILE][S::NT];
  auto window = [&](int s) { return __builtin_amdgcn_readfirstlane(fl->win_j[slot][s]); };
  auto fetch = [&](int s, int t) {
    const int r0 = (tile0 + t) * 16;
    aload<N, RT>(DOWN && window(s) > 1 ? Qin : a.P + (size_t)s * blk, r0 + c, rows, n, g, pa[t]);
    if constexpr (!S::wide) dload<N, RT, F>(a.X + (size_t)a.xidx[s] * blk, r0, rows, n, g, c, xa[t]);
  };
  int s = mask ? __ffsll((long long)mask) - 1 : -1;
  if (s >= 0) {
#pragma unroll
    for (int t = 0; t < NTILE; ++t) fetch(s, t);
  }
  const size_t fam = (size_t)BMS_MAX_WIN * nn;  // one family in Wm
  while (s >= 0) {
    mask &= mask - 1;
    const int s2 = mask ? __ffsll((long long)mask) - 1 : -1;
    const int j = window(s);
    // the window's 2j coefficient matrices into LDS (complex n x n, the X
    // family, then the P family)
    const CF* wm = a.Wm + (size_t)s * 2 * fam;
    lds_copy(wm, lds, j * nn * (int)sizeof(CF), wave, lane);
    lds_copy(wm + fam, lds + SREG, j * nn * (int)sizeof(CF), wave, lane);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const F* bx = (const F*)lds;
    const F* bp = (const F*)(lds + SREG);
    CF* X = a.X + (size_t)a.xidx[s] * blk;
    CF* P = a.P + (size_t)s * blk;
#pragma unroll
    for (int t = 0; t < NTILE; ++t) {
      const int r0 = (tile0 + t) * 16;
      constexpr int NACC = S::wide ? 3 : S::NT;  // accumulators of one product family
      VF pn[NACC], dx[NACC];
#pragma unroll
      for (int nt = 0; nt < NACC; ++nt) {
        pn[nt] = (S::wide || nt >= S::NT) ? VF{0, 0, 0, 0} : qn[t][nt];
        dx[nt] = VF{0, 0, 0, 0};
      }
      // the increment is formed on its own and added to X once, so X (large
      // next to one window's increment) is rounded once
      auto prod = [&](const F(&av)[S::KS], int m) {
        if constexpr (S::wide) {
          mfma_wide<F, N, RT>(dx, av, bx + m * 2 * nn, n, g, c);
          mfma_wide<F, N, RT>(pn, av, bp + m * 2 * nn, n, g, c);
        } else {
          mfma_acc_c<N>(dx, av, bx + m * 2 * nn, g, c);
          mfma_acc_c<N>(pn, av, bp + m * 2 * nn, g, c);
        }
      };
      // P and the ring buffers Q_{k-j+2} .. Q_k, two in flight
      F qa[2][S::KS];
      if constexpr (DOWN) {
        // (the first, Q_k or for j = 1 P, is there)
        auto load = [&](int m, F(&av)[S::KS]) {
          aload<N, RT>(m ? a.Qring + (size_t)((k - j + 1 + m) % win) * blk : P, r0 + c, rows, n, g,
                       av);
        };
#pragma unroll
        for (int i = 0; i < MW; ++i) {
          if (i < j) {
            F(&av)[S::KS] = i & 1 ? qa[0] : pa[t];
            if (i + 1 < j) load(j - 2 - i, i & 1 ? pa[t] : qa[0]);
            prod(av, j - 1 - i);
          }
        }
      } else {
        auto ring = [&](int i) { return a.Qring + (size_t)((k - j + 2 + i) % win) * blk; };
        if (j >= 2) aload<N, RT>(ring(0), r0 + c, rows, n, g, qa[0]);
        prod(pa[t], 0);
#pragma unroll
        for (int i = 0; i < MW - 1; ++i) {
          if (i < j - 1) {
            if (i + 1 < j - 1) aload<N, RT>(ring(i + 1), r0 + c, rows, n, g, qa[(i + 1) & 1]);
            prod(qa[i & 1], i + 1);
          }
        }
      }
      if constexpr (S::wide) {
        dload<N, RT, F>(X, r0, rows, n, g, c, xa[t]);
        xa[t][0] += wide_re(dx);
        xa[t][1] += wide_im(dx);
        const VF pst[S::NT] = {qn[t][0] + wide_re(pn), qn[t][1] + wide_im(pn)};
        dstore<N, RT, F>(X, r0, rows, n, g, c, xa[t]);
        dstore<N, RT, F>(P, r0, rows, n, g, c, pst);
      } else {
#pragma unroll
        for (int nt = 0; nt < S::NT; ++nt) xa[t][nt] += dx[nt];
        dstore<N, RT, F>(X, r0, rows, n, g, c, xa[t]);
        dstore<N, RT, F>(P, r0, rows, n, g, c, pn);
      }
      if (s2 >= 0) fetch(s2, t);
    }
    s = s2;
    __syncthreads();  // every wave is done with this shift's coefficients
  }
}

// Rows r0 .. r0 + 15 of a block as a buffer: accesses past the last row read zero and
// store nothing, so no access of the kernel below sits behind a branch. The waits for
// loads in flight are counted in order with the stores, and a store that may not be
// there would have to be waited for with the next load.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* base, int r0, int rows,
                                                            int rowbytes) {
  const int left = rows - r0;
  const int nr = left < 0 ? 0 : (left < 16 ? left : 16);
  const size_t p = (size_t)base + (size_t)(nr ? r0 : 0) * rowbytes;
  const size_t lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)p);
  const size_t hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(p >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(hi << 32 | lo), 0,
                                           __builtin_amdgcn_readfirstlane(nr * rowbytes),
                                           0x00027000);
}
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));

// aload, dload and dstore on such a tile
template <int N, typename F>
__device__ __forceinline__ void aload_b(__amdgpu_buffer_rsrc_t t, int g, int c,
                                        F (&a)[MfShape<N>::KS]) {
  constexpr int B = MfShape<N>::KS * (int)sizeof(F);  // bytes of a lane's run
  typedef F fv __attribute__((ext_vector_type(16 / sizeof(F))));
#pragma unroll
  for (int h = 0; h < B / 16; ++h) {
    const fv v = __builtin_bit_cast(
        fv, __builtin_amdgcn_raw_buffer_load_b128(t, (4 * c + g) * B + 16 * h, 0, 0));
#pragma unroll
    for (int e = 0; e < (int)(16 / sizeof(F)); ++e) a[h * (int)(16 / sizeof(F)) + e] = v[e];
  }
  if constexpr (B % 16 == 8) {  // FP32 at N = 12
    typedef F f2 __attribute__((ext_vector_type(2)));
    const f2 v = __builtin_bit_cast(
        f2, __builtin_amdgcn_raw_buffer_load_b64(t, (4 * c + g) * B + B - 8, 0, 0));
    a[MfShape<N>::KS - 2] = v[0];
    a[MfShape<N>::KS - 1] = v[1];
  }
}
template <int N, typename F>
__device__ __forceinline__ void dload_b(__amdgpu_buffer_rsrc_t t, int g, int c,
                                        typename Mf<F>::V (&d)[MfShape<N>::NT]) {
  typedef F f2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int o = Mf<F>::row(g, p) * 2 * N * (int)sizeof(F);
    if constexpr (MfShape<N>::wide) {
      f2 v;
      if constexpr (sizeof(F) == 8)
        v = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b128(t, o + c * 16, 0, 0));
      else
        v = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(t, o + c * 8, 0, 0));
      d[0][p] = v.x;
      d[1][p] = v.y;
    } else {
      const int oc = o + (2 * (c % N) + c / N) * (int)sizeof(F);
      if constexpr (sizeof(F) == 8)
        d[0][p] = __builtin_bit_cast(F, __builtin_amdgcn_raw_buffer_load_b64(t, oc, 0, 0));
      else
        d[0][p] = __builtin_bit_cast(F, __builtin_amdgcn_raw_buffer_load_b32(t, oc, 0, 0));
    }
  }
}
template <int N, typename F>
__device__ __forceinline__ void dstore_b(__amdgpu_buffer_rsrc_t t, int g, int c,
                                         const typename Mf<F>::V (&d)[MfShape<N>::NT]) {
  typedef F f2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    // (N = 12: the lanes of columns past 11 store out of range)
    const int o = MfShape<N>::wide && N < 16 && c >= N
                      ? 1 << 30
                      : Mf<F>::row(g, p) * 2 * N * (int)sizeof(F);
    if constexpr (MfShape<N>::wide) {
      const f2 v = {d[0][p], d[1][p]};
      if constexpr (sizeof(F) == 8)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), t, o + c * 16, 0, 0);
      else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), t, o + c * 8, 0, 0);
    } else {
      const int oc = o + (2 * (c % N) + c / N) * (int)sizeof(F);
      const F v = d[0][p];
      if constexpr (sizeof(F) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), t, oc, 0, 0);
      else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), t, oc, 0, 0);
    }
  }
}

// The windows that an update closes together (usually those of every shift but sigma_0),
// after the launch above has formed Q_{k+1}; same products, same order of sums, same bits (at
// n = 12 but for the rounding of adding P's terms).
//
// In k_update_mfma each shift reads the ring tiles again (3 or 7 loads of a wave against
// one each of P and X), 64 rows share a copy of the coefficients, and every wave waits for
// these between shifts. Here a work-group of eight waves holds its 128 rows' ring tiles in
// LDS for all shifts, and the coefficients of the next shift (in registers, then the other
// half of their LDS buffer), its P tile and this shift's X are in flight while a shift is
// computed. That fills the LDS of a compute unit at n = 16 (64 KiB coefficients, 96 KiB
// ring; in FP32 Q_k stays in registers), so one work-group per compute unit walks the row
// blocks. What bounds it then: HBM in FP64 (X and P of every shift read and written, 4.3 TB/s
// of about 4.7), the matrix cores in FP32 (eight products a tile and window). Measured at
// 32^4, n = 16, 20 shifts, full windows, both launches: FP64 9.8 -> 7.8 ms, FP32 8.0 -> 6.7;
// at 16^4, n = 8, 16 shifts: FP64 268 -> 168 us, FP32 no gain (160 and 163: not taken); n = 12,
// 15 shifts, 12 x 14 x 10 x 24 and 16^4: FP64 272 -> 196 and 398 -> 291 us, FP32 203 -> 185 and
// 347 -> 289.
// Slower: the window's products unrolled (FP64 8.0, FP32 7.3), LDS operands read a product
// ahead (FP32 7.2).
template <typename F, int N>
__global__ __launch_bounds__(CL_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
void k_update_close(UpdateArgs<F, F> a) {
  using S = MfShape<N>;
  using CF = cplx<F>;
  using VF = typename Mf<F>::V;
  constexpr int MW = MfWin<F>::MW;
  constexpr bool DOWN = N == 12;  // sums as k_update_mfma of that width adds them
  // Q_k (whose A operand costs FP32 only N / 2 registers) stays in registers in FP32
  constexpr bool QREG = sizeof(F) == 4;
  constexpr int LR = QREG ? MW - 2 : MW - 1;        // ring tiles of a wave in LDS
  constexpr int TB = 16 * N * (int)sizeof(CF);      // bytes of a tile
  constexpr int FAM = MW * N * N * (int)sizeof(CF); // bytes of one coefficient family
  constexpr int CPS = 2 * FAM / 16;                 // 16-byte pieces of a shift, and
  constexpr int CR = (CPS + CL_THREADS - 1) / CL_THREADS;  // of a thread
  // 16-byte units of a row; at a power of two they lie exchanged by the row in LDS, so that
  // the rows of a column do not meet on the same banks
  constexpr int UPR = N * (int)sizeof(CF) / 16;
  constexpr bool SWZ = (UPR & (UPR - 1)) == 0;
  constexpr int USH = UPR == 16 ? 0 : (UPR == 8 ? 1 : 2);
  constexpr int RB = N * (int)sizeof(CF);           // bytes of a row
  static_assert(FAM % 16 == 0 && (!SWZ || (UPR << USH) == 16) && TB % 256 == 0, "shape");
  __shared__ __align__(16) unsigned char lds[4 * FAM + CL_WAVES * LR * TB];
  const SolverFlags* fl = a.flags;
  if (fl->halted) return;
  unsigned long long all;
  windows_due(fl, a.ns, 1, all);
  if (!all) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int rows = a.rows, win = a.win, k = fl->iter - 1, slot = fl->iter & 1;
  const size_t blk = (size_t)rows * N;
  unsigned char* ring = lds + 4 * FAM + wave * (LR * TB);
  // lane s: the iterations in the window of shift s
  const int jl = lane < a.ns ? fl->win_j[slot][lane] : 0;
  auto wj = [&](int s) { return __builtin_amdgcn_readlane(jl, s); };
  int jmax = 0;
  for (unsigned long long m = all; m; m &= m - 1) jmax = max(jmax, wj(__ffsll((long long)m) - 1));

  // coefficients of a shift: loaded by all threads a shift ahead, written to the buffer
  // not in use when the shift before is done
  u4 cr[CR];
  auto cload = [&](int s) {
    const unsigned char* wm = (const unsigned char*)(a.Wm + (size_t)s * 2 * BMS_MAX_WIN * N * N);
#pragma unroll
    for (int u = 0; u < CR; ++u) {
      int q = u * CL_THREADS + tid;
      if (CPS % CL_THREADS && q >= CPS) q = 0;
      const int f = q / (FAM / 16), o = (q % (FAM / 16)) * 16;
      cr[u] = *(const u4*)(wm + (size_t)f * (BMS_MAX_WIN * N * N * sizeof(CF)) + o);
    }
  };
  auto cstore = [&](int b) {
#pragma unroll
    for (int u = 0; u < CR; ++u)
      if (CPS % CL_THREADS == 0 || u * CL_THREADS + tid < CPS)
        *(u4*)(lds + b * 2 * FAM + (u * CL_THREADS + tid) * 16) = cr[u];
  };
  const int sfirst = __ffsll((long long)all) - 1;
  int buf = 0, s = sfirst, j = wj(s);
  cload(s);
  cstore(0);
  __syncthreads();

  F pa[S::KS];
  aload_b<N>(tile_rsrc(a.P + (size_t)s * blk, (blockIdx.x * CL_WAVES + wave) * 16, rows, RB), g, c,
             pa);
  const int nblk = (rows + 16 * CL_WAVES - 1) / (16 * CL_WAVES);
  for (int tb = blockIdx.x; tb < nblk; tb += gridDim.x) {
    const int r0 = (tb * CL_WAVES + wave) * 16;
    // the ring tiles Q_{k-m}, straight to LDS; rows past the end read row 0 (their results
    // are not stored)
    for (int m = QREG ? 1 : 0; m <= jmax - 2; ++m) {
      const unsigned char* q = (const unsigned char*)(a.Qring + (size_t)((k - m) % win) * blk);
#pragma unroll
      for (int i = 0; i < (TB + 1023) / 1024; ++i) {
        const int x = i * 64 + lane, r = x / UPR;
        const int u = SWZ ? (x % UPR) ^ ((r >> USH) & (UPR - 1)) : x % UPR;
        const size_t row = r0 + r < rows ? r0 + r : 0;
        if (TB % 1024 == 0 || x * 16 < TB) __builtin_amdgcn_global_load_lds(
            (glob_void*)(q + row * (N * sizeof(CF)) + u * 16),
            (lds_void*)(ring + (m - (QREG ? 1 : 0)) * TB + i * 1024), 16, 0, 0);
      }
    }
    F qk[QREG ? S::KS : 1];
    if constexpr (QREG)
      aload_b<N>(tile_rsrc(a.Qring + (size_t)(k % win) * blk, r0, rows, RB), g, c, qk);
    VF qn[S::NT];
    dload_b<N, F>(tile_rsrc(a.Qring + (size_t)((k + 1) % win) * blk, r0, rows, RB), g, c, qn);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    unsigned long long mask = all;
    while (mask) {
      mask &= mask - 1;
      const int s2 = mask ? __ffsll((long long)mask) - 1 : sfirst, j2 = wj(s2);
      cload(s2);
      const __amdgpu_buffer_rsrc_t X = tile_rsrc(a.X + (size_t)a.xidx[s] * blk, r0, rows, RB);
      const __amdgpu_buffer_rsrc_t P = tile_rsrc(a.P + (size_t)s * blk, r0, rows, RB);
      VF xa[S::NT];
      dload_b<N, F>(X, g, c, xa);
      const F* bx = (const F*)(lds + buf * 2 * FAM);
      const F* bp = (const F*)(lds + buf * 2 * FAM + FAM);
      constexpr int NACC = S::wide ? 3 : S::NT;
      VF pn[NACC], dx[NACC];
#pragma unroll
      for (int nt = 0; nt < NACC; ++nt) {
        pn[nt] = (S::wide || nt >= S::NT) ? VF{0, 0, 0, 0} : qn[nt];
        dx[nt] = VF{0, 0, 0, 0};
      }
      auto prod = [&](const F(&av)[S::KS], int m) {
        if constexpr (S::wide) {
          mfma_wide<F, N, false>(dx, av, bx + m * 2 * N * N, N, g, c);
          mfma_wide<F, N, false>(pn, av, bp + m * 2 * N * N, N, g, c);
        } else {
          mfma_acc_c<N>(dx, av, bx + m * 2 * N * N, g, c);
          mfma_acc_c<N>(pn, av, bp + m * 2 * N * N, g, c);
        }
      };
      auto rload = [&](int m, F(&av)[S::KS]) {
        const unsigned char* p = ring + (m - (QREG ? 1 : 0)) * TB + c * (N * sizeof(CF));
        if constexpr (SWZ) {
          typedef F fv __attribute__((ext_vector_type(16 / sizeof(F))));
#pragma unroll
          for (int h = 0; h < UPR / 4; ++h) {
            const fv v = *(const fv*)(p + (((g * (UPR / 4) + h) ^ ((c >> USH) & (UPR - 1))) * 16));
#pragma unroll
            for (int e = 0; e < (int)(16 / sizeof(F)); ++e)
              av[h * (int)(16 / sizeof(F)) + e] = v[e];
          }
        } else {
#pragma unroll
          for (int h = 0; h < S::KS / 2; ++h) {
            const CF v = ((const CF*)p)[g * (S::KS / 2) + h];
            av[2 * h] = v.x;
            av[2 * h + 1] = v.y;
          }
        }
      };
      const int rn = mask ? r0 : r0 + (int)gridDim.x * CL_WAVES * 16;
      // the P tile of the next shift, or of the first shift of the next rows, takes this
      // one's registers (DOWN: so P's products come first all the same, but into sums of
      // their own that are added to the others at the end)
      const __amdgpu_buffer_rsrc_t Pn = tile_rsrc(a.P + (size_t)s2 * blk, rn, rows, RB);
      prod(pa, 0);
      aload_b<N>(Pn, g, c, pa);
      VF xp[NACC];
      if constexpr (DOWN) {
#pragma unroll
        for (int i = 0; i < NACC; ++i) {
          xp[i] = dx[i];
          dx[i] = VF{0, 0, 0, 0};
        }
        if constexpr (QREG) prod(qk, j - 1);
        for (int m = QREG ? 1 : 0; m <= j - 2; ++m) {
          F qa[S::KS];
          rload(m, qa);
          prod(qa, j - 1 - m);
        }
#pragma unroll
        for (int i = 0; i < NACC; ++i) dx[i] += xp[i];
      } else {
        for (int m = j - 2; m >= (QREG ? 1 : 0); --m) {
          F qa[S::KS];
          rload(m, qa);
          prod(qa, j - 1 - m);
        }
        if constexpr (QREG) prod(qk, j - 1);
      }
      if constexpr (S::wide) {
        xa[0] += wide_re(dx);
        xa[1] += wide_im(dx);
        const VF pst[S::NT] = {qn[0] + wide_re(pn), qn[1] + wide_im(pn)};
        dstore_b<N, F>(X, g, c, xa);
        dstore_b<N, F>(P, g, c, pst);
      } else {
#pragma unroll
        for (int nt = 0; nt < S::NT; ++nt) xa[nt] += dx[nt];
        dstore_b<N, F>(X, g, c, xa);
        dstore_b<N, F>(P, g, c, pn);
      }
      cstore(buf ^ 1);
      __syncthreads();
      buf ^= 1;
      s = s2;
      j = j2;
    }
  }
}

// The windowed update for 17 <= n <= 32 (N = 24 or 32): the products as in k_update_mfma, the
// output columns in two halves of 16. The window's coefficients (up to 128 KiB at n = 32) pass
// through LDS one iteration at a time, X and P family together; two work-groups share a
// compute unit, and one computes while the other waits for its copy. Columns past n meet a
// zero A operand, output columns past n are not used. On the matrix cores 2 x 2 x 3 N / 4
// steps (FP32 2 x 2 x N) of 16 x 16 x 4 a tile, iteration and shift; X and P are moved once per window, where
// the vector kernel for any n, which this replaces, moved them every iteration. Measured at
// 16^4, 12 shifts none of which converges, FP64, per iteration: n = 32 1484 -> 403 us, n = 24
// 1028 -> 287 (FP32 897 -> 175).
template <typename F, int N>
__global__ __launch_bounds__(BMS_WG) __attribute__((amdgpu_waves_per_eu(2)))
void k_update_wide(UpdateArgs<F, F> a) {
  using S = MfShape<N>;
  using CF = cplx<F>;
  using VF = typename Mf<F>::V;
  constexpr int QREG = (N * N * 16 + 1023) / 1024 * 1024;               // an FP64 matrix
  constexpr int SREG = (N * N * (int)sizeof(CF) + 1023) / 1024 * 1024;  // one in F
  constexpr int TP = 64;                                                // reals of a tile's row
  constexpr int TBYTES = sizeof(F) == 4 ? MF_WAVES * 16 * TP * 8 : 0;
  constexpr int LBYTES = 2 * QREG + 512 > TBYTES ? 2 * QREG + 512 : TBYTES;
  __shared__ __align__(16) unsigned char lds[LBYTES];
  SolverFlags* fl = a.flags;
  if (fl->halted) return;
  const int tid = threadIdx.x;
  const int iter = fl->iter, stop = fl->stop, slot = iter & 1;
  const bool lead = blockIdx.y == 0;
  if (lead && blockIdx.x == 0 && tid == 0) {
    fl->upd_done = iter;
    fl->upd_stop = stop;
  }
  if (lead && blockIdx.x == 0 && tid < 64) log_update(fl, a.upd_log, a.max_iter, a.ns);
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int n = a.n, nn = n * n;
  const int rows = a.rows, win = a.win, k = iter - 1;
  const size_t blk = (size_t)rows * n;
  const CF* Qin = a.Qring + (size_t)(k % win) * blk;
  CF* Qout = a.Qring + (size_t)((k + 1) % win) * blk;
  const int r0 = (blockIdx.x * MF_WAVES + wave) * 16;
  unsigned long long late;
  unsigned long long mask = windows_due(fl, a.ns, 0, late) &
                            __ballot(lane % gridDim.y == blockIdx.y);
  if (!lead && !mask) return;

  lds_copy(a.rhoinv, lds, nn * 16, wave, lane);
  lds_copy(a.arho, lds + QREG, nn * 16, wave, lane);
  dx4 qd[2][2];  // [half][re, im]
  {
    double av[S::KS], wv[S::KS];
    aload<N, true>(Qin, r0 + c, rows, n, g, av);
    aload<N, true>(a.W, r0 + c, rows, n, g, wv);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      dx4 d[2] = {dx4{0.0, 0.0, 0.0, 0.0}, dx4{0.0, 0.0, 0.0, 0.0}};
      mfma_wide<double, N, true>(d, av, (const double*)lds + 32 * h, n, g, c);
      mfma_wide<double, N, true>(d, wv, (const double*)(lds + QREG) + 32 * h, n, g, c);
      qd[h][0] = wide_re(d);
      qd[h][1] = wide_im(d);
    }
  }
  // D layout of output half h: complex column 16 h + c of tile row Mf<>::row(g, p)
  auto put = [&](CF* base, int r, int h, double re, double im) {
    if (r < rows && 16 * h + c < n) {
      CF v;
      v.x = (F)re;
      v.y = (F)im;
      base[(size_t)r * n + 16 * h + c] = v;
    }
  };
  if (lead) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int p = 0; p < 4; ++p)
        put(Qout, r0 + Mf<double>::row(g, p), h, qd[h][0][p], qd[h][1][p]);
  }
  __syncthreads();  // the Q-step LDS is reused below
  VF qn[2][2];
  if constexpr (sizeof(F) == 8) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      qn[h][0] = qd[h][0];
      qn[h][1] = qd[h][1];
    }
  } else {
    double* tq = (double*)lds + wave * (16 * TP);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int p = 0; p < 4; ++p)
          tq[Mf<double>::row(g, p) * TP + h * 32 + i * 16 + c] = qd[h][i][p];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int p = 0; p < 4; ++p)
          qn[h][i][p] = (F)tq[Mf<F>::row(g, p) * TP + h * 32 + i * 16 + c];
  }

  const size_t fam = (size_t)BMS_MAX_WIN * nn;
  for (; mask; mask &= mask - 1) {
    const int s = __ffsll((long long)mask) - 1;
    const int j = __builtin_amdgcn_readfirstlane(fl->win_j[slot][s]);
    const CF* wm = a.Wm + (size_t)s * 2 * fam;
    CF* X = a.X + (size_t)a.xidx[s] * blk;
    CF* P = a.P + (size_t)s * blk;
    constexpr int ACC = sizeof(F) == 4 ? 2 : 3;
    VF dx[2][ACC], dp[2][ACC];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < ACC; ++i) {
        dx[h][i] = VF{0, 0, 0, 0};
        dp[h][i] = VF{0, 0, 0, 0};
      }
    for (int m = j - 1; m >= 0; --m) {
      __syncthreads();  // every wave is done with the matrices before
      lds_copy(wm + (size_t)m * nn, lds, nn * (int)sizeof(CF), wave, lane);
      lds_copy(wm + fam + (size_t)m * nn, lds + SREG, nn * (int)sizeof(CF), wave, lane);
      F av[S::KS];
      // the ring buffers Q_k .. Q_{k-j+2}, then P
      aload<N, true>(m == 0 ? P : a.Qring + (size_t)((k - j + 1 + m) % win) * blk, r0 + c, rows, n,
                     g, av);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        mfma_wide<F, N, true>(dx[h], av, (const F*)lds + 32 * h, n, g, c);
        mfma_wide<F, N, true>(dp[h], av, (const F*)(lds + SREG) + 32 * h, n, g, c);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const VF xr = wide_re(dx[h]), xi = wide_im(dx[h]);
      const VF pr = qn[h][0] + wide_re(dp[h]), pi = qn[h][1] + wide_im(dp[h]);
      CF x[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int r = r0 + Mf<F>::row(g, p);
        x[p] = X[(size_t)(r < rows ? r : 0) * n + (16 * h + c < n ? 16 * h + c : 0)];
      }
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int r = r0 + Mf<F>::row(g, p);
        if (r < rows && 16 * h + c < n) {
          x[p].x += xr[p];
          x[p].y += xi[p];
          X[(size_t)r * n + 16 * h + c] = x[p];
          CF v;
          v.x = pr[p];
          v.y = pi[p];
          P[(size_t)r * n + 16 * h + c] = v;
        }
      }
    }
  }
}

// After the last iteration: every update window still open (the solve ended
// without its update applying it) is applied to X,
//   X += P Cx + sum_{i < j-1} Q_{k-j+2+i} Ex_i
// with the FP64 window state of the last update that ran (k = its iteration).
// One thread per complex entry of a row block.
template <typename F>
__global__ __launch_bounds__(BMS_WG) void k_update_drain(UpdateArgs<F, F> a) {
  using CF = cplx<F>;
  const SolverFlags* fl = a.flags;
  const int u = fl->upd_done;
  if (u < 0 || fl->upd_stop) return;
  const int slot = u & 1, k = u - 1, win = a.win;
  const int n = a.n, ns = a.ns;
  const size_t blk = (size_t)a.rows * n, nn = (size_t)n * n;
  const size_t fam = (size_t)BMS_MAX_WIN * nn;
  const size_t e = (size_t)blockIdx.x * BMS_WG + threadIdx.x;
  if (e >= blk) return;
  const size_t row = e / n;
  const int col = (int)(e - row * n);
  for (int s = 0; s < ns; ++s) {
    const int j = fl->win_j[slot][s];
    if (j == 0 || fl->win_flush[slot][s]) continue;
    const double2* xf = a.wst + (size_t)(slot * ns + s) * 2 * fam;
    const CF* P = a.P + (size_t)s * blk + row * n;
    double2 acc = make_double2(0, 0);
    for (int i = j - 2; i >= 0; --i) {
      const CF* Q = a.Qring + (size_t)((k - j + 2 + i) % win) * blk + row * n;
      const double2* ex = xf + (size_t)(i + 1) * nn;
      for (int kk = 0; kk < n; ++kk) acc = cfma(to_d(Q[kk]), ex[(size_t)kk * n + col], acc);
    }
    for (int kk = 0; kk < n; ++kk) acc = cfma(to_d(P[kk]), xf[(size_t)kk * n + col], acc);
    CF* X = a.X + (size_t)a.xidx[s] * blk + e;
    *X = cadd(*X, from_d<CF>(acc));
  }
}

// The windowed update for n <= 7, where the 16-column tiles of the matrix cores would be
// mostly empty: a lane per (row, column), whole rows inside a wave (64 / N rows, so that
// a wave has read its rows of Q and P before it overwrites any). A lane reads whole rows
// of Q, W, P and the ring (the row's N lanes hit the same lines) and its column of the
// coefficients, the shift's from LDS; the ring rows stay in registers for all shifts.
// Memory bound on large blocks: per shift and window X and P are read and written once, as
// in k_update_mfma. On small ones latency bound, hence the shift groups.
// The sums run from Q_k down and take P last, as in k_update_mfma.
// Measured per launch against the every-iteration form: n = 4 at 8^4 with 12 shifts
// 18.0 -> 5.2 us, n = 1 at 4^4 with 8 shifts 4.5 -> 3.6 us.
// Waves per SIMD: what the registers of the ring leave, asked for where the compiler would
// take a few registers more (FP64 at 16^4, n = 5: 45 -> 41 us).
template <typename F, int N>
__global__ __launch_bounds__(BMS_WG)
__attribute__((amdgpu_waves_per_eu(
    sizeof(F) == 4 ? 1 : (N == 2 ? 6 : (N == 3 ? 5 : (N == 5 ? 4 : 1))))))
void k_update_vec(UpdateArgs<F, F> a) {
  using CF = cplx<F>;
  constexpr int MW = MfWin<F>::MW, RPW = 64 / N, NN = N * N;
  // X loaded after the ring products: its registers are what costs a wave per SIMD (n = 3
  // FP64 21.7 -> 19.5 us; at n = 6, where they fit, late loads cost 49 -> 61)
  constexpr bool XLATE = sizeof(F) == 8 && (N == 3 || N == 5);
  __shared__ CF cf[2][MW * NN];  // one shift's window coefficients: X family, P family
  SolverFlags* fl = a.flags;
  if (fl->halted) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int iter = fl->iter, stop = fl->stop, slot = iter & 1;
  const bool lead = blockIdx.y == 0;
  if (lead && blockIdx.x == 0 && tid == 0) {
    fl->upd_done = iter;
    fl->upd_stop = stop;
  }
  if (lead && blockIdx.x == 0 && tid < 64) log_update(fl, a.upd_log, a.max_iter, a.ns);
  const int rows = a.rows, ns = a.ns, win = a.win, k = iter - 1;
  unsigned long long mask =
      __ballot(lane < ns && lane % gridDim.y == blockIdx.y && fl->win_j[slot][lane] > 0 &&
               (fl->win_flush[slot][lane] || stop));
  if (!lead && !mask) return;
  const size_t blk = (size_t)rows * N;
  const int lr = lane / N, col = lane - lr * N;
  const int row = (blockIdx.x * MF_WAVES + wave) * RPW + lr;
  const bool live = lr < RPW && row < rows;
  const size_t ro = live ? (size_t)row * N : 0;  // dead lanes read row 0 and write nothing
  // Q_{k+1} = Q_k rho^-1 + W (-alpha rho^-1), in FP64
  const CF* Qin = a.Qring + (size_t)(k % win) * blk + ro;
  double2 q = make_double2(0, 0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    q = cfma(to_d(Qin[i]), a.rhoinv[i * N + col], q);
    q = cfma(to_d(a.W[ro + i]), a.arho[i * N + col], q);
  }
  const CF qn = from_d<CF>(q);
  if (lead && live) a.Qring[(size_t)((k + 1) % win) * blk + ro + col] = qn;
  CF ring[MW - 1][N];
  int jr = 1;  // window length the ring rows are loaded for (1: none)
  const size_t fam = (size_t)BMS_MAX_WIN * NN;
  while (mask) {
    const int s = __ffsll((long long)mask) - 1;
    mask &= mask - 1;
    const int j = __builtin_amdgcn_readfirstlane(fl->win_j[slot][s]);
    CF* P = a.P + (size_t)s * blk + ro;
    CF* X = a.X + (size_t)a.xidx[s] * blk + ro + col;
    CF p[N];
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = P[i];
    CF x;
    if (!XLATE) x = *X;
    const CF* wm = a.Wm + (size_t)s * 2 * fam;
    for (int e = tid; e < j * NN; e += BMS_WG) {
      cf[0][e] = wm[e];
      cf[1][e] = wm[fam + e];
    }
    if (j > 1 && j != jr) {
#pragma unroll
      for (int m = 0; m < MW - 1; ++m)
        if (m < j - 1) {
          const CF* Q = a.Qring + (size_t)((k - j + 2 + m) % win) * blk + ro;
#pragma unroll
          for (int i = 0; i < N; ++i) ring[m][i] = Q[i];
        }
      jr = j;
    }
    __syncthreads();
    // the increment is formed on its own and added to X once
    CF dx = czero<CF>(), pn = qn;
#pragma unroll
    for (int m = MW - 2; m >= 0; --m)
      if (m < j - 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
          dx = cfma(ring[m][i], cf[0][(m + 1) * NN + i * N + col], dx);
          pn = cfma(ring[m][i], cf[1][(m + 1) * NN + i * N + col], pn);
        }
      }
    if (XLATE) x = *X;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      dx = cfma(p[i], cf[0][i * N + col], dx);
      pn = cfma(p[i], cf[1][i * N + col], pn);
    }
    if (live) {
      *X = cadd(x, dx);
      P[col] = pn;
    }
    __syncthreads();  // every wave is done with this shift's coefficients
  }
}

// Groups the shifts of an update are dealt to: as many as bring the launch to about
// two work-groups per compute unit, so that a small lattice, whose rows alone leave most of
// the chip idle while each work-group walks its shifts one after the other, spreads the
// shifts too. Measured at 8^4, FP64, 16 shifts, full windows, one group and with this rule:
// n = 4 23.3 and 12.8 us, n = 8 49.9 and 20.2, n = 16 114 and 40.
template <typename F>
int shift_groups(const UpdateArgs<F, F>& a, int blocks) {
  if (a.win < 2) return 1;  // Q is updated in place
  return std::min(a.ns, std::max(1, 2 * a.num_cu / blocks));
}

template <typename F, int N, int NTILE, bool RT>
hipError_t launch_mf(hipStream_t st, const UpdateArgs<F, F>& a) {
  int tiles = (a.rows + 15) / 16;
  int waves = (tiles + NTILE - 1) / NTILE;
  int blocks = (waves + MF_WAVES - 1) / MF_WAVES;
  const dim3 grid(blocks, shift_groups(a, blocks));
  UpdateArgs<F, F> b = a;
  // where the rows alone fill the chip, the windows that close together go to their own
  // kernel (FP32 at n = 8: no gain)
  constexpr bool own = RT ? N == 12 : (N == 16 || sizeof(F) == 8);
  b.closing = own && a.n == N && a.win > 2 && grid.y == 1;
  k_update_mfma<F, N, NTILE, RT><<<grid, BMS_WG, 0, st>>>(b);
  if constexpr (own)
    if (b.closing) {
      // one work-group per compute unit (its LDS holds one at n = 16)
      const int nblk = (a.rows + 16 * CL_WAVES - 1) / (16 * CL_WAVES);
      k_update_close<F, N><<<std::min(nblk, a.num_cu), CL_THREADS, 0, st>>>(b);
    }
  return hipGetLastError();
}

template <typename F, int N>
hipError_t launch_wide(hipStream_t st, const UpdateArgs<F, F>& a) {
  const int blocks = ((a.rows + 15) / 16 + MF_WAVES - 1) / MF_WAVES;
  const dim3 grid(blocks, shift_groups(a, blocks));
  k_update_wide<F, N><<<grid, BMS_WG, 0, st>>>(a);
  return hipGetLastError();
}

template <typename F, int N>
hipError_t launch_vec(hipStream_t st, const UpdateArgs<F, F>& a) {
  constexpr int RPB = MF_WAVES * (64 / N);  // rows per work-group
  const int blocks = (a.rows + RPB - 1) / RPB;
  const dim3 grid(blocks, shift_groups(a, blocks));
  k_update_vec<F, N><<<grid, BMS_WG, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace

bool update_mfma_supported(int n) { return n == 8 || n == 16; }
bool update_windowed(int n) { return n <= 32; }

// (n > 16: the small step's share of a window grows with it, four iterations in FP32 too)
template <typename F>
int update_mfma_max_win(int n) {
  return n > 16 ? 4 : MfWin<F>::MW;
}

// two_tiles: two 16-row tiles per wave instead of one (n = 8 and 16)
template <typename F>
hipError_t launch_update_mfma(hipStream_t st, const UpdateArgs<F, F>& a, bool two_tiles) {
  switch (a.n) {
    case 1: return launch_vec<F, 1>(st, a);
    case 2: return launch_vec<F, 2>(st, a);
    case 3: return launch_vec<F, 3>(st, a);
    case 4: return launch_vec<F, 4>(st, a);
    case 5: return launch_vec<F, 5>(st, a);
    case 6: return launch_vec<F, 6>(st, a);
    case 7: return launch_vec<F, 7>(st, a);
    case 8: return two_tiles ? launch_mf<F, 8, 2, false>(st, a) : launch_mf<F, 8, 1, false>(st, a);
    case 16:
      return two_tiles ? launch_mf<F, 16, 2, false>(st, a) : launch_mf<F, 16, 1, false>(st, a);
    default:
      if (a.n > 32) return hipErrorInvalidValue;
      if (a.n > 16) return a.n <= 24 ? launch_wide<F, 24>(st, a) : launch_wide<F, 32>(st, a);
      return a.n <= 12 ? launch_mf<F, 12, 1, true>(st, a) : launch_mf<F, 16, 1, true>(st, a);
  }
}

template <typename F>
hipError_t launch_update_drain(hipStream_t st, const UpdateArgs<F, F>& a) {
  const size_t blk = (size_t)a.rows * a.n;
  k_update_drain<F><<<(unsigned)((blk + BMS_WG - 1) / BMS_WG), BMS_WG, 0, st>>>(a);
  return hipGetLastError();
}

template hipError_t launch_update_mfma<double>(hipStream_t, const UpdateArgs<double, double>&,
                                               bool);
template hipError_t launch_update_mfma<float>(hipStream_t, const UpdateArgs<float, float>&, bool);
template hipError_t launch_update_drain<double>(hipStream_t, const UpdateArgs<double, double>&);
template hipError_t launch_update_drain<float>(hipStream_t, const UpdateArgs<float, float>&);
template int update_mfma_max_win<double>(int);
template int update_mfma_max_win<float>(int);
