// Gauge-field kernels of an RHMC trajectory (the gauge part of the HMC
// Hamiltonian of Sec. II and its molecular dynamics, Sec. IV):
//   Wilson action   S_g = beta sum_{x, mu<nu} (1 - Re Tr U_mu nu(x) / 3),
//                   U_mu nu(x) = U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
//   gauge force     F^a = -dS_g/d omega^a for U_mu(x) -> exp(i omega^a T^a) U_mu(x),
//                   T^a = lambda_a / 2: with the staple sum A_mu(x) of the six
//                   plaquettes through the link, F^a = -(beta/3) Im Tr(T^a U A),
//                   added into the momenta as P += scale F
//   link update     U <- exp(i eps P^a T^a) U
//   kinetic energy  1/2 sum (P^a)^2
// Links U[mu][idx][3][3] complex128 (lexicographic idx, periodic), momenta
// P[mu][idx][8] float64. One thread per site or link; the two sums finish in
// the fixed-order partial-sum kernel, so they are reproducible.
#include <cmath>

#include "blas.h"
#include "links.h"

namespace {

__device__ __forceinline__ M3 ld(const double2* p) {
  M3 m;
#pragma unroll
  for (int k = 0; k < 9; ++k) m.e[k] = p[k];
  return m;
}

// a b, a b^dag
__device__ __forceinline__ M3 mm(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = make_double2(0, 0);
#pragma unroll
      for (int k = 0; k < 3; ++k) s = cfma(a.e[3 * i + k], b.e[3 * k + j], s);
      r.e[3 * i + j] = s;
    }
  return r;
}
__device__ __forceinline__ M3 mmd(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = make_double2(0, 0);
#pragma unroll
      for (int k = 0; k < 3; ++k) s = cfma(a.e[3 * i + k], cconj(b.e[3 * j + k]), s);
      r.e[3 * i + j] = s;
    }
  return r;
}
__device__ __forceinline__ double re_tr(const M3& a) { return a.e[0].x + a.e[4].x + a.e[8].x; }

struct Lat {
  int L[4];
  int stride[4];
  int vol;
};

__device__ __forceinline__ void coords(const Lat& g, int idx, int* c) {
  c[0] = idx % g.L[0];
  c[1] = (idx / g.L[0]) % g.L[1];
  c[2] = (idx / (g.L[0] * g.L[1])) % g.L[2];
  c[3] = idx / (g.L[0] * g.L[1] * g.L[2]);
}
// lexicographic index of the site k steps from c in direction mu (|k| <= L)
__device__ __forceinline__ int nbr(const Lat& g, int idx, const int* c, int mu, int k) {
  int v = c[mu] + k;
  int d = k;
  if (v < 0) d += g.L[mu];
  if (v >= g.L[mu]) d -= g.L[mu];
  return idx + d * g.stride[mu];
}
__device__ __forceinline__ const double2* lk(const double2* U, const Lat& g, int mu, int idx) {
  return U + ((size_t)mu * g.vol + idx) * 9;
}

__device__ __forceinline__ double block_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int s = BMS_WG / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  return red[0];
}

// per block: sum over its sites of sum_{mu<nu} (1 - Re Tr U_mu nu / 3)
__global__ __launch_bounds__(BMS_WG) void k_wilson(const double2* __restrict__ U, Lat g,
                                                   double2* __restrict__ partials) {
  __shared__ double red[BMS_WG];
  const int idx = blockIdx.x * BMS_WG + threadIdx.x;
  double acc = 0;
  if (idx < g.vol) {
    int c[4];
    coords(g, idx, c);
    for (int mu = 0; mu < 4; ++mu)
      for (int nu = mu + 1; nu < 4; ++nu) {
        const M3 a = mm(ld(lk(U, g, mu, idx)), ld(lk(U, g, nu, nbr(g, idx, c, mu, 1))));
        const M3 b = mm(ld(lk(U, g, nu, idx)), ld(lk(U, g, mu, nbr(g, idx, c, nu, 1))));
        acc += 1.0 - re_tr(mmd(a, b)) / 3.0;
      }
  }
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = make_double2(s, 0);
}

// Im Tr(T^a W) for the eight generators T^a = lambda_a / 2
__device__ __forceinline__ void im_tr_t(const M3& w, double* f) {
  const double2* e = w.e;
  f[0] = 0.5 * (e[3].y + e[1].y);
  f[1] = 0.5 * (-e[3].x + e[1].x);
  f[2] = 0.5 * (e[0].y - e[4].y);
  f[3] = 0.5 * (e[6].y + e[2].y);
  f[4] = 0.5 * (-e[6].x + e[2].x);
  f[5] = 0.5 * (e[7].y + e[5].y);
  f[6] = 0.5 * (-e[7].x + e[5].x);
  f[7] = 0.5 / sqrt(3.0) * (e[0].y + e[4].y - 2.0 * e[8].y);
}

// P[mu][x] += scale * F^a, F^a = -(beta/3) Im Tr(T^a U_mu(x) A_mu(x)).
// A link takes 19 links (18 of them in the six staples), and what bounds the kernel is the
// latency of fetching them. So three lanes share a link, lane i holding row i of every
// product (a row vector times the next factor, which it reads from LDS): with a third of the
// registers four waves per SIMD are resident instead of two, and a staple's three links are
// requested together, while the staple before is multiplied. A wave's 21 links are read as
// whole lines (as in links.h). Work-groups are dealt so that each XCD has one stretch of
// the lattice, the four directions of its sites one after the other: the staples' links
// then meet in its L2. Measured at 16^3 x 32: 197 us with a
// thread per link reading it from memory, 169 with a thread per link and whole lines, 110 so.
constexpr int GF_LINKS = 21;              // links per wave
constexpr int GF_SLOT = 3 * 64;           // LDS of one factor of a wave's links, complex
constexpr int GF_SITES = 4 * GF_LINKS;    // sites per work-group

struct GfBatch {
  double2 e[3][3];  // [factor][load]
};

__global__ __launch_bounds__(BMS_WG, 4) void k_gauge_force(const double2* __restrict__ U, Lat g,
                                                           double beta, double scale,
                                                           double* __restrict__ P) {
  __shared__ double2 stage[BMS_WG / 64][3 * GF_SLOT];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double2* lds = stage[wave];
  // work-group b runs on XCD b % 8
  const int xcd = blockIdx.x & 7, jb = blockIdx.x >> 3, mu = jb & 3;
  const int per = gridDim.x >> 5;  // chunks of GF_SITES sites per XCD
  const int ll = lane < 63 ? lane / 3 : GF_LINKS - 1, i = lane < 63 ? lane - 3 * (lane / 3) : 2;
  const int x0 = (xcd * per + (jb >> 2)) * GF_SITES + wave * GF_LINKS + ll;
  const bool live = x0 < g.vol && lane < 63;
  const int idx = x0 < g.vol ? x0 : g.vol - 1;  // past the end: a valid site, nothing written
  int c[4];
  coords(g, idx, c);
  auto step = [&](int at, int cnu, int nu, int k) {  // at's neighbour, its coordinate cnu
    const int v = cnu + k;
    return at + (v < 0 ? k + g.L[nu] : (v >= g.L[nu] ? k - g.L[nu] : k)) * g.stride[nu];
  };
  auto pick = [&](int nu) { return nu == 0 ? c[0] : (nu == 1 ? c[1] : (nu == 2 ? c[2] : c[3])); };
  // load k of a factor takes entry 63 k + lane of the wave's 189
  int from[3], ent[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int e = min(63 * k + lane, 9 * GF_LINKS - 1), j = (e * 7282) >> 16;  // e / 9
    from[k] = 3 * j;
    ent[k] = e - 9 * j;
  }
  auto fetch = [&](int link, double2 (&r)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) r[k] = wl_ld(U + (size_t)__shfl(link, from[k]) * 9 + ent[k]);
  };
  auto put = [&](const GfBatch& b) {
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        wl_st(lds + f * GF_SLOT + (lane < 63 ? 63 * k + lane : 9 * GF_LINKS + k), b.e[f][k]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  // factor f's entry (r, q) of this lane's link
  auto at = [&](int f, int r, int q) { return wl_ld(lds + f * GF_SLOT + 9 * ll + 3 * r + q); };
  const int cmu = pick(mu), xp = step(idx, cmu, mu, 1);
  // up: U_nu(x+mu), U_mu(x+nu), U_nu(x); down: U_nu(x+mu-nu), U_mu(x-nu), U_nu(x-nu)
  auto request = [&](int s, GfBatch& b) {  // s: staple 0 .. 5 (nu = mu + 1 + s / 2, up then down)
    const int nu = (mu + 1 + (s >> 1)) & 3;
    const int xn = step(idx, pick(nu), nu, s & 1 ? -1 : 1);
    fetch(nu * g.vol + (s & 1 ? step(xn, cmu, mu, 1) : xp), b.e[0]);
    fetch(mu * g.vol + xn, b.e[1]);
    fetch(nu * g.vol + (s & 1 ? xn : idx), b.e[2]);
  };
  double2 A[3] = {{0, 0}, {0, 0}, {0, 0}};
  GfBatch b;
  request(0, b);
#pragma unroll 1
  for (int s = 0; s < 6; ++s) {
    put(b);
    if (s < 5)
      request(s + 1, b);
    else
      fetch(mu * g.vol + idx, b.e[0]);
    __builtin_amdgcn_sched_barrier(0);
    double2 v[3], w[3];
    if (s & 1) {
      // row i of (U_mu(x-nu) U_nu(x+mu-nu))^dag U_nu(x-nu)
#pragma unroll
      for (int k = 0; k < 3; ++k) v[k] = cconj(at(0, k, i));
    } else {
      // row i of U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
#pragma unroll
      for (int k = 0; k < 3; ++k) v[k] = at(0, i, k);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      w[j] = make_double2(0, 0);
#pragma unroll
      for (int k = 0; k < 3; ++k) w[j] = cfma(v[k], cconj(at(1, j, k)), w[j]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        double2 m = at(2, s & 1 ? k : j, s & 1 ? j : k);
        m.y = s & 1 ? m.y : -m.y;
        A[j] = cfma(w[k], m, A[j]);
      }
    __builtin_amdgcn_sched_barrier(0);
  }
  // W = U A: row i from U's row i and the rows of A, then W whole in every lane
#pragma unroll
  for (int k = 0; k < 3; ++k) b.e[1][k] = b.e[2][k] = make_double2(0, 0);
  put(b);
  __builtin_amdgcn_wave_barrier();
  double2* own = lds + GF_SLOT + 9 * ll + 3 * i;
  if (lane < 63) {
#pragma unroll
    for (int k = 0; k < 3; ++k) wl_st(own + k, A[k]);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  double2 wr[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    wr[j] = make_double2(0, 0);
#pragma unroll
    for (int k = 0; k < 3; ++k) wr[j] = cfma(at(0, i, k), at(1, k, j), wr[j]);
  }
  if (lane < 63) {
#pragma unroll
    for (int k = 0; k < 3; ++k) wl_st(own + GF_SLOT + k, wr[k]);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (!live) return;
  M3 w;
#pragma unroll
  for (int e = 0; e < 9; ++e) w.e[e] = wl_ld(lds + 2 * GF_SLOT + 9 * ll + e);
  double f[8];
  im_tr_t(w, f);
  // lane i writes components i, i + 3, i + 6
  double* p = P + ((size_t)mu * g.vol + idx) * 8 + i;
  const double k = -scale * beta / 3.0;
  p[0] += k * (i == 0 ? f[0] : (i == 1 ? f[1] : f[2]));
  p[3] += k * (i == 0 ? f[3] : (i == 1 ? f[4] : f[5]));
  if (i < 2) p[6] += k * (i == 0 ? f[6] : f[7]);
}

// E = exp(i X) for traceless Hermitian X by scaling and squaring: Y = X / 2^s with
// |Y|_F <= 1/4, the Taylor series of exp(i Y) to order 16 (remainder below
// 4^-17 / 17!), then s squarings. Powers of Y reduce to 1, Y, Y^2 by the
// characteristic equation Y^3 = c1 Y + c0 (c1 = tr Y^2 / 2, c0 = det Y, both real), so the
// series is a recurrence of three real numbers and costs one matrix product.
__device__ __forceinline__ M3 exp_i(const M3& X) {
  double nf = 0;
#pragma unroll
  for (int k = 0; k < 9; ++k) nf += X.e[k].x * X.e[k].x + X.e[k].y * X.e[k].y;
  nf = sqrt(nf);
  int s = 0;
  while (nf > 0.25 && s < 60) {
    nf *= 0.5;
    ++s;
  }
  const double sc = ldexp(1.0, -s);
  M3 Y;
#pragma unroll
  for (int k = 0; k < 9; ++k) Y.e[k] = cscale(X.e[k], sc);
  const M3 Y2 = mm(Y, Y);
  const double c1 = 0.5 * re_tr(Y2);
  // det Y = Re sum over row 0 (real for Hermitian Y)
  double c0 = 0;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int b1 = (b + 1) % 3, b2 = (b + 2) % 3;
    const double2 m = csub(cmul(Y.e[3 + b1], Y.e[6 + b2]), cmul(Y.e[3 + b2], Y.e[6 + b1]));
    c0 += Y.e[b].x * m.x - Y.e[b].y * m.y;
  }
  // Y^j / j! = p + q Y + r Y^2, summed into the real (even j) and imaginary parts of the
  // coefficients with the signs of i^j
  double p = 1, q = 0, r = 0, fr[3] = {1, 0, 0}, fi[3] = {0, 0, 0};
#pragma unroll
  for (int j = 1; j <= 16; ++j) {
    const double inv = 1.0 / j, t = r;
    r = q * inv;
    q = fma(t, c1, p) * inv;
    p = t * c0 * inv;
    const double sg = (j >> 1) & 1 ? -1.0 : 1.0;
    double* f = j & 1 ? fi : fr;
    f[0] = fma(sg, p, f[0]);
    f[1] = fma(sg, q, f[1]);
    f[2] = fma(sg, r, f[2]);
  }
  M3 E;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 y = Y.e[k], z = Y2.e[k];
    double2 v = make_double2(k % 4 == 0 ? fr[0] : 0.0, k % 4 == 0 ? fi[0] : 0.0);
    v = cfma(make_double2(fr[1], fi[1]), y, v);
    E.e[k] = cfma(make_double2(fr[2], fi[2]), z, v);
  }
  for (int k = 0; k < s; ++k) E = mm(E, E);
  return E;
}

// two momenta of a link; a caller's P has the alignment of double
typedef double d2a8 __attribute__((ext_vector_type(2), aligned(8)));

// U_mu(x) <- exp(i eps P^a T^a) U_mu(x), one thread per link; bound by reading U and P and
// writing U once, the links as whole lines (links.h). Measured at 16^3 x 32: 56 -> 28 us
// (184 MB, most of it in the Infinity Cache).
__global__ __launch_bounds__(BMS_WG) void k_link_update(double2* __restrict__ U,
                                                        const double* __restrict__ P, int nlink,
                                                        double eps) {
  __shared__ double2 stage[BMS_WG / 64][WL_ENTRIES];
  double2* lds = stage[threadIdx.x >> 6];
  // 4 V links, V a multiple of 16: whole waves leave together
  const int t = blockIdx.x * BMS_WG + threadIdx.x;
  if (t >= nlink) return;
  // the wave's 64 links are one contiguous run: entry 64 k + lane of it in load k
  double2* u = U + (size_t)(t - (int)(threadIdx.x & 63)) * 9 + (threadIdx.x & 63);
  M3 m;
#pragma unroll
  for (int k = 0; k < 9; ++k) m.e[k] = wl_ld(u + 64 * k);
  double p[8];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const d2a8 v = ((const d2a8*)P)[(size_t)t * 4 + a];
    p[2 * a] = v.x;
    p[2 * a + 1] = v.y;
  }
  const double h = 0.5 * eps, r3 = 1.0 / sqrt(3.0);
  M3 X;
  X.e[0] = make_double2(h * (p[2] + r3 * p[7]), 0);
  X.e[4] = make_double2(h * (-p[2] + r3 * p[7]), 0);
  X.e[8] = make_double2(h * (-2.0 * r3 * p[7]), 0);
  X.e[1] = make_double2(h * p[0], -h * p[1]);
  X.e[3] = make_double2(h * p[0], h * p[1]);
  X.e[2] = make_double2(h * p[3], -h * p[4]);
  X.e[6] = make_double2(h * p[3], h * p[4]);
  X.e[5] = make_double2(h * p[5], -h * p[6]);
  X.e[7] = make_double2(h * p[5], h * p[6]);
  const M3 E = exp_i(X);
  const M3 n = wl_spread(mm(E, wl_own(m, lds)), lds);
#pragma unroll
  for (int k = 0; k < 9; ++k) wl_st(u + 64 * k, n.e[k]);
}

// per block: 1/2 sum of squares of its momenta
__global__ __launch_bounds__(BMS_WG) void k_kinetic(const double* __restrict__ P, size_t n,
                                                    double2* __restrict__ partials) {
  __shared__ double red[BMS_WG];
  double acc = 0;
  for (size_t i = (size_t)blockIdx.x * BMS_WG + threadIdx.x; i < n;
       i += (size_t)gridDim.x * BMS_WG)
    acc += P[i] * P[i];
  const double s = block_sum(0.5 * acc, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = make_double2(s, 0);
}

Lat lat_of(const bms_ctx* c) {
  Lat g;
  for (int i = 0; i < 4; ++i) g.L[i] = c->dims[i];
  g.stride[0] = 1;
  g.stride[1] = c->dims[0];
  g.stride[2] = c->dims[0] * c->dims[1];
  g.stride[3] = c->dims[0] * c->dims[1] * c->dims[2];
  g.vol = (int)c->vol;
  return g;
}

constexpr int kKineticBlocks = 1024;

// a one-entry grid reduction read back to the host
int reduce_to_host(bms_ctx* c, double2* partials, int nb, double* out) {
  void* o;
  int rc = scratch_buf(c, S_RES, 64, &o);
  if (rc) return rc;
  HIP_TRY(c, launch_sum_partials(c->stream, partials, nb, 1, (double2*)o, nullptr, nullptr));
  double2 h;
  HIP_TRY(c, hipMemcpyAsync(&h, o, sizeof h, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  *out = h.x;
  return BMS_OK;
}

}  // namespace

int gauge_action_dev(bms_ctx* c, double beta, const void* U, double* S) {
  const Lat g = lat_of(c);
  const int nb = (g.vol + BMS_WG - 1) / BMS_WG;
  void* pp;
  int rc = scratch_buf(c, S_PART, (size_t)nb * sizeof(double2) + 64, &pp);
  if (rc) return rc;
  k_wilson<<<nb, BMS_WG, 0, c->stream>>>((const double2*)U, g, (double2*)pp);
  HIP_TRY(c, hipGetLastError());
  double s;
  if ((rc = reduce_to_host(c, (double2*)pp, nb, &s))) return rc;
  *S = beta * s;
  return BMS_OK;
}

int gauge_force_dev(bms_ctx* c, double beta, const void* U, void* P, double scale) {
  const Lat g = lat_of(c);
  const int per = ((g.vol + GF_SITES - 1) / GF_SITES + 7) / 8;  // chunks of sites per XCD
  k_gauge_force<<<per * 32, BMS_WG, 0, c->stream>>>((const double2*)U, g, beta, scale, (double*)P);
  HIP_TRY(c, hipGetLastError());
  return BMS_OK;
}

int link_update_dev(bms_ctx* c, double eps, const void* P, void* U) {
  const int n = 4 * (int)c->vol;
  k_link_update<<<(n + BMS_WG - 1) / BMS_WG, BMS_WG, 0, c->stream>>>((double2*)U,
                                                                    (const double*)P, n, eps);
  HIP_TRY(c, hipGetLastError());
  return BMS_OK;
}

int kinetic_dev(bms_ctx* c, const void* P, double* K) {
  const size_t n = (size_t)4 * c->vol * 8;
  const int nb = (int)std::min<size_t>(kKineticBlocks, (n + BMS_WG - 1) / BMS_WG);
  void* pp;
  int rc = scratch_buf(c, S_PART, (size_t)nb * sizeof(double2) + 64, &pp);
  if (rc) return rc;
  k_kinetic<<<nb, BMS_WG, 0, c->stream>>>((const double*)P, n, (double2*)pp);
  HIP_TRY(c, hipGetLastError());
  return reduce_to_host(c, (double2*)pp, nb, K);
}

extern "C" int bms_gauge_action(bms_ctx* c, double beta, const void* U, double* S) {
  if (!c) return BMS_EINVAL;
  if (!U || !S) return set_err(c, BMS_EINVAL, "null pointer");
  if (!std::isfinite(beta)) return set_err(c, BMS_EINVAL, "beta not finite");
  int rc = user_stream_begin(c);
  if (rc) return rc;
  UserStream us(c);
  return gauge_action_dev(c, beta, U, S);
}

extern "C" int bms_gauge_force(bms_ctx* c, double beta, const void* U, void* P, double scale) {
  if (!c) return BMS_EINVAL;
  if (!U || !P) return set_err(c, BMS_EINVAL, "null pointer");
  if (!std::isfinite(beta) || !std::isfinite(scale))
    return set_err(c, BMS_EINVAL, "beta or scale not finite");
  int rc = user_stream_begin(c);
  if (rc) return rc;
  UserStream us(c);
  return gauge_force_dev(c, beta, U, P, scale);
}

extern "C" int bms_gauge_update(bms_ctx* c, double eps, const void* P, void* U) {
  if (!c) return BMS_EINVAL;
  if (!U || !P) return set_err(c, BMS_EINVAL, "null pointer");
  if (!std::isfinite(eps)) return set_err(c, BMS_EINVAL, "eps not finite");
  int rc = user_stream_begin(c);
  if (rc) return rc;
  UserStream us(c);
  return link_update_dev(c, eps, P, U);
}

extern "C" int bms_kinetic_energy(bms_ctx* c, const void* P, double* K) {
  if (!c) return BMS_EINVAL;
  if (!P || !K) return set_err(c, BMS_EINVAL, "null pointer");
  int rc = user_stream_begin(c);
  if (rc) return rc;
  UserStream us(c);
  return kinetic_dev(c, P, K);
}
