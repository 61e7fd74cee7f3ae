// Device-side Krylov scalars of the batched GMRES (declarations and the
// algorithm in dgmres.h).  The kernels of the scalars alone run one wavefront
// whose lane r serves system r of the batch; the fused steps for short vectors
// run one workgroup per system.
#include "dgmres.h"

namespace ddamg {

namespace {

__device__ inline double cabs2(double2 a) { return a.x * a.x + a.y * a.y; }
__device__ inline double cabs1(double2 a) { return hypot(a.x, a.y); }
__device__ inline double2 cneg(double2 a) { return make_double2(-a.x, -a.y); }
__device__ inline double2 cdiv(double2 a, double2 b) {
  const double d = b.x * b.x + b.y * b.y;
  return make_double2((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}

__global__ void k_gm_reset(long long* iters, int nb) {
  const int r = threadIdx.x;
  if (r < nb) iters[r] = 0;
}

// lane 0 stores whether any lane's predicate holds; called once by every
// lane of the wavefront, outside divergent code
__device__ inline void set_flag(int* flag, bool pred) {
  const unsigned long long any = __ballot(pred);
  if (threadIdx.x == 0) *flag = any != 0ull;
}

// the per-system bodies return the lane's part of the flag
__device__ inline bool gm_begin_body(DevGmres& d, int r, int m, double tol, int first) {
  GmSys& S = d.sys[r];
  const double beta = sqrt(fmax(d.res[(size_t)r * (KMAX + 1)].x, 0.0));
  if (first == 1) {
    S.target = tol * beta;
    S.active = beta > 0.0;
  } else if (first == 2) {
    S.active = S.active && isfinite(beta) && beta > S.target;
  } else {
    S.active = S.active && !S.conv && beta > 0.0;
  }
  S.conv = 0;
  S.live = S.active;
  S.jend = 0;
  // step j writes rows 0..j+1 of Hessenberg column j and g[j+1], so nothing
  // of an earlier cycle is read again
  S.g[0] = make_double2(S.active ? beta : 0.0, 0.0);
  d.scale[r] = S.active ? 1.0 / beta : 0.0;
  return S.active;
}

__global__ void k_gm_begin(DevGmres d, int m, int nb, double tol, int first) {
  const int r = threadIdx.x;
  const bool live = r < nb ? gm_begin_body(d, r, m, tol, first) : false;
  set_flag(d.flag, live);
}

__global__ void k_gm_cgs1(DevGmres d, int j, int nb) {
  const int r = threadIdx.x;
  if (r >= nb) return;
  GmSys& S = d.sys[r];
  const double2* h = d.res + (size_t)r * (KMAX + 1);
  const double ww = h[j + 1].x;
  double proj = 0;
  for (int i = 0; i <= j; ++i) {
    S.h1[i] = h[i];
    proj += cabs2(h[i]);
  }
  S.ww1 = ww;
  const int again = S.live && !(ww - proj > 0.5 * ww);
  S.again = again;
  for (int i = 0; i <= j; ++i) d.coef[(size_t)r * KMAX + i] = again ? cneg(h[i]) : make_double2(0.0, 0.0);
}

__device__ inline bool gm_step_body(DevGmres& d, int r, int j, int m) {
  GmSys& S = d.sys[r];
  double2* cf = d.coef + (size_t)r * KMAX;
  if (!S.live) {
    for (int i = 0; i <= j; ++i) cf[i] = make_double2(0.0, 0.0);
    d.scale[r] = 0.0;
    return false;
  }
  const double2* h2 = d.res + (size_t)r * (KMAX + 1);
  double proj = 0;
  for (int i = 0; i <= j; ++i) proj += cabs2(S.h1[i]);
  double hn = sqrt(fmax(S.ww1 - proj, 0.0));
  // Hessenberg column j (first pass, plus the second where it ran)
  double2* H = S.H;
  for (int i = 0; i <= j; ++i) {
    double2 hi = S.h1[i];
    if (S.again) hi = cadd(hi, h2[i]);
    H[(size_t)i * m + j] = hi;
    cf[i] = cneg(S.again ? h2[i] : S.h1[i]);
  }
  if (S.again) {
    double nn = h2[j + 1].x;
    for (int i = 0; i <= j; ++i) nn -= cabs2(h2[i]);
    hn = sqrt(fmax(nn, 0.0));
  }
  // Givens rotations of the earlier columns, then the new one
  H[(size_t)(j + 1) * m + j] = make_double2(hn, 0.0);
  for (int i = 0; i < j; ++i) {
    const double2 a = H[(size_t)i * m + j], bq = H[(size_t)(i + 1) * m + j];
    H[(size_t)i * m + j] = cadd(cmul(S.cs[i], a), cmul(S.sn[i], bq));
    H[(size_t)(i + 1) * m + j] = csub(cmul(S.cs[i], bq), cmul(cconj(S.sn[i]), a));
  }
  const double2 a = H[(size_t)j * m + j];
  const double aa = cabs1(a);
  const double rho = sqrt(cabs2(a) + hn * hn);
  if (rho == 0.0) {
    S.cs[j] = make_double2(1.0, 0.0);
    S.sn[j] = make_double2(0.0, 0.0);
  } else if (aa == 0.0) {
    S.cs[j] = make_double2(0.0, 0.0);
    S.sn[j] = make_double2(1.0, 0.0);
  } else {
    S.cs[j] = make_double2(aa / rho, 0.0);
    S.sn[j] = make_double2(a.x / aa * hn / rho, a.y / aa * hn / rho);
  }
  H[(size_t)j * m + j] = cadd(cmul(S.cs[j], a), cscale(S.sn[j], hn));
  H[(size_t)(j + 1) * m + j] = make_double2(0.0, 0.0);
  const double2 gj = S.g[j];
  S.g[j + 1] = cneg(cmul(cconj(S.sn[j]), gj));
  S.g[j] = cmul(S.cs[j], gj);
  const double est = cabs1(S.g[j + 1]);
  ++d.iters[r];
  S.jend = j + 1;
  if (!isfinite(est)) {
    // nothing more for this system; its iterate stays what it was
    S.live = 0;
    S.active = 0;
    S.jend = 0;
  } else if (est <= S.target || hn == 0.0) {
    S.live = 0;
    S.conv = 1;
  }
  d.scale[r] = S.live ? 1.0 / hn : 0.0;
  return S.live;
}

__global__ void k_gm_step(DevGmres d, int j, int m, int nb) {
  const int r = threadIdx.x;
  const bool live = r < nb ? gm_step_body(d, r, j, m) : false;
  set_flag(d.flag, live);
}

__device__ inline bool gm_solve_body(DevGmres& d, int r, int m) {
  GmSys& S = d.sys[r];
  const bool again = S.active && !S.conv;
  double2* y = d.coef + (size_t)r * KMAX;
  for (int i = 0; i < m; ++i) y[i] = make_double2(0.0, 0.0);
  if (!S.active || S.jend == 0) return again;
  const double2* H = S.H;
  for (int i = S.jend - 1; i >= 0; --i) {
    double2 acc = S.g[i];
    for (int k = i + 1; k < S.jend; ++k) acc = csub(acc, cmul(H[(size_t)i * m + k], y[k]));
    y[i] = cdiv(acc, H[(size_t)i * m + i]);
  }
  return again;
}

__global__ void k_gm_solve(DevGmres d, int m, int nb) {
  const int r = threadIdx.x;
  const bool again = r < nb ? gm_solve_body(d, r, m) : false;
  set_flag(d.flag, again);
}

// ---------------------------------------------------------------------------
// Fused steps for short vectors: a coarsest level of 1280 components takes
// longer to launch kernels for than to work on.  One workgroup holds the
// system's w in LDS; each wavefront takes whole inner products, so that one
// costs one wavefront reduction.  A step (norms, Gram-Schmidt twice, Givens
// rotation, next basis vector) in one launch of 10.7 us on average (1280 FP32
// components) instead of five: with the wavefront-per-value second reduction
// pass a solve on 16^3x32 takes 13.3 ms instead of 15.0.  A whole cycle of 24
// steps (FP32), separate launches / fused: 640 components 1230 / 720 us, 2560
// 1260 / 930, 6400 1610 / 1590; 32 systems 3200 / 1910, 3270 / 2390, 4770 / 4290.
// ---------------------------------------------------------------------------
constexpr int GM_WG = 512, GM_W = GM_WG / 64;

__device__ inline double gsum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// hd[i] = <V_i, w> (i <= j), hd[j + 1] = <w, w>; w in LDS; starts and ends with
// a barrier
template <typename T>
__device__ inline void gm_dots(const C<T>* V, long long vs, const C<T>* w, int n, int j, double2* hd) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  for (int i = wv; i <= j + 1; i += GM_W) {
    double2 a = czero<double>();
    if (i <= j) {
      const C<T>* Vi = V + i * vs;
#pragma unroll 8
      for (int e = lane; e < n; e += 64) cjfma(a, ccast<double>(Vi[e]), ccast<double>(w[e]));
    } else {
      for (int e = lane; e < n; e += 64) {
        const double2 v = ccast<double>(w[e]);
        a.x = rfma(v.x, v.x, rfma(v.y, v.y, a.x));
      }
    }
    a.x = gsum(a.x);
    a.y = gsum(a.y);
    if (lane == 0) hd[i] = a;
  }
  __syncthreads();
}

// w + sum_{i <= j} c_i V_i at element e, rounded to T
template <typename T>
__device__ inline C<T> gm_combine(const C<T>* V, long long vs, C<T> w, int e, int j, const double2* c) {
  double2 a = ccast<double>(w);
  for (int i0 = 0; i0 <= j; i0 += 8) {
    C<T> v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = V[min(i0 + u, j) * vs + e];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i0 + u <= j) cfma(a, c[i0 + u], ccast<double>(v[u]));
  }
  return ccast<T>(a);
}

template <typename T> __device__ inline C<T> gm_scaled(C<T> v, double sc) {
  return sc == 0.0 ? czero<T>() : ccast<T>(cscale(ccast<double>(v), sc));
}

template <typename T>
__global__ void __launch_bounds__(GM_WG) k_gm_start(DevGmres d, const C<T>* __restrict__ r0, C<T>* __restrict__ V,
                                                    long long n, int m, double tol, int first) {
  extern __shared__ unsigned char smem_raw[];
  C<T>* w = reinterpret_cast<C<T>*>(smem_raw);
  __shared__ double part[GM_W];
  __shared__ double sc;
  const int r = blockIdx.x, t = threadIdx.x;
  double ww = 0.0;
  for (int e = t; e < n; e += GM_WG) {
    w[e] = r0[r * n + e];
    const double2 v = ccast<double>(w[e]);
    ww = rfma(v.x, v.x, rfma(v.y, v.y, ww));
  }
  ww = gsum(ww);
  if ((t & 63) == 0) part[t >> 6] = ww;
  __syncthreads();
  if (t == 0) {
    for (int q = 1; q < GM_W; ++q) ww += part[q];
    d.res[(size_t)r * (KMAX + 1)] = make_double2(ww, 0.0);
    const bool live = gm_begin_body(d, r, m, tol, first);
    d.flag[1 + r] = live;
    sc = d.scale[r];
  }
  __syncthreads();
  for (int e = t; e < n; e += GM_WG) V[r * n + e] = gm_scaled<T>(w[e], sc);
}

template <typename T>
__global__ void __launch_bounds__(GM_WG) k_gm_arnoldi(DevGmres d, C<T>* V, long long vs, const C<T>* __restrict__ wv,
                                                      long long n, int j, int m) {
  extern __shared__ unsigned char smem_raw[];
  C<T>* w = reinterpret_cast<C<T>*>(smem_raw);
  __shared__ double2 h1[KMAX + 1], h2[KMAX + 1], cf[KMAX + 1], cs[KMAX], sn[KMAX];
  __shared__ double sc;
  const int r = blockIdx.x, t = threadIdx.x;
  GmSys& S = d.sys[r];
  V += r * n;
  C<T>* Vn = V + (j + 1) * vs;
  if (!S.live) {
    if (t == 0) d.flag[1 + r] = 0;
    if (j + 1 < m)
      for (int e = t; e < n; e += GM_WG) Vn[e] = czero<T>();
    return;
  }
  for (int e = t; e < n; e += GM_WG) w[e] = wv[r * n + e];
  if (t < j) {
    cs[t] = S.cs[t];
    sn[t] = S.sn[t];
  }
  gm_dots<T>(V, vs, w, (int)n, j, h1);
  double proj = 0.0;
  for (int i = 0; i <= j; ++i) proj += cabs2(h1[i]);
  const double ww = h1[j + 1].x;
  const bool again = !(ww - proj > 0.5 * ww);
  if (again) {
    if (t <= j) cf[t] = cneg(h1[t]);
    __syncthreads();
    for (int e = t; e < n; e += GM_WG) w[e] = gm_combine<T>(V, vs, w[e], e, j, cf);
    gm_dots<T>(V, vs, w, (int)n, j, h2);
  }
  if (t <= j) cf[t] = cneg(again ? h2[t] : h1[t]);
  if (t == 0) {
    double hn = sqrt(fmax(ww - proj, 0.0));
    if (again) {
      double nn = h2[j + 1].x;
      for (int i = 0; i <= j; ++i) nn -= cabs2(h2[i]);
      hn = sqrt(fmax(nn, 0.0));
    }
    // Hessenberg column j under the earlier rotations, then the new one
    double2* H = S.H;
    double2 a = again ? cadd(h1[0], h2[0]) : h1[0];
    for (int i = 0; i < j; ++i) {
      const double2 b = again ? cadd(h1[i + 1], h2[i + 1]) : h1[i + 1];
      H[(size_t)i * m + j] = cadd(cmul(cs[i], a), cmul(sn[i], b));
      a = csub(cmul(cs[i], b), cmul(cconj(sn[i]), a));
    }
    const double aa = cabs1(a), rho = sqrt(cabs2(a) + hn * hn);
    double2 c, q;
    if (rho == 0.0) {
      c = make_double2(1.0, 0.0);
      q = make_double2(0.0, 0.0);
    } else if (aa == 0.0) {
      c = make_double2(0.0, 0.0);
      q = make_double2(1.0, 0.0);
    } else {
      c = make_double2(aa / rho, 0.0);
      q = make_double2(a.x / aa * hn / rho, a.y / aa * hn / rho);
    }
    S.cs[j] = c;
    S.sn[j] = q;
    H[(size_t)j * m + j] = cadd(cmul(c, a), cscale(q, hn));
    H[(size_t)(j + 1) * m + j] = make_double2(0.0, 0.0);
    const double2 gj = S.g[j], gn = cneg(cmul(cconj(q), gj));
    S.g[j + 1] = gn;
    S.g[j] = cmul(c, gj);
    const double est = cabs1(gn);
    ++d.iters[r];
    int live = 1;
    if (!isfinite(est)) {
      // nothing more for this system; its iterate stays what it was
      live = 0;
      S.active = 0;
      S.jend = 0;
    } else {
      S.jend = j + 1;
      if (est <= S.target || hn == 0.0) {
        live = 0;
        S.conv = 1;
      }
    }
    S.live = live;
    sc = live ? 1.0 / hn : 0.0;
    d.flag[1 + r] = live;
  }
  __syncthreads();
  if (j + 1 < m)
    for (int e = t; e < n; e += GM_WG) Vn[e] = gm_scaled<T>(gm_combine<T>(V, vs, w[e], e, j, cf), sc);
}

template <typename T>
__global__ void __launch_bounds__(GM_WG) k_gm_finish(DevGmres d, const C<T>* V, long long vs, C<T>* __restrict__ x,
                                                     long long n, int m, int first) {
  __shared__ double2 H[KMAX][KMAX], y[KMAX];
  const int r = blockIdx.x, t = threadIdx.x;
  GmSys& S = d.sys[r];
  const int je = S.active ? S.jend : 0;
  if (t == 0) d.flag[1 + r] = S.active && !S.conv;
  for (int e = t; e < je * je; e += GM_WG) H[e / je][e % je] = S.H[(size_t)(e / je) * m + e % je];
  if (t < je) y[t] = S.g[t];
  __syncthreads();
  // back substitution, column by column
  for (int i = je - 1; i >= 0; --i) {
    if (t == i) y[i] = cdiv(y[i], H[i][i]);
    __syncthreads();
    if (t < i) y[t] = csub(y[t], cmul(H[t][i], y[i]));
    __syncthreads();
  }
  x += r * n;
  for (int e = t; e < n; e += GM_WG) {
    const C<T> x0 = first ? czero<T>() : x[e];
    x[e] = je > 0 ? gm_combine<T>(V + r * n, vs, x0, e, je - 1, y) : x0;
  }
}

}  // namespace

void gm_reset(const DevGmres& d, int nb, hipStream_t s) {
  k_gm_reset<<<1, 64, 0, s>>>(d.iters, nb);
  DD_LAUNCH_CHECK();
}

void gm_begin(const DevGmres& d, int m, int nb, double tol, int first, hipStream_t s) {
  DD_REQUIRE(m >= 1 && m <= KMAX && nb >= 1 && nb <= NBMAX && NBMAX <= 64, "bad device GMRES shape");
  k_gm_begin<<<1, 64, 0, s>>>(d, m, nb, tol, first);
  DD_LAUNCH_CHECK();
}

void gm_cgs1(const DevGmres& d, int j, int nb, hipStream_t s) {
  k_gm_cgs1<<<1, 64, 0, s>>>(d, j, nb);
  DD_LAUNCH_CHECK();
}

void gm_step(const DevGmres& d, int j, int m, int nb, hipStream_t s) {
  DD_REQUIRE(j >= 0 && j < m && m <= KMAX, "bad device GMRES step");
  k_gm_step<<<1, 64, 0, s>>>(d, j, m, nb);
  DD_LAUNCH_CHECK();
}

void gm_solve(const DevGmres& d, int m, int nb, hipStream_t s) {
  k_gm_solve<<<1, 64, 0, s>>>(d, m, nb);
  DD_LAUNCH_CHECK();
}

template <typename T>
void gm_start(const DevGmres& d, const C<T>* r0, C<T>* V, long long n, int m, int nb, double tol, int first,
              hipStream_t s) {
  DD_REQUIRE(m >= 1 && m <= KMAX && nb >= 1 && nb <= NBMAX && gm_short<T>(n), "bad device GMRES shape");
  k_gm_start<T><<<nb, GM_WG, n * sizeof(C<T>), s>>>(d, r0, V, n, m, tol, first);
  DD_LAUNCH_CHECK();
}
template <typename T>
void gm_arnoldi(const DevGmres& d, C<T>* V, long long vs, const C<T>* w, long long n, int j, int m, int nb,
                hipStream_t s) {
  DD_REQUIRE(j >= 0 && j < m && m <= KMAX && nb >= 1 && nb <= NBMAX && gm_short<T>(n), "bad device GMRES step");
  k_gm_arnoldi<T><<<nb, GM_WG, n * sizeof(C<T>), s>>>(d, V, vs, w, n, j, m);
  DD_LAUNCH_CHECK();
}
template <typename T>
void gm_finish(const DevGmres& d, const C<T>* V, long long vs, C<T>* x, long long n, int m, int nb, bool first,
               hipStream_t s) {
  DD_REQUIRE(m >= 1 && m <= KMAX && nb >= 1 && nb <= NBMAX && gm_short<T>(n), "bad device GMRES shape");
  k_gm_finish<T><<<nb, GM_WG, 0, s>>>(d, V, vs, x, n, m, first);
  DD_LAUNCH_CHECK();
}
#define DD_INST(T)                                                                                            \
  template void gm_start<T>(const DevGmres&, const C<T>*, C<T>*, long long, int, int, double, int, hipStream_t); \
  template void gm_arnoldi<T>(const DevGmres&, C<T>*, long long, const C<T>*, long long, int, int, int, hipStream_t); \
  template void gm_finish<T>(const DevGmres&, const C<T>*, long long, C<T>*, long long, int, int, bool, hipStream_t);
DD_INST(double)
DD_INST(float)
#undef DD_INST

}  // namespace ddamg
