// CGNR: conjugate gradients on the normal equations D^H D z = D^H b with the
// residual r = b - D z, entirely in FP64 -- the Krylov method the paper
// compares DD-alpha-AMG against and whose iteration count it uses as the
// conditioning indicator of a configuration (Sec. 4, Tab. 2 and Tab. 5).
// D^H is applied as Gamma5 D Gamma5 (gamma5-hermiticity of the
// Wilson-clover operator).  A batch of systems advances together with its
// own scalars and stopping test per system.
//
// The scalars stay on the device, so that an iteration is four kernels (six
// where the stencil's norm parts are folded first) and, after the first few, no
// host round trip:
//   w = D p and parts of <w, w>;
//   alpha = gamma / <w, w>, r -= alpha w and parts of <r, r>;
//   z = D^H r and parts of <z, z>;
//   stopping test, beta = <z, z> / gamma, x += alpha p, p = z + beta p.
// Every workgroup of an update sums the parts it needs itself, in the same
// order.  Bound by memory: 12 vectors and twice the FP64 operator per
// iteration.  16^3x32, one system: 151 us per iteration, against 236 us with
// separate Gamma5, axpy, scaling and norm kernels and three host
// synchronisations per iteration.
#include <chrono>
#include <cmath>
#include <complex>
#include <vector>

#include "cgnr.h"

namespace ddamg {

namespace {

void norms2(Reducer& red, const double2* v, long long n, int nb, std::vector<double>& out, hipStream_t s) {
  red.bdots<double>(nullptr, v, 0, 0, const_cast<double2*>(v), n, nb, s);
  std::vector<std::complex<double>> r(nb);
  red.bfetch(1, nb, r.data(), s);
  out.resize(nb);
  for (int k = 0; k < nb; ++k) out[k] = r[k].real();
}

// one system's scalars; gamma and live are double-buffered by iteration (an
// update kernel reads one and its first workgroup writes the other)
struct CgSys {
  double gamma[2];
  int live[2];
  double alpha, stop;    // stop: tol^2 ||b||^2
  int iters, status;
};
constexpr int CG_WG = 256;
constexpr int CG_PARTS = 1024;   // most parts an update's workgroups sum themselves
constexpr int CG_RING = 4;       // iterations the host runs ahead of the stopping test, plus one
// Iterations whose stopping test is read before the next is issued: a run of k
// iterations that the host is ahead of issues k + 2, which a short one (a warm
// start, a loose tolerance) would not make up for.  A call of one iteration on
// 8^4 340 us with host scalars, 500 with the host ahead, 330 so; on 32^3x64 9.8,
// 12.6, 8.2 ms.
constexpr int CG_EAGER = 8;

// the sum of n parts, the same in every thread and in every workgroup
__device__ double sum_parts(const double* __restrict__ p, int n, double* lds) {
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += CG_WG) s += p[i];
  s = group_sum<64>(s);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = s;
  __syncthreads();
  s = (lds[0] + lds[1]) + (lds[2] + lds[3]);
  __syncthreads();
  return s;
}

// many parts of each system summed into one (blockIdx.x = system)
__global__ void __launch_bounds__(CG_WG) k_cg_fold(const double* __restrict__ parts, int n, double* __restrict__ out) {
  __shared__ double lds[4];
  const double s = sum_parts(parts + (long long)blockIdx.x * n, n, lds);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

__global__ void __launch_bounds__(CG_WG) k_cg_residual(CgSys* __restrict__ sys, int cur, const double* __restrict__ ww,
                                                       int nww, const double2* __restrict__ w, double2* __restrict__ r,
                                                       long long n, double* __restrict__ rr) {
  __shared__ double lds[4];
  const int k = blockIdx.y;
  const double del = sum_parts(ww + (long long)k * nww, nww, lds);
  const double alpha = sys[k].live[cur] && del > 0.0 ? sys[k].gamma[cur] / del : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) sys[k].alpha = alpha;
  w += k * n;
  r += k * n;
  double s = 0.0;
  const long long S = (long long)gridDim.x * CG_WG;
#pragma unroll 4
  for (long long i = (long long)blockIdx.x * CG_WG + threadIdx.x; i < n; i += S) {
    const double2 a = w[i];
    double2 b = r[i];
    b.x = rfma(-alpha, a.x, b.x);
    b.y = rfma(-alpha, a.y, b.y);
    r[i] = b;
    s = rfma(b.x, b.x, s);
    s = rfma(b.y, b.y, s);
  }
  s = group_sum<64>(s);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) rr[(long long)k * gridDim.x + blockIdx.x] = (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

// flag (host): whether the system goes on after this iteration; count (host):
// its iterations and status so far
__global__ void __launch_bounds__(CG_WG) k_cg_direction(CgSys* __restrict__ sys, int cur, const double* __restrict__ rr,
                                                        int nrr, const double* __restrict__ zz, int nzz,
                                                        const double2* __restrict__ z, double2* __restrict__ p,
                                                        double2* __restrict__ x, long long n, int* __restrict__ flag,
                                                        int2* __restrict__ count) {
  __shared__ double lds[4];
  const int k = blockIdx.y, was = sys[k].live[cur];
  const double rho = sum_parts(rr + (long long)k * nrr, nrr, lds), gam1 = sum_parts(zz + (long long)k * nzz, nzz, lds);
  const double gam = sys[k].gamma[cur], alpha = sys[k].alpha;
  const bool finite = isfinite(rho), live = was && finite && !(rho <= sys[k].stop);
  const double beta = live && gam > 0.0 ? gam1 / gam : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sys[k].gamma[cur ^ 1] = gam1;
    sys[k].live[cur ^ 1] = live;
    if (was) {
      ++sys[k].iters;
      if (!live) sys[k].status = finite ? DDAMG_OK : DDAMG_ENONFINITE;
      count[k] = make_int2(sys[k].iters, sys[k].status);
    }
    flag[k] = live;
  }
  if (!was) return;   // a system that has ended keeps its iterate
  z += k * n;
  p += k * n;
  x += k * n;
  const long long S = (long long)gridDim.x * CG_WG;
#pragma unroll 4
  for (long long i = (long long)blockIdx.x * CG_WG + threadIdx.x; i < n; i += S) {
    const double2 a = p[i], b = z[i];
    double2 c = x[i];
    c.x = rfma(alpha, a.x, c.x);
    c.y = rfma(alpha, a.y, c.y);
    x[i] = c;
    p[i] = make_double2(rfma(beta, a.x, b.x), rfma(beta, a.y, b.y));
  }
}

struct Events {
  hipEvent_t ev[CG_RING] = {};
  Events() {
    for (auto& e : ev) DD_CHECK_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  }
  ~Events() {
    for (auto& e : ev)
      if (e) (void)hipEventDestroy(e);
  }
  Events(const Events&) = delete;
  Events& operator=(const Events&) = delete;
};

}  // namespace

void cgnr(Context& ctx, const double2* b, double2* x, int nb, double tol, int max_iter, ddamg_solve_stats* st,
          hipStream_t s) {
  DD_REQUIRE(nb >= 1 && nb <= NBMAX, "batch out of range");
  const FineGeom& g = ctx.g;
  const long long n = (long long)g.nblk * 192, vs = n * nb;
  const FineOpView<double> D = ctx.view<double>();
  Reducer red;
  DevArray<double2> r, p, w, z;
  r.alloc(vs);
  p.alloc(vs);
  w.alloc(vs);
  z.alloc(vs);
  // parts of the norms: the stencil's per workgroup, folded into one where
  // they are many, and one per workgroup of the residual update
  const int nd = dslash_norm_parts(g.nblk), np = nd > CG_PARTS ? 1 : nd;
  const int grid = (int)std::min<long long>(CG_PARTS, (n + 4 * CG_WG - 1) / (4 * CG_WG));
  static_assert(sizeof(CgSys) % sizeof(double) == 0, "the norms follow the systems' records");
  DevArray<double> small;   // one allocation: a call on a small lattice notices each
  const size_t sw = sizeof(CgSys) / sizeof(double);
  small.alloc(nb * (sw + nd + 1 + grid));
  CgSys* sys = reinterpret_cast<CgSys*>(small.p);
  double *dparts = small.p + nb * sw, *sums = dparts + (size_t)nb * nd, *rparts = sums + nb;
  const double* parts = np == 1 ? sums : dparts;
  auto apply = [&](const double2* v, double2* out, bool g5) {
    dslash_norm(D, v, out, g5, dparts, s, nb);
    if (np == 1) {
      k_cg_fold<<<nb, CG_WG, 0, s>>>(dparts, nd, sums);
      DD_LAUNCH_CHECK();
    }
  };
  std::vector<double> bn, rho, gam;
  norms2(red, b, n, nb, bn, s);
  // r = b - D x, z = D^H r, p = z
  dslash<double>(D, x, r.p, s, nb);
  vbmy<double>(b, r.p, vs, s);
  apply(r.p, z.p, true);
  vcopy<double, double>(z.p, p.p, vs, s);
  norms2(red, r.p, n, nb, rho, s);
  norms2(red, z.p, n, nb, gam, s);
  std::vector<CgSys> h(nb);
  bool any = false;
  for (int k = 0; k < nb; ++k) {
    st[k] = ddamg_solve_stats{};
    h[k] = CgSys{};
    h[k].status = DDAMG_ENOCONV;
    h[k].stop = tol * tol * bn[k];
    if (!std::isfinite(bn[k]) || !std::isfinite(rho[k])) h[k].status = DDAMG_ENONFINITE;
    else if (rho[k] <= h[k].stop) h[k].status = DDAMG_OK;
    h[k].live[0] = h[k].status == DDAMG_ENOCONV;
    h[k].gamma[0] = gam[k];
    any = any || h[k].live[0];
  }
  const int2* count = nullptr;   // host words: complete when the stream has drained
  if (any && max_iter > 0) {
    DD_CHECK_HIP(hipMemcpyAsync(sys, h.data(), sizeof(CgSys) * nb, hipMemcpyHostToDevice, s));
    Events done;
    int *host = nullptr, *dev = nullptr;
    red.host_words(&host, &dev, (2 + CG_RING) * nb);
    count = reinterpret_cast<const int2*>(host);
    const int* flag_host = host + 2 * nb;
    int* flag_dev = dev + 2 * nb;
    for (int it = 0; it < max_iter; ++it) {
      const int cur = it & 1, slot = it % CG_RING;
      // the flags of `ahead` iterations ago decide whether to go on: the
      // iterations issued past the last system's stopping test change nothing
      const int ahead = it <= CG_EAGER ? 1 : CG_RING - 1;
      if (it >= ahead) {
        const int old = (it - ahead) % CG_RING;
        DD_CHECK_HIP(hipEventSynchronize(done.ev[old]));
        bool more = false;
        for (int k = 0; k < nb; ++k) more = more || static_cast<const volatile int*>(flag_host)[old * nb + k] != 0;
        if (!more) break;
      }
      apply(p.p, w.p, false);
      k_cg_residual<<<dim3(grid, nb), CG_WG, 0, s>>>(sys, cur, parts, np, w.p, r.p, n, rparts);
      DD_LAUNCH_CHECK();
      apply(r.p, z.p, true);
      k_cg_direction<<<dim3(grid, nb), CG_WG, 0, s>>>(sys, cur, rparts, grid, parts, np, z.p, p.p, x, n,
                                                      flag_dev + slot * nb, reinterpret_cast<int2*>(dev));
      DD_LAUNCH_CHECK();
      DD_CHECK_HIP(hipEventRecord(done.ev[slot], s));
    }
  }
  // the true residual of every system
  dslash<double>(D, x, r.p, s, nb);
  vbmy<double>(b, r.p, vs, s);
  norms2(red, r.p, n, nb, rho, s);
  for (int k = 0; k < nb; ++k) {
    const double rel = bn[k] > 0 ? std::sqrt(std::max(rho[k], 0.0) / bn[k]) : 0.0;
    const int2 c = count && h[k].live[0] ? count[k] : make_int2(0, h[k].status);
    st[k].outer_iters = c.x;
    st[k].true_relres = rel;
    st[k].status = c.y == DDAMG_OK && !(rel <= tol) ? DDAMG_ENOCONV : c.y;
  }
}

}  // namespace ddamg
