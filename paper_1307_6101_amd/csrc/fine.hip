// Fine-lattice kernels: layout conversion, clover construction, the
// Wilson-clover stencil and the red-black SAP colour pass with block MR.
//
// Operator (the paper's eq. (1); definition of D as in the two-level
// predecessor, textbook Sheikholeslami-Wohlert form):
//   (D psi)(x) = A(x) psi(x) - 1/2 sum_mu [ (1-g_mu) U_mu(x) psi(x+mu)
//                                         + (1+g_mu) U_mu(x-mu)^H psi(x-mu) ]
//   A(x) = (m0+4) - c_sw/16 sum_{mu<nu} g_mu g_nu (x) (Q_mu,nu - Q_mu,nu^H),
// chiral gamma basis, Gamma5 = diag(1,1,-1,-1): A(x) is block diagonal with
// one Hermitian 6x6 block per chirality.
//
// Spin projection.  With g_mu = [[0, B_mu],[B_mu^H, 0]], (1 -+ g_mu) psi is
// fixed by its upper half h = (psi_0 + c0 psi_j0, psi_1 + c1 psi_j1), with
// (j0, c0, j1, c1) = (3, i, 2, i), (3, 1, 2, -1), (2, i, 3, -i), (2, -1, 3, -1)
// for mu = 0..3 in the forward hop and c -> -c in the backward hop; the lower
// half is rebuilt as out_j0 += conj(c0) chi_0, out_j1 += conj(c1) chi_1 with
// chi = U h.  So each hop moves 6 instead of 12 complex numbers through the
// SU(3) multiply.
#include "fine.h"
#include "fine_dev.h"

#include <type_traits>

#include <vector>

namespace ddamg {

FineGeom make_fine_geom(const int dims[4]) {
  FineGeom g;
  g.V = 1;
  g.nblk = 1;
  for (int mu = 0; mu < 4; ++mu) {
    DD_REQUIRE(dims[mu] % 4 == 0, "every lattice extent must be a multiple of 4");
    g.dims[mu] = dims[mu];
    g.nb[mu] = dims[mu] / 2;
    g.V *= dims[mu];
    g.nblk *= g.nb[mu];
  }
  return g;
}

void fine_tables(const FineGeom& g, int* nbr_blk, int* colour_blocks) {
  int n[2] = {0, 0};
  const int half = g.nblk / 2;
  for (int b = 0; b < g.nblk; ++b) {
    int c[4];
    block_decode(g.nb, b, c);
    for (int mu = 0; mu < 4; ++mu) {
      for (int dir = 0; dir < 2; ++dir) {
        int cc[4] = {c[0], c[1], c[2], c[3]};
        cc[mu] = (cc[mu] + (dir == 0 ? 1 : g.nb[mu] - 1)) % g.nb[mu];
        nbr_blk[b * 8 + 2 * mu + dir] = block_encode(g.nb, cc);
      }
    }
    int col = (c[0] + c[1] + c[2] + c[3]) & 1;
    colour_blocks[col * half + n[col]++] = b;
  }
}

// ---------------------------------------------------------------------------
// index helpers
// ---------------------------------------------------------------------------
struct DevGeom {
  int X, Y, Z, T;
  int nb[4];
  long long V;
};
static DevGeom devgeom(const FineGeom& g) {
  return DevGeom{g.dims[0], g.dims[1], g.dims[2], g.dims[3], {g.nb[0], g.nb[1], g.nb[2], g.nb[3]}, g.V};
}

__device__ inline void canonical_to_native(const DevGeom& g, long long i, int& blk, int& loc) {
  int x = (int)(i % g.X);
  long long r = i / g.X;
  int y = (int)(r % g.Y);
  r /= g.Y;
  int z = (int)(r % g.Z);
  int t = (int)(r / g.Z);
  const int b[4] = {x >> 1, y >> 1, z >> 1, t >> 1};
  blk = block_encode(g.nb, b);
  loc = (x & 1) | ((y & 1) << 1) | ((z & 1) << 2) | ((t & 1) << 3);
}

__device__ inline long long canon_index(const DevGeom& g, int x, int y, int z, int t) {
  x = (x + g.X) % g.X;
  y = (y + g.Y) % g.Y;
  z = (z + g.Z) % g.Z;
  t = (t + g.T) % g.T;
  return x + (long long)g.X * (y + (long long)g.Y * (z + (long long)g.Z * t));
}

// ---------------------------------------------------------------------------
// conversions
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_to_native(DevGeom g, const double2* __restrict__ in, C<T>* __restrict__ out) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= g.V) return;
  const long long off = (long long)blockIdx.y * g.V * 12;
  int blk, loc;
  canonical_to_native(g, i, blk, loc);
#pragma unroll
  for (int c = 0; c < 12; ++c)
    out[off + ((long long)blk * 12 + c) * 16 + loc] = ccast<T>(in[off + i * 12 + c]);
}

template <typename T>
__global__ void k_from_native(DevGeom g, const C<T>* __restrict__ in, double2* __restrict__ out) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= g.V) return;
  const long long off = (long long)blockIdx.y * g.V * 12;
  int blk, loc;
  canonical_to_native(g, i, blk, loc);
#pragma unroll
  for (int c = 0; c < 12; ++c)
    out[off + i * 12 + c] = ccast<double>(in[off + ((long long)blk * 12 + c) * 16 + loc]);
}

__global__ void k_links_to_native(DevGeom g, const double2* __restrict__ in, double2* __restrict__ out) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= g.V) return;
  int blk, loc;
  canonical_to_native(g, i, blk, loc);
  for (int e = 0; e < 36; ++e) out[((long long)blk * 36 + e) * 16 + loc] = in[i * 36 + e];
}

template <typename S> __device__ inline S op_round(double2 v);
template <> __device__ inline float2 op_round<float2>(double2 v) { return make_float2((float)v.x, (float)v.y); }
template <> __device__ inline __half2 op_round<__half2>(double2 v) {
  return __floats2half2_rn((float)v.x, (float)v.y);
}
// one thread per (block, chunk, site): FP64 entries in, one chunk out
template <typename S>
__global__ void k_op_store(const double2* __restrict__ in, S* __restrict__ out, long long n) {
  constexpr int N = OpChunk<S>::N, NQ = 36 / N;
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int loc = (int)(i & 15);
  const long long bq = i >> 4, blk = bq / NQ;
  const int q = (int)(bq - blk * NQ);
  OpChunk<S> c;
#pragma unroll
  for (int k = 0; k < N; ++k) c.v[k] = op_round<S>(in[(blk * 36 + q * N + k) * 16 + loc]);
  reinterpret_cast<OpChunk<S>*>(out)[i] = c;
}

template <typename T>
void fine_to_native(const FineGeom& g, const double2* in, C<T>* out, int nrhs, hipStream_t s) {
  dim3 grid(nblocks(g.V, 256), nrhs);
  k_to_native<T><<<grid, 256, 0, s>>>(devgeom(g), in, out);
  DD_LAUNCH_CHECK();
}
template <typename T>
void fine_from_native(const FineGeom& g, const C<T>* in, double2* out, int nrhs, hipStream_t s) {
  dim3 grid(nblocks(g.V, 256), nrhs);
  k_from_native<T><<<grid, 256, 0, s>>>(devgeom(g), in, out);
  DD_LAUNCH_CHECK();
}
void links_to_native(const FineGeom& g, const double2* links, double2* out, hipStream_t s) {
  k_links_to_native<<<nblocks(g.V, 256), 256, 0, s>>>(devgeom(g), links, out);
  DD_LAUNCH_CHECK();
}
template <typename S>
void op_store(const FineGeom& g, const double2* in, S* out, hipStream_t s) {
  const long long n = g.V * (36 / OpChunk<S>::N);
  k_op_store<S><<<nblocks(n, 256), 256, 0, s>>>(in, out, n);
  DD_LAUNCH_CHECK();
}
template void op_store<float2>(const FineGeom&, const double2*, float2*, hipStream_t);
template void op_store<__half2>(const FineGeom&, const double2*, __half2*, hipStream_t);

// ---------------------------------------------------------------------------
// clover construction (FP64, canonical links in, native packed out)
// ---------------------------------------------------------------------------
struct M3 { double2 e[9]; };

__device__ inline M3 load_link(const double2* L, long long site, int mu) {
  M3 m;
#pragma unroll
  for (int k = 0; k < 9; ++k) m.e[k] = L[(site * 4 + mu) * 9 + k];
  return m;
}
// a * b, a^H * b, a * b^H
__device__ inline M3 mm(const M3& a, const M3& b) {
  M3 c;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = czero<double>();
#pragma unroll
      for (int k = 0; k < 3; ++k) cfma(s, a.e[i * 3 + k], b.e[k * 3 + j]);
      c.e[i * 3 + j] = s;
    }
  return c;
}
__device__ inline M3 mhm(const M3& a, const M3& b) {
  M3 c;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = czero<double>();
#pragma unroll
      for (int k = 0; k < 3; ++k) cjfma(s, a.e[k * 3 + i], b.e[k * 3 + j]);
      c.e[i * 3 + j] = s;
    }
  return c;
}
__device__ inline M3 mmh(const M3& a, const M3& b) {
  M3 c;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = czero<double>();
#pragma unroll
      for (int k = 0; k < 3; ++k) cfma(s, a.e[i * 3 + k], cconj(b.e[j * 3 + k]));
      c.e[i * 3 + j] = s;
    }
  return c;
}

// chiral-basis gamma matrices, entries as (re, im)
__constant__ double c_gamma[4][4][4][2] = {
    {{{0, 0}, {0, 0}, {0, 0}, {0, -1}}, {{0, 0}, {0, 0}, {0, -1}, {0, 0}},
     {{0, 0}, {0, 1}, {0, 0}, {0, 0}}, {{0, 1}, {0, 0}, {0, 0}, {0, 0}}},
    {{{0, 0}, {0, 0}, {0, 0}, {-1, 0}}, {{0, 0}, {0, 0}, {1, 0}, {0, 0}},
     {{0, 0}, {1, 0}, {0, 0}, {0, 0}}, {{-1, 0}, {0, 0}, {0, 0}, {0, 0}}},
    {{{0, 0}, {0, 0}, {0, -1}, {0, 0}}, {{0, 0}, {0, 0}, {0, 0}, {0, 1}},
     {{0, 1}, {0, 0}, {0, 0}, {0, 0}}, {{0, 0}, {0, -1}, {0, 0}, {0, 0}}},
    {{{0, 0}, {0, 0}, {1, 0}, {0, 0}}, {{0, 0}, {0, 0}, {0, 0}, {1, 0}},
     {{1, 0}, {0, 0}, {0, 0}, {0, 0}}, {{0, 0}, {1, 0}, {0, 0}, {0, 0}}}};

__device__ inline double2 gam(int mu, int a, int b) {
  return mk<double>(c_gamma[mu][a][b][0], c_gamma[mu][a][b][1]);
}

__global__ void k_clover(DevGeom g, const double2* __restrict__ L, double m0, double csw,
                         double2* __restrict__ out) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= g.V) return;
  int xc[4];
  {
    long long r = i;
    xc[0] = (int)(r % g.X); r /= g.X;
    xc[1] = (int)(r % g.Y); r /= g.Y;
    xc[2] = (int)(r % g.Z); xc[3] = (int)(r / g.Z);
  }
  auto nbr = [&](int mu, int smu, int nu, int snu) {
    int c[4] = {xc[0], xc[1], xc[2], xc[3]};
    c[mu] += smu;
    c[nu] += snu;
    return canon_index(g, c[0], c[1], c[2], c[3]);
  };
  // A_chi[6][6], chi = 0 (spins 0,1), 1 (spins 2,3)
  double2 A[2][6][6];
  for (int h = 0; h < 2; ++h)
    for (int a = 0; a < 6; ++a)
      for (int b = 0; b < 6; ++b) A[h][a][b] = czero<double>();
  if (csw != 0.0) {
    for (int mu = 0; mu < 4; ++mu)
      for (int nu = mu + 1; nu < 4; ++nu) {
        M3 Um = load_link(L, i, mu), Un = load_link(L, i, nu);
        M3 Um_pn = load_link(L, nbr(nu, 1, mu, 0), mu);      // U_mu(x+nu)
        M3 Un_pm = load_link(L, nbr(mu, 1, nu, 0), nu);      // U_nu(x+mu)
        M3 Um_mm = load_link(L, nbr(mu, -1, nu, 0), mu);     // U_mu(x-mu)
        M3 Un_mm = load_link(L, nbr(mu, -1, nu, 0), nu);     // U_nu(x-mu)
        M3 Um_pnmm = load_link(L, nbr(mu, -1, nu, 1), mu);   // U_mu(x+nu-mu)
        M3 Um_mmmn = load_link(L, nbr(mu, -1, nu, -1), mu);  // U_mu(x-mu-nu)
        M3 Un_mmmn = load_link(L, nbr(mu, -1, nu, -1), nu);  // U_nu(x-mu-nu)
        M3 Um_mn = load_link(L, nbr(nu, -1, mu, 0), mu);     // U_mu(x-nu)
        M3 Un_mn = load_link(L, nbr(nu, -1, mu, 0), nu);     // U_nu(x-nu)
        M3 Un_mnpm = load_link(L, nbr(mu, 1, nu, -1), nu);   // U_nu(x-nu+mu)
        // four counter-clockwise leaves at x
        M3 q1 = mmh(mmh(mm(Um, Un_pm), Um_pn), Un);
        // Un(x) Um(x+nu-mu)^H Un(x-mu)^H Um(x-mu)
        M3 q2 = mm(mmh(mmh(Un, Um_pnmm), Un_mm), Um_mm);
        // leaf 3: Um(x-mu)^H Un(x-mu-nu)^H Um(x-mu-nu) Un(x-nu)
        M3 t3 = mhm(Un_mmmn, mm(Um_mmmn, Un_mn));           // Un(x-mu-nu)^H Um(x-mu-nu) Un(x-nu)
        M3 l3 = mhm(Um_mm, t3);
        // leaf 4: Un(x-nu)^H Um(x-nu) Un(x-nu+mu) Um(x)^H
        M3 l4 = mmh(mhm(Un_mn, mm(Um_mn, Un_mnpm)), Um);
        M3 F;
#pragma unroll
        for (int k = 0; k < 9; ++k) F.e[k] = cadd(cadd(q1.e[k], q2.e[k]), cadd(l3.e[k], l4.e[k]));
        // F <- Q - Q^H
        M3 Fa;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
          for (int b = 0; b < 3; ++b) Fa.e[a * 3 + b] = csub(F.e[a * 3 + b], cconj(F.e[b * 3 + a]));
        // sigma = g_mu g_nu (block diagonal in chirality)
        for (int h = 0; h < 2; ++h)
          for (int s = 0; s < 2; ++s)
            for (int sp = 0; sp < 2; ++sp) {
              double2 sg = czero<double>();
              for (int k = 0; k < 4; ++k) cfma(sg, gam(mu, 2 * h + s, k), gam(nu, k, 2 * h + sp));
              sg = cscale(sg, -csw / 16.0);
              for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b) cfma(A[h][s * 3 + a][sp * 3 + b], sg, Fa.e[a * 3 + b]);
            }
      }
  }
  int blk, loc;
  canonical_to_native(g, i, blk, loc);
  double2* o = out + (long long)blk * 36 * 16 + loc;
  for (int h = 0; h < 2; ++h) {
    double d[6];
    for (int a = 0; a < 6; ++a) d[a] = A[h][a][a].x + (m0 + 4.0);
    for (int k = 0; k < 3; ++k) o[(h * 18 + k) * 16] = mk<double>(d[2 * k], d[2 * k + 1]);
    int e = 3;
    for (int a = 0; a < 6; ++a)
      for (int b = a + 1; b < 6; ++b) o[(h * 18 + e++) * 16] = A[h][a][b];
  }
}

void clover_build(const FineGeom& g, const double2* links, double m0, double csw, double2* out,
                  hipStream_t s) {
  k_clover<<<nblocks(g.V, 128), 128, 0, s>>>(devgeom(g), links, m0, csw, out);
  DD_LAUNCH_CHECK();
}

// the eight neighbour blocks of `blk` (2*mu + 0: +mu, 2*mu + 1: -mu), two
// 16-byte loads issued together so that no later load waits on an index
struct Nbr8 {
  int v[8];
};
__device__ inline Nbr8 load_nbr8(const int* __restrict__ nbr, int blk) {
  const int4* p = reinterpret_cast<const int4*>(nbr + (size_t)blk * 8);
  const int4 a = p[0], b = p[1];
  return Nbr8{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}

// Completes the arithmetic that produces acc before the statements that
// follow (empty asm statements that read and write it), so that the next
// hop's loads are not issued ahead of it: those of all eight hops on canonical
// fields would need more registers than two wavefronts per SIMD have.
template <typename T> __device__ inline void pin12(C<T> (&acc)[12]) {
#pragma unroll
  for (int c = 0; c < 12; ++c) asm volatile("" : "+v"(acc[c].x), "+v"(acc[c].y));
}

// A stencil kernel reads its input spinors through one of these: a native
// field of storage V (C<T>, or FP16 with site scales)
template <typename T, typename V>
struct NativeIn {
  static constexpr bool EAGER = false;
  const V* in;
  const float* ins;
  __device__ inline void site(int blk, int loc, C<T> v[12]) const { load_site<T, V>(in, ins, blk, loc, v); }
  // the spinor at the site's neighbour in direction MU, which lies in block nb
  template <int MU, bool FWD> __device__ inline void hop(int nb, int loc, C<T> v[12]) const {
    site(nb, loc ^ (1 << MU), v);
  }
};

// or from a canonical complex128 field
template <typename T>
struct CanonIn {
  static constexpr bool EAGER = true;
  // field f, the site with index t (block * 16 + local) in the tile at tc
  __device__ inline void place(const DevGeom& g, const double2* f, const int (&tc)[4], int t) {
    in = f;
    dims[0] = g.X, dims[1] = g.Y, dims[2] = g.Z, dims[3] = g.T;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) c[mu] = 4 * tc[mu] + 2 * ((t >> (4 + mu)) & 1) + ((t >> mu) & 1);
    own = c[0] + (long long)g.X * (c[1] + (long long)g.Y * (c[2] + (long long)g.Z * c[3]));
  }
  const double2* in;
  int c[4], dims[4];     // the site's coordinates, the lattice
  long long own;         // its canonical index
  __device__ inline void at(long long i, C<T> v[12]) const {
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = ccast<T>(in[i * 12 + k]);
  }
  __device__ inline void site(int, int, C<T> v[12]) const { at(own, v); }
  template <int MU, bool FWD> __device__ inline void hop(int, int, C<T> v[12]) const {
    long long st = 1;
#pragma unroll
    for (int mu = 0; mu < MU; ++mu) st *= dims[mu];
    if constexpr (FWD) at(c[MU] + 1 == dims[MU] ? own - (dims[MU] - 1) * st : own + st, v);
    else at(c[MU] == 0 ? own + (dims[MU] - 1) * st : own - st, v);
  }
};

// Completes a hop before the next one's loads are issued where nothing else
// (an index to wait for) spaces them out and they would not fit the registers
template <typename T, typename In> __device__ inline void hop_done(C<T> (&acc)[12]) {
  if constexpr (In::EAGER) {
    pin12<T>(acc);
    asm volatile("" ::: "memory");
  }
}

// both hops of direction MU
template <typename T, typename S, int MU, typename In>
__device__ inline void hops_mu(const FineOpView<T, S>& op, const In& in, int blk, int loc, const Nbr8& nb8,
                               C<T> (&acc)[12]) {
  constexpr int bit = 1 << MU;
  C<T> psi[12], u[9];
  // forward: psi(x+mu), U_mu(x)
  {
    const int nb = (loc & bit) ? nb8.v[2 * MU] : blk;
    in.template hop<MU, true>(nb, loc, psi);
    load_link<T, MU, S>(op.U, blk, loc, u);
    hop_apply<T, MU, true>(psi, u, acc);
    hop_done<T, In>(acc);
  }
  // backward: psi(x-mu), U_mu(x-mu)^H
  {
    const int nb = (loc & bit) ? blk : nb8.v[2 * MU + 1];
    in.template hop<MU, false>(nb, loc, psi);
    load_link<T, MU, S>(op.U, nb, loc ^ bit, u);
    hop_apply<T, MU, false>(psi, u, acc);
    hop_done<T, In>(acc);
  }
}

// acc = (D in)(x) at one site
template <typename T, typename S, bool NT, typename In>
__device__ inline void dslash_site(const FineOpView<T, S>& op, const In& in, int blk, int loc, C<T> (&acc)[12]) {
  const Nbr8 nb8 = load_nbr8(op.nbr, blk);
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = czero<T>();
  hops_mu<T, S, 0>(op, in, blk, loc, nb8, acc);
  hops_mu<T, S, 1>(op, in, blk, loc, nb8, acc);
  hops_mu<T, S, 2>(op, in, blk, loc, nb8, acc);
  hops_mu<T, S, 3>(op, in, blk, loc, nb8, acc);
  C<T> psi[12], av[12];
  in.site(blk, loc, psi);
  clover_apply<T, S, NT>(op.A, blk, loc, psi, av);
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = mk<T>(av[c].x - T(0.5) * acc[c].x, av[c].y - T(0.5) * acc[c].y);
}

// Whether one field's pass reads its operator data past the caches: where it
// does not fit the last-level cache it would only push out what is reused
// (the faces' spinors).  FP64 stencil on 32^3x64: 893 -> 837 us; where it fits
// (16^3x32, FP32) a repeated call finds it there: 21.0 us against 23.1.
constexpr double LLC_BYTES = 256e6;
template <typename S> inline bool op_streams(int nblk, int nb) {
  return nb == 1 && 72.0 * sizeof(S) * 16 * nblk > LLC_BYTES;
}

// One site per thread.  A batch of nb fields runs over a one-dimensional
// grid of gx * nb workgroups with the XCD-aware batch mapping.  The result is
// written past the caches, which keep the spinors and links that neighbouring
// workgroups share: 12 fields of 16^3x32 in FP32 218 -> 209 us (inputs not in the
// last-level cache; 193 -> 168 us where they are), one FP64 field of 32^3x64 843
// -> 820 us.  (Several fields per thread on one load of the links cost occupancy:
// 12 fields 204 us one by one, 208 two and 267 four at a time.)
template <typename T, typename S, typename V, bool NT>
__global__ void __launch_bounds__(256) k_dslash(FineOpView<T, S> op, const V* __restrict__ in,
                                                const float* __restrict__ ins, C<T>* __restrict__ out,
                                                long long fs, int gx, int nb) {
  int x, r;
  xcd_slab_rhs<S>(blockIdx.x, gx, nb, x, r);
  const int tid = x * blockDim.x + threadIdx.x;
  const int blk = tid >> 4, loc = tid & 15;
  if (blk >= op.nblk) return;
  const long long off = (long long)r * fs;
  C<T> o[12];
  dslash_site<T, S, NT>(op, NativeIn<T, V>{in + off, std::is_same<V, __half2>::value ? ins + off / 12 : nullptr}, blk,
                        loc, o);
  C<T>* p = out + off + (long long)blk * 192 + loc;
#pragma unroll
  for (int c = 0; c < 12; ++c) store_nt(p + c * 16, o[c]);
}

// D, or with G5 its adjoint Gamma5 D Gamma5 (the signs of the lower spins
// applied as they are loaded and stored), on native FP64 fields, and per
// workgroup the sum of |out|^2 (partial[field * gx + chunk])
struct NativeG5In : NativeIn<double, double2> {
  __device__ inline void site(int blk, int loc, double2 v[12]) const {
    NativeIn<double, double2>::site(blk, loc, v);
#pragma unroll
    for (int c = 6; c < 12; ++c) v[c] = make_double2(-v[c].x, -v[c].y);
  }
  template <int MU, bool FWD> __device__ inline void hop(int nb, int loc, double2 v[12]) const {
    site(nb, loc ^ (1 << MU), v);
  }
};
template <bool G5, bool NT>
__global__ void __launch_bounds__(256) k_dslash_norm(FineOpView<double> op, const double2* __restrict__ in,
                                                     double2* __restrict__ out, double* __restrict__ partial,
                                                     long long fs, int gx, int nb) {
  __shared__ double sums[4];
  int x, r;
  xcd_slab_rhs<double2>(blockIdx.x, gx, nb, x, r);
  const int blk = x * 16 + (threadIdx.x >> 4), loc = threadIdx.x & 15;   // nblk is a multiple of 16
  const long long off = (long long)r * fs;
  double2 o[12];
  using In = std::conditional_t<G5, NativeG5In, NativeIn<double, double2>>;
  In f;
  f.in = in + off;
  f.ins = nullptr;
  dslash_site<double, double2, NT>(op, f, blk, loc, o);
  double2* p = out + off + (long long)blk * 192 + loc;
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    s = rfma(o[c].x, o[c].x, s);
    s = rfma(o[c].y, o[c].y, s);
    p[c * 16] = G5 && c >= 6 ? make_double2(-o[c].x, -o[c].y) : o[c];
  }
  s = group_sum<64>(s);
  if ((threadIdx.x & 63) == 0) sums[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) partial[(long long)r * gx + x] = (sums[0] + sums[1]) + (sums[2] + sums[3]);
}

void dslash_norm(const FineOpView<double>& op, const double2* in, double2* out, bool g5, double* partial,
                 hipStream_t s, int nb) {
  const long long fs = (long long)op.nblk * 192;
  const int gx = dslash_norm_parts(op.nblk);
  const bool nt = op_streams<double2>(op.nblk, nb);
  const auto k = g5 ? (nt ? k_dslash_norm<true, true> : k_dslash_norm<true, false>)
                    : (nt ? k_dslash_norm<false, true> : k_dslash_norm<false, false>);
  k<<<gx * nb, 256, 0, s>>>(op, in, out, partial, fs, gx, nb);
  DD_LAUNCH_CHECK();
}

// The stencil on canonical complex128 fields, without native copies of them:
// a site's spinor is 192 contiguous bytes to read, and the workgroup's 4^4
// tile of results goes through LDS to be written in rows of four sites (768
// bytes).  FP64 on 48^3x96: 4334 us, against 6829 us with a conversion
// before and after the native stencil (1264 and 1063 us).
template <typename T, typename S, bool NT>
__global__ void __launch_bounds__(256) k_dslash_canonical(FineOpView<T, S> op, DevGeom g,
                                                          const double2* in, double2* out, int gx, int nb) {
  constexpr int PITCH = 13;
  __shared__ C<T> tile[256 * PITCH];
  int x, r;
  xcd_slab_rhs<S>(blockIdx.x, gx, nb, x, r);
  const int t = threadIdx.x, blk = x * 16 + (t >> 4), loc = t & 15;
  const int nt[4] = {g.nb[0] >> 1, g.nb[1] >> 1, g.nb[2] >> 1, g.nb[3] >> 1};
  int tc[4];
  tile_decode(nt, x, tc);
  CanonIn<T> f;
  f.place(g, in + (long long)r * g.V * 12, tc, t);
  C<T> o[12];
  dslash_site<T, S, NT>(op, f, blk, loc, o);
#pragma unroll
  for (int c = 0; c < 12; ++c) tile[t * PITCH + c] = o[c];
  __syncthreads();
  out += (long long)r * g.V * 12;
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const int e = 256 * k + t, row = e / 48, q = e - 48 * row, xs = q / 12, c = q - 12 * xs;
    const int ys = row & 3, zs = (row >> 2) & 3, ts = row >> 4;
    const int src = (xs & 1) | (ys & 1) << 1 | (zs & 1) << 2 | (ts & 1) << 3 | (xs >> 1) << 4 | (ys >> 1) << 5 |
                    (zs >> 1) << 6 | (ts >> 1) << 7;
    const long long site = 4 * tc[0] + (long long)g.X * (4 * tc[1] + ys + (long long)g.Y * (4 * tc[2] + zs + (long long)g.Z * (4 * tc[3] + ts)));
    store_nt(out + site * 12 + q, ccast<double>(tile[src * PITCH + c]));
  }
}

// The stencil of a small lattice: four wavefronts share 64 sites, wavefront mu
// doing both hops of direction mu (and two of them a chirality of the clover
// each), summed through LDS.  w: the wavefront, lane: its site; on return
// acc[3 w .. 3 w + 2] are those components of (D in)(x).
template <typename T, typename S, typename In>
__device__ inline void dslash_split_site(const FineOpView<T, S>& op, const In& f, int w, int lane, int blk, int loc,
                                         C<T> (*part)[12][64], C<T> (&acc)[12]) {
  const Nbr8 nb8 = load_nbr8(op.nbr, blk);
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = czero<T>();
  if (w == 0) hops_mu<T, S, 0>(op, f, blk, loc, nb8, acc);
  else if (w == 1) hops_mu<T, S, 1>(op, f, blk, loc, nb8, acc);
  else if (w == 2) hops_mu<T, S, 2>(op, f, blk, loc, nb8, acc);
  else hops_mu<T, S, 3>(op, f, blk, loc, nb8, acc);
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = cscale(acc[c], T(-0.5));
  if (w < 2) {
    C<T> psi[12], av[6];
    f.site(blk, loc, psi);
    C<T> v[6];
    S e[18];
    if (w) load_entries<18, 18>(op.A, blk, loc, e);
    else load_entries<0, 18>(op.A, blk, loc, e);
#pragma unroll
    for (int c = 0; c < 6; ++c) v[c] = w ? psi[6 + c] : psi[c];
    clover_block<T>(0, [&](int k) { return ldc<T, S>(e[k]); }, v, av);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      if (w) acc[6 + c] = cadd(acc[6 + c], av[c]);
      else acc[c] = cadd(acc[c], av[c]);
    }
  }
  // wavefront w sums components 3w .. 3w + 2, its own from registers
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    const int o = c / 3;
    if (o != w) part[o < w ? w - 1 : w][c][lane] = acc[c];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 12; ++c)
    if (c / 3 == w)
#pragma unroll
      for (int k = 0; k < 3; ++k) acc[c] = cadd(acc[c], part[k][c][lane]);
}

// (grid: gx groups of four blocks per field; nblk is a multiple of 16)
template <typename T, typename S, typename V>
__global__ void __launch_bounds__(256) k_dslash_split(FineOpView<T, S> op, const V* __restrict__ in,
                                                      const float* __restrict__ ins, C<T>* __restrict__ out,
                                                      long long fs, int gx) {
  __shared__ C<T> part[3][12][64];
  const int x = blockIdx.x % gx, r = blockIdx.x / gx;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int blk = x * 4 + (lane >> 4), loc = lane & 15;
  const long long off = r * fs;
  C<T> acc[12];
  dslash_split_site<T, S>(op, NativeIn<T, V>{in + off, std::is_same<V, __half2>::value ? ins + off / 12 : nullptr}, w,
                          lane, blk, loc, part, acc);
  C<T>* po = out + off + (long long)blk * 192 + loc;
#pragma unroll
  for (int c = 0; c < 12; ++c)
    if (c / 3 == w) po[c * 16] = acc[c];
}
// the same on canonical fields
template <typename T, typename S>
__global__ void __launch_bounds__(256) k_dslash_split_canonical(FineOpView<T, S> op, DevGeom g, const double2* in,
                                                                double2* out, int gx) {
  __shared__ C<T> part[3][12][64];
  const int x = blockIdx.x % gx, r = blockIdx.x / gx;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int blk = x * 4 + (lane >> 4), loc = lane & 15;
  const int nt[4] = {g.nb[0] >> 1, g.nb[1] >> 1, g.nb[2] >> 1, g.nb[3] >> 1};
  int tc[4];
  tile_decode(nt, x >> 2, tc);
  CanonIn<T> f;
  f.place(g, in + (long long)r * g.V * 12, tc, (blk & 15) * 16 + loc);
  C<T> acc[12];
  dslash_split_site<T, S>(op, f, w, lane, blk, loc, part, acc);
  double2* po = out + ((long long)r * g.V + f.own) * 12;
#pragma unroll
  for (int c = 0; c < 12; ++c)
    if (c / 3 == w) po[c] = ccast<double>(acc[c]);
}

// Largest grid (in workgroups of 256 sites) that is split: below it the device
// is not filled and a call takes as long as one site's chain of loads.  Kernel
// and launch in us, one site per thread / split, FP64: 4096 sites 9.3 / 7.4,
// 16384 sites 10.1 / 8.8, 32768 sites 13.8 / 16.2.
constexpr unsigned DSLASH_SPLIT = 64;

template <typename T, typename S, typename V>
static void dslash_launch(const FineOpView<T, S>& op, const V* in, const float* ins, C<T>* out, hipStream_t s, int nb) {
  const long long fs = (long long)op.nblk * 192;
  const unsigned gx = nblocks((size_t)op.nblk * 16, 256);
  if (gx * nb <= DSLASH_SPLIT) {
    const unsigned g4 = op.nblk / 4;
    k_dslash_split<T, S, V><<<g4 * nb, 256, 0, s>>>(op, in, ins, out, fs, (int)g4);
  } else if (op_streams<S>(op.nblk, nb)) {
    k_dslash<T, S, V, true><<<gx * nb, 256, 0, s>>>(op, in, ins, out, fs, (int)gx, nb);
  } else {
    k_dslash<T, S, V, false><<<gx * nb, 256, 0, s>>>(op, in, ins, out, fs, (int)gx, nb);
  }
  DD_LAUNCH_CHECK();
}

template <typename T, typename S>
void dslash_canonical(const FineGeom& g, const FineOpView<T, S>& op, const double2* in, double2* out, hipStream_t s,
                      int nb) {
  const unsigned gx = op.nblk / 16;
  // (the same line as for native fields: both give the same bits)
  if (gx * nb <= DSLASH_SPLIT)
    k_dslash_split_canonical<T, S><<<4 * gx * nb, 256, 0, s>>>(op, devgeom(g), in, out, (int)(4 * gx));
  else if (op_streams<S>(op.nblk, nb))
    k_dslash_canonical<T, S, true><<<gx * nb, 256, 0, s>>>(op, devgeom(g), in, out, (int)gx, nb);
  else
    k_dslash_canonical<T, S, false><<<gx * nb, 256, 0, s>>>(op, devgeom(g), in, out, (int)gx, nb);
  DD_LAUNCH_CHECK();
}
template void dslash_canonical<double, double2>(const FineGeom&, const FineOpView<double>&, const double2*, double2*,
                                                hipStream_t, int);
template void dslash_canonical<float, float2>(const FineGeom&, const FineOpView<float>&, const double2*, double2*,
                                              hipStream_t, int);
template void dslash_canonical<float, __half2>(const FineGeom&, const FineOpView<float, __half2>&, const double2*,
                                               double2*, hipStream_t, int);

template <typename T, typename S>
void dslash(const FineOpView<T, S>& op, const C<T>* in, C<T>* out, hipStream_t s, int nb) {
  dslash_launch<T, S, C<T>>(op, in, nullptr, out, s, nb);
}

void dslash_hs(const FineOpView<double>& op, const __half2* in, const float* ins, double2* out, hipStream_t s,
               int nb) {
  dslash_launch<double, double2, __half2>(op, in, ins, out, s, nb);
}

// ---------------------------------------------------------------------------
// SAP colour pass.  Two lanes per site: lanes 0-15 of a 32-lane group take a 2^4
// block's sites with p = 0, lanes 16-31 the same sites with p = 1; a wavefront
// holds two blocks and is a workgroup by itself, so no wave waits for another.
// A batch of fields runs one field per workgroup with the XCD-aware mapping.
// r = b - D z with the full operator (the blocks' z staged in LDS: the in-block
// neighbours come from there, the others from memory), then mr_iters minimal
// residual steps on the Dirichlet block operator D_i (self term + the four
// in-block hops, partner spinors exchanged through LDS, block sums of the step
// sizes by DPP row moves), z += x.
//
// Lane p of a site holds its chirality p (six components) and that half of the
// clover, and computes the hops of directions x, y (p = 0) or z, t (p = 1) for
// all four spins; the partial sums of the other chirality then change lanes
// (row swaps).  x and z both project with phases +-i, y and t with +-1, so both
// lanes run the same instructions with signs of their own, and links are
// loaded and turned (U for the lower site of a pair, U^H for the upper one)
// once per site, not once per lane.  A lane keeps its links, and with FP16
// storage its clover, in registers for the pass.
// ---------------------------------------------------------------------------
constexpr int SAP_WG = 64;

// (a, b) of lane rows (16 lanes) r and r + 1, r even: a of row r + 1 changes
// places with b of row r
__device__ inline void row_swap(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ inline void row_swap(double& a, double& b) {
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  a = __hiloint2double((int)hi[0], (int)lo[0]);
  b = __hiloint2double((int)hi[1], (int)lo[1]);
}

// the sum of v over the 32 lanes of a block, in each of them
template <typename T> __device__ inline T block_sum(T v) {
  T a = sum16<T>(v), b = a;
  row_swap(a, b);
  return a + b;
}

// NE operator entries of a site from E0 (lane p = 0) or E0 + 18 (p = 1)
template <int E0, int NE, bool NT = false, typename S>
__device__ inline void load_entries_pair(const S* __restrict__ d, int blk, int loc, int p, S (&e)[NE]) {
  constexpr int N = OpChunk<S>::N, Q0 = E0 / N, Q1 = (E0 + 18) / N, O0 = E0 % N, O1 = (E0 + 18) % N;
  constexpr int NQ = ((O0 > O1 ? O0 : O1) + NE + N - 1) / N;
  static_assert(Q1 + NQ <= 36 / N, "past the site's entries");
  S raw[NQ * N];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = (p ? Q1 : Q0) + q;
    const OpChunk<S> c = NT ? load_chunk_nt<S>(d, blk, loc, i) : load_chunk<S>(d, blk, loc, i);
#pragma unroll
    for (int k = 0; k < N; ++k) raw[q * N + k] = c.v[k];
  }
#pragma unroll
  for (int k = 0; k < NE; ++k) {
    if constexpr (O0 == O1) e[k] = raw[O0 + k];
    else e[k] = p ? raw[O1 + k] : raw[O0 + k];
  }
}

// o = dag ? e^H : e for a stored 3x3 link: a select with a negated source for
// each real and imaginary part; FP16 pairs in one select and a sign flip
template <typename S> __device__ inline void orient(const S (&e)[9], bool dag, S (&o)[9]) {
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      S v = dag ? e[b * 3 + a] : e[a * 3 + b];
      if constexpr (std::is_same<S, __half2>::value)
        v = __builtin_bit_cast(S, __builtin_bit_cast(unsigned, v) ^ (dag ? 0x80000000u : 0u));
      else
        v.y = dag ? -v.y : v.y;
      o[a * 3 + b] = v;
    }
}

// The direction of step ST (0: x or z, 1: y or t) as a bit of the site index
__device__ inline int pair_bit(int ST, int p) { return (p ? 4 : 1) << ST; }

// A lane's partial sums of the hops: spins 2 and 3 (l1, l2), and the upper
// spins they are projected with: u1 spin 1 - p, u2 spin p
template <typename T> struct PairAcc {
  C<T> u1[3], u2[3], l1[3], l2[3];
};

// One projected hop of step ST; psi(i, a): i = 0, 1 the spins of u1, u2, i = 2,
// 3 spins 2, 3.  sg = 1 (forward) or -1; the phases of the first pair are sg
// i (x and z) or -sg (y and t), those of the second +-sg i, +-sg, - for p = 1.
// The result is multiplied by m (the scale of FP16 spinors: applied in the
// accumulation it costs nothing) and added to acc, or replaces it (FIRST).
// MIX: links in FP16, which enter an fma unconverted, so there is no product
// without one.
template <typename T, int ST, bool FIRST, bool SCALED, bool MIX, typename G>
__device__ inline void pair_hop(G&& psi, T sg, int p, const C<T> (&u)[9], T m, PairAcc<T>& acc) {
  const T s1 = ST ? -sg : sg, s2 = p ? -sg : sg;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const T s = i ? s2 : s1;
    C<T>(&up)[3] = i ? acc.u2 : acc.u1;
    C<T>(&lo)[3] = i ? acc.l2 : acc.l1;
    C<T> h[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const C<T> v = psi(i, a);
      const C<T> w = ST ? psi(2 + i, a) : cmuli(psi(2 + i, a));
      h[a] = mk<T>(fma(s, w.x, v.x), fma(s, w.y, v.y));
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      C<T> v;
      if constexpr (MIX) {
        v = czero<T>();
        cfma(v, u[a * 3], h[0]);
      } else {
        v = cmul(u[a * 3], h[0]);
      }
      cfma(v, u[a * 3 + 1], h[1]);
      cfma(v, u[a * 3 + 2], h[2]);
      const C<T> w = ST ? v : cmulmi(v);
      const T sm = SCALED ? s * m : s;
      if constexpr (FIRST) {
        up[a] = SCALED ? cscale(v, m) : v;
        lo[a] = cscale(w, sm);
      } else {
        up[a] = SCALED ? mk<T>(fma(m, v.x, up[a].x), fma(m, v.y, up[a].y)) : cadd(up[a], v);
        lo[a] = mk<T>(fma(sm, w.x, lo[a].x), fma(sm, w.y, lo[a].y));
      }
    }
  }
}

// the sum of both lanes' partial sums, each lane its chirality
template <typename T> __device__ inline void pair_total(PairAcc<T>& acc, int p, C<T> (&o)[6]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    // afterwards (p = 0 | 1): u1 spin 1 | 3, l2 spin 0 | 3, u2 spin 0 | 2, l1 spin 1 | 2
    row_swap(acc.u1[a].x, acc.l2[a].x);
    row_swap(acc.u1[a].y, acc.l2[a].y);
    row_swap(acc.u2[a].x, acc.l1[a].x);
    row_swap(acc.u2[a].y, acc.l1[a].y);
    o[a] = cadd(acc.u2[a], p ? acc.l1[a] : acc.l2[a]);
    o[3 + a] = cadd(acc.u1[a], p ? acc.l2[a] : acc.l1[a]);
  }
}

// the in-block hop of step ST from the components staged in LDS (rs: the block's
// [12][16]) with the link as the site applies it
template <typename T, int ST, bool FIRST, typename S>
__device__ inline void pair_inblock(const C<T>* rs, int loc, int p, const S (&o)[9], PairAcc<T>& acc) {
  const int bit = pair_bit(ST, p);
  const C<T>* r = rs + (loc ^ bit);
  C<T> u[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) u[k] = ldc<T, S>(o[k]);
  const int f1 = p ? 0 : 48, f2 = p ? 48 : 0;
  pair_hop<T, ST, FIRST, false, std::is_same<S, __half2>::value>(
      [&](int i, int a) { return r[i >= 2 ? (3 * i + a) * 16 : (i ? f2 : f1) + a * 16]; },
      (loc & bit) ? T(-1) : T(1), p, u, T(1), acc);
}

// The in-block link of step ST as the site applies it: the link joining loc and
// loc ^ bit belongs to the lower site, which applies U; the upper site applies
// U^H (the transposed entries, conjugated).
template <int ST, typename S>
__device__ inline void pair_link(const S* __restrict__ U, int blk, int loc, int p, S (&o)[9]) {
  const int bit = pair_bit(ST, p);
  S e[9];
  load_entries_pair<9 * ST, 9>(U, blk, loc & ~bit, p, e);
  orient(e, (loc & bit) != 0, o);
}

// The out-of-block hop of step ST in the residual of a block site: the
// neighbour outside the block is x+mu for the upper site of the pair (link
// U_mu(x), the site's own) and x-mu for the lower one (link U_mu(x-mu) of the
// neighbour block's site, applied as U^H).
template <typename T, typename S, typename V, int ST>
__device__ inline void pair_outer(const FineOpView<T, S>& op, const V* __restrict__ in, const float* __restrict__ ins,
                                  int blk, int loc, int p, int nbf, int nbb, PairAcc<T>& acc) {
  const int bit = pair_bit(ST, p);
  const bool up = loc & bit;
  const int nb = up ? nbf : nbb;
  const V* f = in + (long long)nb * 192 + (loc ^ bit);
  const int f1 = p ? 0 : 48, f2 = p ? 48 : 0;
  V raw[12];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int a = 0; a < 3; ++a) raw[3 * i + a] = f[i >= 2 ? (3 * i + a) * 16 : (i ? f2 : f1) + a * 16];
  float m = 1.f;
  if constexpr (std::is_same<V, __half2>::value) m = ins[(long long)nb * 16 + (loc ^ bit)];
  S e[9], o[9];
  load_entries_pair<9 * ST, 9>(op.U, up ? blk : nb, up ? loc : loc ^ bit, p, e);
  orient(e, !up, o);
  C<T> u[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) u[k] = ldc<T, S>(o[k]);
  pair_hop<T, ST, ST == 0, std::is_same<V, __half2>::value, std::is_same<S, __half2>::value>(
      [&](int i, int a) { return ldc<T, V>(raw[3 * i + a]); }, up ? T(1) : T(-1), p, u, T(m), acc);
}

// Whether a colour pass keeps its clover entries in registers for the MR steps
// (FP16 storage: 18 registers) or reads them again at every step
template <typename S> struct ClKeep : std::false_type {};
template <> struct ClKeep<__half2> : std::true_type {};

// One workgroup per (two blocks, field of the batch), gx pairs of blocks;
// b and z in spinor storage V (bs, zs: their site scales for FP16).
//
// Bound by its vector instructions on batches (about 2500 a lane, two lanes a
// site, at three waves per SIMD; one lane a site: 4335 at two), by memory for
// one field of a large lattice, by latency on a small one, where the two lanes
// double the wavefronts.  Five sweeps, one lane a site in workgroups of four wavefronts / of one / this:
// 32^3x64 FP16 operators 2264 / 2128 / 1915 us; 16^3x32 x 12 FP32 fields 1496 /
// 1410 / 1358; per pass, 12 FP16 fields of 24^3x48 682 / 666 / 667, one FP32
// field of 16^3x32 24.5 / 22.9 / 19.5; FP64 (two sweeps, 5 fields) - / 650 / 543.
// Held to three waves per SIMD in FP32 (two: FP16 12-field pass 718).
//
// What is read once in a pass (b) goes past the caches, and with NT (op_streams)
// the result and the clover that is kept too: two sweeps on one field of 32^4
// with FP16 operators 375 -> 360 us, of 32^3x64 779 -> 752 (a batch's z is found
// again in the last-level cache: 4 fields of 24^4 413 us, 439 if not).
template <typename T, typename S, typename V, bool NT>
__global__ void __launch_bounds__(SAP_WG, sizeof(T) == 8 ? 2 : 3)
k_sap_colour(FineOpView<T, S> op, const int* __restrict__ cblk,
             int mr_iters, const V* __restrict__ b, const float* __restrict__ bs, V* __restrict__ z,
             float* __restrict__ zs, int nb, long long fs, int gx) {
  __shared__ C<T> rsm[2 * 192];
  constexpr bool HS = std::is_same<V, __half2>::value;
  constexpr bool KEEP = !std::is_same<T, double>::value;
  constexpr bool CK = ClKeep<S>::value;
  const int t = threadIdx.x, loc = t & 15, p = (t >> 4) & 1;
  int xw, rw;
  xcd_slab_rhs<S>(blockIdx.x, gx, nb, xw, rw);
  b += (long long)rw * fs;
  z += (long long)rw * fs;
  if constexpr (HS) {
    bs += (long long)rw * (fs / 12);
    zs += (long long)rw * (fs / 12);
  }
  const int blk = cblk[xw * 2 + (t >> 5)];
  C<T>* rs = rsm + (t >> 5) * 192;           // the block's components [12][16]
  C<T>* own = rs + p * 96 + loc;             // the lane's: own[c * 16]
  const long long so = (long long)blk * 192 + p * 96 + loc, sc = (long long)blk * 16 + loc;

  V zkeep[6];
  float zsk = 1.f, bsk = 1.f;
#pragma unroll
  for (int c = 0; c < 6; ++c) zkeep[c] = z[so + c * 16];
  if constexpr (HS) zsk = zs[sc];
  S ul[KEEP ? 2 : 1][9];
  if constexpr (KEEP) {
    pair_link<0>(op.U, blk, loc, p, ul[0]);
    pair_link<1>(op.U, blk, loc, p, ul[1]);
  }
  S ce[18];
  if constexpr (CK) load_entries_pair<0, 18, NT>(op.A, blk, loc, p, ce);
  const int* nbr = op.nbr + (long long)blk * 8 + (p ? 4 : 0);
  const int4 nb4 = *reinterpret_cast<const int4*>(nbr);
  V braw[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) braw[c] = load_nt(b + so + c * 16);
  if constexpr (HS) bsk = bs[sc];

  auto decode = [&](V v, float m) {
    C<T> w = ldc<T, V>(v);
    if constexpr (HS) w = mk<T>(w.x * T(m), w.y * T(m));
    return w;
  };
  // acc (+)= the in-block hops of what is staged; q = A (own) - 1/2 total
  PairAcc<T> acc;
  auto inblock = [&](auto first) {
    constexpr bool F = decltype(first)::value;
    if constexpr (!KEEP) pair_link<0>(op.U, blk, loc, p, ul[0]);
    pair_inblock<T, 0, F>(rs, loc, p, ul[0], acc);
    if constexpr (!KEEP) pair_link<1>(op.U, blk, loc, p, ul[0]);
    pair_inblock<T, 1, false>(rs, loc, p, ul[KEEP ? 1 : 0], acc);
  };
  auto diag = [&](const C<T> (&v)[6], C<T> (&o)[6]) {
    if constexpr (!CK) load_entries_pair<0, 18>(op.A, blk, loc, p, ce);
    clover_block<T>(0, [&](int k) { return ldc<T, S>(ce[k]); }, v, o);
    C<T> h[6];
    pair_total<T>(acc, p, h);
#pragma unroll
    for (int c = 0; c < 6; ++c) o[c] = mk<T>(rfma(T(-0.5), h[c].x, o[c].x), rfma(T(-0.5), h[c].y, o[c].y));
  };

  C<T> rho[6], x[6], q[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    rho[c] = decode(zkeep[c], zsk);
    own[c * 16] = rho[c];
    x[c] = czero<T>();
  }
  __syncthreads();
  pair_outer<T, S, V, 0>(op, z, zs, blk, loc, p, nb4.x, nb4.y, acc);
  pair_outer<T, S, V, 1>(op, z, zs, blk, loc, p, nb4.z, nb4.w, acc);
  inblock(std::false_type{});
  diag(rho, q);
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    const C<T> bb = decode(braw[c], bsk);
    rho[c] = mk<T>(bb.x - q[c].x, bb.y - q[c].y);
  }

  for (int it = 0; it < mr_iters; ++it) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 6; ++c) own[c * 16] = rho[c];
    __syncthreads();
    inblock(std::true_type{});
    diag(rho, q);
    T qr_re = 0, qr_im = 0, qq = 0;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      qr_re = rfma(q[c].x, rho[c].x, qr_re);
      qr_re = rfma(q[c].y, rho[c].y, qr_re);
      qr_im = rfma(q[c].x, rho[c].y, qr_im);
      qr_im = rfma(-q[c].y, rho[c].x, qr_im);
      qq = rfma(q[c].x, q[c].x, qq);
      qq = rfma(q[c].y, q[c].y, qq);
    }
    qr_re = block_sum<T>(qr_re);
    qr_im = block_sum<T>(qr_im);
    qq = block_sum<T>(qq);
    const T iq = qq > T(0) ? T(1) / qq : T(0);
    const C<T> alpha = mk<T>(qr_re * iq, qr_im * iq);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      cfma(x[c], alpha, rho[c]);
      cfma(rho[c], mk<T>(-alpha.x, -alpha.y), q[c]);
    }
  }
  // z + x (for FP16 spinors re-encoded with the site's new scale)
#pragma unroll
  for (int c = 0; c < 6; ++c) x[c] = cadd(decode(zkeep[c], zsk), x[c]);
  if constexpr (HS) {
    float m = 0.f;
#pragma unroll
    for (int c = 0; c < 6; ++c) m = fmaxf(m, fmaxf(fabsf(x[c].x), fabsf(x[c].y)));
    float m2 = m;
    row_swap(m, m2);
    m = fmaxf(m, m2);
    const float inv = m > 0.f ? 1.f / m : 0.f;
    if (p == 0) zs[sc] = m;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const __half2 h = __floats2half2_rn(x[c].x * inv, x[c].y * inv);
      if constexpr (NT) store_nt(z + so + c * 16, h);
      else z[so + c * 16] = h;
    }
  } else {
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      if constexpr (NT) store_nt(z + so + c * 16, x[c]);
      else z[so + c * 16] = x[c];
    }
  }
}


template <typename T, typename S>
void sap_colour(const FineOpView<T, S>& op, const int* colour_blocks, int colour, int mr_iters,
                const C<T>* b, C<T>* z, hipStream_t s, int nb) {
  const int ncb = op.nblk / 2;
  const long long fs = (long long)op.nblk * 192;
  const unsigned gx = ncb / 2;   // (extents are multiples of 4: a colour has 8k blocks)
  const auto k = op_streams<S>(op.nblk, nb) ? k_sap_colour<T, S, C<T>, true> : k_sap_colour<T, S, C<T>, false>;
  k<<<gx * nb, SAP_WG, 0, s>>>(op, colour_blocks + colour * ncb, mr_iters, b, nullptr, z, nullptr, nb, fs, (int)gx);
  DD_LAUNCH_CHECK();
}

void sap_colour_hs(const FineOpView<float, __half2>& op, const int* colour_blocks, int colour, int mr_iters,
                   const __half2* b, const float* bs, __half2* z, float* zs, hipStream_t s, int nb) {
  const int ncb = op.nblk / 2;
  const long long fs = (long long)op.nblk * 192;
  const unsigned gx = ncb / 2;   // (extents are multiples of 4: a colour has 8k blocks)
  const auto k = op_streams<__half2>(op.nblk, nb) ? k_sap_colour<float, __half2, __half2, true>
                                                  : k_sap_colour<float, __half2, __half2, false>;
  k<<<gx * nb, SAP_WG, 0, s>>>(op, colour_blocks + colour * ncb, mr_iters, b, bs, z, zs, nb, fs, (int)gx);
  DD_LAUNCH_CHECK();
}

// explicit instantiations
#define DD_INST(T)                                                                              \
  template void fine_to_native<T>(const FineGeom&, const double2*, C<T>*, int, hipStream_t);   \
  template void fine_from_native<T>(const FineGeom&, const C<T>*, double2*, int, hipStream_t); \
  template void dslash<T, C<T>>(const FineOpView<T, C<T>>&, const C<T>*, C<T>*, hipStream_t, int); \
  template void sap_colour<T, C<T>>(const FineOpView<T, C<T>>&, const int*, int, int, const C<T>*, \
                                    C<T>*, hipStream_t, int);
DD_INST(double)
DD_INST(float)
#undef DD_INST
template void dslash<float, __half2>(const FineOpView<float, __half2>&, const float2*, float2*, hipStream_t,
                                    int);
template void sap_colour<float, __half2>(const FineOpView<float, __half2>&, const int*, int, int, const float2*,
                                         float2*, hipStream_t, int);

// one thread per site and field: largest |re|, |im| of the 12 components,
// the components divided by it rounded to FP16, and their decoded FP64 value
__global__ void k_encode_sites(const float2* __restrict__ in, __half2* __restrict__ half, float* __restrict__ scale,
                               double2* __restrict__ dec, int nblk) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int blk = tid >> 4, loc = tid & 15;
  if (blk >= nblk) return;
  const long long fs = (long long)nblk * 192, off = (long long)blockIdx.y * fs + (long long)blk * 192 + loc;
  float2 v[12];
  float m = 0.f;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    v[c] = in[off + c * 16];
    m = fmaxf(m, fmaxf(fabsf(v[c].x), fabsf(v[c].y)));
  }
  const float inv = m > 0.f ? 1.f / m : 0.f;
  scale[(long long)blockIdx.y * nblk * 16 + (long long)blk * 16 + loc] = m;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    const __half2 h = __floats2half2_rn(v[c].x * inv, v[c].y * inv);
    half[off + c * 16] = h;
    const float2 r = __half22float2(h);
    dec[off + c * 16] = make_double2((double)r.x * m, (double)r.y * m);
  }
}

void encode_sites(const FineGeom& g, const float2* in, __half2* half, float* scale, double2* dec, int nb,
                  hipStream_t s) {
  k_encode_sites<<<dim3(nblocks((size_t)g.nblk * 16, 256), nb), 256, 0, s>>>(in, half, scale, dec, g.nblk);
  DD_LAUNCH_CHECK();
}

template <typename T>
__global__ void k_encode_h(const C<T>* __restrict__ in, __half2* __restrict__ half, float* __restrict__ scale,
                           int nblk) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int blk = tid >> 4, loc = tid & 15;
  if (blk >= nblk) return;
  const long long fs = (long long)nblk * 192, ss = (long long)nblk * 16, r = blockIdx.y;
  C<T> v[12];
  load_spinor<T>(in + r * fs, blk, loc, v);
  store_site<T, __half2>(half + r * fs, scale + r * ss, blk, loc, v);
}
template <typename T>
__global__ void k_decode_h(const __half2* __restrict__ half, const float* __restrict__ scale, C<T>* __restrict__ out,
                           int nblk) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int blk = tid >> 4, loc = tid & 15;
  if (blk >= nblk) return;
  const long long fs = (long long)nblk * 192, ss = (long long)nblk * 16, r = blockIdx.y;
  C<T> v[12];
  load_site<T, __half2>(half + r * fs, scale + r * ss, blk, loc, v);
  C<T>* o = out + r * fs + (long long)blk * 192 + loc;
#pragma unroll
  for (int c = 0; c < 12; ++c) o[c * 16] = v[c];
}
template <typename T>
void encode_h(const FineGeom& g, const C<T>* in, __half2* half, float* scale, int nb, hipStream_t s) {
  k_encode_h<T><<<dim3(nblocks((size_t)g.nblk * 16, 256), nb), 256, 0, s>>>(in, half, scale, g.nblk);
  DD_LAUNCH_CHECK();
}
template <typename T>
void decode_h(const FineGeom& g, const __half2* half, const float* scale, C<T>* out, int nb, hipStream_t s) {
  k_decode_h<T><<<dim3(nblocks((size_t)g.nblk * 16, 256), nb), 256, 0, s>>>(half, scale, out, g.nblk);
  DD_LAUNCH_CHECK();
}
template void encode_h<double>(const FineGeom&, const double2*, __half2*, float*, int, hipStream_t);
template void encode_h<float>(const FineGeom&, const float2*, __half2*, float*, int, hipStream_t);
template void decode_h<double>(const FineGeom&, const __half2*, const float*, double2*, int, hipStream_t);
template void decode_h<float>(const FineGeom&, const __half2*, const float*, float2*, int, hipStream_t);

}  // namespace ddamg
