// Matrix-core kernels of the coarse level (see coarse_mfma.h).
#pragma once

#include <algorithm>
#include <type_traits>

#include "coarse_dev.h"
#include "coarse_mfma.h"
#include "fine_dev.h"

namespace ddamg {

// ---------------------------------------------------------------------------
// Batches on the matrix cores (FP32 arithmetic, up to 16 right-hand sides per
// launch chunk).  Per site the product is a complex GEMM
//   out (d x nr) = [K_k, k in mask] (d x ns d)  *  [in(nbr_k); ..] (ns d x nr),
// done as real 16x16x4 MFMA tiles: rows i of a 16-row tile, right-hand side r
// in the 16 columns, four complex GEMM columns per step and four real
// products per step (Cr += Ar Br - Ai Bi, Ci += Ar Bi + Ai Br).  A workgroup
// is one site with G wavefronts per row tile that share the site's operator
// blocks (mfma_shape says how many); the first of them gets the sum (mfma_join)
// and holds its rows of the result complete in registers, where the epilogue
// works on them.  The A operand goes from memory straight to registers, several blocks in
// flight before the workgroup waits for its input vectors; the B operand
// (the input vectors of every right-hand side) is staged in LDS with
// contiguous reads along a site's components, the pitch odd so that neither
// the staging writes (components along the lanes) nor the operand reads
// (right-hand sides along the lanes) meet on a bank (even only where the tile
// would not fit otherwise).
// Operand layout of v_mfma_f32_16x16x4f32: lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16]; result register v of lane l is D[4 (l / 16) + v][l % 16].
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int MFMA_NB = 16;        // right-hand sides per launch chunk

// the s-th set bit of a block mask, -1 past the last
__device__ inline int mask_slot(unsigned mask, int s) {
  for (; s > 0; --s) mask &= mask - 1u;
  return mask ? __builtin_ctz(mask) : -1;
}
// the index of this wavefront in its workgroup, in a scalar register
__device__ inline int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// One wavefront's 16 rows of every G-th operator block of a site from the g-th
// on: a ring of DEP blocks in registers, the next block loaded where one has
// been applied (deeper rings cost a wavefront per SIMD: 7 % slower)
template <typename S, int NJ, int G>
struct MfmaRows {
  static constexpr int DEP = 2;
  S a[DEP][NJ];
  const S* Kx;
  unsigned mask;
  int ns, d, lo, kk, g;
  __device__ __forceinline__ void load(int u, int s) {
    const S* Kb = Kx + (unsigned)(mask_slot(mask, s) * d * d);
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
      // columns past d repeat column d - 1 (they meet zero rows of B)
      const unsigned o = (t + 1) * 4 <= d ? (unsigned)(lo + (4 * t + kk) * d) : (unsigned)(lo + min(4 * t + kk, d - 1) * d);
      a[u][t] = Kb[o];
    }
  }
  __device__ __forceinline__ void prefetch(const S* __restrict__ Kx_, unsigned mask_, int row, int kk_, int d_, int g_) {
    Kx = Kx_;
    mask = mask_;
    ns = __builtin_popcount(mask_);
    d = d_;
    lo = row;
    kk = kk_;
    g = g_;
#pragma unroll
    for (int u = 0; u < DEP; ++u)
      if (g + u * G < ns) load(u, g + u * G);
  }
  // lds_b: [ns][4 NJ][pitch], this lane's column rl
  __device__ __forceinline__ void apply(const float2* lds_b, int pitch, int rl, f32x4& cr, f32x4& ci) {
    cr = {0.f, 0.f, 0.f, 0.f};
    ci = {0.f, 0.f, 0.f, 0.f};
    const float2* bt = lds_b + kk * pitch + rl;
#pragma unroll 1
    for (int s0 = g; s0 < ns; s0 += DEP * G) {
#pragma unroll
      for (int u = 0; u < DEP; ++u)
        if (s0 + u * G < ns) {
          // summed per block, then over the blocks: shorter chains of FP32
          // additions than one running sum over all columns
          f32x4 br = {0.f, 0.f, 0.f, 0.f}, bi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int t = 0; t < NJ; ++t) {
            const float2 av = ldc<float, S>(a[u][t]);
            const float2 bv = bt[((s0 + u * G) * 4 * NJ + 4 * t) * pitch];
            br = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, br, 0, 0, 0);
            bi = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.y, bi, 0, 0, 0);
            br = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.y, bv.y, br, 0, 0, 0);
            bi = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.x, bi, 0, 0, 0);
          }
          cr += br;
          ci += bi;
          if (s0 + (u + DEP) * G < ns) load(u, s0 + (u + DEP) * G);
        }
    }
  }
};

// FP16 storage.  The matrix cores multiply FP16 numbers 16 times as fast as FP32
// ones and sum the exact products in FP32, so the operator enters as it is
// stored and an input vector x in two FP16 parts of a common power of two per
// (block, right-hand side), hi = fp16(x s) and mid = fp16(2^11 (x s - hi)):
// together 23 bits of x, one unit in its last FP32 place, and entries far below
// the largest of their (block, right-hand side) to 2^-50 of that (see split_row).
// A lane's four columns t, each (re, im), are eight consecutive k of
// v_mfma_f32_16x16x32_f16 in both operands: lane l supplies A[l % 16][8 (l / 16)
// ..] and B[8 (l / 16) ..][l % 16], the result as for the FP32 instruction.  The real part's B holds
// (re, -im), the imaginary part's (im, re).  Error against 64 bits of five SAP
// sweeps, vector kernels / FP32 products / this: d = 16 1.71e-7 / 1.36e-7 /
// 1.10e-7, d = 40 2.64e-7 / 1.96e-7 / 1.28e-7, d = 64 3.37e-7 / 2.43e-7 /
// 1.34e-7, the same where the components of a field spread over six decades;
// five sweeps on 12 fields of 8^3x16 sites 4090 us with FP32 products, 3410 so.
template <int NJ, int G>
struct MfmaRows<__half2, NJ, G> {
  static constexpr int DEP = 2;
  unsigned a[DEP][NJ];
  const unsigned* Kx;
  unsigned mask;
  int ns, d, lo, kk, g;
  __device__ __forceinline__ void load(int u, int s) {
    const unsigned* Kb = Kx + (unsigned)(mask_slot(mask, s) * d * d);
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
      // columns past d repeat column d - 1 (they meet zero rows of B)
      const unsigned o = (t + 1) * 4 <= d ? (unsigned)(lo + (4 * t + kk) * d) : (unsigned)(lo + min(4 * t + kk, d - 1) * d);
      a[u][t] = Kb[o];
    }
  }
  __device__ __forceinline__ void prefetch(const __half2* __restrict__ Kx_, unsigned mask_, int row, int kk_, int d_, int g_) {
    Kx = reinterpret_cast<const unsigned*>(Kx_);
    mask = mask_;
    ns = __builtin_popcount(mask_);
    d = d_;
    lo = row;
    kk = kk_;
    g = g_;
#pragma unroll
    for (int u = 0; u < DEP; ++u)
      if (g + u * G < ns) load(u, g + u * G);
  }
  // lds_b: [ns][4 NJ][pitch] pairs (hi, mid), behind them the inverse scales
  // [ns][pitch]
  __device__ __forceinline__ void apply(const float2* lds_b, int pitch, int rl, f32x4& cr, f32x4& ci) {
    typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    cr = {0.f, 0.f, 0.f, 0.f};
    ci = {0.f, 0.f, 0.f, 0.f};
    const uint2* bt = reinterpret_cast<const uint2*>(lds_b) + kk * pitch + rl;
    const float* sc = reinterpret_cast<const float*>(lds_b + ns * 4 * NJ * pitch) + rl;
#pragma unroll 1
    for (int s0 = g; s0 < ns; s0 += DEP * G) {
#pragma unroll
      for (int u = 0; u < DEP; ++u)
        if (s0 + u * G < ns) {
          f32x4 hr = {0.f, 0.f, 0.f, 0.f}, hi = hr, mr = hr, mi = hr;
#pragma unroll
          for (int t0 = 0; t0 < NJ; t0 += 4) {
            u32x4 av = {0, 0, 0, 0}, h0 = av, h1 = av, m0 = av, m1 = av;
#pragma unroll
            for (int t = t0; t < NJ && t < t0 + 4; ++t) {
              const uint2 bv = bt[((s0 + u * G) * 4 * NJ + 4 * t) * pitch];
              av[t - t0] = a[u][t];
              h0[t - t0] = bv.x ^ 0x80000000u;
              h1[t - t0] = __builtin_amdgcn_alignbit(bv.x, bv.x, 16);
              m0[t - t0] = bv.y ^ 0x80000000u;
              m1[t - t0] = __builtin_amdgcn_alignbit(bv.y, bv.y, 16);
            }
            const f16x8 A = __builtin_bit_cast(f16x8, av);
            hr = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, __builtin_bit_cast(f16x8, h0), hr, 0, 0, 0);
            hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, __builtin_bit_cast(f16x8, h1), hi, 0, 0, 0);
            mr = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, __builtin_bit_cast(f16x8, m0), mr, 0, 0, 0);
            mi = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, __builtin_bit_cast(f16x8, m1), mi, 0, 0, 0);
          }
          const float sv = sc[(s0 + u * G) * pitch];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            cr[v] = rfma(sv, rfma(0x1p-11f, mr[v], hr[v]), cr[v]);
            ci[v] = rfma(sv, rfma(0x1p-11f, mi[v], hi[v]), ci[v]);
          }
          if (s0 + (u + DEP) * G < ns) load(u, s0 + (u + DEP) * G);
        }
    }
  }
};

// The two FP16 parts of this lane's element f of a row that LR lanes hold: scaled by the power of two that takes the row's largest |re|, |im| to [2^14,
// 2^15) (rows below 2^-100 as if that were theirs); inv its inverse
template <int LR>
__device__ __forceinline__ uint2 split_row(float2 f, float& inv) {
  float m = fmaxf(fabsf(f.x), fabsf(f.y));
  m = fmaxf(m, dpp_mov<0xB1>(m));
  m = fmaxf(m, dpp_mov<0x4E>(m));
  m = fmaxf(m, dpp_mov<0x141>(m));
  if constexpr (LR > 8) m = fmaxf(m, dpp_mov<0x140>(m));
  if constexpr (LR > 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    m = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  if constexpr (LR > 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    m = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  const unsigned e = max(__float_as_uint(m) >> 23, 27u);
  const float s = __uint_as_float((268u - e) << 23);
  inv = __uint_as_float((e - 14u) << 23);
  f = make_float2(f.x * s, f.y * s);
  const __half2 h = __floats2half2_rn(f.x, f.y);
  const float2 hf = __half22float2(h);
  const __half2 l = __floats2half2_rn((f.x - hf.x) * 2048.f, (f.y - hf.y) * 2048.f);
  return make_uint2(__builtin_bit_cast(unsigned, h), __builtin_bit_cast(unsigned, l));
}

// Stages the input vectors of a site: row (k, r), slot k of the mask and
// right-hand side r, is a contiguous read of LR lanes (8 to 64, as d needs),
// so that a wavefront reads 64 / LR right-hand sides of a slot at once, U such
// reads in flight at a time; get(r, o) loads element o of right-hand side r,
// fin(r, v) turns what was loaded into the staged value, and mid() runs once
// after the first loads are issued.  The neighbour of slot k is read once into
// lane k and broadcast from there, so that no row waits on an index.  Rows past
// d of a slot are zeroed (they meet the repeated operator columns).  For FP16
// storage (H) a row is split as its product takes it.
template <bool H, int NJ, typename G, typename F, typename M>
__device__ __forceinline__ void mfma_stage(float2* lds_b, int pitch, unsigned mask, const int* __restrict__ nb9, int w,
                                           int nw, int lane, int d, int nr, G&& get, F&& fin, M&& mid) {
  constexpr int U = 8, LR = NJ <= 2 ? 8 : NJ <= 4 ? 16 : NJ <= 8 ? 32 : 64, RP = 64 / LR;
  const int ns = __builtin_popcount(mask), np = ns * ((nr + RP - 1) / RP);
  const int c = lane & (LR - 1), lc = min(c, d - 1), sub = lane / LR;
  int nbr = 0;
  if (lane < ns) nbr = nb9[mask_slot(mask, lane)];
  const int dr = nw / ns, dk = nw - dr * ns;
  int r = w / ns, k = w - r * ns;   // (r counts groups of RP right-hand sides)
  if (w >= np) mid();   // a wavefront without a row still meets mid()'s barrier
  for (int p0 = w; p0 < np; p0 += U * nw) {
    decltype(get(0, 0u)) v[U];
    int r1 = r, k1 = k;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u] = get(min(r1 * RP + sub, nr - 1), (unsigned)(__builtin_amdgcn_readlane(nbr, k1) * d + lc));
      r1 += dr;
      k1 += dk;
      if (k1 >= ns) k1 -= ns, ++r1;
    }
    if (p0 == w) mid();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r * RP < nr) {
        const int rs = r * RP + sub;
        const float2 f = fin(min(rs, nr - 1), v[u]);
        if constexpr (H) {
          float inv;
          const uint2 h = split_row<LR>(f, inv);
          if (rs < nr) {
            if (c < 4 * NJ)
              reinterpret_cast<uint2*>(lds_b)[(k * 4 * NJ + c) * pitch + rs] = c < d ? h : make_uint2(0u, 0u);
            if (c == 0) reinterpret_cast<float*>(lds_b + ns * 4 * NJ * pitch)[k * pitch + rs] = inv;
          }
        } else if (rs < nr && c < 4 * NJ) {
          lds_b[(k * 4 * NJ + c) * pitch + rs] = c < d ? f : make_float2(0.f, 0.f);
        }
      }
      r += dr;
      k += dk;
      if (k >= ns) k -= ns, ++r;
    }
  }
}

// The sum over the groups of wavefronts of a row tile's results, in group 0
// (through the B tile's LDS, which every wavefront has finished reading)
template <int G>
__device__ __forceinline__ void mfma_join(float2* lds_b, int mt, int nmt, int g, int lane, f32x4& cr, f32x4& ci) {
  if constexpr (G > 1) {
    f32x4* part = reinterpret_cast<f32x4*>(lds_b) + lane;
    __syncthreads();
    if (g > 0) {
      part[((g - 1) * nmt + mt) * 128] = cr;
      part[((g - 1) * nmt + mt) * 128 + 64] = ci;
    }
    __syncthreads();
    if (g == 0)
#pragma unroll
      for (int v = 0; v < G - 1; ++v) {
        cr += part[(v * nmt + mt) * 128];
        ci += part[(v * nmt + mt) * 128 + 64];
      }
  }
}

// Rows 4 (l / 16) .. + 3 of the tile and right-hand side l % 16 belong to
// lane l: calls f(v, o) for each row that exists, o its offset in the field
template <typename F>
__device__ __forceinline__ void mfma_rows(int mt, int lane, int d, F&& f) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = mt * 16 + 4 * (lane >> 4) + v;
    if (i < d) f(v, i);
  }
}

// out = K in over the sites of `sites` (nullptr: every site), or with b
// given out = b - K in (the residual of a SAP colour pass)
template <typename S, int NJ, int G>
__global__ void __launch_bounds__(64 * G * ((NJ + 3) / 4), 4) k_capply_mfma(CoarseOpView<float, S> op, const int* __restrict__ sites,
                                                               const float2* __restrict__ in,
                                                               const float2* __restrict__ b, float2* __restrict__ out,
                                                               long long n, int nb, int per, int pitch) {
  extern __shared__ __align__(16) float2 lds_b[];
  const int wg = xcd_slab_index(blockIdx.x, gridDim.x);
  const int site = sites ? sites[wg] : wg, d = op.d;
  const int w = wave_id(), lane = threadIdx.x & 63;
  constexpr int nmt = (NJ + 3) / 4;
  const long long off = (long long)blockIdx.y * per * n;
  in += off;
  out += off;
  const int nr = min(per, nb - (int)blockIdx.y * per);
  const int kk = lane >> 4, rl = min(lane & 15, nr - 1), g = G > 1 ? w / nmt : 0, mt = w - g * nmt;
  MfmaRows<S, NJ, G> mr;
  mfma_stage<std::is_same<S, __half2>::value, NJ>(
      lds_b, pitch, 0x1FFu, op.nbr9 + (size_t)site * 9, w, nmt * G, lane, d, nr,
      [&](int r, unsigned o) { return in[r * n + o]; }, [](int, float2 v) { return v; },
      [&] { mr.prefetch(op.K + (size_t)site * 9 * d * d, 0x1FFu, min(mt * 16 + (lane & 15), d - 1), kk, d, g); });
  const long long own = (long long)site * d + rl * n;
  float2 bv[4];
  if (b && g == 0) mfma_rows(mt, lane, d, [&](int v, int i) { bv[v] = b[off + own + i]; });
  __syncthreads();
  f32x4 cr, ci;
  mr.apply(lds_b, pitch, rl, cr, ci);
  mfma_join<G>(lds_b, mt, nmt, g, lane, cr, ci);
  if (g == 0 && (lane & 15) < nr)
    mfma_rows(mt, lane, d, [&](int v, int i) {
      float2 o = make_float2(cr[v], ci[v]);
      if (b) o = csub(bv[v], o);
      out[own + i] = o;
    });
}

// sums over each group of 16 lanes of the step-size sums of field r0 + lane /
// 16 in one block (block-major per-site partials): every lane of the group
// gets the step size
__device__ inline float2 block_alpha_row(const float* __restrict__ part, int blk, int bs, int lane) {
  float s0 = 0.f, s1 = 0.f, s2 = 0.f;
  for (int v = lane & 15; v < bs; v += 16) {
    const float* p = part + ((size_t)blk * bs + v) * 4;
    s0 += p[0];
    s1 += p[1];
    s2 += p[2];
  }
  s0 = row_sum16(s0);
  s1 = row_sum16(s1);
  s2 = row_sum16(s2);
  return s2 > 0.f ? make_float2(s0 / s2, s1 / s2) : czero<float>();
}

// The MR step of a batch on the matrix cores (the product as in
// k_capply_mfma, over the in-block operator blocks of a site).  Workgroups
// are mapped so that the sites of a block run on one XCD, whose L2 then
// serves the block's vectors to all of them.  Bound by the number of its load
// instructions and the latency of the chain step size, inputs, product, with
// FP32 storage by the matrix cores' FP32 rate too: 12 fields on 4096 sites, d =
// 40, FP16 storage 230 us on the vector units, 86 with FP32 products, 79 with
// FP16 ones and 77 so with registers held to four waves per SIMD; the residual
// (k_capply_mfma) 194, 136, 112, 109 us, and 103 with its inputs requested ahead
// of the operator (the same order makes this kernel spill and costs it 0-20 %).
template <typename S, int NJ, int G>
__global__ void __launch_bounds__(64 * G * ((NJ + 3) / 4), 4) k_sap_q_mfma(CoarseOpView<float, S> op, const int* __restrict__ csites,
                                                              SapTables tb, int pos0, int step,
                                                              const float2* __restrict__ rho_prev,
                                                              const float2* __restrict__ q_prev,
                                                              const float* __restrict__ part_prev,
                                                              float2* __restrict__ rho_cur,
                                                              float2* __restrict__ q_cur, float* __restrict__ part_cur,
                                                              float2* __restrict__ z, long long n, int nb, int per, int pitch) {
  extern __shared__ __align__(16) float2 lds_b[];
  constexpr int nmt = (NJ + 3) / 4;
  constexpr bool H = std::is_same<S, __half2>::value;
  __shared__ float2 alpha_s[MFMA_NB];
  __shared__ float dot_s[nmt][3][MFMA_NB];
  const int x = xcd_slab_index(blockIdx.x, gridDim.x);
  const int site = csites[x], d = op.d;
  const int w = wave_id(), lane = threadIdx.x & 63;
  const long long off = (long long)blockIdx.y * per * n, pn = (long long)op.V * 4;
  const long long poff = (long long)blockIdx.y * per * pn;
  rho_prev += off;
  q_prev += off;
  rho_cur += off;
  q_cur += off;
  z += off;
  part_prev += poff;
  part_cur += poff;
  const int nr = min(per, nb - (int)blockIdx.y * per);
  const int kk = lane >> 4, rl = min(lane & 15, nr - 1), g = G > 1 ? w / nmt : 0, mt = w - g * nmt;
  const int pos = pos0 + x, blk = pos / tb.bs;
  const unsigned mask = __builtin_amdgcn_readfirstlane(tb.inmask[pos]);
  MfmaRows<S, NJ, G> mr;
  mr.prefetch(op.K + (size_t)site * 9 * d * d, mask, min(mt * 16 + (lane & 15), d - 1), kk, d, g);
  const int* nb9 = op.nbr9 + (size_t)site * 9;
  // the site's own rows of the previous residual and of z, for z += alpha rho
  const long long own = (long long)site * d + rl * n;
  // (H: and the new residual, which the staged rows hold in parts)
  float2 zown[4], rown[4], qown[4];
  if (H && step == 0 && g == 0) mfma_rows(mt, lane, d, [&](int v, int i) { rown[v] = rho_prev[own + i]; });
  if (step > 0) {
    if (g == 0)
      mfma_rows(mt, lane, d, [&](int v, int i) {
        zown[v] = z[own + i];
        rown[v] = rho_prev[own + i];
        if constexpr (H) qown[v] = q_prev[own + i];
      });
    mfma_stage<H, NJ>(
        lds_b, pitch, mask, nb9, w, nmt * G, lane, d, nr,
        [&](int r, unsigned o) {
          const float2 a = rho_prev[r * n + o], b = q_prev[r * n + o];
          return make_float4(a.x, a.y, b.x, b.y);
        },
        [&](int r, float4 v) { return csub(make_float2(v.x, v.y), cmul(alpha_s[r], make_float2(v.z, v.w))); },
        [&] {
          for (int r0 = 4 * w; r0 < nr; r0 += 4 * nmt * G) {
            const int r = min(r0 + (lane >> 4), nr - 1);
            const float2 al = block_alpha_row(part_prev + r * pn, blk, tb.bs, lane);
            if ((lane & 15) == 0) alpha_s[r] = al;
          }
          __syncthreads();
        });
  } else {
    mfma_stage<H, NJ>(
        lds_b, pitch, mask, nb9, w, nmt * G, lane, d, nr, [&](int r, unsigned o) { return rho_prev[r * n + o]; },
        [](int, float2 v) { return v; }, [] {});
  }
  __syncthreads();
  f32x4 cr, ci;
  mr.apply(lds_b, pitch, rl, cr, ci);
  // (FP32 storage: the tile's rows of the new residual, before the join takes the B tile's place)
  float2 keep[4];
  if constexpr (!H && G > 1)
    if (g == 0) mfma_rows(mt, lane, d, [&](int v, int i) { keep[v] = lds_b[i * pitch + rl]; });
  mfma_join<G>(lds_b, mt, nmt, g, lane, cr, ci);
  if (g == 0) {
    float a0 = 0.f, a1 = 0.f, a2 = 0.f;
    const bool live = (lane & 15) < nr;
    mfma_rows(mt, lane, d, [&](int v, int i) {
      float2 rho;
      if constexpr (H) rho = step > 0 ? csub(rown[v], cmul(alpha_s[rl], qown[v])) : rown[v];
      else if constexpr (G > 1) rho = keep[v];
      else rho = lds_b[i * pitch + rl];
      const float2 q = make_float2(cr[v], ci[v]);
      a0 = rfma(q.x, rho.x, rfma(q.y, rho.y, a0));
      a1 = rfma(q.x, rho.y, rfma(-q.y, rho.x, a1));
      a2 = rfma(q.x, q.x, rfma(q.y, q.y, a2));
      if (live) {
        rho_cur[own + i] = rho;
        q_cur[own + i] = q;
        if (step > 0) {
          cfma(zown[v], alpha_s[rl], rown[v]);
          z[own + i] = zown[v];
        }
      }
    });
    // over the four row groups of the tile, then over the row tiles
    a0 += __shfl_xor(a0, 16, 64);
    a1 += __shfl_xor(a1, 16, 64);
    a2 += __shfl_xor(a2, 16, 64);
    a0 += __shfl_xor(a0, 32, 64);
    a1 += __shfl_xor(a1, 32, 64);
    a2 += __shfl_xor(a2, 32, 64);
    if (lane < 16) {
      dot_s[mt][0][lane] = a0;
      dot_s[mt][1][lane] = a1;
      dot_s[mt][2][lane] = a2;
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 3 * nr; e += 64 * G * nmt) {
    const int c = e / nr, r = e - c * nr;
    float t = 0.f;
#pragma unroll
    for (int v = 0; v < nmt; ++v) t += dot_s[v][c][r];
    part_cur[r * pn + (size_t)pos * 4 + c] = t;
  }
}

template <int LO, int HI, typename F>
inline void with_int(int v, F&& f) {
  if constexpr (LO <= HI) {
    if (v == LO) f(std::integral_constant<int, LO>{});
    else with_int<LO + 1, HI>(v, f);
  } else {
    throw Error(-1, "unsupported size");
  }
}

// The launch of a batch of nb fields on d components with ns staged blocks on
// `sites` sites: chunks of `per` right-hand sides (equal chunks of at most 16,
// fewer where the B tile would pass the LDS a workgroup has), the B tile's
// pitch, the groups of wavefronts and the LDS bytes (H: with the scales)
struct MfmaShape {
  int per, nch, nmt, nj, pitch;
  int g;       // groups of wavefronts that share the operator blocks
  size_t lds;
};
inline MfmaShape mfma_shape(int d, int nb, int ns, int sites, bool H, int lds_limit) {
  MfmaShape m;
  m.nj = (d + 3) / 4;
  m.nmt = (m.nj + 3) / 4;
  const int row = ns * (4 * m.nj * (int)sizeof(float2) + (H ? (int)sizeof(float) : 0));
  const int cap = std::min(MFMA_NB, lds_limit / row);
  m.nch = (nb + cap - 1) / cap;
  m.per = (nb + m.nch - 1) / m.nch;
  m.pitch = (m.per | 1) * row <= lds_limit ? m.per | 1 : m.per;   // odd where it fits
  // More groups shorten a workgroup's chain of staging and products but hold
  // more of the device for each site: they pay where the sites do not fill it,
  // and for few row tiles also where many right-hand sides are staged.  One SAP
  // sweep with FP16 storage in us, 1 / 2 / 4 groups (3 for d = 40): 12 fields of
  // d = 16 on 256 sites 85 / 68 / 60, 2048 110 / 91 / 86, 4096 138 / 127 / 143; d =
  // 32 on 256 95 / 74 / 67, 2048 147 / 130 / 160, 4096 240 / 223 / 286; d = 40 on
  // 256 120 / 96 / 86, 1024 152 / 140 / 162, 4096 388 / 527 / 604; d = 56 on 256
  // 132 / 110 / -, 4096 583 / 667 / -; operator apply, 12 fields of d = 16 on 4096
  // sites 34 / 26 / 20, of d = 32 65 / 45 / 57, 3 fields 32 / 32 / 48.
  const long long wgs = (long long)sites * m.nch;
  const bool many = ns == 9 && m.per >= 8;
  if (m.nmt == 1) m.g = wgs <= 1024 || many ? 4 : 2;
  else if (m.nmt == 2) m.g = wgs <= 256 ? 4 : wgs <= 1024 || many ? 2 : 1;
  else m.g = wgs <= (m.nmt == 3 ? 512 : 256) ? 2 : 1;
  m.lds = std::max((size_t)m.pitch * row, (size_t)(m.g - 1) * m.nmt * 2048);
  return m;
}

// f(NJ, G) as compile-time numbers
template <typename F>
inline void with_mfma_shape(const MfmaShape& m, F&& f) {
  with_int<1, 16>(m.nj, [&](auto nj) {
    constexpr int nmt = (decltype(nj)::value + 3) / 4;
    if constexpr (nmt <= 2)
      if (m.g == 4) return f(nj, std::integral_constant<int, 4>{});
    if (m.g == 2) return f(nj, std::integral_constant<int, 2>{});
    if constexpr (nmt >= 2) f(nj, std::integral_constant<int, 1>{});
  });
}

template <typename S>
void coarse_apply_mfma(const CoarseOpView<float, S>& op, const int* sites, int nsites, const float2* in,
                       const float2* b, float2* out, hipStream_t s, int nb) {
  const long long n = (long long)op.V * op.d;
  const MfmaShape m = mfma_shape(op.d, nb, 9, nsites, std::is_same<S, __half2>::value, 65536);
  with_mfma_shape(m, [&](auto nj, auto g) {
    constexpr int NJ = decltype(nj)::value, G = decltype(g)::value;
    k_capply_mfma<S, NJ, G><<<dim3(nsites, m.nch), 64 * G * m.nmt, m.lds, s>>>(op, sites, in, b, out, n, nb, m.per,
                                                                              m.pitch);
  });
  DD_LAUNCH_CHECK();
}

template <typename S>
void coarse_sap_q_mfma(const CoarseOpView<float, S>& op, const SapTables& tb, const int* csites, int nsites, int pos0,
                       int step, float2* z, const SapScratch<float>& ws, hipStream_t s, int nb) {
  const long long n = (long long)op.V * op.d;
  // (alpha_s and dot_s next to the B tile)
  const MfmaShape m = mfma_shape(op.d, nb, tb.kmax, nsites, std::is_same<S, __half2>::value, 65536 - 1024);
  const int pp = (step + 1) & 1, cc = step & 1;   // previous / current buffers
  with_mfma_shape(m, [&](auto nj, auto g) {
    constexpr int NJ = decltype(nj)::value, G = decltype(g)::value;
    k_sap_q_mfma<S, NJ, G><<<dim3(nsites, m.nch), 64 * G * m.nmt, m.lds, s>>>(
        op, csites, tb, pos0, step, ws.rho[pp], ws.q[pp], ws.part[pp], ws.rho[cc], ws.q[cc], ws.part[cc], z, n, nb,
        m.per, m.pitch);
  });
  DD_LAUNCH_CHECK();
}

}  // namespace ddamg
