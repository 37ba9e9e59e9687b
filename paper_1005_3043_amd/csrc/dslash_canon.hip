// The fine operator D (Eq. 2) directly on the boundary's canonical arrays
// (lexicographic sites, a site's components innermost, complex128), for
// wilson_apply: one kernel instead of packing the links and the input into
// the internal layout, applying the stencil there and unpacking.  A stateless
// call reads its inputs once, so the packed copies never paid: on 32^3 x 64
// in FP64 with one right-hand side 1.88 ms went into 0.58 (links) + 0.34
// (input) packing, 0.55 stencil and 0.39 unpacking, and each call allocated
// and freed the copies.
//
// Bound by memory (32^3 x 64, FP64 x 1 and FP32 x 12: 7.1 to 7.4 TB/s of reads
// past L2 and writes), in the binary16 class by the vector units' rounding and
// conversions (24^3 x 48 x 12: at least 68 % busy).  A site's 12 spinor
// components (192 bytes) and 9 link entries (144 bytes) are contiguous, which
// one thread per site would read in strides; instead a wavefront reads the
// entries of its 64 consecutive sites (or of their neighbours, contiguous up to
// the lattice's edges) as one flat run, 1 KiB per load, and hands them to the
// threads through LDS, rounded to the arithmetic type on the way.  Rows of 13
// spinor and 9 link entries make the per-thread reads free of bank conflicts
// (an odd number of 8- or 16-byte units).  The output leaves the same way.
//
// Per site the hops are added in the order of k_dslash and with its hop code,
// so every precision gives k_dslash's bits on the same rounded inputs.
#include <type_traits>

#include "canon_order.h"
#include "kernels.h"
#include "wilson_site.h"

namespace mg {
namespace {

constexpr int SROW = 13;  // LDS entries per site of a spinor (12 used)
constexpr int LROW = 9;   // LDS entries per site of a link
constexpr int LTILE = 66 * LROW;  // a tile's links and the spare row (even number of entries)

struct CanonGeom {
  int L[4];
  uint32_t S[4];  // stride of each direction in sites
  uint32_t V, ntile;
  FastDiv f[3];
  int antiperiodic;
  CanonOrder order;  // of the streaming form
};

typedef double double2v __attribute__((ext_vector_type(2)));

// Flat run of a tile's spinor entries: load i of lane l is entry e = 64 i + l,
// component e % 12 of site e / 12.  64 * 3 = 16 * 12, so three (site,
// component) pairs per lane serve all twelve loads, 16 sites apart.
struct Flat12 {
  uint32_t j[3], c[3];
  __device__ __forceinline__ explicit Flat12(uint32_t lane) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint32_t e = 64u * q + lane;
      j[q] = e / 12;
      c[q] = e - 12 * j[q];
    }
  }
  __device__ __forceinline__ uint32_t site(int i) const { return j[i % 3] + 16u * (i / 3); }
  __device__ __forceinline__ uint32_t comp(int i) const { return c[i % 3]; }
  __device__ __forceinline__ uint32_t row(int i) const { return j[i % 3] * SROW + c[i % 3] + 16u * SROW * (i / 3); }
};
// Links: seven sites (63 lanes) per load, ten loads per tile.  Every lane
// loads and stages without a condition (under one the compiler would move the
// loads behind the spinor's staging): lane 63 repeats the next load's first
// entry, and what lies past the tile goes to a spare row.
constexpr int LSITES = 7, LLOADS = 10;


__device__ __forceinline__ void coords_of(const CanonGeom &g, uint32_t s, int (&x)[4]) {
#pragma unroll
  for (int mu = 0; mu < 3; ++mu) {
    const uint32_t q = g.f[mu].div(s);
    x[mu] = (int)(s - q * (uint32_t)g.L[mu]);
    s = q;
  }
  x[3] = (int)s;
}
__device__ __forceinline__ uint32_t nbr_of(const CanonGeom &g, uint32_t s, const int (&x)[4], int mu, bool fwd) {
  if (fwd) return x[mu] + 1 < g.L[mu] ? s + g.S[mu] : s - (uint32_t)(g.L[mu] - 1) * g.S[mu];
  return x[mu] > 0 ? s - g.S[mu] : s + (uint32_t)(g.L[mu] - 1) * g.S[mu];
}

// The values a binary16 spinor (per-site scale) holds for v: store_site's
// rounding for h16 without the store.
template <typename C> __device__ __forceinline__ void h16_values(C (&v)[12], float m) {
  const float inv = m > 0.f ? 1.0f / m : 0.f;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    float x = (float)v[c].x * inv, y = (float)v[c].y * inv;
    // the quotient is an FP32 number in the storage's definition: without
    // this the compiler rounds the product to binary16 directly (fma_mixlo)
    asm("" : "+v"(x), "+v"(y));
    v[c] = mk<C>((float)(_Float16)x * m, (float)(_Float16)y * m);
  }
}
template <int N, typename C> __device__ __forceinline__ float h16_max(const C (&v)[N]) {
  float m = 0.f;
#pragma unroll
  for (int c = 0; c < N; ++c) m = fmaxf(m, fmaxf(fabsf((float)v[c].x), fabsf((float)v[c].y)));
  return m;
}

// (float)(_Float16)d, rounded once.  The hardware has no such conversion and
// the compiler's takes some 30 instructions; going through FP32 rounds twice,
// which only differs where the FP32 value is a midpoint of binary16 (or its
// result is subnormal).  Those take the compiler's conversion.
__device__ __forceinline__ float via_half(double d) {
  const float f = (float)d;
  const bool sure = (__builtin_bit_cast(uint32_t, f) & 0x1fffu) != 0x1000u && fabsf(f) >= 6.103515625e-05f;
  float h = (float)(_Float16)f;
  if (!sure) h = (float)(_Float16)d;
  return h;
}

// Link entries in the class's storage: as they are, or rounded to binary16.
template <bool Q16, typename C> __device__ __forceinline__ C link_value(double2 v) {
  if constexpr (Q16) return mk<C>(via_half(v.x), via_half(v.y));
  else return cvt<C>(v);
}

// Workgroup -> position in the visiting order: XCD k (dispatch order modulo
// 8) takes the k-th contiguous share of it.
__device__ __forceinline__ uint32_t xcd_share(uint32_t bid, uint32_t n) {
  const uint32_t k = bid & 7u, q = n >> 3, rem = n & 7u;
  return k * q + (k < rem ? k : rem) + (bid >> 3);
}

template <typename C> __device__ __forceinline__ void store_flat(double2 *out, size_t at, C v) {
  const double2v d = {(double)v.x, (double)v.y};
  __builtin_nontemporal_store(d, reinterpret_cast<double2v *>(out + at));
}

// Streaming form: one site per thread.  WR = 1: each wavefront takes a tile
// of 64 sites of one right-hand side and stages its own links.  WR > 1: the
// WR wavefronts of a workgroup take the same tile for WR right-hand sides and
// stage the links together, so that a link is read once per group; the groups
// of a tile are consecutive on one XCD, whose L2 then holds them.  In FP32 on
// 32^3 x 64 with 12 right-hand sides the links would otherwise be 6 of every
// 16 bytes read.
template <typename R, bool Q16, int WR>
__global__ __launch_bounds__(256, 2) void k_dslash_canon(CanonGeom g, const double2 *__restrict__ U,
                                                         const double2 *__restrict__ in, double2 *__restrict__ out,
                                                         R diag, int nrhs, uint32_t ngrp) {
  using C = c_t<R>;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  C *sp = reinterpret_cast<C *>(lds_raw) + (size_t)wv * 64 * SROW;
  C *lk = WR > 1 ? reinterpret_cast<C *>(lds_raw) + (size_t)nw * 64 * SROW : sp;
  uint32_t *nb = reinterpret_cast<uint32_t *>(reinterpret_cast<C *>(lds_raw) + (size_t)nw * 64 * SROW +
                                              (WR > 1 ? LTILE : 0)) +
                 (WR > 1 ? 0 : wv * 9 * 64);
  const uint32_t pos = xcd_share(blockIdx.x, gridDim.x);
  uint32_t tile, rhs;
  if constexpr (WR > 1) {
    tile = pos / ngrp;
    rhs = (pos % ngrp) * WR + wv;
  } else {
    tile = pos * nw + wv;
    rhs = 0;
    if (tile >= g.ntile) return;  // whole wavefronts; no barrier in this form
  }
  const bool live = rhs < (uint32_t)nrhs;
  const double2 *vin = in + (size_t)(live ? rhs : nrhs - 1) * 12 * g.V;
  const uint32_t n0 = tile * 64, s = site_at(g.order, min(n0 + lane, g.V - 1));
  int x[4];
  coords_of(g, s, x);
#pragma unroll
  for (int h = 0; h < 8; ++h)
    if (WR == 1 || (h % WR) == wv) nb[h * 64 + lane] = nbr_of(g, s, x, h >> 1, (h & 1) == 0);
  if (WR == 1 || wv == 0) nb[8 * 64 + lane] = s;
  if constexpr (WR > 1) __syncthreads();
  else __builtin_amdgcn_wave_barrier();
  C acc[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = mk<C>(0, 0);
  constexpr int NL = (LLOADS + WR - 1) / WR;  // link loads per thread
  const Flat12 f(lane);
  const uint32_t lj = lane / LROW, lc = lane - LROW * lj;
  // In FP32 a hop's loads are issued while the hop before it is computed (one
  // load round trip per hop otherwise stands between the staging barriers:
  // 12 right-hand sides on 32^3 x 64 4.54 -> 3.79 ms); the ninth set is the
  // centre.
  double2 a[12], b[NL];
  auto issue = [&](int h) {
    const uint32_t *nh = nb + h * 64;
#pragma unroll
    for (int i = 0; i < 12; ++i) a[i] = vin[(size_t)nh[f.site(i)] * 12 + f.comp(i)];
    if (h < 8) {
      const double2 *Um = U + (size_t)(h >> 1) * g.V * 9;
      const uint32_t *nl = (h & 1) ? nh : nb + 8 * 64;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const uint32_t j = min((uint32_t)((WR > 1 ? i * WR + wv : i) * LSITES) + lj, 63u);
        b[i] = Um[(size_t)nl[j] * 9 + lc];
      }
    }
  };
  // (FP64 has no registers left for it: it spills a hundred and more)
  constexpr bool AHEAD = sizeof(R) == 4;
  if constexpr (AHEAD) issue(0);
#pragma unroll 1
  for (int mu = 0; mu < 4; ++mu) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      if constexpr (!AHEAD) issue(2 * mu + d);
      if constexpr (WR > 1) __syncthreads();  // the previous hop's links have been read
#pragma unroll
      for (int i = 0; i < 12; ++i) sp[f.row(i)] = cvt<C>(a[i]);
      __builtin_amdgcn_wave_barrier();
      C p[12], u[9];
      if constexpr (WR == 1) {  // the links pass through the same LDS after the spinor
#pragma unroll
        for (int c = 0; c < 12; ++c) p[c] = sp[lane * SROW + c];
        __builtin_amdgcn_wave_barrier();
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const uint32_t j = min((uint32_t)((WR > 1 ? i * WR + wv : i) * LSITES) + lj, 64u);
        lk[j * LROW + lc] = link_value<Q16, C>(b[i]);
      }
      if constexpr (WR > 1) __syncthreads();
      else __builtin_amdgcn_wave_barrier();
      if constexpr (AHEAD) issue(2 * mu + d + 1);
      if constexpr (WR > 1) {
#pragma unroll
        for (int c = 0; c < 12; ++c) p[c] = sp[lane * SROW + c];
      }
#pragma unroll
      for (int c = 0; c < 9; ++c) u[c] = lk[lane * LROW + c];
      __builtin_amdgcn_wave_barrier();
      if constexpr (Q16) h16_values(p, h16_max(p));
      R eta = 1;
      if (mu == 3 && g.antiperiodic && x[3] == (d == 0 ? g.L[3] - 1 : 0)) eta = -1;
      if (d == 0) hop_dispatch<true>(mu, acc, p, u, eta);
      else hop_dispatch<false>(mu, acc, p, u, eta);
    }
  }
  // centre, result, and back through LDS
  if constexpr (!AHEAD) issue(8);
#pragma unroll
  for (int i = 0; i < 12; ++i) sp[f.row(i)] = cvt<C>(a[i]);
  __builtin_amdgcn_wave_barrier();
  C r[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) r[c] = sp[lane * SROW + c];
  if constexpr (Q16) h16_values(r, h16_max(r));
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    r[c].x = fma(diag, r[c].x, (R)-0.5 * acc[c].x);
    r[c].y = fma(diag, r[c].y, (R)-0.5 * acc[c].y);
  }
  if constexpr (Q16) h16_values(r, h16_max(r));
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int c = 0; c < 12; ++c) sp[lane * SROW + c] = r[c];
  __builtin_amdgcn_wave_barrier();
  if (!live) return;
  double2 *vout = out + (size_t)rhs * 12 * g.V;
  const uint32_t ns = min(64u, g.V - n0);
#pragma unroll
  for (int i = 0; i < 12; ++i)
    if (f.site(i) < ns) store_flat(vout, (size_t)nb[8 * 64 + f.site(i)] * 12 + f.comp(i), sp[f.row(i)]);
}

// Latency form, for calls with too few tiles to fill the device: the eight
// hops of a tile run on eight wavefronts at once (one load round trip instead
// of eight) and leave their contributions in LDS, where four wavefronts add
// three components each in the streaming form's order.
template <typename R, bool Q16>
__global__ __launch_bounds__(512) void k_dslash_canon_split(CanonGeom g, const double2 *__restrict__ U,
                                                            const double2 *__restrict__ in,
                                                            double2 *__restrict__ out, R diag) {
  using C = c_t<R>;
  extern __shared__ __align__(16) unsigned char lds_raw[];  // [8][64][SROW]
  __shared__ uint32_t nbt[8][64];
  __shared__ float mx[4][64];
  const int lane = threadIdx.x & 63, h = threadIdx.x >> 6;
  C *all = reinterpret_cast<C *>(lds_raw), *sp = all + (size_t)h * 64 * SROW;
  const uint32_t s0 = blockIdx.x * 64, last = g.V - 1, s = min(s0 + lane, last);
  const double2 *vin = in + (size_t)blockIdx.y * 12 * g.V;
  const int mu = h >> 1;
  const bool fwd = (h & 1) == 0;
  int x[4];
  coords_of(g, s, x);
  switch (mu) {  // constant coordinate indices
    case 0: nbt[h][lane] = nbr_of(g, s, x, 0, fwd); break;
    case 1: nbt[h][lane] = nbr_of(g, s, x, 1, fwd); break;
    case 2: nbt[h][lane] = nbr_of(g, s, x, 2, fwd); break;
    default: nbt[h][lane] = nbr_of(g, s, x, 3, fwd); break;
  }
  __builtin_amdgcn_wave_barrier();
  // four wavefronts also fetch three components of the centre
  double2 cen[3];
  if (h < 4) {
#pragma unroll
    for (int c = 0; c < 3; ++c) cen[c] = vin[(size_t)s * 12 + 3 * h + c];
  }
  const Flat12 f(lane);
  double2 a[12], b[9];
#pragma unroll
  for (int i = 0; i < 12; ++i) a[i] = vin[(size_t)nbt[h][f.site(i)] * 12 + f.comp(i)];
  const double2 *Um = U + (size_t)mu * g.V * 9;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const uint32_t e = i * 64 + lane, j = e / 9;
    b[i] = Um[(size_t)(fwd ? min(s0 + j, last) : nbt[h][j]) * 9 + (e - 9 * j)];
  }
#pragma unroll
  for (int i = 0; i < 12; ++i) sp[f.row(i)] = cvt<C>(a[i]);
  __builtin_amdgcn_wave_barrier();
  C p[12], u[9], acc[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    p[c] = sp[lane * SROW + c];
    acc[c] = mk<C>(0, 0);
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < 9; ++i) sp[i * 64 + lane] = link_value<Q16, C>(b[i]);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int c = 0; c < 9; ++c) u[c] = sp[lane * LROW + c];
  __builtin_amdgcn_wave_barrier();
  if constexpr (Q16) h16_values(p, h16_max(p));
  R eta = 1;
  if (mu == 3 && g.antiperiodic && x[3] == (fwd ? g.L[3] - 1 : 0)) eta = -1;
  if (fwd) hop_dispatch<true>(mu, acc, p, u, eta);
  else hop_dispatch<false>(mu, acc, p, u, eta);
#pragma unroll
  for (int c = 0; c < 12; ++c) sp[lane * SROW + c] = acc[c];
  C ctr[3];
  if (h < 4) {
#pragma unroll
    for (int c = 0; c < 3; ++c) ctr[c] = cvt<C>(cen[c]);
    if constexpr (Q16) mx[h][lane] = h16_max(ctr);
  }
  __syncthreads();
  C r[3];
  if (h < 4) {
    if constexpr (Q16) {
      const float m = fmaxf(fmaxf(mx[0][lane], mx[1][lane]), fmaxf(mx[2][lane], mx[3][lane]));
      C w[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) w[c] = c < 3 ? ctr[c] : mk<C>(0, 0);
      h16_values(w, m);
#pragma unroll
      for (int c = 0; c < 3; ++c) ctr[c] = w[c];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      C t = all[lane * SROW + 3 * h + c];
#pragma unroll
      for (int q = 1; q < 8; ++q) t = cadd(t, all[((size_t)q * 64 + lane) * SROW + 3 * h + c]);
      r[c].x = fma(diag, ctr[c].x, (R)-0.5 * t.x);
      r[c].y = fma(diag, ctr[c].y, (R)-0.5 * t.y);
    }
  }
  __syncthreads();
  if (h < 4) {
    if constexpr (Q16) mx[h][lane] = h16_max(r);
#pragma unroll
    for (int c = 0; c < 3; ++c) all[lane * SROW + 3 * h + c] = r[c];
  }
  __syncthreads();
  if constexpr (Q16) {
    if (h == 0) {
      const float m = fmaxf(fmaxf(mx[0][lane], mx[1][lane]), fmaxf(mx[2][lane], mx[3][lane]));
      C w[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) w[c] = all[lane * SROW + c];
      h16_values(w, m);
#pragma unroll
      for (int c = 0; c < 12; ++c) all[lane * SROW + c] = w[c];
    }
    __syncthreads();
  }
  const size_t o = ((size_t)blockIdx.y * g.V + s0) * 12;
  const uint32_t ne = min(64u, g.V - s0) * 12;
  for (uint32_t e = threadIdx.x; e < ne; e += 512) {
    const uint32_t j = e / 12;
    store_flat(out, o + e, all[j * SROW + (e - 12 * j)]);
  }
}

// Up to this many tiles times right-hand sides the latency form is taken: two
// of its workgroups per CU at most, all resident at once.  7 x 10 x 13 x 18
// with five right-hand sides (1 280): 16.3 us streaming, 19.3 us this way;
// 8^4 with one (64): 9.4 us, and 14.9 us the stencil alone in one wavefront
// per tile.
constexpr uint64_t SPLIT_MAX = 512;

template <typename R, bool Q16>
hipError_t launch(const CanonGeom &g0, const double2 *U, const double2 *in, double2 *out, double diag, int nrhs,
                  hipStream_t st) {
  using C = c_t<R>;
  CanonGeom g = g0;
  const size_t row = sizeof(C) * 64 * SROW;
  if ((uint64_t)g.ntile * nrhs <= SPLIT_MAX) {
    hipLaunchKernelGGL((k_dslash_canon_split<R, Q16>), dim3(g.ntile, nrhs), dim3(512), 8 * row, st, g, U, in, out,
                       (R)diag);
    return hipGetLastError();
  }
  g.order = canon_order(g.L, nrhs);
  if (nrhs == 1) {
    const int nw = 4;
    const uint32_t nblk = (g.ntile + nw - 1) / nw;
    hipLaunchKernelGGL((k_dslash_canon<R, Q16, 1>), dim3(nblk), dim3(64 * nw), nw * (row + 9 * 64 * 4), st, g, U, in,
                       out, (R)diag, 1, 1u);
    return hipGetLastError();
  }
  const uint32_t ngrp = (uint32_t)(nrhs + 3) / 4;
  const int wr = (nrhs + (int)ngrp - 1) / (int)ngrp;
  const size_t lds = wr * row + sizeof(C) * LTILE + 9 * 64 * 4;
  const dim3 grid(g.ntile * ngrp), block(64 * wr);
  if (wr == 2)
    hipLaunchKernelGGL((k_dslash_canon<R, Q16, 2>), grid, block, lds, st, g, U, in, out, (R)diag, nrhs, ngrp);
  else if (wr == 3)
    hipLaunchKernelGGL((k_dslash_canon<R, Q16, 3>), grid, block, lds, st, g, U, in, out, (R)diag, nrhs, ngrp);
  else
    hipLaunchKernelGGL((k_dslash_canon<R, Q16, 4>), grid, block, lds, st, g, U, in, out, (R)diag, nrhs, ngrp);
  return hipGetLastError();
}

}  // namespace

hipError_t dslash_canon(const int L[4], int antiperiodic, const double2 *U, double mass, const double2 *in,
                        double2 *out, int nrhs, mg_prec_t prec, hipStream_t st) {
  CanonGeom g{};
  uint32_t v = 1;
  for (int mu = 0; mu < 4; ++mu) {
    g.L[mu] = L[mu];
    g.S[mu] = v;
    v *= (uint32_t)L[mu];
    if (mu < 3) g.f[mu] = FastDiv((uint32_t)L[mu]);
  }
  g.V = v;
  g.ntile = (v + 63) / 64;
  g.antiperiodic = antiperiodic;
  const double diag = 4.0 + mass;
  if (prec == MG_F64) return launch<double, false>(g, U, in, out, diag, nrhs, st);
  if (prec == MG_F32) return launch<float, false>(g, U, in, out, diag, nrhs, st);
  return launch<float, true>(g, U, in, out, diag, nrhs, st);
}

}  // namespace mg
