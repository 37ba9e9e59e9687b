// FP64 restriction r_c = P^dag r and prolongation e (+)= P e_c of the fine
// level (Eq. 4, Eq. 8) for up to 16 right-hand sides at a time, as complex
// GEMMs on the FP64 matrix cores (16x16x4, four real products per complex
// one).  One workgroup per aggregate reads its P once for all of them; per
// chirality h the restriction is C = P_h^dag F (M = Nv, N = nrhs, K = 6 |B|)
// and the prolongation F = P_h E (M = 6 |B|, N = nrhs, K = Nv).
//
// The fine vectors are either internal or the caller's canonical arrays
// (CANON), so that a call at the boundary needs no packed copy: 16 sites of
// every right-hand side at a time pass through LDS, rows of 13 entries per
// site and an odd number per right-hand side (no bank conflicts in either
// direction).  Wavefront w takes components 3 w .. 3 w + 2 (w / 2 = chirality).
//
// Bound by P: 3.06 GB for Nv = 24 on 24^3 x 48 against 1.53 GB of vectors.  The
// vector kernels read P once per four right-hand sides and reduced every
// inner product over the wavefront: 12 right-hand sides there took 2.91 ms
// (restriction) and 2.06 ms (prolongation), with 1.45 and 1.53 ms of packing
// and unpacking around them.
//
// MFMA lane layouts (16x16x4, FP64): A lane l = (row l % 16, k l / 16); B lane
// l = (k l / 16, column l % 16); C lane l, register v = (row 4 v + l / 16,
// column l % 16).
#include "kernels.h"

namespace mg {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int TF_SITES = 16;           // sites per chunk
constexpr int TF_ROW = 13;             // LDS entries per site (12 used)
constexpr int TF_VEC = TF_SITES * TF_ROW + 1;  // LDS entries per right-hand side
constexpr int TF_VB = 256;             // largest aggregate
constexpr int TF_NR = 16;              // right-hand sides per workgroup (N of the MFMA)
constexpr int TF_TOT = TF_SITES * 12;  // entries of a chunk per right-hand side

__device__ __forceinline__ uint32_t coarse_site(const Geom &gc, uint32_t B) {
  const int x[4] = {(int)(B % gc.L[0]), (int)((B / gc.L[0]) % gc.L[1]), (int)((B / (gc.L[0] * gc.L[1])) % gc.L[2]),
                    (int)(B / (gc.L[0] * gc.L[1] * gc.L[2]))};
  return encode(gc, x);
}

// Entry e of a chunk's n right-hand sides, in the order the fine array holds
// them: (right-hand side, local site, component) and its offset in memory.
template <bool CANON>
__device__ __forceinline__ size_t chunk_entry(const Geom &g, uint32_t s0, int l0, const uint32_t *ci, int e, int &r,
                                              int &j, int &c) {
  r = e / TF_TOT;
  const int f = e - r * TF_TOT;
  if constexpr (CANON) {
    j = f / 12;
    c = f - 12 * j;
    return (size_t)ci[min(l0 + j, (int)g.vb - 1)] * 12 + c;
  } else {
    c = f / TF_SITES;
    j = f - TF_SITES * c;
    return fidx(s0 + min(l0 + j, (int)g.vb - 1), c, 12);
  }
}

template <bool CANON, int MT>
__global__ __launch_bounds__(256, 2) void k_restrict_f64(Geom g, Geom gc, int nv, int nrhs, int per,
                                                      const double2 *__restrict__ P,
                                                      const double2 *__restrict__ fine, double2 *__restrict__ coarse) {
  extern __shared__ double2 sF[];  // [n][TF_VEC], then the wavefronts' sums
  __shared__ uint32_t ci[TF_VB];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, q = lane >> 4, col = lane & 15;
  const uint32_t B = blockIdx.x, s0 = B * g.vb;
  const int r0 = blockIdx.y * per, n = min(per, nrhs - r0), vb = (int)g.vb;
  const size_t vs = (size_t)12 * (CANON ? g.V : g.Vpad);
  fine += (size_t)r0 * vs;
  if constexpr (CANON)
    for (int l = tid; l < vb; l += 256) ci[l] = canon_index(g, decode(g, s0 + l));
  const int colc = min(col, n - 1);
  const double2 *Pm[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) Pm[m] = P + (size_t)min(16 * m + col, nv - 1) * 12 * g.Vpad;
  double2 a[3][MT][4];
  auto load_p = [&](int c3, int ch) {  // k-step u takes site 4 u + q of the chunk
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t o = fidx(s0 + min(ch * TF_SITES + 4 * u + q, vb - 1), 3 * wv + c3, 12);
#pragma unroll
      for (int m = 0; m < MT; ++m) a[c3][m][u] = Pm[m][o];
    }
  };
#pragma unroll
  for (int c3 = 0; c3 < 3; ++c3) load_p(c3, 0);
  // Sums as short as the vector kernel's, a tree over threads of 12 products
  // each: a matrix instruction adds four products from zero, the four k-steps
  // of a component are added, and two chunks at a time join the total.  All
  // 768 products of a wavefront in one accumulator rounded 7 times as much
  // (4^4 aggregates, relative to extended precision: 1.3e-15 against 1.9e-16,
  // 1.9e-16 this way).  The additions cost 4 % of a restriction and
  // prolongation of 12 vectors on 24^3 x 48 (1.92 -> 1.99 ms).
  doublex4 re[MT], im[MT], sre[MT], sim[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) re[m] = im[m] = sre[m] = sim[m] = doublex4{0.0, 0.0, 0.0, 0.0};
  const doublex4 zero = {0.0, 0.0, 0.0, 0.0};
  const int nch = (vb + TF_SITES - 1) / TF_SITES, tot = n * TF_TOT;
  for (int ch = 0; ch < nch; ++ch) {
    __syncthreads();  // ci is there; the previous chunk has been read
    for (int e0 = tid; e0 < tot; e0 += 4 * 256) {
      double2 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        int r, j, c;
        const size_t o = chunk_entry<CANON>(g, s0, ch * TF_SITES, ci, min(e0 + 256 * k, tot - 1), r, j, c);
        v[k] = fine[(size_t)r * vs + o];
        if (ch * TF_SITES + j >= vb) v[k] = make_double2(0.0, 0.0);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        int r, j, c;
        chunk_entry<CANON>(g, s0, ch * TF_SITES, ci, min(e0 + 256 * k, tot - 1), r, j, c);
        sF[r * TF_VEC + j * TF_ROW + c] = v[k];
      }
    }
    __syncthreads();
    if ((ch & 1) == 0) {  // a new pair of chunks
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        sre[m] += re[m];
        sim[m] += im[m];
        re[m] = im[m] = doublex4{0.0, 0.0, 0.0, 0.0};
      }
    }
#pragma unroll
    for (int c3 = 0; c3 < 3; ++c3) {
      const double2 *bp = sF + colc * TF_VEC + q * TF_ROW + 3 * wv + c3;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        doublex4 qr, qi;
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // conj(P) F
          const double2 p = a[c3][m][u], f = bp[4 * u * TF_ROW];
          const doublex4 xx = __builtin_amdgcn_mfma_f64_16x16x4f64(p.x, f.x, zero, 0, 0, 0);
          const doublex4 xy = __builtin_amdgcn_mfma_f64_16x16x4f64(p.x, f.y, zero, 0, 0, 0);
          const doublex4 yy = __builtin_amdgcn_mfma_f64_16x16x4f64(p.y, f.y, zero, 0, 0, 0);
          const doublex4 yx = __builtin_amdgcn_mfma_f64_16x16x4f64(p.y, f.x, zero, 0, 0, 0);
          qr = u == 0 ? xx + yy : qr + (xx + yy);
          qi = u == 0 ? xy - yx : qi + (xy - yx);
        }
        re[m] += qr;
        im[m] += qi;
        // added here: the compiler would keep the products of all tiles until
        // the chunk's end, past the registers it has
        asm volatile("" : "+v"(re[m]), "+v"(im[m]));
      }
      if (ch + 1 < nch) load_p(c3, ch + 1);
    }
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    re[m] += sre[m];
    im[m] += sim[m];
  }
  __syncthreads();
  // the odd wavefront of each chirality hands its sums to the even one
  if (wv & 1) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v) sF[(((wv >> 1) * MT + m) * 4 + v) * 64 + lane] = make_double2(re[m][v], im[m][v]);
  }
  __syncthreads();
  if ((wv & 1) || col >= n) return;
  double2 *out = coarse + ((size_t)(r0 + col) * gc.V + coarse_site(gc, B)) * (2 * nv) + (wv >> 1) * nv;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * m + 4 * v + q;
      const double2 o = sF[(((wv >> 1) * MT + m) * 4 + v) * 64 + lane];
      if (i < nv) out[i] = make_double2(re[m][v] + o.x, im[m][v] + o.y);
    }
}

// KS = ceil(Nv / 4) k-steps, at most KM.
template <bool CANON, int KM>
__global__ __launch_bounds__(256) void k_prolong_f64(Geom g, Geom gc, int nv, int nrhs, int per,
                                                     const double2 *__restrict__ P,
                                                     const double2 *__restrict__ coarse, double2 *__restrict__ fine,
                                                     int accumulate) {
  extern __shared__ double2 sF[];  // [n][TF_VEC], then E [2][4 KM][n]
  __shared__ uint32_t ci[TF_VB];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, q = lane >> 4, col = lane & 15;
  const uint32_t B = blockIdx.x, s0 = B * g.vb;
  const int r0 = blockIdx.y * per, n = min(per, nrhs - r0), vb = (int)g.vb, h = wv >> 1;
  const size_t vs = (size_t)12 * (CANON ? g.V : g.Vpad);
  fine += (size_t)r0 * vs;
  double2 *sE = sF + (size_t)n * TF_VEC;
  if constexpr (CANON)
    for (int l = tid; l < vb; l += 256) ci[l] = canon_index(g, decode(g, s0 + l));
  const uint32_t ic = coarse_site(gc, B);
  for (int e = tid; e < 2 * 4 * KM * n; e += 256) {
    const int r = e / (8 * KM), k = e - r * 8 * KM, hh = k / (4 * KM), i = k - hh * 4 * KM;
    const double2 v = coarse[((size_t)(r0 + r) * gc.V + ic) * (2 * nv) + hh * nv + min(i, nv - 1)];
    sE[k * n + r] = i < nv ? v : make_double2(0.0, 0.0);
  }
  const int KS = (nv + 3) >> 2, colc = min(col, n - 1);
  double2 a[3][KM];
  auto load_p = [&](int c3, int ch) {  // row = site of the chunk
    const size_t o = fidx(s0 + min(ch * TF_SITES + col, vb - 1), 3 * wv + c3, 12);
#pragma unroll
    for (int k = 0; k < KM; ++k) a[c3][k] = P[(size_t)min(4 * min(k, KS - 1) + q, nv - 1) * 12 * g.Vpad + o];
  };
#pragma unroll
  for (int c3 = 0; c3 < 3; ++c3) load_p(c3, 0);
  __syncthreads();
  const int nch = (vb + TF_SITES - 1) / TF_SITES, tot = n * TF_TOT;
  for (int ch = 0; ch < nch; ++ch) {
#pragma unroll
    for (int c3 = 0; c3 < 3; ++c3) {
      doublex4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        if (k >= KS) break;
        const double2 p = a[c3][k], b = sE[(h * 4 * KM + 4 * k + q) * n + colc];
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(p.x, b.x, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(p.x, b.y, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(-p.y, b.y, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(p.y, b.x, im, 0, 0, 0);
      }
      if (ch + 1 < nch) load_p(c3, ch + 1);
      if (col < n) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          sF[col * TF_VEC + (4 * v + q) * TF_ROW + 3 * wv + c3] = make_double2(re[v], im[v]);
      }
    }
    __syncthreads();
    for (int e = tid; e < tot; e += 256) {
      int r, j, c;
      const size_t o = chunk_entry<CANON>(g, s0, ch * TF_SITES, ci, e, r, j, c);
      if (ch * TF_SITES + j >= vb) continue;
      double2 v = sF[r * TF_VEC + j * TF_ROW + c];
      double2 *p = fine + (size_t)r * vs + o;
      if (accumulate) v = cadd(*p, v);
      *p = v;
    }
    __syncthreads();
  }
}

template <typename F> hipError_t groups(int nrhs, F &&f) {
  const int ng = (nrhs + TF_NR - 1) / TF_NR, per = (nrhs + ng - 1) / ng;
  f(ng, per);
  return hipGetLastError();
}

}  // namespace

// Where the vector kernels (transfer.hip) stay: one workgroup of theirs, for
// an aggregate and up to four right-hand sides, is done before this file's
// chain of 16-site chunks (5 us each at Nv = 24, 3 at Nv = 8), which counts
// while there are few workgroups; and one right-hand side leaves 15 of 16
// matrix columns empty.  Whole calls on canonical vectors in us, this way / the
// vector kernels with their packing, 4^4 aggregates.  Restriction of one
// vector, Nv = 8 / 24: 8^4 50 / 87 and 32 / 41; 24^3 x 48 411 / 820 and 327 /
// 675.  Several, Nv = 24: 16 aggregates x 2 93 / 64; 64 x 12 114 / 82; 256 x 4
// 114 / 107; 128 x 12 116 / 171; Nv = 8: 256 x 4 64 / 58, 128 x 12 87 / 90.
// Aggregates of 128 sites, 32 x 12, 61 / 69.
bool restrict_takes_mma_f64(const Geom &g, int nrhs) {
  return nrhs > 1 && (g.vb <= 128 || (uint64_t)g.Vc * nrhs > 1024);
}
// Prolongation, Nv = 24: one vector, 16 / 162 / 256 aggregates 60 / 67 / 84 and
// 37 / 63 / 94; several, 64 x 12 82 / 68, 162 x 4 71 / 70, 128 x 12 84 / 121,
// 256 x 2 89 / 95.  Aggregates of 192 sites, 32 x 1, 50 / 52.
bool prolong_takes_mma_f64(const Geom &g, int nrhs) {
  return g.vb <= 192 || g.Vc >= 256 || g.Vc * nrhs > 768;
}

template <bool CANON>
hipError_t restrict_fine_f64(const Geom &g, const Geom &gc, int nv, const double2 *P, const double2 *fine,
                             double2 *coarse, int nrhs, hipStream_t st) {
  return groups(nrhs, [&](int ng, int per) {
    const int mt = (nv + 15) / 16;
    size_t lds = sizeof(double2) * (size_t)per * TF_VEC;
    const size_t sums = sizeof(double2) * 2 * mt * 4 * 64;
    if (lds < sums) lds = sums;
    const dim3 grid(g.Vc, ng);
    if (mt == 1)
      hipLaunchKernelGGL((k_restrict_f64<CANON, 1>), grid, dim3(256), lds, st, g, gc, nv, nrhs, per, P, fine, coarse);
    else
      hipLaunchKernelGGL((k_restrict_f64<CANON, 2>), grid, dim3(256), lds, st, g, gc, nv, nrhs, per, P, fine, coarse);
  });
}
template <bool CANON>
hipError_t prolong_fine_f64(const Geom &g, const Geom &gc, int nv, const double2 *P, const double2 *coarse,
                            double2 *fine, int nrhs, int accumulate, hipStream_t st) {
  return groups(nrhs, [&](int ng, int per) {
    const dim3 grid(g.Vc, ng);
#define MG_PF(KM)                                                                                            \
  hipLaunchKernelGGL((k_prolong_f64<CANON, KM>), grid, dim3(256),                                            \
                     sizeof(double2) * (size_t)per * (TF_VEC + 8 * KM), st, g, gc, nv, nrhs, per, P, coarse, \
                     fine, accumulate)
    if (nv <= 8) MG_PF(2);
    else if (nv <= 16) MG_PF(4);
    else if (nv <= 24) MG_PF(6);
    else MG_PF(8);
#undef MG_PF
  });
}
template hipError_t restrict_fine_f64<false>(const Geom &, const Geom &, int, const double2 *, const double2 *,
                                             double2 *, int, hipStream_t);
template hipError_t restrict_fine_f64<true>(const Geom &, const Geom &, int, const double2 *, const double2 *,
                                            double2 *, int, hipStream_t);
template hipError_t prolong_fine_f64<false>(const Geom &, const Geom &, int, const double2 *, const double2 *,
                                            double2 *, int, int, hipStream_t);
template hipError_t prolong_fine_f64<true>(const Geom &, const Geom &, int, const double2 *, const double2 *,
                                           double2 *, int, int, hipStream_t);

}  // namespace mg
