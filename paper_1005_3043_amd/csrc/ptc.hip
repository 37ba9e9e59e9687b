// Learned near-null-vector proposal: a two-layer gauge-equivariant network of
// parallel-transport convolutions (an extension of the adaptive setup of
// "Adaptive Multigrid"; the paper has no such network).
//
// Hop operators T_k, k = 0..8: T_0 = 1; k = 1 + 2 mu + dir transports the
// neighbour value along the link of the hopping term of Eq. 2 (dir 0:
// eta U_mu(x) psi(x+mu); dir 1: eta U_mu(x-mu)^dag psi(x-mu)), eta = -1
// across the antiperiodic time boundary.  A layer is
//   out_a(x) = sum_{b,k} W_abk (T_k in_b)(x),   W_abk a complex 4x4 spin matrix.
// Forward and backward passes are split into a transport stage (H_bk = T_k
// in_b, stored for the weight gradient) and site-local channel mixing; the
// adjoint transport uses T_{+mu}^dag = T_{-mu}.  The training loss is the
// subspace fit of target vectors per chirality-split aggregate (the blocks
// on which P is built, Eq. 4), solved by Cholesky of the 24 x 24 Gram
// matrices in FP64.  FP32 weights and arithmetic; fields in the fine
// tile-interleaved layout [channel][12 * Vpad].
#include <algorithm>
#include <type_traits>

#include "ptc.h"

namespace mg {

__device__ __forceinline__ float2 cf(float x, float y) { return make_float2(x, y); }
__device__ __forceinline__ float2 cfmaf(float2 a, float2 b, float2 c) {
  return cf(fmaf(a.x, b.x, fmaf(-a.y, b.y, c.x)), fmaf(a.x, b.y, fmaf(a.y, b.x, c.y)));
}
// conj(a) * b + c
__device__ __forceinline__ float2 cfmacf(float2 a, float2 b, float2 c) {
  return cf(fmaf(a.x, b.x, fmaf(a.y, b.y, c.x)), fmaf(a.x, b.y, fmaf(-a.y, b.x, c.y)));
}

// h = T_KK psi at site s (12 complex: spin-major 3 s + c).  The hop is a
// constant: with a running one the coordinate arrays went to LDS.
template <int KK>
__device__ __forceinline__ void transport_site(float2 (&h)[12], const Geom &g, uint32_t s, const Coords &k,
                                               const float2 *__restrict__ U, const float2 *__restrict__ psi) {
  if constexpr (KK == 0) {
#pragma unroll
    for (int c = 0; c < 12; ++c) h[c] = psi[fidx(s, c, 12)];
  } else {
    constexpr int mu = (KK - 1) >> 1;
    constexpr bool back = ((KK - 1) & 1) != 0;
    const uint32_t sn = back ? nbr_bwd(g, s, k, mu) : nbr_fwd(g, s, k, mu), sl = back ? sn : s;
    float eta = 1.f;
    if (mu == 3 && g.antiperiodic) {
      if (!back && k.o[3] == g.b[3] - 1 && k.c[3] == g.C[3] - 1) eta = -1.f;
      if (back && k.o[3] == 0 && k.c[3] == 0) eta = -1.f;
    }
    float2 u[9], p[12];
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = U[fidx(sl, mu * 9 + e, 36)];
#pragma unroll
    for (int c = 0; c < 12; ++c) p[c] = psi[fidx(sn, c, 12)];
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        float2 acc = cf(0.f, 0.f);
#pragma unroll
        for (int b = 0; b < 3; ++b)
          acc = back ? cfmacf(u[b * 3 + a], p[sp * 3 + b], acc) : cfmaf(u[a * 3 + b], p[sp * 3 + b], acc);
        h[sp * 3 + a] = cf(eta * acc.x, eta * acc.y);
      }
  }
}
// f(constant 0), .., f(constant 8)
template <int KK = 0, typename F> __device__ __forceinline__ void each_hop(F &&f) {
  if constexpr (KK < PTC_HOPS) {
    f(std::integral_constant<int, KK>{});
    each_hop<KK + 1>(f);
  }
}

constexpr int adjoint_hop(int kk) { return kk == 0 ? 0 : (((kk - 1) & 1) ? kk - 1 : kk + 1); }

// H[b * 9 + k] = T_k in[b]
__global__ __launch_bounds__(256) void k_ptc_transport(Geom g, const float2 *__restrict__ U,
                                                       const float2 *__restrict__ in, float2 *__restrict__ H) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= g.V) return;
  const int b = blockIdx.y;
  const size_t F = (size_t)12 * g.Vpad;
  const Coords k = decode(g, s);
  const float2 *src = in + b * F;
  each_hop([&](auto kk) {
    float2 h[12];
    transport_site<kk>(h, g, s, k, U, src);
    float2 *dst = H + ((size_t)b * PTC_HOPS + kk) * F;
#pragma unroll
    for (int c = 0; c < 12; ++c) dst[fidx(s, c, 12)] = h[c];
  });
}

// ------------------------------------------------------------ channel mixing
// Both mixings are one complex GEMM on the FP32 matrix cores (16x16x4 MFMA,
// four real products per complex one), columns = (site, colour):
//   forward  out[(a, s), x] = sum_{(bk, t)} W_abk[s][t] H[(bk, t), x]
//   adjoint  A[(bk, t), x] = sum_{(a, s)} conj(W_abk[s][t]) G[(a, s), x]
// A k-step is the four spins of one channel, so lane (row, t) of the first
// operand reads one entry of a 4x4 spin matrix, and lane (t, site) of the
// second one entry of a spinor plane; lane (q, site) of the result holds the
// four spins of one output channel.  A wavefront takes MIX_M row tiles (24
// channels at most) of 32 sites of one colour: the fields are read once per 24
// output channels, the weights come from L2.  Bound by the matrix cores: 8 -> 24
// channels on 16^3 x 32 is 87 GFLOP, 0.80 and 0.88 ms with them 72 and 64 %
// busy and 1.2 and 1.8 GB moved.  In vector code (each thread its site's
// twelve components, four output channels at a time) the forward product took
// 1.4 ms and the adjoint 1.56.
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int MIX_MMAX = 6;  // row tiles per wavefront at most
constexpr int MIX_N = 2;     // 16-site column tiles per wavefront

template <bool ADJ, int MIX_M>
__global__ __launch_bounds__(256, 2) void k_ptc_mix(Geom g, int nrow, int nk, int cin, const float2 *__restrict__ W,
                                                    const float2 *__restrict__ in, float2 *__restrict__ out) {
  const int lane = threadIdx.x & 63, q = lane >> 4, col = lane & 15;
  const size_t F = (size_t)12 * g.Vpad;
  const uint32_t item = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;  // (tile, colour, half of the tile)
  const uint32_t tile = item / 6, c = (item % 6) >> 1, s0 = (item & 1) * 32;
  if (tile >= g.Vpad / TILE) return;
  const int m0 = blockIdx.y * MIX_M;
  // row r of the product: (channel r / 4, spin r % 4)
  const float2 *wr[MIX_M];
#pragma unroll
  for (int m = 0; m < MIX_M; ++m) {
    const int r = min((m0 + m) * 16 + col, 4 * nrow - 1), ch = r >> 2, sp = r & 3;
    wr[m] = ADJ ? W + (size_t)ch * 16 + q * 4 + sp : W + (size_t)ch * cin * PTC_HOPS * 16 + sp * 4 + q;
  }
  const size_t wk = ADJ ? (size_t)cin * PTC_HOPS * 16 : 16;  // from one summed channel to the next
  const float2 *src = in + ((size_t)tile * 12 + q * 3 + c) * TILE + s0 + col;
  floatx4 re[MIX_M][MIX_N], im[MIX_M][MIX_N];
#pragma unroll
  for (int m = 0; m < MIX_M; ++m)
#pragma unroll
    for (int n = 0; n < MIX_N; ++n) re[m][n] = im[m][n] = floatx4{0.f, 0.f, 0.f, 0.f};
  float2 an[MIX_M], bn[MIX_N];
  auto load = [&](int k) {
#pragma unroll
    for (int n = 0; n < MIX_N; ++n) bn[n] = src[(size_t)k * F + 16 * n];
#pragma unroll
    for (int m = 0; m < MIX_M; ++m) an[m] = wr[m][(size_t)k * wk];
  };
  load(0);
  for (int k = 0; k < nk; ++k) {
    float2 a[MIX_M], b[MIX_N];
#pragma unroll
    for (int m = 0; m < MIX_M; ++m) a[m] = an[m];
#pragma unroll
    for (int n = 0; n < MIX_N; ++n) b[n] = bn[n];
    load(min(k + 1, nk - 1));
#pragma unroll
    for (int m = 0; m < MIX_M; ++m) {
      const float ay = ADJ ? -a[m].y : a[m].y, my = -ay;
#pragma unroll
      for (int n = 0; n < MIX_N; ++n) {
        re[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m].x, b[n].x, re[m][n], 0, 0, 0);
        im[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m].x, b[n].y, im[m][n], 0, 0, 0);
        re[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(my, b[n].y, re[m][n], 0, 0, 0);
        im[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(ay, b[n].x, im[m][n], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int m = 0; m < MIX_M; ++m) {
    const int ch = (m0 + m) * 4 + q;
    if (ch >= nrow) break;
    float2 *dst = out + (size_t)ch * F + ((size_t)tile * 12 + c) * TILE + s0 + col;
#pragma unroll
    for (int n = 0; n < MIX_N; ++n)
#pragma unroll
      for (int sp = 0; sp < 4; ++sp) dst[(size_t)sp * 3 * TILE + 16 * n] = cf(re[m][n][sp], im[m][n][sp]);
  }
}

// gin[b] = sum_k T_k^dag A[b*9+k]
__global__ __launch_bounds__(256) void k_ptc_transport_adj(Geom g, const float2 *__restrict__ U,
                                                           const float2 *__restrict__ A, float2 *__restrict__ gin) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= g.V) return;
  const int b = blockIdx.y;
  const size_t F = (size_t)12 * g.Vpad;
  const Coords k = decode(g, s);
  float2 acc[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = cf(0.f, 0.f);
  each_hop([&](auto kk) {
    float2 h[12];
    transport_site<adjoint_hop(kk)>(h, g, s, k, U, A + ((size_t)b * PTC_HOPS + kk) * F);
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = cf(acc[c].x + h[c].x, acc[c].y + h[c].y);
  });
  float2 *dst = gin + (size_t)b * F;
#pragma unroll
  for (int c = 0; c < 12; ++c) dst[fidx(s, c, 12)] = acc[c];
}

// Weight gradient gW[(a, s), (bk, t)] = sum over sites and colours of G_a[s][c]
// conj(H_bk[t][c]), another complex GEMM on the FP32 matrix cores with the
// sites as the summed index.  A wavefront holds WG_M x WG_N result tiles (12
// channels by 12 hops at most) and walks its share of the 16-site blocks; lane (row,
// q) reads the four consecutive sites 4 q .. 4 q + 3 of its row's plane in one
// access and uses them in four k-steps (the sum does not depend on their
// order).  Each of the workgroup's four wavefronts sums its own share in FP32,
// the shares are added in FP64: part[chunk][row][column].  (One (a, bk) pair
// per workgroup in vector code read G and H once per pair, 43 GB through L2,
// and took 4.3 ms; this takes 0.95 for 8 -> 24 channels on 16^3 x 32, 87 GFLOP
// with the matrix cores 59 % busy and 3.6 GB fetched.)
constexpr int WG_MMAX = 3, WG_N = 3;
template <int WG_M>
__global__ __launch_bounds__(256, 2) void k_ptc_wgrad(Geom g, int nrow, int ncol, int ngn, const float2 *__restrict__ G,
                                                      const float2 *__restrict__ H, double2 *__restrict__ part) {
  __shared__ double2 sh[4][64][WG_N * 4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, q = lane >> 4, col = lane & 15;
  const size_t F = (size_t)12 * g.Vpad;
  const int mg = blockIdx.y / ngn * WG_M, ng = blockIdx.y % ngn * WG_N;
  const float2 *ga[WG_M], *hb[WG_N];
#pragma unroll
  for (int m = 0; m < WG_M; ++m) {
    const int r = min((mg + m) * 16 + col, 4 * nrow - 1);
    ga[m] = G + (size_t)(r >> 2) * F + (size_t)(r & 3) * 3 * TILE + 4 * q;
  }
#pragma unroll
  for (int n = 0; n < WG_N; ++n) {
    const int r = min((ng + n) * 16 + col, 4 * ncol - 1);
    hb[n] = H + (size_t)(r >> 2) * F + (size_t)(r & 3) * 3 * TILE + 4 * q;
  }
  // Each item (16 sites of one colour) is summed by itself in FP32 and then
  // added in FP64, so that no FP32 sum is longer than 32 products however large
  // the lattice and however few the chunks.
  double sre[WG_M][WG_N][4], sim[WG_M][WG_N][4];
#pragma unroll
  for (int m = 0; m < WG_M; ++m)
#pragma unroll
    for (int n = 0; n < WG_N; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) sre[m][n][v] = sim[m][n][v] = 0.0;
  // (tile, colour, 16-site block) items, dealt to the chunks' wavefronts in turn
  const uint32_t nitem = g.Vpad / TILE * 12, step = gridDim.x * 4;
  float4 an[WG_M][2], bn[WG_N][2];
  auto load = [&](uint32_t it) {
    const uint32_t tile = it / 12, rem = it % 12;
    const size_t o = ((size_t)tile * 12 + (rem >> 2)) * TILE + (rem & 3) * 16;
#pragma unroll
    for (int m = 0; m < WG_M; ++m) {
      an[m][0] = reinterpret_cast<const float4 *>(ga[m] + o)[0];
      an[m][1] = reinterpret_cast<const float4 *>(ga[m] + o)[1];
    }
#pragma unroll
    for (int n = 0; n < WG_N; ++n) {
      bn[n][0] = reinterpret_cast<const float4 *>(hb[n] + o)[0];
      bn[n][1] = reinterpret_cast<const float4 *>(hb[n] + o)[1];
    }
  };
  uint32_t it = blockIdx.x * 4 + wv;
  if (it < nitem) load(it);
  for (; it < nitem; it += step) {
    float2 a[WG_M][4], b[WG_N][4];
#pragma unroll
    for (int m = 0; m < WG_M; ++m)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        a[m][2 * u] = cf(an[m][u].x, an[m][u].y);
        a[m][2 * u + 1] = cf(an[m][u].z, an[m][u].w);
      }
#pragma unroll
    for (int n = 0; n < WG_N; ++n)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        b[n][2 * u] = cf(bn[n][u].x, bn[n][u].y);
        b[n][2 * u + 1] = cf(bn[n][u].z, bn[n][u].w);
      }
    load(it + step < nitem ? it + step : it);
#pragma unroll
    for (int m = 0; m < WG_M; ++m) {
      floatx4 re[WG_N], im[WG_N];
#pragma unroll
      for (int n = 0; n < WG_N; ++n) re[n] = im[n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float mx = -a[m][u].x;
#pragma unroll
        for (int n = 0; n < WG_N; ++n) {
          re[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m][u].x, b[n][u].x, re[n], 0, 0, 0);
          im[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m][u].y, b[n][u].x, im[n], 0, 0, 0);
          re[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m][u].y, b[n][u].y, re[n], 0, 0, 0);
          im[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(mx, b[n][u].y, im[n], 0, 0, 0);
        }
      }
#pragma unroll
      for (int n = 0; n < WG_N; ++n)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          sre[m][n][v] += re[n][v];
          sim[m][n][v] += im[n][v];
        }
    }
  }
  const int nc = 4 * ncol;
#pragma unroll
  for (int m = 0; m < WG_M; ++m) {
    __syncthreads();
#pragma unroll
    for (int n = 0; n < WG_N; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) sh[wv][lane][n * 4 + v] = make_double2(sre[m][n][v], sim[m][n][v]);
    __syncthreads();
    // wavefront v sums register v of every column tile
    for (int n = 0; n < WG_N; ++n) {
      double2 t = make_double2(0.0, 0.0);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const double2 x = sh[w][lane][n * 4 + wv];
        t.x += x.x;
        t.y += x.y;
      }
      const int r = (mg + m) * 16 + 4 * q + wv, cc = (ng + n) * 16 + col;
      if (r < 4 * nrow && cc < nc) part[((size_t)blockIdx.x * 4 * nrow + r) * nc + cc] = t;
    }
  }
}

// gW[a][bk][s][t] from the chunks' sums
__global__ __launch_bounds__(256) void k_ptc_wgrad_final(int nrow, int ncol, int nchunk,
                                                         const double2 *__restrict__ part, float2 *__restrict__ gW) {
  __shared__ double2 sh[8][32];
  // 32 outputs per workgroup, eight threads each
  const int n = 16 * nrow * ncol, o = blockIdx.x * 32 + (threadIdx.x & 31), sub = threadIdx.x >> 5;
  double2 t = make_double2(0.0, 0.0);
  if (o < n)
    for (int c = sub; c < nchunk; c += 8) {
      const double2 v = part[(size_t)c * n + o];
      t.x += v.x;
      t.y += v.y;
    }
  sh[sub][threadIdx.x & 31] = t;
  __syncthreads();
  if (sub != 0 || o >= n) return;
#pragma unroll
  for (int q = 1; q < 8; ++q) {
    t.x += sh[q][threadIdx.x].x;
    t.y += sh[q][threadIdx.x].y;
  }
  const int r = o / (4 * ncol), cc = o - r * 4 * ncol;
  gW[(((size_t)(r >> 2) * ncol + (cc >> 2)) * 4 + (r & 3)) * 4 + (cc & 3)] = cf((float)t.x, (float)t.y);
}

// ------------------------------------------------------------ subspace fit
// Block (aggregate B, chirality chi): rows r = (site l of B, component
// 6 chi + j), j < 6.  Gram G = Y^dag Y (ny x ny) and R = Y^dag V (ny x nv),
// FP64 on the matrix cores (16x16x4, the FP32 entries widened): row tiles of
// Y, column tiles of [Y V], summed over the block's rows.  Lane (row, q) reads
// the four consecutive sites 4 q .. 4 q + 3 of a component plane (in one access
// where the block is whole groups of four sites) and uses them in four
// k-steps; the four wavefronts' shares of the sum are added in LDS.  In vector
// code from LDS rows the 24 x 48 products of 16^3 x 32 took 0.98 ms.
typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int GR_NMAX = 3;  // column tiles per workgroup at most

template <int GR_N>
__global__ __launch_bounds__(256) void k_fit_gram(Geom g, int ny, int nv, int ngn, const float2 *__restrict__ Y,
                                                  const float2 *__restrict__ V, double2 *__restrict__ GR) {
  __shared__ double sh[4][64][8];
  const uint32_t B = blockIdx.x;
  const int chi = blockIdx.y, mt = blockIdx.z / ngn, n0 = blockIdx.z % ngn * GR_N;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, q = lane >> 4, col = lane & 15;
  const int nc = ny + nv, vb = (int)g.vb, KB = (vb + 15) / 16;  // 16-site blocks of a component
  const size_t F = (size_t)12 * g.Vpad;
  const float2 *ya = Y + (size_t)min(mt * 16 + col, ny - 1) * F;
  const float2 *xb[GR_N];
#pragma unroll
  for (int n = 0; n < GR_N; ++n) {
    const int j = min((n0 + n) * 16 + col, nc - 1);
    xb[n] = j < ny ? Y + (size_t)j * F : V + (size_t)(j - ny) * F;
  }
  doublex4 re[GR_N], im[GR_N];
#pragma unroll
  for (int n = 0; n < GR_N; ++n) re[n] = im[n] = doublex4{0.0, 0.0, 0.0, 0.0};
  const bool whole = vb % 4 == 0;  // four sites 4 q .. stay in one tile and start 32-byte aligned
  auto load4 = [&](const float2 *f, int comp, int l, float2 (&o)[4]) {
    const uint32_t s = B * g.vb + l;
    if (whole) {
      const bool in = l < vb;
      const float4 *p = reinterpret_cast<const float4 *>(f + fidx(in ? s : B * g.vb, comp, 12));
      const float4 a = p[0], b = p[1];
      const float z = in ? 1.f : 0.f;
      o[0] = cf(a.x * z, a.y * z);
      o[1] = cf(a.z * z, a.w * z);
      o[2] = cf(b.x * z, b.y * z);
      o[3] = cf(b.z * z, b.w * z);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        o[u] = f[fidx(l + u < vb ? s + u : B * g.vb, comp, 12)];
        if (l + u >= vb) o[u] = cf(0.f, 0.f);
      }
    }
  };
  for (int it = wv; it < 6 * KB; it += 4) {
    const int comp = 6 * chi + it / KB, l = (it % KB) * 16 + 4 * q;
    float2 a[4], b[GR_N][4];
    load4(ya, comp, l, a);
#pragma unroll
    for (int n = 0; n < GR_N; ++n) load4(xb[n], comp, l, b[n]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double ax = a[u].x, ay = a[u].y;
#pragma unroll
      for (int n = 0; n < GR_N; ++n) {  // conj(y) x
        const double bx = b[n][u].x, by = b[n][u].y;
        re[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax, bx, re[n], 0, 0, 0);
        im[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax, by, im[n], 0, 0, 0);
        re[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(ay, by, re[n], 0, 0, 0);
        im[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ay, bx, im[n], 0, 0, 0);
      }
    }
  }
  // FP64 result layout: lane (q, col) register v holds row 4 v + q
  double2 *out = GR + ((size_t)B * 2 + chi) * ny * nc;
#pragma unroll
  for (int n = 0; n < GR_N; ++n) {
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      sh[wv][lane][2 * v] = re[n][v];
      sh[wv][lane][2 * v + 1] = im[n][v];
    }
    __syncthreads();
    double2 t = make_double2(0.0, 0.0);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      t.x += sh[w][lane][2 * wv];
      t.y += sh[w][lane][2 * wv + 1];
    }
    const int i = mt * 16 + 4 * wv + q, j = (n0 + n) * 16 + col;
    if (i < ny && j < nc) out[(size_t)i * nc + j] = t;
  }
}

// C = G^{-1} R per block by Cholesky (G = L L^dag), FP64 in LDS.  A
// non-positive pivot marks the block (flag = 1) and leaves C = 0.
__global__ __launch_bounds__(64) void k_fit_solve(int ny, int nv, const double2 *__restrict__ GR,
                                                  double2 *__restrict__ Cout, int *__restrict__ flag) {
  extern __shared__ double2 sm[];  // G [ny][ny], R [ny][nv]
  const int blk = blockIdx.x;
  const int nc = ny + nv;
  double2 *G = sm, *R = sm + ny * ny;
  const double2 *src = GR + (size_t)blk * ny * nc;
  for (int o = threadIdx.x; o < ny * nc; o += blockDim.x) {
    const int i = o / nc, j = o % nc;
    if (j < ny) G[i * ny + j] = src[o];
    else R[i * nv + (j - ny)] = src[o];
  }
  __syncthreads();
  // in-place Cholesky, lower triangle of G holds L; every lane forms the
  // pivot, lane i the entry of row i below it (one thread doing all of it
  // took 0.3 ms for 1 024 blocks)
  bool bad = false;
  for (int j = 0; j < ny; ++j) {
    double d = G[j * ny + j].x;
    for (int p = 0; p < j; ++p) d -= G[j * ny + p].x * G[j * ny + p].x + G[j * ny + p].y * G[j * ny + p].y;
    if (!(d > 0.0)) {
      bad = true;
      break;
    }
    const double ljj = sqrt(d);
    const int i = j + 1 + (int)threadIdx.x;  // ny <= 32 rows
    if (i < ny) {
      double2 a = G[i * ny + j];
      for (int p = 0; p < j; ++p) {  // a -= L[i][p] conj(L[j][p])
        const double2 x = G[i * ny + p], y = G[j * ny + p];
        a.x -= x.x * y.x + x.y * y.y;
        a.y -= x.y * y.x - x.x * y.y;
      }
      G[i * ny + j] = make_double2(a.x / ljj, a.y / ljj);
    }
    __syncthreads();
    if (threadIdx.x == 0) G[j * ny + j] = make_double2(ljj, 0.0);
    __syncthreads();
  }
  double2 *C = Cout + (size_t)blk * ny * nv;
  if (bad) {
    if (threadIdx.x == 0) atomicOr(flag, 1);
    for (int o = threadIdx.x; o < ny * nv; o += blockDim.x) C[o] = make_double2(0.0, 0.0);
    return;
  }
  // one column of R per thread: L z = r, then L^dag c = z
  for (int j = threadIdx.x; j < nv; j += blockDim.x) {
    for (int i = 0; i < ny; ++i) {
      double2 a = R[i * nv + j];
      for (int p = 0; p < i; ++p) {
        const double2 l = G[i * ny + p], z = R[p * nv + j];
        a.x -= l.x * z.x - l.y * z.y;
        a.y -= l.x * z.y + l.y * z.x;
      }
      const double d = G[i * ny + i].x;
      R[i * nv + j] = make_double2(a.x / d, a.y / d);
    }
    for (int i = ny - 1; i >= 0; --i) {
      double2 a = R[i * nv + j];
      for (int p = i + 1; p < ny; ++p) {  // a -= conj(L[p][i]) c[p]
        const double2 l = G[p * ny + i], z = R[p * nv + j];
        a.x -= l.x * z.x + l.y * z.y;
        a.y -= l.x * z.y - l.y * z.x;
      }
      const double d = G[i * ny + i].x;
      R[i * nv + j] = make_double2(a.x / d, a.y / d);
    }
    for (int i = 0; i < ny; ++i) C[i * nv + j] = R[i * nv + j];
  }
}

// Residual E = V - Y C, loss partial sum |E|^2 per block and the gradient
// gY = -(2 / Z) E C^dag, two products on the FP32 matrix cores with the
// block's rows (site, component) as columns: E^T = V^T - C^T Y^T, 16 targets at
// a time; lane (q, row) of that result holds targets 4 q .. 4 q + 3, which is
// what it has to supply as the second operand of gY^T = conj(C) E^T when its
// k-step u takes target 4 q + u, so E never leaves its registers.  (One thread
// per row with Y and gY rows in registers spilled and took 3.6 ms.)
__global__ __launch_bounds__(256) void k_fit_resid(Geom g, int ny, int nv, const float2 *__restrict__ Y,
                                                   const float2 *__restrict__ V, const double2 *__restrict__ Cm,
                                                   const double *__restrict__ Z, float2 *__restrict__ gY,
                                                   double *__restrict__ part) {
  extern __shared__ float2 cs[];  // C [ny][ldc] in FP32, zero past nv
  __shared__ double lds[4];
  const uint32_t B = blockIdx.x;
  const int chi = blockIdx.y;
  const size_t F = (size_t)12 * g.Vpad;
  const int IT = (ny + 15) >> 4, JT = (nv + 15) >> 4, ldc = JT * 16 + 1;
  const double2 *C = Cm + ((size_t)B * 2 + chi) * ny * nv;
  for (int o = threadIdx.x; o < ny * ldc; o += blockDim.x) {
    const int i = o / ldc, j = o - i * ldc;
    cs[o] = j < nv ? cf((float)C[i * nv + j].x, (float)C[i * nv + j].y) : cf(0.f, 0.f);
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, q = lane >> 4, col = lane & 15;
  const float sc = (float)(-2.0 / Z[0]);
  const int KB = ((int)g.vb + 15) / 16;
  double t[1] = {0.0};
  for (int it = wv; it < 6 * KB; it += 4) {
    const int comp = 6 * chi + it / KB, l = (it % KB) * 16 + col;
    const bool on = l < (int)g.vb;
    const size_t off = fidx(B * g.vb + (on ? l : 0), comp, 12);
    float2 y[8];  // lane (q, row): Y_{4 u + q}
#pragma unroll
    for (int u = 0; u < 8; ++u) y[u] = Y[(size_t)min(4 * u + q, ny - 1) * F + off];
    floatx4 gr[2], gi[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) gr[m] = gi[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int jt = 0; jt < JT; ++jt) {
      // Y C is summed by itself and then taken from V: its partial sums are
      // smaller than V and round less
      floatx4 er = {0.f, 0.f, 0.f, 0.f}, ei = {0.f, 0.f, 0.f, 0.f};
      float2 x[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = V[(size_t)min(16 * jt + 4 * q + v, nv - 1) * F + off];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (4 * u >= ny) break;
        float2 c = cs[min(4 * u + q, ny - 1) * ldc + 16 * jt + col];
        if (4 * u + q >= ny) c = cf(0.f, 0.f);
        er = __builtin_amdgcn_mfma_f32_16x16x4f32(c.x, y[u].x, er, 0, 0, 0);
        ei = __builtin_amdgcn_mfma_f32_16x16x4f32(c.x, y[u].y, ei, 0, 0, 0);
        er = __builtin_amdgcn_mfma_f32_16x16x4f32(-c.y, y[u].y, er, 0, 0, 0);
        ei = __builtin_amdgcn_mfma_f32_16x16x4f32(c.y, y[u].x, ei, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool in = 16 * jt + 4 * q + v < nv;
        er[v] = in ? x[v].x - er[v] : 0.f;
        ei[v] = in ? x[v].y - ei[v] : 0.f;
      }
      if (on) {
#pragma unroll
        for (int v = 0; v < 4; ++v) t[0] += (double)er[v] * er[v] + (double)ei[v] * ei[v];
      }
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        if (m >= IT) break;
#pragma unroll
        for (int v = 0; v < 4; ++v) {  // e conj(c)
          const float2 c = cs[min(16 * m + col, ny - 1) * ldc + 16 * jt + 4 * q + v];
          gr[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.x, er[v], gr[m], 0, 0, 0);
          gi[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.x, ei[v], gi[m], 0, 0, 0);
          gr[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.y, ei[v], gr[m], 0, 0, 0);
          gi[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(-c.y, er[v], gi[m], 0, 0, 0);
        }
      }
    }
    if (on) {
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = 16 * m + 4 * q + v;
          if (i < ny) gY[(size_t)i * F + off] = cf(sc * gr[m][v], sc * gi[m][v]);
        }
    }
  }
  block_sum<1>(t, lds);
  if (threadIdx.x == 0) part[(size_t)B * 2 + chi] = t[0];
}

__global__ void k_ptc_sum(const double *__restrict__ p, int n, double *__restrict__ out) {
  __shared__ double lds[4];
  double t[1] = {0.0};
  for (int i = threadIdx.x; i < n; i += blockDim.x) t[0] += p[i];
  block_sum<1>(t, lds);
  if (threadIdx.x == 0) out[0] = t[0];
}

__global__ __launch_bounds__(256) void k_ptc_norm2(const float2 *__restrict__ x, size_t n, double *__restrict__ part) {
  __shared__ double lds[4];
  double t[1] = {0.0};
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    t[0] += (double)x[i].x * x[i].x + (double)x[i].y * x[i].y;
  block_sum<1>(t, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = t[0];
}

// Adam on the real and imaginary parts of complex parameters.
__global__ __launch_bounds__(256) void k_ptc_adam(float2 *__restrict__ W, const float2 *__restrict__ gW,
                                                  float2 *__restrict__ m, float2 *__restrict__ v, size_t n, float lr,
                                                  float b1, float b2, float eps, float c1, float c2) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float2 g = gW[i];
  float2 mi = m[i], vi = v[i];
  mi = cf(b1 * mi.x + (1.f - b1) * g.x, b1 * mi.y + (1.f - b1) * g.y);
  vi = cf(b2 * vi.x + (1.f - b2) * g.x * g.x, b2 * vi.y + (1.f - b2) * g.y * g.y);
  m[i] = mi;
  v[i] = vi;
  const float2 w = W[i];
  W[i] = cf(w.x - lr * (mi.x / c1) / (sqrtf(vi.x / c2) + eps), w.y - lr * (mi.y / c1) / (sqrtf(vi.y / c2) + eps));
}

// ---------------------------------------------------------------- launchers
hipError_t ptc_transport(const Geom &g, const float2 *U, const float2 *in, int cin, float2 *H, hipStream_t st) {
  hipLaunchKernelGGL(k_ptc_transport, dim3(div_up(g.V, 256), cin), dim3(256), 0, st, g, U, in, H);
  return hipGetLastError();
}
// nrow output channels from nk summed ones; the row tiles in as few equal
// groups of at most MIX_MMAX as they make.  With six always, a network of two
// channels on 16^3 x 32 computed five empty tiles: forward pass 462 us, 301 in
// vector code, 249 this way (24 output channels, six tiles: 1.4 ms).
template <bool ADJ>
static hipError_t mix(const Geom &g, int nrow, int nk, int cin, const float2 *W, const float2 *in, float2 *out,
                      hipStream_t st) {
  const int tiles = div_up(4 * nrow, 16), ng = div_up(tiles, MIX_MMAX);
  const dim3 grid(div_up((long)g.Vpad / TILE * 6, 4), ng);
  switch (div_up(tiles, ng)) {
#define MG_MIX(M)                                                                                              \
  case M:                                                                                                      \
    hipLaunchKernelGGL((k_ptc_mix<ADJ, M>), grid, dim3(256), 0, st, g, nrow, nk, cin, W, in, out);             \
    break;
    MG_MIX(1) MG_MIX(2) MG_MIX(3) MG_MIX(4) MG_MIX(5) MG_MIX(6)
#undef MG_MIX
  }
  return hipGetLastError();
}
hipError_t ptc_mix(const Geom &g, int cin, int cout, const float2 *W, const float2 *H, float2 *out, hipStream_t st) {
  return mix<false>(g, cout, cin * PTC_HOPS, cin, W, H, out, st);
}
hipError_t ptc_mix_adj(const Geom &g, int cin, int cout, const float2 *W, const float2 *G, float2 *A,
                       hipStream_t st) {
  return mix<true>(g, cin * PTC_HOPS, cout, cin, W, G, A, st);
}
hipError_t ptc_transport_adj(const Geom &g, const float2 *U, const float2 *A, int cin, float2 *gin, hipStream_t st) {
  hipLaunchKernelGGL(k_ptc_transport_adj, dim3(div_up(g.V, 256), cin), dim3(256), 0, st, g, U, A, gin);
  return hipGetLastError();
}
// Chunks of the weight gradient's site sum: enough workgroups for the device,
// and no more partial sums than that takes.
int ptc_wchunks(int cin, int cout) {
  const int groups = div_up(4 * cout, 16 * WG_MMAX) * div_up(4 * cin * PTC_HOPS, 16 * WG_N);
  return std::max(1, std::min(256, div_up(1024, groups)));
}
hipError_t ptc_wgrad(const Geom &g, int cin, int cout, const float2 *G, const float2 *H, double2 *part, float2 *gW,
                     hipStream_t st) {
  const int ncol = cin * PTC_HOPS, nchunk = ptc_wchunks(cin, cout);
  const int tiles = div_up(4 * cout, 16), ngm = div_up(tiles, WG_MMAX), ngn = div_up(4 * ncol, 16 * WG_N);
  const dim3 grid(nchunk, ngm * ngn);
  // equal groups of row tiles, none of them empty: two channels on 16^3 x 32
  // 142 us with three always, 125 in vector code, 69 this way
  switch (div_up(tiles, ngm)) {
#define MG_WG(M)                                                                                        \
  case M:                                                                                               \
    hipLaunchKernelGGL(k_ptc_wgrad<M>, grid, dim3(256), 0, st, g, cout, ncol, ngn, G, H, part);         \
    break;
    MG_WG(1) MG_WG(2) MG_WG(3)
#undef MG_WG
  }
  hipLaunchKernelGGL(k_ptc_wgrad_final, dim3(div_up(16 * cout * ncol, 32)), dim3(256), 0, st, cout, ncol, nchunk, part,
                     gW);
  return hipGetLastError();
}
hipError_t ptc_fit(const Geom &g, int ny, int nv, const float2 *Y, const float2 *V, const double *Z, double2 *GR,
                   double2 *C, int *flag, float2 *gY, double *part, double *loss, hipStream_t st) {
  const int nc = ny + nv, tiles = div_up(nc, 16), ngn = div_up(tiles, GR_NMAX);
  const dim3 grid(g.Vc, 2, div_up(ny, 16) * ngn);
  // equal groups again: two channels 206 us with three always, 77 in vector
  // code, 79 this way
  switch (div_up(tiles, ngn)) {
#define MG_GR(N)                                                                                \
  case N:                                                                                       \
    hipLaunchKernelGGL(k_fit_gram<N>, grid, dim3(256), 0, st, g, ny, nv, ngn, Y, V, GR);        \
    break;
    MG_GR(1) MG_GR(2) MG_GR(3)
#undef MG_GR
  }
  hipLaunchKernelGGL(k_fit_solve, dim3(g.Vc * 2), dim3(64), sizeof(double2) * ny * nc, st, ny, nv, GR, C, flag);
  const size_t lds = sizeof(float2) * ny * (div_up(nv, 16) * 16 + 1);
  hipLaunchKernelGGL(k_fit_resid, dim3(g.Vc, 2), dim3(256), lds, st, g, ny, nv, Y, V, C, Z, gY, part);
  hipLaunchKernelGGL(k_ptc_sum, dim3(1), dim3(256), 0, st, part, (int)(g.Vc * 2), loss);
  return hipGetLastError();
}
hipError_t ptc_norm2(const float2 *x, size_t n, double *part, double *out, hipStream_t st) {
  hipLaunchKernelGGL(k_ptc_norm2, dim3(PTC_NBLOCKS), dim3(256), 0, st, x, n, part);
  hipLaunchKernelGGL(k_ptc_sum, dim3(1), dim3(256), 0, st, part, PTC_NBLOCKS, out);
  return hipGetLastError();
}
hipError_t ptc_adam_k(float2 *W, const float2 *gW, float2 *m, float2 *v, size_t n, int step, double lr, double b1,
                      double b2, double eps, hipStream_t st) {
  const float c1 = (float)(1.0 - pow(b1, step)), c2 = (float)(1.0 - pow(b2, step));
  hipLaunchKernelGGL(k_ptc_adam, dim3(div_up((long)n, 256)), dim3(256), 0, st, W, gW, m, v, n, (float)lr, (float)b1,
                     (float)b2, (float)eps, c1, c2);
  return hipGetLastError();
}

}  // namespace mg
