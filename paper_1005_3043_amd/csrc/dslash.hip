// Fine-level Wilson-Dirac operator, Eq. (2):
//   (D psi)(x) = (4+m) psi(x) - 1/2 sum_mu [ eta (1-gamma_mu) U_mu(x) psi(x+mu)
//                                          + eta (1+gamma_mu) U_mu(x-mu)^dag psi(x-mu) ]
// eta = -1 on hops across an antiperiodic time boundary.
//
// The spin projection (wilson_site.h) reduces each hop to a half spinor and
// two SU(3) mat-vecs: 1320 flops per site for all eight hops.
//
// One thread per site of the site-blocked, tile-interleaved layout (two or
// three right-hand sides per thread when there are several).  The loop over mu
// is rolled (wave-uniform).  Links are either stored in full (9 complex) or as
// their first two rows (6 complex, NL = 6); the third row of an SU(3) matrix is
// the complex conjugate of the cross product of the first two, which trades 42
// flops per link for a third less link traffic.
#include <type_traits>

#include "kernels.h"
#include "wilson_site.h"

namespace mg {

template <typename C> __host__ __device__ __forceinline__ void reconstruct_row2(C (&u)[9]) {
  // row 2 = conj(row0 x row1)
  const C a = csub(cmul(u[1], u[5]), cmul(u[2], u[4]));
  const C b = csub(cmul(u[2], u[3]), cmul(u[0], u[5]));
  const C c = csub(cmul(u[0], u[4]), cmul(u[1], u[3]));
  u[6] = mk<C>(a.x, -a.y);
  u[7] = mk<C>(b.x, -b.y);
  u[8] = mk<C>(c.x, -c.y);
}

template <int NL, typename C, typename S>
__device__ __forceinline__ void load_link_t(C (&u)[9], const S *__restrict__ U, int mu, uint32_t s) {
#pragma unroll
  for (int e = 0; e < NL; ++e) u[e] = cvt<C>(U[fidx(s, mu * NL + e, 4 * NL)]);
  if constexpr (NL == 6) reconstruct_row2(u);
}

// A 256-site workgroup's copy of its own input, each thread one site, in the
// storage type and the layout of the field.
template <typename TI> __device__ __forceinline__ void stage_sites(TI *sh, const TI *__restrict__ in, uint32_t s) {
  constexpr int NS = SiteSlots<TI>::n;
#pragma unroll
  for (int c = 0; c < NS; ++c) sh[fidx(threadIdx.x, c, NS)] = in[fidx(s, c, NS)];
}

// The stencil at one site for K right-hand sides (input stride vs between
// them): each direction's two links are loaded once and applied to all K.
// Only the first kv are distinct; the spare slots repeat the last of them.
//
// Bound by the bytes that miss L2: the wavefronts in flight on an XCD hold
// more spinors and links than its 4 MB, so a site's spinor was fetched again
// by most hops that read it (12 right-hand sides on 32^3 x 64 read 28.1 GB in
// FP64 and 12.7 GB in FP32; with the copy 18.2 and 10.7 GB).
// The workgroup's own 256 sites are therefore copied to LDS once (sh), and a
// hop that stays inside them reads there: with 4^4 aggregates two thirds of
// all hops.  The choice is one address select per hop in front of flat loads;
// loads in two divergent branches measured 2.42 ms, one select 2.22, no copy
// 2.38.  Per launch, before / after: one right-hand side FP64 494 / 386 us,
// FP32 264 / 236, FP16 class 162 / 139; twelve FP64 4.49 / 3.99 ms, FP32 2.39
// / 2.18, FP16 class 1.67 / 1.58, the MR q-recursion forms 3.29 / 3.03 and
// 2.32 / 2.21.  On 16^3 x 32 one FP32 right-hand side took 27.7 us with the
// coordinates in an indexed array (memory), 15.5 with selects.
template <int K, int NL, typename C, typename S, typename TI>
__device__ __forceinline__ void dslash_site_k(C (&res)[K][12], C (&ctr)[K][12], const Geom &g, uint32_t s,
                                              const S *__restrict__ U, const TI *__restrict__ in, size_t vs, int kv,
                                              decltype(C::x) diag, const TI *sh) {
  using R = decltype(C::x);
  constexpr int NS = SiteSlots<TI>::n;
  // component c at 64 c behind this, in the workgroup's copy or in memory
  auto site = [&](int k, uint32_t t) -> const TI * {
    return (t ^ s) < 256 ? sh + k * 256 * NS + fidx(t & 255u, 0, NS)
                         : in + (size_t)(k < kv ? k : kv - 1) * vs + fidx(t, 0, NS);
  };
  const Coords kk = decode(g, s);
  C acc[K][12];
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int i = 0; i < 12; ++i) acc[k][i] = mk<C>(0, 0);
#pragma unroll 1
  for (int mu = 0; mu < 4; ++mu) {
    // selects, not an indexed array (which would live in memory)
    const int o = mu == 0 ? kk.o[0] : mu == 1 ? kk.o[1] : mu == 2 ? kk.o[2] : kk.o[3];
    const int cc = mu == 0 ? kk.c[0] : mu == 1 ? kk.c[1] : mu == 2 ? kk.c[2] : kk.c[3];
    const uint32_t sf = nbr_fwd(g, s, o, cc, mu), sb = nbr_bwd(g, s, o, cc, mu);
    R ef = 1, eb = 1;
    if (mu == 3 && g.antiperiodic) {
      if (kk.o[3] == g.b[3] - 1 && kk.c[3] == g.C[3] - 1) ef = -1;
      if (kk.o[3] == 0 && kk.c[3] == 0) eb = -1;
    }
    C u[9];
    load_link_t<NL>(u, U, mu, s);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      C p[12];
      load_site(p, site(k, sf), 0);
      hop_dispatch<true>(mu, acc[k], p, u, ef);
    }
    load_link_t<NL>(u, U, mu, sb);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      C p[12];
      load_site(p, site(k, sb), 0);
      hop_dispatch<false>(mu, acc[k], p, u, eb);
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    load_site(ctr[k], sh + k * 256 * NS, s & 255u);
#pragma unroll
    for (int i = 0; i < 12; ++i) {
      res[k][i].x = fma(diag, ctr[k][i].x, (R)-0.5 * acc[k][i].x);
      res[k][i].y = fma(diag, ctr[k][i].y, (R)-0.5 * acc[k][i].y);
    }
  }
}

// Block of `per` consecutive sites that workgroup bid of nblk visits.  The
// hardware deals workgroups to the eight XCDs round-robin; xcd_remap gives
// each XCD a contiguous range of the visiting order.  Where aggregates are
// whole blocks and the coarse z extent is divisible by 8, XCD k takes the
// aggregates of the z layers k C_z/8 .. (k+1) C_z/8 - 1 and walks them x
// fastest, then y, then t: the t neighbours of an aggregate are visited one
// x-y layer apart on the same XCD (L2), and the XCDs move through t in step,
// so the z neighbours another XCD needs are read at about the same time.
// (The aggregate-major order walks x, y, z, then t, with each XCD owning a
// t range; on 32^3 x 64 the visiting order above is 3-6 % faster, and
// walking 4x4-aggregate x-y quadrants in t or in z instead is 5-13 % slower.)
// Otherwise the order is the storage order.
__device__ __forceinline__ uint32_t visit_pos(uint32_t q, uint32_t nblk, const Geom &g, uint32_t per) {
  const uint32_t sub = g.vb / per;
  const uint32_t C0 = (uint32_t)g.C[0], C1 = (uint32_t)g.C[1], C2 = (uint32_t)g.C[2], C3 = (uint32_t)g.C[3];
  if ((nblk & 7u) == 0 && C2 % 8 == 0 && sub * per == g.vb && nblk == g.Vc * sub) {
    const uint32_t per_xcd = nblk >> 3, xcd = q / per_xcd, r0 = q - xcd * per_xcd;
    const uint32_t j = r0 % sub;
    uint32_t r = r0 / sub;
    const uint32_t cx = r % C0;
    r /= C0;
    const uint32_t cy = r % C1;
    r /= C1;
    const uint32_t ct = r % C3;
    const uint32_t cz = xcd * (C2 >> 3) + r / C3;
    return (cx + C0 * (cy + C1 * (cz + C2 * ct))) * sub + j;
  }
  return q;
}
__device__ __forceinline__ uint32_t visit_block(uint32_t bid, uint32_t nblk, const Geom &g, uint32_t per) {
  return visit_pos(xcd_remap(bid, nblk), nblk, g, per);
}

// Minimum waves per SIMD requested from the register allocator (0 = none).
#ifndef MG_DSLASH_WAVES_F64
#define MG_DSLASH_WAVES_F64 0
#endif
#ifndef MG_DSLASH_WAVES_F32
#define MG_DSLASH_WAVES_F32 0
#endif
template <typename R> constexpr int dslash_waves() {
  return sizeof(R) == 8 ? MG_DSLASH_WAVES_F64 : MG_DSLASH_WAVES_F32;
}

// The MR step of the q recursion (DS_MRQ) at one site: res = D q_k and
// ctr = q_k on entry; q_{k+1} = q_k - a D q_k is written to qout and left in
// res, r_{k+1} = rprev - a q_k to rout and left in ctr (values as stored).
// rprev is read once by the launch: non-temporal loads keep L2 for the
// neighbour spinors and links (12-RHS FP32 3.37 -> 3.31 ms, FP16 class 2.41
// -> 2.33 ms on 32^3 x 64); likewise b of the residual form.
template <typename C, typename TO>
__device__ __forceinline__ void mrq_site(C (&res)[12], C (&ctr)[12], const TO *rprev, TO *qout, TO *rout,
                                         uint32_t s, double2 ad) {
  using R = decltype(C::x);
  const C ma = mk<C>((R)-ad.x, (R)-ad.y);
  C rp[12];
  load_site_nt(rp, rprev, s);
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const C t = res[i];
    res[i] = cfma(ma, t, ctr[i]);
    rp[i] = cfma(ma, ctr[i], rp[i]);
  }
  store_site<true>(qout, s, res);
  store_site<true>(rout, s, rp);
#pragma unroll
  for (int i = 0; i < 12; ++i) ctr[i] = rp[i];
}

// One site per thread, one right-hand side per grid row.  Input spinors
// are stored as TI, the output (and b of the residual mode) as TO: complex
// FP64 / FP32, or binary16 with a per-site scale (h16).
template <typename R, int MODE, int NL, typename S, typename TI, typename TO>
__global__ __launch_bounds__(256, dslash_waves<R>()) void k_dslash(Geom g, const S *__restrict__ U,
                                                const TI *__restrict__ in, TO *__restrict__ out,
                                                const TO *__restrict__ b, R diag,
                                                double *__restrict__ partials, MrqArgs<TO> mq) {
  using C = c_t<R>;
  in += (size_t)blockIdx.y * site_slots<TI>() * g.Vpad;
  const size_t off = (size_t)blockIdx.y * site_slots<TO>() * g.Vpad;
  out += off;
  const uint32_t s = visit_block(blockIdx.x, gridDim.x, g, 256) * 256 + threadIdx.x;
  __shared__ TI sh[256 * SiteSlots<TI>::n];
  stage_sites(sh, in, s < g.V ? s : g.V - 1);
  __syncthreads();
  double red[3] = {0.0, 0.0, 0.0};
  if (s < g.V) {
    C res1[1][12], ctr1[1][12];
    dslash_site_k<1, NL, C>(res1, ctr1, g, s, U, in, 0, 1, diag, sh);
    C(&res)[12] = res1[0], (&ctr)[12] = ctr1[0];
    if constexpr (MODE == DS_RESID) {
      C bb[12];
      load_site_nt(bb, b + off, s);
#pragma unroll
      for (int i = 0; i < 12; ++i) res[i] = csub(bb[i], res[i]);
    }
    // the output is not read again by this launch: non-temporal stores leave
    // L2 to the neighbour spinors and links that are
    if constexpr (MODE == DS_MRQ) mrq_site(res, ctr, mq.rprev + off, out, mq.rout + off, s, mq.alpha[blockIdx.y]);
    else store_site<true>(out, s, res);
    if constexpr (MODE == DS_MR || MODE == DS_MRQ) {
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        // <q, r> = sum conj(q) r with q = D r (as stored), r = centre (DS_MRQ:
        // q_{k+1} and r_{k+1} as stored)
        red[0] += (double)res[i].x * ctr[i].x + (double)res[i].y * ctr[i].y;
        red[1] += (double)res[i].x * ctr[i].y - (double)res[i].y * ctr[i].x;
        red[2] += (double)res[i].x * res[i].x + (double)res[i].y * res[i].y;
      }
    }
  }
  if constexpr (MODE == DS_MR || MODE == DS_MRQ) {
    __shared__ double lds[16 * 3];
    block_sum<3>(red, lds);
    if (threadIdx.x == 0) {
      double *p = partials + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 3;
      p[0] = red[0];
      p[1] = red[1];
      p[2] = red[2];
    }
  }
}

// Several right-hand sides: K per thread (256-site workgroups), so that
// each direction's links are loaded once for all K; the workgroups of one
// group of K right-hand sides cover the lattice, grid.y = groups (K from
// take_three below).  K = 2 against one per thread, 12 right-hand sides on
// 32^3 x 64: FP32 2.25 / 2.60 ms.  Running the groups of one block back to
// back on an XCD is slower (links from L2, but the spinor neighbours further
// apart).  A ragged last group repeats its last right-hand side in the spare
// slots and stores only the valid ones.
// Tile blocks per chunk of the right-hand-side-group order below (0: the
// groups one after another over the whole lattice).  On 32^3 x 64 with 12
// right-hand sides, 512 blocks (16 chunks, 25 MB of FP32 links each):
// FP32 2.52 -> 2.42 ms, FP16 class 1.74 -> 1.70 ms, FP64 4.77 -> 4.69 ms
// per launch before the LDS copy, the MR q-recursion forms within 1 %; 128 and
// 2048 blocks gained less or lost, and with the copy 256 blocks lose 2-3 %
// against 512 (FP32 2.31 / 2.25 ms, FP64 4.07 / 3.99).
#ifndef MG_DSLASH_CHUNK
#define MG_DSLASH_CHUNK 512
#endif
template <typename R, int MODE, int NL, typename S, int K, typename TI, typename TO>
__global__ __launch_bounds__(256, dslash_waves<R>()) void k_dslash_rb(Geom g, const S *__restrict__ U, const TI *__restrict__ in,
                                                   TO *__restrict__ out, const TO *__restrict__ b, R diag,
                                                   double *__restrict__ partials, int nrhs, MrqArgs<TO> mq) {
  using C = c_t<R>;
  // Right-hand-side groups in chunks of the lattice: the workgroups of the
  // launch (in dispatch order) take the groups of one chunk of RHS_CHUNK
  // tile blocks in turn before the next chunk, so that a chunk's links are
  // read again by the other groups while they are still in the last-level
  // cache.  The chunk is a multiple of 8 blocks: a workgroup's XCD (dispatch
  // order modulo 8) is the one its tile block belongs to.
  uint32_t bid = blockIdx.x;
  int grp = blockIdx.y;
  constexpr uint32_t CH = MG_DSLASH_CHUNK;
  if (CH > 0 && gridDim.x % CH == 0) {
    const uint32_t lin = blockIdx.y * gridDim.x + blockIdx.x, span = CH * gridDim.y;
    const uint32_t c = lin / span, rem = lin - c * span;
    grp = (int)(rem / CH);
    bid = c * CH + rem % CH;
  }
  const int r0 = grp * K;
  const uint32_t slot = bid, nslot = gridDim.x;
  const int kv = nrhs - r0 < K ? nrhs - r0 : K;
  const size_t vsi = (size_t)site_slots<TI>() * g.Vpad, vso = (size_t)site_slots<TO>() * g.Vpad;
  const uint32_t s = visit_block(bid, gridDim.x, g, 256) * 256 + threadIdx.x;
  __shared__ TI sh[K * 256 * SiteSlots<TI>::n];
#pragma unroll
  for (int k = 0; k < K; ++k)
    stage_sites(sh + k * 256 * SiteSlots<TI>::n, in + (size_t)(r0 + (k < kv ? k : kv - 1)) * vsi,
                s < g.V ? s : g.V - 1);
  __syncthreads();
  double red[K][3];
#pragma unroll
  for (int k = 0; k < K; ++k) red[k][0] = red[k][1] = red[k][2] = 0.0;
  if (s < g.V) {
    C res[K][12], ctr[K][12];
    dslash_site_k<K, NL, C>(res, ctr, g, s, U, in + (size_t)r0 * vsi, vsi, kv, diag, sh);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (k >= kv) break;
      const size_t off = (size_t)(r0 + k) * vso;
      if constexpr (MODE == DS_RESID) {
        C bb[12];
        load_site_nt(bb, b + off, s);
#pragma unroll
        for (int i = 0; i < 12; ++i) res[k][i] = csub(bb[i], res[k][i]);
      }
      if constexpr (MODE == DS_MRQ)
        mrq_site(res[k], ctr[k], mq.rprev + off, out + off, mq.rout + off, s, mq.alpha[r0 + k]);
      else
        store_site<true>(out + off, s, res[k]);
      if constexpr (MODE == DS_MR || MODE == DS_MRQ) {
#pragma unroll
        for (int i = 0; i < 12; ++i) {
          red[k][0] += (double)res[k][i].x * ctr[k][i].x + (double)res[k][i].y * ctr[k][i].y;
          red[k][1] += (double)res[k][i].x * ctr[k][i].y - (double)res[k][i].y * ctr[k][i].x;
          red[k][2] += (double)res[k][i].x * res[k][i].x + (double)res[k][i].y * res[k][i].y;
        }
      }
    }
  }
  if constexpr (MODE == DS_MR || MODE == DS_MRQ) {
    __shared__ double lds[4 * 3 * K];
    double v[3 * K];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int q = 0; q < 3; ++q) v[3 * k + q] = red[k][q];
    block_sum<3 * K>(v, lds);
    if (threadIdx.x == 0) {
      for (int k = 0; k < kv; ++k) {
        double *p = partials + ((size_t)(r0 + k) * nslot + slot) * 3;
        p[0] = v[3 * k];
        p[1] = v[3 * k + 1];
        p[2] = v[3 * k + 2];
      }
    }
  }
}

// Right-hand sides per thread of the multi-RHS stencil: each link is loaded
// once per group, and a ragged last group computes its spare slots.  Three
// where that computes no more slots than two would, two otherwise (both at
// two waves per SIMD).  32^3 x 64, two / three: 12 right-hand sides FP32 2.25
// / 2.18 ms, binary16 spinors 1.68 / 1.58 ms; four right-hand sides FP32 0.77
// / 0.99 ms, binary16 0.59 / 0.73 ms.  FP64 spinors spill with three; FP64
// arithmetic on FP32-stored vectors (256 registers, no spill, one wave per
// SIMD) follows the rule.
template <typename R, typename TI> bool take_three(int nrhs) {
  return !(sizeof(R) == 8 && std::is_same<TI, double2>::value) && (nrhs + 2) / 3 * 3 <= (nrhs + 1) / 2 * 2;
}

// Latency form: the eight hops of a 64-site tile run on eight wavefronts at
// once (one round trip of loads instead of eight) and leave their
// contributions in LDS, where four wavefronts add three components each in
// the order of the other kernels (bit-identical results); the first wavefront
// finishes the sites.  Sums: one partial per tile.  Bound by latency: of its
// 4.7 us (8^4, FP64; 10.9 with the hops in turn) about 2 are the loads.
template <typename R, int MODE, int NL, typename S, typename TI, typename TO>
__global__ __launch_bounds__(512, 2) void k_dslash_split(Geom g, const S *__restrict__ U, const TI *__restrict__ in,
                                                         TO *__restrict__ out, const TO *__restrict__ b, R diag,
                                                         double *__restrict__ partials, MrqArgs<TO> mq) {
  using C = c_t<R>;
  __shared__ C hop[8][12][64];
  const int lane = threadIdx.x & 63, h = threadIdx.x >> 6;
  in += (size_t)blockIdx.y * site_slots<TI>() * g.Vpad;
  const size_t off = (size_t)blockIdx.y * site_slots<TO>() * g.Vpad;
  out += off;
  const uint32_t s0 = blockIdx.x * 64 + lane;
  const bool live = s0 < g.V;
  const uint32_t s = live ? s0 : g.V - 1;
  C ctr[12];
  if (h == 0) load_site(ctr, in, s);
  {
    const Coords k = decode(g, s);
    const int mu = h >> 1;
    const bool fwd = (h & 1) == 0;
    const int o = mu == 0 ? k.o[0] : mu == 1 ? k.o[1] : mu == 2 ? k.o[2] : k.o[3];
    const int c = mu == 0 ? k.c[0] : mu == 1 ? k.c[1] : mu == 2 ? k.c[2] : k.c[3];
    const uint32_t sn = fwd ? nbr_fwd(g, s, o, c, mu) : nbr_bwd(g, s, o, c, mu);
    R eta = 1;
    if (mu == 3 && g.antiperiodic && (fwd ? o == g.b[3] - 1 && c == g.C[3] - 1 : o == 0 && c == 0)) eta = -1;
    C p[12], u[9], acc[12];
    load_site(p, in, sn);
    load_link_t<NL>(u, U, mu, fwd ? s : sn);
#pragma unroll
    for (int i = 0; i < 12; ++i) acc[i] = mk<C>(0, 0);
    if (fwd) hop_dispatch<true>(mu, acc, p, u, eta);
    else hop_dispatch<false>(mu, acc, p, u, eta);
#pragma unroll
    for (int i = 0; i < 12; ++i) hop[h][i][lane] = acc[i];
  }
  __syncthreads();
  if (h < 4) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      C t = hop[0][3 * h + i][lane];
#pragma unroll
      for (int q = 1; q < 8; ++q) t = cadd(t, hop[q][3 * h + i][lane]);
      hop[0][3 * h + i][lane] = t;  // read by this lane only
    }
  }
  __syncthreads();
  if (h != 0) return;
  C res[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const C a = hop[0][i][lane];
    res[i].x = fma(diag, ctr[i].x, (R)-0.5 * a.x);
    res[i].y = fma(diag, ctr[i].y, (R)-0.5 * a.y);
  }
  double red[3] = {0.0, 0.0, 0.0};
  if (live) {
    if constexpr (MODE == DS_RESID) {
      C bb[12];
      load_site_nt(bb, b + off, s);
#pragma unroll
      for (int i = 0; i < 12; ++i) res[i] = csub(bb[i], res[i]);
    }
    if constexpr (MODE == DS_MRQ) mrq_site(res, ctr, mq.rprev + off, out, mq.rout + off, s, mq.alpha[blockIdx.y]);
    else store_site(out, s, res);
    if constexpr (MODE == DS_MR || MODE == DS_MRQ) {
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        red[0] += (double)res[i].x * ctr[i].x + (double)res[i].y * ctr[i].y;
        red[1] += (double)res[i].x * ctr[i].y - (double)res[i].y * ctr[i].x;
        red[2] += (double)res[i].x * res[i].x + (double)res[i].y * res[i].y;
      }
    }
  }
  if constexpr (MODE == DS_MR || MODE == DS_MRQ) {
#pragma unroll
    for (int q = 0; q < 3; ++q) red[q] = wave_sum(red[q]);
    if (lane == 0) {
      double *p = partials + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 3;
      p[0] = red[0];
      p[1] = red[1];
      p[2] = red[2];
    }
  }
}

// Tiles (all right-hand sides together) up to which the latency form runs:
// beyond, its traffic and the single finishing wavefront cost more than the
// round trips.  This form / the others, in us: 64 tiles FP64 4.7 / 10.9, FP32
// 4.4 / 9.7, FP16 class 4.2 / 9.2; 324 tiles 9.0 / 12.7, 5.8 / 9.8, 5.1 / 9.3;
// 512 tiles 11.2 / 11.9, 6.3 / 10.0, 5.3 / 9.4; 1024 tiles 21 / 15, 11.3 /
// 10.6, 8.9 / 9.4.  Several right-hand sides: 64 x 12 tiles 14 / 19, 8.3 / 22,
// 7.8 / 19; 128 x 12 tiles FP64 26 / 22.  One line for all types, since the
// number of partial sums follows it.
static bool take_split(const Geom &g, int nrhs) {
  return (uint64_t)div_up(g.V, 64) * nrhs <= (nrhs == 1 ? 512u : 768u);
}

int dslash_blocks(const Geom &g) { return div_up(g.V, 256); }
int dslash_partials(const Geom &g, int nrhs) { return take_split(g, nrhs) ? div_up(g.V, 64) : dslash_blocks(g); }

// Modes that exist for a pair of storage types: FP64 arithmetic on FP32
// spinors is only applied plainly (dslash_in32), a binary16 output of FP32
// spinors is only the residual, the q recursion is not taken in FP64.
template <typename R, typename TI, typename TO> constexpr bool has_mode(DslashMode m) {
  if (!std::is_same<TI, TO>::value) return m == (sizeof(R) == 8 ? DS_PLAIN : DS_RESID);
  return m != DS_MRQ || sizeof(R) == 4;
}
// f(constant mode)
template <typename R, typename TI, typename TO, typename F> static hipError_t with_mode(DslashMode mode, F &&f) {
  switch (mode) {
#define MG_MODE(M)                                         \
  case M:                                                  \
    if constexpr (has_mode<R, TI, TO>(M)) {                \
      f(std::integral_constant<int, M>());                 \
      return hipGetLastError();                            \
    }                                                      \
    break;
    MG_MODE(DS_PLAIN) MG_MODE(DS_RESID) MG_MODE(DS_MR) MG_MODE(DS_MRQ)
#undef MG_MODE
  }
  return hipErrorInvalidValue;
}

template <typename R, int NL, typename S, int K, typename TI, typename TO>
static hipError_t launch_rb(const Geom &g, const S *U, const TI *in, TO *out, const TO *b, double diag, int nrhs,
                            DslashMode mode, double *partials, hipStream_t st, MrqArgs<TO> mq) {
  const dim3 grid(dslash_blocks(g), (nrhs + K - 1) / K);
  return with_mode<R, TI, TO>(mode, [&](auto m) {
    hipLaunchKernelGGL((k_dslash_rb<R, decltype(m)::value, NL, S, K, TI, TO>), grid, dim3(256), 0, st, g, U, in, out,
                       b, (R)diag, partials, nrhs, mq);
  });
}

template <typename R, int NL, typename S, typename TI, typename TO>
static hipError_t launch(const Geom &g, const S *U, const TI *in, TO *out, const TO *b, double diag, int nrhs,
                         DslashMode mode, double *partials, hipStream_t st, MrqArgs<TO> mq) {
  if (take_split(g, nrhs))
    return with_mode<R, TI, TO>(mode, [&](auto m) {
      hipLaunchKernelGGL((k_dslash_split<R, decltype(m)::value, NL, S, TI, TO>), dim3(div_up(g.V, 64), nrhs),
                         dim3(512), 0, st, g, U, in, out, b, (R)diag, partials, mq);
    });
  if (nrhs > 1) {
    if constexpr (!(sizeof(R) == 8 && std::is_same<TI, double2>::value))
      if (take_three<R, TI>(nrhs))
        return launch_rb<R, NL, S, 3>(g, U, in, out, b, diag, nrhs, mode, partials, st, mq);
    return launch_rb<R, NL, S, 2>(g, U, in, out, b, diag, nrhs, mode, partials, st, mq);
  }
  return with_mode<R, TI, TO>(mode, [&](auto m) {
    hipLaunchKernelGGL((k_dslash<R, decltype(m)::value, NL, S, TI, TO>), dim3(dslash_blocks(g), nrhs), dim3(256), 0,
                       st, g, U, in, out, b, (R)diag, partials, mq);
  });
}

template <typename R, typename S, typename TI, typename TO>
hipError_t dslash(const Geom &g, const S *U, int nl, const TI *in, TO *out, const typename same_t<TO>::type *b,
                  double diag, int nrhs, DslashMode mode, double *partials, hipStream_t st,
                  MrqArgs<typename same_t<TO>::type> mq) {
  if (nl == 6) return launch<R, 6, S>(g, U, in, out, b, diag, nrhs, mode, partials, st, mq);
  return launch<R, 9, S>(g, U, in, out, b, diag, nrhs, mode, partials, st, mq);
}

// Plain stencil in FP64 arithmetic on FP32-stored input spinors (the
// flexible GCR applies D to the preconditioner's FP32 output this way).
hipError_t dslash_in32(const Geom &g, const double2 *U, int nl, const float2 *in, double2 *out, double diag,
                       int nrhs, hipStream_t st) {
  return dslash<double, double2, float2, double2>(g, U, nl, in, out, nullptr, diag, nrhs, DS_PLAIN, nullptr, st);
}

// ---------------------------------------------------------------- links
// Copy of the first two rows of every link (NL = 6 layout), and the largest
// deviation |row2 - conj(row0 x row1)| over all links (per-block maxima).
template <typename S>
__global__ __launch_bounds__(256) void k_compress_links(Geom g, const double2 *__restrict__ U,
                                                        S *__restrict__ Uc, double *__restrict__ blockmax) {
  __shared__ double lds[4];
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  double dev = 0.0;
  if (s < g.V) {
    for (int mu = 0; mu < 4; ++mu) {
      double2 u[9], w[9];
#pragma unroll
      for (int e = 0; e < 9; ++e) u[e] = U[fidx(s, mu * 9 + e, 36)];
#pragma unroll
      for (int e = 0; e < 9; ++e) w[e] = u[e];
      reconstruct_row2(w);
      for (int e = 6; e < 9; ++e) dev = fmax(dev, fabs(w[e].x - u[e].x) + fabs(w[e].y - u[e].y));
#pragma unroll
      for (int e = 0; e < 6; ++e) Uc[fidx(s, mu * 6 + e, 24)] = cvt<S>(u[e]);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) dev = fmax(dev, __shfl_xor(dev, off, 64));
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = dev;
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = lds[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = fmax(m, lds[w]);
    blockmax[blockIdx.x] = m;
  }
}

template <typename S>
hipError_t compress_links(const Geom &g, const double2 *U, S *Uc, double *blockmax, hipStream_t st) {
  hipLaunchKernelGGL(k_compress_links<S>, dim3(div_up(g.V, 256)), dim3(256), 0, st, g, U, Uc, blockmax);
  return hipGetLastError();
}

#define DSLASH_INST(R, S, TI, TO)                                                                      \
  template hipError_t dslash<R, S, TI, TO>(const Geom &, const S *, int, const TI *, TO *,                        \
                                           const typename same_t<TO>::type *, double, int, DslashMode, double *,   \
                                           hipStream_t, MrqArgs<typename same_t<TO>::type>);
DSLASH_INST(double, double2, double2, double2)
DSLASH_INST(float, float2, float2, float2)
DSLASH_INST(float, chalf, float2, float2)
DSLASH_INST(float, chalf, h16, h16)
DSLASH_INST(float, chalf, float2, h16)
#undef DSLASH_INST
template hipError_t compress_links<double2>(const Geom &, const double2 *, double2 *, double *, hipStream_t);
template hipError_t compress_links<float2>(const Geom &, const double2 *, float2 *, double *, hipStream_t);
template hipError_t compress_links<chalf>(const Geom &, const double2 *, chalf *, double *, hipStream_t);

}  // namespace mg
