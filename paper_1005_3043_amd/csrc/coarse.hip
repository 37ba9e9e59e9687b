// Coarse operator D_c = P^dag D P applied as a 9-point stencil of n x n
// complex blocks (n = 2 Nv):
//   out(x) = X(x) v(x) + sum_mu [ Y_{+mu}(x) v(x+mu) + Y_{-mu}(x) v(x-mu) ]
// and its adjoint D_c^dag = sigma_3 D_c sigma_3 (gamma_5-Hermiticity carried to
// the coarse grid by the chirality split, P^dag gamma_5 = sigma_3 P^dag).
//
// Storage: coarse vectors are site-major (AoS), v[site][n]; the operator is
// L[site][slot][j][i] with slot 0 = X, slot 1 + (2 mu + dir) = Y, each block
// stored column-major so that the n rows of one column are contiguous.
//
// RS workgroups per coarse site, each owning n / RS consecutive rows: the nine input vectors are staged in LDS; thread (i, g) owns RW
// consecutive rows (RW = 2 in FP32 so every load is 16 bytes) and a strided
// subset g, g+G, ... of the 9n (slot, column) pairs, so each group streams one
// contiguous column segment and the workgroup reads a contiguous window of the
// site's entries per step (coalesced, bandwidth-bound).  The first chunk of
// operator loads is issued before the input vectors are staged so the two
// memory phases overlap.  The G partial row sums are combined in LDS in a
// fixed order (deterministic).
//
// The matrix-core variant (k_coarse_mma) handles all right-hand sides of a
// site in one workgroup: out[:, 0:nrhs] = A [B_0 .. B_8], a complex GEMM with
// M = n rows, N = nrhs (padded to 16) and K = 9n, where A is the site's
// operator (loaded once for every right-hand side) and B the nine staged
// input blocks.  Each complex product is three real 16x16x4 FP32 MFMAs.
#include <type_traits>

#include "solver.h"

namespace mg {

constexpr int CO_CHUNK = 8;   // operator loads in flight per thread
constexpr int CO_PARTS = 8;   // first-stage partial sums per row of the group reduction

// 16-byte (or 8-byte) load of RW consecutive operator entries in storage S.
template <typename S, int RW> struct OpVec;
template <> struct OpVec<double2, 1> {
  using V = double2;
  template <typename C> __device__ static void get(const V &v, C (&o)[1]) { o[0] = cvt<C>(v); }
};
template <> struct OpVec<float2, 2> {
  using V = float4;
  template <typename C> __device__ static void get(const V &v, C (&o)[2]) {
    o[0] = mk<C>(v.x, v.y);
    o[1] = mk<C>(v.z, v.w);
  }
};
template <> struct OpVec<chalf, 2> {
  using V = chalf2;
  template <typename C> __device__ static void get(const V &v, C (&o)[2]) {
    o[0] = cvt<C>(v.v[0]);
    o[1] = cvt<C>(v.v[1]);
  }
};
template <> struct OpVec<chalf, 4> {
  using V = chalf4;
  template <typename C> __device__ static void get(const V &v, C (&o)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = cvt<C>(v.v[q]);
  }
};

// Site read by stencil slot `slot` of coarse site s: slot 0 = s, slot
// 1 + 2 mu + dir = the neighbour in direction mu (dir 0 forward, 1 backward).
// The switch keeps every coordinate index a constant (no private arrays).
__device__ __forceinline__ uint32_t slot_site(const Geom &g, uint32_t s, int slot) {
  const Coords k = decode(g, s);
  switch (slot) {
    case 1: return nbr_fwd(g, s, k, 0);
    case 2: return nbr_bwd(g, s, k, 0);
    case 3: return nbr_fwd(g, s, k, 1);
    case 4: return nbr_bwd(g, s, k, 1);
    case 5: return nbr_fwd(g, s, k, 2);
    case 6: return nbr_bwd(g, s, k, 2);
    case 7: return nbr_fwd(g, s, k, 3);
    case 8: return nbr_bwd(g, s, k, 3);
    default: return s;
  }
}

// |v|^2 with the roundings written out: left to the compiler they differ from
// kernel to kernel, and the CGNR's two forms in FP64 with them (in the FP32
// classes the products are exact).
template <typename C> __device__ __forceinline__ double norm2_of(C v) {
  const double x = v.x, y = v.y;
  return fma(x, x, y * y);
}

// Sums of up to three partial arrays over the workgroup in one pass: out[0]
// = sum a[0..na), out[1] = sum b[0..nb), out[2] = sum c[0..nb) (NULL arrays
// give 0).  Fixed order; result in every thread.
__device__ __forceinline__ void block_allsum3(const double *__restrict__ a, int na, const double *__restrict__ b,
                                              const double *__restrict__ c, int nb, double (&out)[3],
                                              double *lds) {
  double v[3] = {0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < na; i += blockDim.x) v[0] += a[i];
  for (int i = threadIdx.x; i < nb; i += blockDim.x) {
    v[1] += b[i];
    v[2] += c[i];
  }
  const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int q = 0; q < 3; ++q) v[q] = wave_sum(v[q]);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int q = 0; q < 3; ++q) lds[w * 3 + q] = v[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    double t = 0.0;
    for (int k = 0; k < nw; ++k) t += lds[k * 3 + q];
    out[q] = t;
  }
  __syncthreads();
}

// Sum of np partials over the workgroup; result in every thread.
__device__ __forceinline__ double block_allsum_partials(const double *__restrict__ p, int np, double *lds) {
  double a = 0.0;
  for (int i = threadIdx.x; i < np; i += blockDim.x) a += p[i];
  a = wave_sum(a);
  const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds[w] = a;
  __syncthreads();
  double t = 0.0;
  for (int q = 0; q < nw; ++q) t += lds[q];
  __syncthreads();
  return t;
}


// Workgroup i of a per-RHS launch -> (logical workgroup ws of its right-hand
// side, rhs).  Workgroups go round-robin to the 8 XCDs; when the per-RHS
// count is a multiple of 8, XCD x takes the contiguous workgroup range
// [x nbx / 8, (x + 1) nbx / 8) (neighbouring sites share L2) and runs the
// right-hand sides of one workgroup back to back, so that a site's operator
// blocks come from HBM once and from that XCD's L2 for the other RHS.
__device__ __forceinline__ void block_rhs_of(uint32_t i, uint32_t nbx, uint32_t nrhs, uint32_t &ws, int &rhs) {
  if ((nbx & 7u) == 0u) {
    const uint32_t t = i >> 3;
    ws = (i & 7u) * (nbx >> 3) + t / nrhs;
    rhs = (int)(t % nrhs);
  } else {
    ws = i / nrhs;
    rhs = (int)(i % nrhs);
  }
}

template <typename R, typename S, int RW>
__global__ __launch_bounds__(512) void k_coarse(Geom g, int n, const S *__restrict__ L,
                                                 const c_t<R> *__restrict__ in, c_t<R> *__restrict__ out,
                                                 int nrhs, int dagger, double *__restrict__ partials, int pw,
                                                 const int *__restrict__ done, CgCheck chk, CgFuse fz) {
  using C = c_t<R>;
  using VT = typename OpVec<S, RW>::V;
  __shared__ C vin[9 * COARSE_NMAX];
  __shared__ C red[512 * RW];
  __shared__ C red2[CO_PARTS * COARSE_NMAX];
  __shared__ double wred[8 * 4];
  const uint32_t nbx = gridDim.x / (uint32_t)nrhs;  // workgroups per right-hand side
  uint32_t ws;
  int rhs;
  block_rhs_of(blockIdx.x, nbx, (uint32_t)nrhs, ws, rhs);
  if (done != nullptr && done[rhs]) return;
  const int RS = (int)(nbx / g.V);
  const uint32_t s = ws / RS;
  const int nr = n / RS, r0 = (int)(ws - s * RS) * nr;
  const size_t rhs_off = (size_t)rhs * g.V * n;
  in += rhs_off;
  out += rhs_off;
  const int tid = threadIdx.x;
  const int npr = nr / RW;  // row units of this workgroup
  const int G = (int)blockDim.x / npr;
  const int ip = tid % npr, grp = tid / npr;
  const int nP = 9 * n;
  const int nu = n / RW;    // row units per column
  const VT *Ls = reinterpret_cast<const VT *>(L + (size_t)s * 9 * n * n + r0) + ip;
  // Issue the first chunk of operator loads before staging the input vectors
  // so that the two memory phases overlap.  Every load is issued
  // unconditionally (a lane without an entry of its own reads entry 0 and
  // never uses it): a load under a lane mask gets a basic block of its own,
  // where the compiler waits for it before the next one is issued.
  VT lv[CO_CHUNK];
  const bool on = grp < G;
#pragma unroll
  for (int q = 0; q < CO_CHUNK; ++q) {
    const int p = grp + q * G;
    lv[q] = Ls[(size_t)((on && p < nP) ? p : 0) * nu];
  }
  __shared__ uint32_t nbs[9];
  if (tid < 9) nbs[tid] = slot_site(g, s, tid);
  // Scalars of this launch, summed from per-workgroup partials in one pass
  // (one round trip): the CGNR convergence test on the residual of the
  // update just made, and the fused update's coefficient.
  const bool check = chk.part_r != nullptr;
  const bool first = fz.kind == 1 && fz.it0[rhs] == 0;
  const bool coef_on = fz.kind != 0 && !first;
  R coef = 0;
  if (check || coef_on) {
    const double *pa = check ? chk.part_r + (size_t)rhs * chk.np_r : nullptr;
    const double *pn = coef_on ? fz.num + (size_t)rhs * fz.np : nullptr;
    const double *pd = coef_on ? fz.den + (size_t)rhs * fz.np : nullptr;
    double sums[3];
    block_allsum3(pa, check ? chk.np_r : 0, pn, pd, coef_on ? fz.np : 0, sums, wred);
    if (check) {
      const double rr = sums[0];
      const double *cg = chk.cg + (size_t)rhs * CG_NS;
      const int iter = chk.it_in[rhs];
      bool conv;
      if (chk.fused) conv = (iter > 0 && !(rr > cg[4] * cg[3])) || iter >= chk.maxit;
      else conv = !(rr > cg[4] * cg[3]) || iter + 1 >= chk.maxit;
      if (ws == 0 && threadIdx.x == 0) {
        chk.it_out[rhs] = (chk.fused && conv) ? iter : iter + 1;
        if (conv) chk.done[rhs] = 1;
      }
      if (conv) return;
    }
    if (coef_on) {
      if (!(sums[2] > 0.0)) {
        if (fz.kind == 2) {
          if (ws == 0 && tid == 0) fz.done_w[rhs] = 1;
          return;
        }
      } else {
        coef = (R)(sums[1] / sums[2]);
      }
    }
  }
  __syncthreads();
  double own_sq = 0.0;
  if (fz.kind == 0) {
    for (int idx = tid; idx < nP; idx += blockDim.x) {
      const int slot = idx / n, j = idx - slot * n;
      C v = in[(size_t)nbs[slot] * n + j];
      if (dagger && j >= (n >> 1)) v = mk<C>(-v.x, -v.y);
      vin[idx] = v;
    }
  } else {
    const C *fa = reinterpret_cast<const C *>(fz.a) + rhs_off;
    const C *fb = reinterpret_cast<const C *>(fz.b) + rhs_off;
    const R sc = fz.kind == 1 ? coef : -coef;
    for (int idx = tid; idx < nP; idx += blockDim.x) {
      const int slot = idx / n, j = idx - slot * n;
      const size_t o = (size_t)nbs[slot] * n + j;
      C v = cfma(mk<C>(sc, 0), fb[o], fa[o]);
      if (slot == 0) {
        reinterpret_cast<C *>(fz.own)[rhs_off + o] = v;
        if (fz.kind == 2) {
          C *e = reinterpret_cast<C *>(fz.e) + rhs_off;
          const C *pp = reinterpret_cast<const C *>(fz.p) + rhs_off;
          e[o] = cfma(mk<C>(coef, 0), pp[o], e[o]);
          own_sq += norm2_of(v);
        }
      }
      if (dagger && j >= (n >> 1)) v = mk<C>(-v.x, -v.y);
      vin[idx] = v;
    }
  }
  __syncthreads();
  C acc[RW];
#pragma unroll
  for (int q = 0; q < RW; ++q) acc[q] = mk<C>(0, 0);
  for (int base = grp; on && base < nP; base += CO_CHUNK * G) {
    if (base != grp) {
#pragma unroll
      for (int q = 0; q < CO_CHUNK; ++q) {
        const int p = base + q * G;
        lv[q] = Ls[(size_t)(p < nP ? p : 0) * nu];
      }
    }
#pragma unroll
    for (int q = 0; q < CO_CHUNK; ++q) {
      const int p = base + q * G;
      if (p < nP) {
        const C x = vin[p];
        C o[RW];
        OpVec<S, RW>::get(lv[q], o);
#pragma unroll
        for (int t = 0; t < RW; ++t) acc[t] = cfma(o[t], x, acc[t]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < RW; ++q) red[tid * RW + q] = acc[q];
  __syncthreads();
  // Sum of the G group partials of every row in two fixed-order stages:
  // CO_PARTS threads per row add every CO_PARTS-th group, then one thread
  // per row adds the CO_PARTS results (short dependent chains in LDS).
  if (tid < nr * CO_PARTS) {
    const int i = tid % nr, part = tid / nr;
    const int ipr = i / RW, sub = i % RW;
    C sum = mk<C>(0, 0);
    for (int q = part; q < G; q += CO_PARTS) sum = cadd(sum, red[(q * npr + ipr) * RW + sub]);
    red2[part * COARSE_NMAX + i] = sum;
  }
  __syncthreads();
  // partials (pw = 1): ||out||^2;  (pw = 3): <out, in>, ||out||^2 (in = centre)
  double t[3] = {0.0, 0.0, 0.0};
  if (tid < nr) {
    const int row = r0 + tid;
    C sum = red2[tid];
#pragma unroll
    for (int q = 1; q < CO_PARTS; ++q) sum = cadd(sum, red2[q * COARSE_NMAX + tid]);
    if (dagger && row >= (n >> 1)) sum = mk<C>(-sum.x, -sum.y);
    out[(size_t)s * n + row] = sum;
    const C c = vin[row];
    t[0] = (double)sum.x * c.x + (double)sum.y * c.y;
    t[1] = (double)sum.x * c.y - (double)sum.y * c.x;
    t[2] = norm2_of(sum);
  }
  if (partials != nullptr || fz.kind == 2) {
    double v4[4] = {t[0], t[1], t[2], own_sq};
    block_sum<4>(v4, wred);
    if (tid == 0) {
      if (partials != nullptr) {
        double *p = partials + ((size_t)rhs * nbx + ws) * pw;
        if (pw == 1) {
          p[0] = v4[2];
        } else {
          p[0] = v4[0];
          p[1] = v4[1];
          p[2] = v4[2];
        }
      }
      if (fz.kind == 2) fz.part_own[(size_t)rhs * nbx + ws] = v4[3];
    }
  }
}

// ------------------------------------------------------------ persistent CGNR
// The whole coarsest-level CGNR of one right-hand side in one cooperative
// launch: the fused two-phase iteration of k_coarse (phase 1: p = z + beta
// p_old staged, w = A p; phase 2: r = r_old - alpha w staged, e += alpha p,
// z = A^dag r) with a grid-wide exchange after each phase instead of a kernel
// boundary, its start (r = b, z = A^dag b, ||b||^2) included.  Each workgroup
// (one coarse site) loads its operator rows once into registers and keeps
// them for every iteration; a kernel boundary would drop the L2 and fetch the
// operator again.  It also keeps p and r of its site and the eight neighbours
// and repeats their updates, so that only w and z travel, and e of its site.
// Every workgroup computes the same scalars from the same partials in the same
// order, so all of them take the same exit.  A wait is bounded: a workgroup
// that gives up sets *fail and leaves, so the grid always drains.
//
// Bound by the latency of an exchange (store, acknowledge, announce, poll,
// load).  16^3 x 32, n = 40, FP16 storage, 512 sites, 45 iterations: 835 us a
// launch with p and r exchanged as well and the sums acknowledged after the
// vectors, 570 us with that gone, and about 460 us (5 us per phase) with the
// rows' sums on the first wavefront and the reads of apply in flight together.
// 8^4, n = 16, FP64, 16 sites: a solve of 47 ms as chunks of launches takes
// 24.4 ms.
constexpr int CGP_PMAX = 16;          // most operator entries per thread kept in registers

// Data exchanged between workgroups inside the launch is read and written as
// agent-scope relaxed atomics: the loads skip the XCD's non-coherent L2 and
// the stores write through it, so an exchange needs only each thread's stores
// acknowledged before its announcement, and no L2 write-back or invalidation
// (which cost about 80 us per barrier here).
__device__ __forceinline__ unsigned long long xld(const void *p) {
  return __hip_atomic_load(reinterpret_cast<unsigned long long *>(const_cast<void *>(p)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void xst(void *p, unsigned long long v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 cld(const float2 *p) { return __builtin_bit_cast(float2, xld(p)); }
__device__ __forceinline__ void cst(float2 *p, float2 v) { xst(p, __builtin_bit_cast(unsigned long long, v)); }
__device__ __forceinline__ double2 cld(const double2 *p) {
  return make_double2(__builtin_bit_cast(double, xld(&p->x)), __builtin_bit_cast(double, xld(&p->y)));
}
__device__ __forceinline__ void cst(double2 *p, double2 v) {
  xst(&p->x, __builtin_bit_cast(unsigned long long, v.x));
  xst(&p->y, __builtin_bit_cast(unsigned long long, v.y));
}

// The exchange at the end of a phase: everybody's two partial sums, and with
// them the knowledge that everybody's vector entries are there.
//
// Few workgroups (CGP_DIRECT at most): every 64-bit word that travels, of the
// sums and of the vector entries, carries 32 value bits under a 32-bit tag (the
// launch's epoch plus the phase number), and whoever needs it polls it until it
// carries the phase's tag: one way from the store to the reader, with no
// acknowledgement, no arrival and no load after it.  A sum or an entry of z or
// w is written again two phases later, which its writer only reaches after
// everybody has announced the phase between, that is, has read it (the sums
// alternate between two sets, z and w between phases).  8^4, 16 workgroups:
// 3.4 us per phase with the entries acknowledged, announced and then loaded,
// 3.0 us now, of which 2.1 are the exchange (one agent-scope load takes 0.7).
// With every thread polling, also those without an entry, 4.6 us; with 512
// workgroups every poll of everybody's sums moves 8 MB and a solve takes 1.3
// times as long as with the counters below.
//
// More: the sums and entries are stored, then an arrival is counted, and the first
// wavefront polls the counters; the sums are loaded after that, beside the
// vector entries of the next phase.  Arrivals are spread over CGP_NC counters
// on separate 256-byte lines, so that no address takes every workgroup's
// atomic.
//
// Why relaxed atomics order that form: every value another workgroup reads was stored
// with an agent-scope atomic store (written through to the agent's coherence
// point) and is read with an agent-scope atomic load (which bypasses the XCD's
// L2 and reads at that point).  s_waitcnt(0) holds each thread until its stores
// are acknowledged, i.e. performed at agent scope; the workgroup barrier then
// puts all of them before the announcement.  A reader issues its loads only
// after its workgroup has seen every announcement (the loop exit and the
// workgroup barrier order them after the polls).  A release / acquire pair
// would give the same order with an L2 write-back and invalidate per phase;
// with no exchanged data ever held in L2 they are not needed.
constexpr int CGP_NC = 64;  // arrival counters: 8, 16, 32 and 64 measured alike

// The set of a phase: tagged words first, bare sums (which could look like a
// tag) behind them.
template <bool DIRECT> __device__ __forceinline__ size_t cgp_set(uint32_t nblk, uint32_t tag) {
  return DIRECT ? (size_t)(tag & 1u) * 4 * nblk : 8 * CGP_DIRECT + (size_t)(tag & 1u) * 2 * nblk;
}

template <bool DIRECT>
__device__ __forceinline__ void cgp_announce(double (&v)[2], unsigned long long *words, unsigned *bar, uint32_t nblk,
                                             uint32_t tag) {
  // the rows of a site (n <= 64), so its sums and entries, are the first
  // wavefront's; adding the other wavefronts' zeros would change nothing
  if (threadIdx.x >= 64) return;
  const double s0 = wave_sum(v[0]), s1 = wave_sum(v[1]);
  unsigned long long *set = words + cgp_set<DIRECT>(nblk, tag);
  const int q = (threadIdx.x >> 1) & 1;  // direct: thread 2 q + h announces half h of sum q
  const unsigned long long u = __builtin_bit_cast(unsigned long long, q ? s1 : s0);
  if constexpr (DIRECT) {
    const unsigned long long half = (threadIdx.x & 1) ? u >> 32 : u & 0xffffffffull;
    if (threadIdx.x < 4) xst(set + (size_t)threadIdx.x * nblk + blockIdx.x, (unsigned long long)tag << 32 | half);
  } else {
    if (threadIdx.x < 4 && (threadIdx.x & 1) == 0) xst(set + (size_t)q * nblk + blockIdx.x, u);
    __builtin_amdgcn_s_waitcnt(0);  // the vector entries and the sums, acknowledged together
    __builtin_amdgcn_wave_barrier();
    if (threadIdx.x == 0)
      __hip_atomic_fetch_add(bar + (blockIdx.x % CGP_NC) * 64, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// A vector entry as tagged words (a site's, word by word: the words of a
// wavefront's entries are contiguous), and the wait for up to two of them.
template <typename C> constexpr int CGP_CW = sizeof(C) / 4;
template <typename C>
__device__ __forceinline__ void cgp_put(unsigned long long *w, C v, uint32_t tag) {
  struct W {
    uint32_t u[CGP_CW<C>];
  };
  const W x = __builtin_bit_cast(W, v);
#pragma unroll
  for (int j = 0; j < CGP_CW<C>; ++j) xst(w + j, (unsigned long long)tag << 32 | x.u[j]);
}
template <typename C>
__device__ __forceinline__ bool cgp_take(const unsigned long long *w0, const unsigned long long *w1, bool two, C &x0,
                                         C &x1, uint32_t tag, unsigned spin_max) {
  constexpr int NW = CGP_CW<C>;
  struct W {
    uint32_t u[NW];
  } a, b;
  for (unsigned spins = 0;;) {
    unsigned long long u[2 * NW];
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      u[j] = xld(w0 + j);
      u[NW + j] = two ? xld(w1 + j) : u[j];
    }
    bool all = true;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      all = all && (uint32_t)(u[j] >> 32) == tag && (uint32_t)(u[NW + j] >> 32) == tag;
      a.u[j] = (uint32_t)u[j];
      b.u[j] = (uint32_t)u[NW + j];
    }
    if (all) break;
    if (++spins > spin_max) return false;
    __builtin_amdgcn_s_sleep(1);
  }
  x0 = __builtin_bit_cast(C, a);
  x1 = __builtin_bit_cast(C, b);
  return true;
}

// Waits for every workgroup's announcement of `tag` (the phase-th of the
// launch), calls pre() (which fetches the next phase's entries; false when its
// wait gave up) and sums the values in block_allsum3's order, so that each sum
// equals the chunked path's of the same array.  False, for the whole
// workgroup, when a wait gave up.  Tagged words: the last
// wavefront, which holds no entries of small sites, polls the sums.  *bad: zero until a wait gives up.
template <bool DIRECT, typename F>
__device__ __forceinline__ bool cgp_gather(const unsigned long long *words, unsigned *bar, uint32_t nblk,
                                           uint32_t tag, uint32_t phase, double (&out)[2], double *lds, int *bad,
                                           int *fail, unsigned spin_max, F &&pre) {
  const unsigned long long *set = words + cgp_set<DIRECT>(nblk, tag);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  unsigned spins = 0;
  if constexpr (DIRECT) {
    static_assert(CGP_DIRECT <= 128, "two announcements per lane");
    int ok = 1;
    if (w == nw - 1) {
      double v[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t i = lane + 64 * j;
        if (i >= nblk) continue;
        for (;;) {
          unsigned long long u[4];
          bool all = true;
#pragma unroll
          for (int q = 0; q < 4; ++q) u[q] = xld(set + (size_t)q * nblk + i);
#pragma unroll
          for (int q = 0; q < 4; ++q) all = all && (uint32_t)(u[q] >> 32) == tag;
          v[j][0] = __builtin_bit_cast(double, (u[0] & 0xffffffffull) | (u[1] << 32));
          v[j][1] = __builtin_bit_cast(double, (u[2] & 0xffffffffull) | (u[3] << 32));
          if (all) break;
          if (++spins > spin_max) {
            ok = 0;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
      }
      double t0 = wave_sum(v[0][0]), t1 = wave_sum(v[0][1]);
      if (nblk > 64) {
        t0 += wave_sum(v[1][0]);
        t1 += wave_sum(v[1][1]);
      }
      if (lane == 0) {
        lds[0] = t0;
        lds[1] = t1;
      }
    }
    if (!pre()) ok = 0;
    if (!ok) {
      *bad = 1;
      __hip_atomic_store(fail, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __syncthreads();
    out[0] = lds[0];
    out[1] = lds[1];
    return *bad == 0;
  } else {
    if (w == 0) {
      const unsigned target = phase * nblk;
      for (;;) {
        unsigned c = __hip_atomic_load(bar + lane * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        c = wave_sum(c);
        if ((int)(c - target) >= 0) break;  // (both modulo 2^32)
        if (++spins > spin_max) {
          if (lane == 0) {
            *bad = 1;
            __hip_atomic_store(fail, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          }
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __syncthreads();
    if (*bad != 0) return false;
    pre();
    double v[2] = {0.0, 0.0};
    for (uint32_t i = threadIdx.x; i < nblk; i += blockDim.x) {
      v[0] += __builtin_bit_cast(double, xld(set + i));
      v[1] += __builtin_bit_cast(double, xld(set + nblk + i));
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) v[q] = wave_sum(v[q]);
    if (lane == 0) {
      lds[w * 2] = v[0];
      lds[w * 2 + 1] = v[1];
    }
    __syncthreads();
    out[0] = out[1] = 0.0;
    for (int k = 0; k < nw; ++k) {
      out[0] += lds[k * 2];
      out[1] += lds[k * 2 + 1];
    }
    return true;
  }
}

// The operator entries a thread holds in registers for the whole solve, where
// they are half precision: converted at each use.  Left alone the compiler
// converts them once, outside the iteration, and spills the doubled registers.
template <typename S, int RW>
__device__ __forceinline__ typename OpVec<S, RW>::V kept_packed(const typename OpVec<S, RW>::V &v) {
  if constexpr (sizeof(S) == 4) {
    struct W {
      uint32_t w[RW];
    } u = __builtin_bit_cast(W, v);
#pragma unroll
    for (int t = 0; t < RW; ++t) asm volatile("" : "+v"(u.w[t]));
    return __builtin_bit_cast(typename OpVec<S, RW>::V, u);
  } else {
    return v;
  }
}

// DIRECT: at most CGP_DIRECT workgroups, one per CU, so two wavefronts' worth
// of registers per SIMD lane.
template <typename R, typename S, int RW, int PM, bool DIRECT>
__global__ __launch_bounds__(512, DIRECT || (sizeof(S) == 16 && PM == 16) ? 2 : 4) void k_cgnr_persistent(Geom g, int n, const S *__restrict__ L,
                                                            CgPersist<c_t<R>> a) {
  using C = c_t<R>;
  using VT = typename OpVec<S, RW>::V;
  __shared__ C vin[9 * COARSE_NMAX], ploc[9 * COARSE_NMAX], rloc[9 * COARSE_NMAX];
  __shared__ C red[512 * RW];
  __shared__ C red2[CO_PARTS * COARSE_NMAX];
  __shared__ double gsum[2][16];
  __shared__ int bad;
  __shared__ uint32_t nbs[9];
  const uint32_t s = blockIdx.x, nblk = gridDim.x;
  const int tid = threadIdx.x;
  const int npr = n / RW, G = (int)blockDim.x / npr;
  const int ip = tid % npr, grp = tid / npr;
  const int nP = 9 * n, half = n >> 1;
  const bool on = grp < G;
  const VT *Ls = reinterpret_cast<const VT *>(L + (size_t)s * 9 * n * n) + ip;
  VT lv[PM];
#pragma unroll
  for (int q = 0; q < PM; ++q) {
    const int p = grp + q * G;
    lv[q] = Ls[(size_t)((on && p < nP) ? p : 0) * n / RW];
    if (!(on && p < nP)) lv[q] = VT{};
  }
  if (tid < 9) nbs[tid] = slot_site(g, s, tid);
  if (tid == 0) bad = 0;
  __syncthreads();
  // where this thread's staged entries tid and tid + blockDim come from
  const int i0 = tid, i1 = tid + (int)blockDim.x;  // 9 n <= 2 blockDim
  const bool h0 = i0 < nP, h1 = i1 < nP;
  const uint32_t o0 = h0 ? nbs[i0 / n] * n + i0 % n : 0, o1 = h1 ? nbs[i1 / n] * n + i1 % n : 0;
  const bool neg0 = i0 % n >= half, neg1 = i1 % n >= half;
  const uint32_t own = s * n + tid;
  unsigned *bar = a.bar + (size_t)(a.launch & 1u) * CGP_NC * 64;
  if (s == 0 && tid < CGP_NC)  // the next launch's counters
    __hip_atomic_store(a.bar + (size_t)((a.launch + 1) & 1u) * CGP_NC * 64 + tid * 64, 0u, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  // rows of this workgroup times the staged vector, summed over the groups in
  // the fixed two-stage order of k_coarse; returns the row sum (tid < n)
  auto apply = [&]() -> C {
    __syncthreads();
    C acc[RW];
#pragma unroll
    for (int t = 0; t < RW; ++t) acc[t] = mk<C>(0, 0);
#pragma unroll
    for (int q = 0; q < PM; ++q) {
      const int p = grp + q * G;
      // spare entries of the operator are zero: no branch, so that the reads of
      // all entries are in flight together
      const C x = vin[p < nP ? p : nP - 1];
      C o[RW];
      OpVec<S, RW>::get(kept_packed<S, RW>(lv[q]), o);
#pragma unroll
      for (int t = 0; t < RW; ++t) acc[t] = cfma(o[t], x, acc[t]);
    }
#pragma unroll
    for (int t = 0; t < RW; ++t) red[tid * RW + t] = acc[t];
    __syncthreads();
    if (tid < n * CO_PARTS) {
      const int i = tid % n, part = tid / n;
      const int ipr = i / RW, sub = i % RW;
      C sum = mk<C>(0, 0);
      for (int q = part; q < G; q += CO_PARTS) sum = cadd(sum, red[(q * npr + ipr) * RW + sub]);
      red2[part * COARSE_NMAX + i] = sum;
    }
    __syncthreads();
    C sum = mk<C>(0, 0);
    if (tid < n) {
      sum = red2[tid];
#pragma unroll
      for (int q = 1; q < CO_PARTS; ++q) sum = cadd(sum, red2[q * COARSE_NMAX + tid]);
    }
    return sum;
  };
  // r = b, p = 0, e = 0
  double sq = 0.0;
  {
    const C b0 = h0 ? a.b[o0] : mk<C>(0, 0), b1 = h1 ? a.b[o1] : mk<C>(0, 0);
    if (h0) {
      rloc[i0] = b0;
      ploc[i0] = mk<C>(0, 0);
      vin[i0] = neg0 ? mk<C>(-b0.x, -b0.y) : b0;
    }
    if (h1) {
      rloc[i1] = b1;
      ploc[i1] = mk<C>(0, 0);
      vin[i1] = neg1 ? mk<C>(-b1.x, -b1.y) : b1;
    }
    if (tid < n) sq = norm2_of(b0);
  }
  C e = mk<C>(0, 0), x0 = e, x1 = e;
  // the entries of z (which 0) and w (1): tagged words, or the arrays themselves
  constexpr int CW = CGP_CW<C>;
  unsigned long long *ew = a.words + CGP_WORDS;
  const size_t ews = (size_t)CGP_DIRECT * COARSE_NMAX * 4;
  const uint32_t p0 = h0 ? o0 : s * n, p1 = h1 ? o1 : p0;
  auto put = [&](C *arr, int which, C v, uint32_t ph) {
    if constexpr (DIRECT) cgp_put(ew + which * ews + (size_t)own * CW, v, a.epoch + ph);
    else cst(arr + own, v);
  };
  auto take = [&](const C *arr, int which, uint32_t ph) -> bool {
    if constexpr (DIRECT) {
      return !h0 || cgp_take(ew + which * ews + (size_t)p0 * CW, ew + which * ews + (size_t)p1 * CW, h1, x0, x1,
                             a.epoch + ph, a.spin);
    } else {
      x0 = cld(arr + p0);
      x1 = h1 ? cld(arr + p1) : x0;
      return true;
    }
  };
  double sums[2], gam = 0.0, tol2b2 = 0.0;  // gam: ||z_k||^2
  int k = 0, final_it = 0;
  unsigned phase = 0;
  for (;;) {
    // ---- z = A^dag r; ||z||^2 and ||r||^2 (of the update just made; at first ||b||^2)
    {
      C zv = apply();
      double v[2] = {0.0, sq};
      if (tid < n) {
        if (tid >= half) zv = mk<C>(-zv.x, -zv.y);
        put(a.z, 0, zv, phase + 1);
        v[0] = norm2_of(zv);
      }
      ++phase;
      cgp_announce<DIRECT>(v, a.words, bar, nblk, a.epoch + phase);
    }
    if (!cgp_gather<DIRECT>(a.words, bar, nblk, a.epoch + phase, phase, sums, gsum[0], &bad, a.fail, a.spin, [&]() {
          return take(a.z, 0, phase);
        }))
      break;
    R beta = 0;
    if (phase == 1) {
      tol2b2 = a.tol2 * sums[1];
      if (!(sums[1] > 0.0)) break;  // zero right-hand side: no iteration, e = 0
    } else {
      if (!(sums[1] > tol2b2)) {
        final_it = k;
        break;
      }
      beta = gam > 0.0 ? (R)(sums[0] / gam) : (R)0;
    }
    gam = sums[0];
    if (k >= a.maxit) {
      final_it = k;
      break;
    }
    // ---- p = z + beta p_old, w = A p; ||w||^2
    if (h0) vin[i0] = ploc[i0] = cfma(mk<C>(beta, 0), ploc[i0], x0);
    if (h1) vin[i1] = ploc[i1] = cfma(mk<C>(beta, 0), ploc[i1], x1);
    {
      const C wv = apply();
      double v[2] = {0.0, 0.0};
      if (tid < n) {
        put(a.w, 1, wv, phase + 1);
        v[0] = norm2_of(wv);
      }
      ++phase;
      cgp_announce<DIRECT>(v, a.words, bar, nblk, a.epoch + phase);
    }
    if (!cgp_gather<DIRECT>(a.words, bar, nblk, a.epoch + phase, phase, sums, gsum[1], &bad, a.fail, a.spin, [&]() {
          return take(a.w, 1, phase);
        }))
      break;
    if (!(sums[0] > 0.0)) {
      final_it = k + 1;
      break;
    }
    // ---- r = r_old - alpha w, e += alpha p
    const R alpha = (R)(gam / sums[0]);
    if (h0) {
      const C v = cfma(mk<C>(-alpha, 0), x0, rloc[i0]);
      rloc[i0] = v;
      vin[i0] = neg0 ? mk<C>(-v.x, -v.y) : v;
      if (tid < n) {
        e = cfma(mk<C>(alpha, 0), ploc[tid], e);
        sq = norm2_of(v);
      }
    }
    if (h1) {
      const C v = cfma(mk<C>(-alpha, 0), x1, rloc[i1]);
      rloc[i1] = v;
      vin[i1] = neg1 ? mk<C>(-v.x, -v.y) : v;
    }
    ++k;
  }
  if (tid < n) a.e[own] = e;
  if (s == 0 && tid < 2) __hip_atomic_store(a.it + tid, final_it, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <typename R, typename S>
hipError_t cgnr_persistent(const Geom &g, int n, const S *L, const CgPersist<c_t<R>> &a, hipStream_t st) {
  const int rs = coarse_split(n, g.V);
  if (rs != 1 || n > COARSE_NMAX) return hipErrorInvalidValue;
  const int th = coarse_threads(n, g.V);
  // rows per thread as of k_coarse in this storage
  const int RW = sizeof(S) == 16 ? 1 : sizeof(S) == 4 && n % 4 == 0 ? 4 : 2;
  if (n % RW != 0) return hipErrorInvalidValue;
  const int G = th / (n / RW), pm = (9 * n + G - 1) / G;
  if (pm > CGP_PMAX || th > 512 || 9 * n > 2 * th || n * CO_PARTS > th) return hipErrorInvalidValue;
  CgPersist<c_t<R>> args = a;
  Geom gg = g;
  const S *LL = L;
  int nn = n;
  void *kargs[] = {&gg, &nn, &LL, &args};
  // entries per thread decide the register array: 8 where they fit
  const bool p8 = pm <= 8;
  auto pick = [&](auto direct) -> const void * {
    constexpr bool D = decltype(direct)::value;
    if constexpr (sizeof(S) == 4) {
      if (RW == 4 && !p8) return nullptr;  // 16 four-row entries would spill
      if (RW == 4) return reinterpret_cast<const void *>(&k_cgnr_persistent<R, S, 4, 8, D>);
    }
    constexpr int W = sizeof(S) == 16 ? 1 : 2;
    return p8 ? reinterpret_cast<const void *>(&k_cgnr_persistent<R, S, W, 8, D>)
              : reinterpret_cast<const void *>(&k_cgnr_persistent<R, S, W, 16, D>);
  };
  const void *fn = g.V <= CGP_DIRECT ? pick(std::true_type()) : pick(std::false_type());
  if (fn == nullptr) return hipErrorInvalidValue;
  return hipLaunchCooperativeKernel(fn, dim3(g.V), dim3(th), kargs, 0, st);
}
template hipError_t cgnr_persistent<float, chalf>(const Geom &, int, const chalf *, const CgPersist<float2> &,
                                                  hipStream_t);
template hipError_t cgnr_persistent<float, float2>(const Geom &, int, const float2 *, const CgPersist<float2> &,
                                                   hipStream_t);
template hipError_t cgnr_persistent<double, double2>(const Geom &, int, const double2 *, const CgPersist<double2> &,
                                                     hipStream_t);

// ------------------------------------------------------------ matrix cores
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Four consecutive operator entries (16-byte aligned) in their storage type.
template <typename S> struct Op4;
template <> struct Op4<chalf> {
  chalf4 v;
  __device__ __forceinline__ void load(const chalf *p) { v = *reinterpret_cast<const chalf4 *>(p); }
  __device__ __forceinline__ void set(int q, chalf e) { v.v[q] = e; }
  __device__ __forceinline__ float2 get(int q) const { return cvt<float2>(v.v[q]); }
};
template <> struct Op4<float2> {
  float2 v[4];
  __device__ __forceinline__ void load(const float2 *p) {
    const float4 a = reinterpret_cast<const float4 *>(p)[0], b = reinterpret_cast<const float4 *>(p)[1];
    v[0] = make_float2(a.x, a.y);
    v[1] = make_float2(a.z, a.w);
    v[2] = make_float2(b.x, b.y);
    v[3] = make_float2(b.z, b.w);
  }
  __device__ __forceinline__ void set(int q, float2 e) { v[q] = e; }
  __device__ __forceinline__ float2 get(int q) const { return v[q]; }
};

constexpr int MMA_NR = 16;  // right-hand sides per GEMM tile (N of the MFMA)

// The convergence prologue for all right-hand sides of a workgroup (rsum:
// LDS); true when every one has converged.  ||r||^2 of right-hand side r by
// wavefront r mod nw, then lane r of every wavefront tests right-hand side r
// (one after another, their loads alone took a round trip each).
__device__ __forceinline__ bool cg_check_all(const CgCheck &chk, int nrhs, double *rsum) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int r = wv; r < nrhs; r += nw) {
    double t = 0.0;
    for (int i = lane; i < chk.np_r; i += 64) t += chk.part_r[(size_t)r * chk.np_r + i];
    t = wave_sum(t);
    if (lane == 0) rsum[r] = t;
  }
  const int r = min(lane, nrhs - 1);
  const double *cg = chk.cg + (size_t)r * CG_NS;
  const double lim = cg[4] * cg[3];
  const int was = chk.done[r], iter = chk.it_in[r];
  __syncthreads();
  const bool conv = was != 0 || !(rsum[r] > lim) || iter + 1 >= chk.maxit;
  if (blockIdx.x == 0 && wv == 0 && lane < nrhs && was == 0) {
    chk.it_out[r] = iter + 1;
    if (conv) chk.done[r] = 1;
  }
  return __all(conv);
}

// One workgroup per coarse site.  Every wavefront accumulates all MT =
// ceil(n / 16) row tiles of all right-hand sides over its share of the K
// range: blocks of 16 of the 9n (slot, column) pairs, block b to wavefront b
// mod nw.  MFMA lane layouts (16x16x4, FP32): A lane l = (row l % 16, k l /
// 16); B lane l = (k l / 16, column l % 16); C lane l = (rows 4 (l / 16) +
// 0..3, column l % 16).
//
// What it is bound by: the matrix cores and the operator's bytes come to
// about the same time (24^3 x 48, n = 48, 12 right-hand sides, binary16: 34
// us of MFMA, 215 MB), so nothing else may sit in the loop.  With one row
// tile per wavefront and range checks on every operand it issued twelve
// vector instructions per MFMA, 49 us of vector work, 127 us in all.  Here an
// input entry is read (and its Gauss sum formed) once for all row tiles, and
// no operand is checked: rows past n repeat row n - 1 and columns past nrhs
// column 0, whose results are not stored, and the inputs past K are zero.
// 127 -> 76 us there; FP32 storage 127 -> 101 us, and on level 1 of 32^3 x 64
// 0.367 -> 0.310 ms (1.4 GB of operator and vectors, 4.5 TB/s).
template <typename S, int MT, bool RM>
__global__ __launch_bounds__(512) void k_coarse_mma(Geom g, int n, const S *__restrict__ L,
                                                    const float2 *__restrict__ in, float2 *__restrict__ out,
                                                    int nrhs, int dagger, double *__restrict__ part, int pw,
                                                    const int *__restrict__ done, CgCheck chk) {
  extern __shared__ __align__(16) float2 bl[];  // staged inputs [16 KB][nrhs | 1], then the wavefronts' sums
  __shared__ double rsum[MMA_NR];
  __shared__ double pr[MT][64][3];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = blockDim.x >> 6;
  if (done != nullptr) {
    const int d = lane < nrhs ? done[lane] : 1;
    if (__all(d != 0)) return;
  }
  if (chk.part_r != nullptr && cg_check_all(chk, nrhs, rsum)) return;
  const uint32_t s = xcd_remap(blockIdx.x, gridDim.x);
  const int K = 9 * n, half = n >> 1, KB = (K + 15) >> 4, ldb = nrhs | 1;
  const int kq = lane >> 4, col = lane & 15;
  const int colc = col < nrhs ? col : 0;
  // Column-major operator (RM false): lane (row, kq) takes column 16 b + 4 u +
  // kq of its row in k-step u, rows contiguous.  Row-major copy (RM true): the
  // four consecutive columns 16 b + 4 kq .. + 3 in one access, column 16 b + 4
  // kq + u in k-step u (the sum over K does not depend on the order).
  const S *La[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int row = min(16 * m + (lane & 15), n - 1);
    La[m] = L + (size_t)s * K * n + (RM ? (size_t)row * K : (size_t)row);
  }
  Op4<S> abuf[2][MT];
  auto load_block = [&](Op4<S> (&dst)[MT], int b) {
    if constexpr (RM) {
      const int k0 = min(16 * b + 4 * kq, K - 4);
#pragma unroll
      for (int m = 0; m < MT; ++m) dst[m].load(La[m] + k0);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const size_t o = (size_t)min(16 * b + 4 * u + kq, K - 1) * n;
#pragma unroll
        for (int m = 0; m < MT; ++m) dst[m].set(u, La[m][o]);
      }
    }
  };
  // the first blocks are under way before the inputs are staged
  if (wv < KB) load_block(abuf[0], wv);
  if (wv + nw < KB) load_block(abuf[1], wv + nw);
  {
    // Input block (slot, right-hand side) t to wavefront t mod nw, lanes along
    // the components: the addresses are scalar but for the lane's part.  SU
    // entries are loaded before any is stored, so that their round trips
    // overlap.
    constexpr int SU = 9;
    const uint32_t nb = slot_site(g, s, lane < 9 ? lane : 0);
    const int nt = 9 * nrhs, inv = (65536 + nrhs - 1) / nrhs;  // t / nrhs = t inv >> 16 for t < 9 * 16
    const int j = lane < n ? lane : n - 1;
    const bool neg = dagger && j >= half;
    for (int t0 = __builtin_amdgcn_readfirstlane(wv); t0 < nt; t0 += SU * nw) {
      float2 v[SU];
#pragma unroll
      for (int u = 0; u < SU; ++u) {
        const int t = min(t0 + u * nw, nt - 1), slot = t * inv >> 16;
        const uint32_t sn = __builtin_amdgcn_readlane(nb, slot);
        v[u] = in[((size_t)(t - slot * nrhs) * g.V + sn) * n + j];
      }
#pragma unroll
      for (int u = 0; u < SU; ++u) {
        const int t = min(t0 + u * nw, nt - 1), slot = t * inv >> 16;
        bl[(slot * n + j) * ldb + (t - slot * nrhs)] = neg ? make_float2(-v[u].x, -v[u].y) : v[u];
      }
    }
    for (int i = K * ldb + tid; i < KB * 16 * ldb; i += blockDim.x) bl[i] = make_float2(0.f, 0.f);
  }
  __syncthreads();
  // Complex products with three real MFMAs each (Gauss): cre = sum a.x b.x,
  // c2 = sum a.y b.y, cim = sum (a.x + a.y)(b.x + b.y); then re = cre - c2
  // and im = cim - cre - c2.
  floatx4 cre[MT], cim[MT], c2[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) cre[m] = cim[m] = c2[m] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int b0 = wv; b0 < KB; b0 += 2 * nw) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int b = b0 + h * nw;
      if (b >= KB) break;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = 16 * b + (RM ? 4 * kq + u : 4 * u + kq);
        const float2 bv = bl[k * ldb + colc];
        const float bs = bv.x + bv.y;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const float2 av = abuf[h][m].get(u);
          cre[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, cre[m], 0, 0, 0);
          c2[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.y, c2[m], 0, 0, 0);
          cim[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x + av.y, bs, cim[m], 0, 0, 0);
        }
      }
      if (b + 2 * nw < KB) load_block(abuf[h], b + 2 * nw);
    }
  }
  // centre inputs of the rows this thread stores (for the <out, in> partial)
  const int mo = wv;  // wavefront m stores row tile m (MT <= nw or several each)
  __syncthreads();
  float2 ctr[MT][4];
#pragma unroll
  for (int m = 0; m < MT; ++m)
    if (m % nw == mo) {
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) ctr[m][r4] = bl[min(16 * m + 4 * kq + r4, n - 1) * ldb + colc];
    }
  __syncthreads();
  float4 *red = reinterpret_cast<float4 *>(bl);  // [nw][MT][2][64]
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const floatx4 im = cim[m] - cre[m] - c2[m], re = cre[m] - c2[m];
    red[((wv * MT + m) * 2 + 0) * 64 + lane] = make_float4(re[0], re[1], re[2], re[3]);
    red[((wv * MT + m) * 2 + 1) * 64 + lane] = make_float4(im[0], im[1], im[2], im[3]);
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if (m % nw != mo) continue;
    float4 re = red[(m * 2 + 0) * 64 + lane], im = red[(m * 2 + 1) * 64 + lane];
    for (int q = 1; q < nw; ++q) {
      const float4 x = red[((q * MT + m) * 2 + 0) * 64 + lane], y = red[((q * MT + m) * 2 + 1) * 64 + lane];
      re.x += x.x; re.y += x.y; re.z += x.z; re.w += x.w;
      im.x += y.x; im.y += y.y; im.z += y.z; im.w += y.w;
    }
    const float rr[4] = {re.x, re.y, re.z, re.w}, ii[4] = {im.x, im.y, im.z, im.w};
    double t0 = 0.0, t1 = 0.0, t2 = 0.0;
    if (col < nrhs) {
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int row = 16 * m + 4 * kq + r4;
        if (row < n) {
          float2 o = make_float2(rr[r4], ii[r4]);
          if (dagger && row >= half) o = make_float2(-o.x, -o.y);
          out[((size_t)col * g.V + s) * n + row] = o;
          const float2 c = ctr[m][r4];
          t0 += (double)o.x * c.x + (double)o.y * c.y;
          t1 += (double)o.x * c.y - (double)o.y * c.x;
          t2 += (double)o.x * o.x + (double)o.y * o.y;
        }
      }
    }
    pr[m][lane][0] = t0;
    pr[m][lane][1] = t1;
    pr[m][lane][2] = t2;
  }
  if (part == nullptr) return;
  __syncthreads();
  if (tid < nrhs) {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int m = 0; m < MT; ++m)
      for (int g4 = 0; g4 < 4; ++g4) {
        a0 += pr[m][g4 * 16 + tid][0];
        a1 += pr[m][g4 * 16 + tid][1];
        a2 += pr[m][g4 * 16 + tid][2];
      }
    double *p = part + ((size_t)tid * gridDim.x + blockIdx.x) * pw;
    if (pw == 1) {
      p[0] = a2;
    } else {
      p[0] = a0;
      p[1] = a1;
      p[2] = a2;
    }
  }
}

// FP64: the same product on the FP64 matrix cores (16x16x4; C lane l, register
// v = row 4 v + l / 16).  One workgroup of three wavefronts per coarse site and
// group of right-hand sides; wavefront w takes stencil slots w, w + 3, w + 6,
// stages a slot's vectors in its own LDS and reads its operator block once, so
// no barrier stands between the slots.  Bound by the operator's bytes: with
// one workgroup per right-hand side (k_coarse) 12 of them on 24^3 x 48 (n =
// 48, 860 MB) took 626 us; this takes 193, 4.7 TB/s of operator and vectors.
// Three wavefronts per SIMD: with two, whole workgroups of three leave a
// quarter of the slots empty (n = 48: 228 us against 189 before the short
// chains).  Four row tiles do not fit that and take two (n = 64: 352 us; 400
// with 200 bytes spilled).
typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int MF_WAVES = 3;

template <int MT>
__global__ __launch_bounds__(64 * MF_WAVES, MT == 4 ? 2 : 3) void k_coarse_mma_f64(Geom g, int n, const double2 *__restrict__ L,
                                                                  const double2 *__restrict__ in,
                                                                  double2 *__restrict__ out, int nrhs, int per,
                                                                  int dagger, double *__restrict__ part, int pw,
                                                                  const int *__restrict__ done, CgCheck chk) {
  extern __shared__ __align__(16) double2 bl64[];  // [MF_WAVES][4 KP][ldb], then the wavefronts' sums
  __shared__ double rsum[MMA_NR];
  __shared__ double pr[MT][64][3];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r0 = blockIdx.y * per, nr = min(per, nrhs - r0);
  if (done != nullptr) {
    const int d = lane < nr ? done[r0 + lane] : 1;
    if (__all(d != 0)) return;
  }
  if (chk.part_r != nullptr && cg_check_all(chk, nrhs, rsum)) return;
  const uint32_t s = xcd_remap(blockIdx.x, gridDim.x);
  constexpr int U = 4;  // k-steps per load batch
  const int half = n >> 1, KS = (n + 3) >> 2, ldb = nr | 1;
  const int q = lane >> 4, col = lane & 15, colc = col < nr ? col : 0;
  const int KP = (KS + U - 1) / U * U;  // staged k-steps, zero from n on
  double2 *bw = bl64 + (size_t)wv * 4 * KP * ldb;
  uint32_t row[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) row[m] = min(16 * m + col, n - 1);
  const uint32_t nb = slot_site(g, s, lane < 9 ? lane : 0);
  const int j = min(lane, n - 1);
  const bool neg = dagger && j >= half;
  doublex4 re[MT], im[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) re[m] = im[m] = doublex4{0.0, 0.0, 0.0, 0.0};
  double2 a[U][MT];
  // A batch's products (two k-steps' where there are few rows) are one chain
  // from zero, added to the sum when done: one accumulator over a wavefront's
  // three slots rounded 1.7 times as much as k_coarse (n = 48, relative to
  // extended precision: 7.4e-16 against 4.3e-16; 2.4e-16 this way).  24^3 x 48,
  // n = 48, 12 right-hand sides 186 -> 193 us, n = 64 356 -> 352.
  const doublex4 zero = {0.0, 0.0, 0.0, 0.0};
  for (int slot = wv; slot < 9; slot += MF_WAVES) {
    const double2 *Ls = L + ((size_t)s * 9 + slot) * n * n;
    auto load = [&](int k0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t o = (uint32_t)(min(4 * (k0 + u) + q, n - 1) * n);
#pragma unroll
        for (int m = 0; m < MT; ++m) a[u][m] = Ls[o + row[m]];
      }
    };
    load(0);
    {
      const double2 *src = in + ((size_t)r0 * g.V + __builtin_amdgcn_readlane(nb, slot)) * n + j;
      const size_t vs = (size_t)g.V * n;
      __builtin_amdgcn_wave_barrier();
      for (int t0 = 0; t0 < nr; t0 += 4) {
        double2 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = src[(size_t)min(t0 + u, nr - 1) * vs];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          bw[j * ldb + min(t0 + u, nr - 1)] = neg ? make_double2(-v[u].x, -v[u].y) : v[u];
      }
      for (int i = n * ldb + lane; i < 4 * KP * ldb; i += 64) bw[i] = make_double2(0.0, 0.0);
      __builtin_amdgcn_wave_barrier();
    }
    // NK k-steps from k0 on, and the loads of the next batch
    auto batch = [&](auto nk, int k0) {
      constexpr int NK = decltype(nk)::value, CH = MT > 2 ? NK : 2;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
#pragma unroll
        for (int h = 0; h < NK / CH; ++h) {
          doublex4 tr = zero, ti = zero;
#pragma unroll
          for (int v = 0; v < CH; ++v) {
            const int u = CH * h + v;
            const double2 p = a[u][m], b = bw[(4 * (k0 + u) + q) * ldb + colc];
            tr = __builtin_amdgcn_mfma_f64_16x16x4f64(p.x, b.x, tr, 0, 0, 0);
            ti = __builtin_amdgcn_mfma_f64_16x16x4f64(p.x, b.y, ti, 0, 0, 0);
            tr = __builtin_amdgcn_mfma_f64_16x16x4f64(-p.y, b.y, tr, 0, 0, 0);
            ti = __builtin_amdgcn_mfma_f64_16x16x4f64(p.y, b.x, ti, 0, 0, 0);
          }
          if (NK == U && k0 + U < KS) {  // the next batch takes the chain's registers
#pragma unroll
            for (int v = 0; v < CH; ++v)
              a[CH * h + v][m] = Ls[(uint32_t)(min(4 * (k0 + U + CH * h + v) + q, n - 1) * n) + row[m]];
          }
          re[m] += tr;
          im[m] += ti;
          asm volatile("" : "+v"(re[m]), "+v"(im[m]));  // added here, not kept for all tiles
        }
      }
    };
    int k0 = 0;
    for (; k0 + 2 < KS; k0 += U) batch(std::integral_constant<int, U>(), k0);
    if (k0 < KS) batch(std::integral_constant<int, 2>(), k0);
  }
  // sums of wavefronts 1 and 2 to wavefront 0; slot 0, the centre, was wavefront 0's first
  __syncthreads();
  if (wv > 0) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v) bl64[(((wv - 1) * MT + m) * 4 + v) * 64 + lane] = make_double2(re[m][v], im[m][v]);
  }
  __syncthreads();
  if (wv == 0) {
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      double t0 = 0.0, t1 = 0.0, t2 = 0.0;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double2 o = make_double2(re[m][v], im[m][v]);
        for (int w = 0; w < MF_WAVES - 1; ++w) o = cadd(o, bl64[((w * MT + m) * 4 + v) * 64 + lane]);
        const int i = 16 * m + 4 * v + q;
        if (i < n && col < nr) {
          if (dagger && i >= half) o = make_double2(-o.x, -o.y);
          const size_t at = ((size_t)(r0 + col) * g.V + s) * n + i;
          out[at] = o;
          if (part != nullptr) {
            double2 c = make_double2(0.0, 0.0);
            if (pw == 3) c = in[at];  // (not taken under dagger)
            t0 += o.x * c.x + o.y * c.y;
            t1 += o.x * c.y - o.y * c.x;
            t2 += o.x * o.x + o.y * o.y;
          }
        }
      }
      pr[m][lane][0] = t0;
      pr[m][lane][1] = t1;
      pr[m][lane][2] = t2;
    }
  }
  if (part == nullptr) return;
  __syncthreads();
  if (tid < nr) {
    double t[3] = {0.0, 0.0, 0.0};
    for (int m = 0; m < MT; ++m)
      for (int g4 = 0; g4 < 4; ++g4)
#pragma unroll
        for (int c = 0; c < 3; ++c) t[c] += pr[m][g4 * 16 + tid][c];
    double *p = part + ((size_t)(r0 + tid) * gridDim.x + blockIdx.x) * pw;
    if (pw == 1) {
      p[0] = t[2];
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) p[c] = t[c];
    }
  }
}

static hipError_t coarse_mma_f64(const Geom &g, int n, const double2 *L, const double2 *in, double2 *out, int nrhs,
                                 int dagger, const CoarseArgs &a, const CgCheck &c, hipStream_t st) {
  const int ng = (nrhs + MMA_NR - 1) / MMA_NR, per = (nrhs + ng - 1) / ng, mt = (n + 15) / 16;
  size_t lds = sizeof(double2) * MF_WAVES * ((n + 15) / 16 * 16) * (per | 1);
  const size_t sums = sizeof(double2) * (MF_WAVES - 1) * mt * 4 * 64;
  if (lds < sums) lds = sums;
#define MG_MF(M)                                                                                                    \
  hipLaunchKernelGGL(k_coarse_mma_f64<M>, dim3(g.V, ng), dim3(64 * MF_WAVES), lds, st, g, n, L, in, out, nrhs, per, \
                     dagger, a.part, a.pw, a.done, c)
  if (mt == 1) MG_MF(1);
  else if (mt == 2) MG_MF(2);
  else if (mt == 3) MG_MF(3);
  else MG_MF(4);
#undef MG_MF
  return hipGetLastError();
}

// Whether several FP64 right-hand sides take the matrix cores, one workgroup
// per site, or k_coarse, one workgroup per site and right-hand side.  The
// former takes 20 us for a site at n = 48 (6 at n = 16) however few there are,
// the latter 9 us (5) while its workgroups fit the device, about 1 024 of them,
// half as many where the number of sites is not a multiple of 8 and a site's
// operator goes to every XCD's L2.  Matrix cores / k_coarse in us, n = 48: 64
// sites x 12 right-hand sides 23 / 18; 128 x 8 25 / 22, x 12 26 / 31; 256 x 4
// 27 / 23, x 6 28 / 32; 81 x 6 24 / 26, x 8 25 / 33; 162 x 4 25 / 33.  n = 16:
// 64 x 12 8.0 / 8.7, 16 x 12 7.9 / 5.4.  On many sites two or three right-hand
// sides share the reads of the operator in k_coarse too: 2 592 sites x 2, n =
// 64 / 48 / 40 / 16 311, 177, 143, 24 / 268, 171, 129, 41; x 3, n = 64 / 48 / 40
// 316, 179, 144 / 333, 218, 163; 512 sites, n = 40, x 3 34 / 26, x 4 34 / 32.
static bool take_mma_f64(const Geom &g, int n, int nrhs) {
  const int least = g.V < 1024u ? 4 : n > 16 ? 3 : 2;
  return nrhs >= least && (uint64_t)g.V * nrhs > ((g.V & 7u) ? 512u : 1024u);
}

// Wavefronts per workgroup of variant ks (or 8 + ks): the K range in 2 ks shares.
static int mma_waves(int ks) { return 2 * ks; }
static size_t mma_lds_bytes(int n, int nrhs, int ks) {
  const size_t b = (size_t)((9 * n + 15) / 16 * 16) * (nrhs | 1) * sizeof(float2);
  const size_t r = (size_t)mma_waves(ks) * ((n + 15) / 16) * 2 * 64 * sizeof(float4);
  return b > r ? b : r;
}

// Which products the variants take.  The bound on the staged vectors leaves a
// workgroup at most 72 KB of the CU's 160 KB of LDS: n = 64 with 12 right-hand
// sides on eight wavefronts, 64 KB of sums (60 KB of vectors before them) and 6
// KB of partial products.
bool coarse_mma_ok(int n, int nrhs, int variant) {
  const int ks = variant & 7;
  if (n > COARSE_NMAX || nrhs < 1 || nrhs > MMA_NR) return false;
  if (variant != ks && (variant != (ks | 8) || n % 4 != 0)) return false;  // row-major copy: 16-byte rows
  if (ks != 1 && ks != 2 && ks != 4) return false;
  return (size_t)9 * n * nrhs * sizeof(float2) <= 56 * 1024;
}

// Workgroups per coarse site.  Splitting a site's rows over several
// workgroups was measured slower at every coarse-lattice size here (it halves
// the contiguous column segments), so each site is one workgroup; the
// general form is kept for the row bookkeeping of the kernel.
int coarse_split(int, uint32_t) { return 1; }

// Threads per workgroup: G groups of the workgroup's rows (FP64 count), up to
// 512 threads (measured best against 256 and 1024) and at most 64 groups.
int coarse_threads(int n, uint32_t V) {
  const int nr = n / coarse_split(n, V);
  int G = 512 / nr;
  if (G > 64) G = 64;
  if (G < 1) G = 1;
  return (G * nr + 63) / 64 * 64;
}

template <typename R, typename S>
hipError_t coarse_apply_k(const Geom &g, int n, const S *L, const c_t<R> *in, c_t<R> *out, int nrhs, int dagger,
                          const CoarseArgs &a, hipStream_t st) {
  CgCheck c{};
  if (a.chk) c = *a.chk;
  if constexpr (sizeof(R) == 4) {
    if (a.variant > 0) {
      if (a.fuse && a.fuse->kind) return hipErrorInvalidValue;  // fusion is per-RHS kernel only
      const int ks = a.variant & 7;
      const bool rm = (a.variant & 8) != 0;
      if (!coarse_mma_ok(n, nrhs, a.variant)) return hipErrorInvalidValue;
      if (rm && a.lt == nullptr) return hipErrorInvalidValue;
      const S *Lk = rm ? static_cast<const S *>(a.lt) : L;
      const dim3 block(64 * mma_waves(ks));
      const size_t lds = mma_lds_bytes(n, nrhs, ks);
#define MG_MMA_LAUNCH(MTV, RMV)                                                                                 \
  hipLaunchKernelGGL((k_coarse_mma<S, MTV, RMV>), dim3(g.V), block, lds, st, g, n, Lk, in, out, nrhs, dagger, \
                     a.part, a.pw, a.done, c)
      switch ((n + 15) / 16) {
        case 1: if (rm) MG_MMA_LAUNCH(1, true); else MG_MMA_LAUNCH(1, false); break;
        case 2: if (rm) MG_MMA_LAUNCH(2, true); else MG_MMA_LAUNCH(2, false); break;
        case 3: if (rm) MG_MMA_LAUNCH(3, true); else MG_MMA_LAUNCH(3, false); break;
        default: if (rm) MG_MMA_LAUNCH(4, true); else MG_MMA_LAUNCH(4, false); break;
      }
#undef MG_MMA_LAUNCH
      return hipGetLastError();
    }
  } else {
    if (a.variant > 0) return hipErrorInvalidValue;
    // Not where the CGNR updates are fused in.
    if (take_mma_f64(g, n, nrhs) && !(a.fuse && a.fuse->kind) && (c.part_r == nullptr || nrhs <= MMA_NR))
      return coarse_mma_f64(g, n, L, in, out, nrhs, dagger, a, c, st);
  }
  const dim3 grid(g.V * coarse_split(n, g.V) * nrhs);
  dim3 block(coarse_threads(n, g.V));
  CgFuse f{};
  if (a.fuse) f = *a.fuse;
  if constexpr (sizeof(S) == 16) {
    hipLaunchKernelGGL((k_coarse<R, S, 1>), grid, block, 0, st, g, n, L, in, out, nrhs, dagger, a.part, a.pw, a.done,
                       c, f);
  } else if constexpr (sizeof(S) == 8) {
    hipLaunchKernelGGL((k_coarse<R, S, 2>), grid, block, 0, st, g, n, L, in, out, nrhs, dagger, a.part, a.pw, a.done,
                       c, f);
  } else {
    // half storage: four rows per 16-byte load when the rows of a workgroup
    // come in multiples of four, else two rows per 8-byte load
    if ((n / coarse_split(n, g.V)) % 4 == 0)
      hipLaunchKernelGGL((k_coarse<R, S, 4>), grid, block, 0, st, g, n, L, in, out, nrhs, dagger, a.part, a.pw, a.done,
                         c, f);
    else
      hipLaunchKernelGGL((k_coarse<R, S, 2>), grid, block, 0, st, g, n, L, in, out, nrhs, dagger, a.part, a.pw, a.done,
                         c, f);
  }
  return hipGetLastError();
}

template hipError_t coarse_apply_k<double, double2>(const Geom &, int, const double2 *, const double2 *, double2 *,
                                                    int, int, const CoarseArgs &, hipStream_t);
template hipError_t coarse_apply_k<float, float2>(const Geom &, int, const float2 *, const float2 *, float2 *, int,
                                                  int, const CoarseArgs &, hipStream_t);
template hipError_t coarse_apply_k<float, chalf>(const Geom &, int, const chalf *, const float2 *, float2 *, int,
                                                 int, const CoarseArgs &, hipStream_t);

}  // namespace mg
