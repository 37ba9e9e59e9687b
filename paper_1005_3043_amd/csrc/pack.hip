// Layout conversion between the boundary's canonical complex128 arrays
// (lexicographic sites, components innermost) and the internal site-blocked
// structure-of-arrays planes, with an optional precision change.
#include "solver.h"

namespace mg {

// A wavefront converts one 64-site tile.  On the canonical side a site's
// components are contiguous (192 bytes of a spinor, 144 of a link), which a
// thread per site reads and writes in strides; here 64 lanes move one flat run
// of the tile's entries (contiguous over an aggregate's x extent) and LDS
// turns it into component planes.  24 vectors of 24^3 x 48 in FP64 2.48 -> 1.19
// ms (6.1 GB), in FP32 on 16^3 x 32 0.45 -> 0.16 ms (0.9 GB); the links of 24^3 x
// 48 in FP64 0.20 -> 0.17 ms.
constexpr int PK_WAVES = 4;

// N components per site, rows of ROW entries in LDS (odd: no bank conflicts).
// Load i of lane l is entry 64 i + l of the tile's flat run.
template <int N> __device__ __forceinline__ uint32_t flat_site(int i, uint32_t lane) { return (64u * i + lane) / N; }

template <typename T, int N>
__device__ __forceinline__ void pack_tile(const Geom &g, const double2 *__restrict__ src, c_t<T> *__restrict__ dst,
                                          const uint32_t *ci, c_t<T> *row, uint32_t lane) {
  constexpr int ROW = N | 1;
  double2 v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t j = flat_site<N>(i, lane);
    v[i] = src[(size_t)ci[j] * N + (64u * i + lane - N * j)];
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t j = flat_site<N>(i, lane);
    row[j * ROW + (64u * i + lane - N * j)] = mk<c_t<T>>((T)v[i].x, (T)v[i].y);
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int c = 0; c < N; ++c) dst[c * TILE + lane] = row[lane * ROW + c];
  __builtin_amdgcn_wave_barrier();
}

// Canonical index of every site of the wavefront's tile into ci; false where
// the tile lies past the lattice.
__device__ __forceinline__ bool tile_sites(const Geom &g, uint32_t tile, uint32_t *ci, uint32_t lane) {
  if (tile * TILE >= g.Vpad) return false;
  const uint32_t s = min(tile * TILE + lane, g.V - 1);
  ci[lane] = canon_index(g, decode(g, s));
  __builtin_amdgcn_wave_barrier();
  return true;
}

// (Padding sites of the last tile receive a copy of the last site on the way
// through LDS; their entries are left as they are.)
template <typename T>
__global__ __launch_bounds__(64 * PK_WAVES) void k_pack(Geom g, const double2 *__restrict__ canon,
                                                        c_t<T> *__restrict__ internal) {
  __shared__ c_t<T> rows[PK_WAVES][64 * 13];
  __shared__ uint32_t ci[PK_WAVES][64];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6, tile = blockIdx.x * PK_WAVES + wv;
  if (!tile_sites(g, tile, ci[wv], lane)) return;
  const double2 *src = canon + (size_t)blockIdx.y * g.V * 12;
  c_t<T> *dst = internal + ((size_t)blockIdx.y * g.Vpad + (size_t)tile * TILE) * 12;
  if ((tile + 1) * TILE <= g.V) {
    pack_tile<T, 12>(g, src, dst, ci[wv], rows[wv], lane);
  } else if (tile * TILE + lane < g.V) {
    for (int c = 0; c < 12; ++c) {
      const double2 v = src[(size_t)ci[wv][lane] * 12 + c];
      dst[c * TILE + lane] = mk<c_t<T>>((T)v.x, (T)v.y);
    }
  }
}

template <typename T>
__global__ __launch_bounds__(64 * PK_WAVES) void k_unpack(Geom g, const c_t<T> *__restrict__ internal,
                                                          double2 *__restrict__ canon) {
  __shared__ c_t<T> rows[PK_WAVES][64 * 13];
  __shared__ uint32_t ci[PK_WAVES][64];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6, tile = blockIdx.x * PK_WAVES + wv;
  if (!tile_sites(g, tile, ci[wv], lane)) return;
  double2 *dst = canon + (size_t)blockIdx.y * g.V * 12;
  const c_t<T> *src = internal + ((size_t)blockIdx.y * g.Vpad + (size_t)tile * TILE) * 12;
  c_t<T> v[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) v[c] = src[c * TILE + lane];
#pragma unroll
  for (int c = 0; c < 12; ++c) rows[wv][lane * 13 + c] = v[c];
  __builtin_amdgcn_wave_barrier();
  const uint32_t ns = min((uint32_t)TILE, g.V - tile * TILE);
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const uint32_t j = flat_site<12>(i, lane), c = 64u * i + lane - 12 * j;
    const c_t<T> e = rows[wv][j * 13 + c];
    if (j < ns) dst[(size_t)ci[wv][j] * 12 + c] = make_double2((double)e.x, (double)e.y);
  }
}

template <typename T>
hipError_t pack_field(const Geom &g, const double2 *canon, c_t<T> *internal, int nvec, hipStream_t st) {
  if (nvec <= 0 || g.V == 0) return hipSuccess;
  dim3 grid(div_up(g.Vpad / TILE, PK_WAVES), nvec);
  hipLaunchKernelGGL(k_pack<T>, grid, dim3(64 * PK_WAVES), 0, st, g, canon, internal);
  return hipGetLastError();
}

template <typename T>
hipError_t unpack_field(const Geom &g, const c_t<T> *internal, double2 *canon, int nvec, hipStream_t st) {
  if (nvec <= 0 || g.V == 0) return hipSuccess;
  dim3 grid(div_up(g.Vpad / TILE, PK_WAVES), nvec);
  hipLaunchKernelGGL(k_unpack<T>, grid, dim3(64 * PK_WAVES), 0, st, g, internal, canon);
  return hipGetLastError();
}

// Gauge field: canonical U[mu][lex site][3][3] -> internal 36-component
// fine field, component mu * 9 + (3 a + b); blockIdx.y = mu.
template <typename T>
__global__ __launch_bounds__(64 * PK_WAVES) void k_pack_gauge(Geom g, const double2 *__restrict__ canon,
                                                              c_t<T> *__restrict__ internal) {
  __shared__ c_t<T> rows[PK_WAVES][64 * 9];
  __shared__ uint32_t ci[PK_WAVES][64];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6, tile = blockIdx.x * PK_WAVES + wv;
  if (!tile_sites(g, tile, ci[wv], lane)) return;
  const double2 *src = canon + (size_t)blockIdx.y * g.V * 9;
  c_t<T> *dst = internal + ((size_t)tile * 36 + blockIdx.y * 9) * TILE;
  if ((tile + 1) * TILE <= g.V) {
    pack_tile<T, 9>(g, src, dst, ci[wv], rows[wv], lane);
  } else if (tile * TILE + lane < g.V) {
    for (int e = 0; e < 9; ++e) {
      const double2 v = src[(size_t)ci[wv][lane] * 9 + e];
      dst[e * TILE + lane] = mk<c_t<T>>((T)v.x, (T)v.y);
    }
  }
}
template <typename T> hipError_t pack_gauge(const Geom &g, const double2 *canon, c_t<T> *internal, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_gauge<T>, dim3(div_up(g.Vpad / TILE, PK_WAVES), 4), dim3(64 * PK_WAVES), 0, st, g, canon,
                     internal);
  return hipGetLastError();
}
template hipError_t pack_gauge<double>(const Geom &, const double2 *, double2 *, hipStream_t);
template hipError_t pack_gauge<float>(const Geom &, const double2 *, float2 *, hipStream_t);

// Site-major (coarse) vectors: canonical [vec][lex site][n] <-> internal
// [vec][site-blocked s][n].
template <typename T>
__global__ __launch_bounds__(256) void k_pack_aos(Geom g, const double2 *__restrict__ canon,
                                                  c_t<T> *__restrict__ internal, int ncomp) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)g.V * ncomp) return;
  const uint32_t s = (uint32_t)(e / ncomp);
  const int c = (int)(e - (size_t)s * ncomp);
  const Coords k = decode(g, s);
  const uint32_t i = canon_index(g, k);
  const size_t vec = (size_t)blockIdx.y * g.V * ncomp;
  const double2 v = canon[vec + (size_t)i * ncomp + c];
  internal[vec + e] = mk<c_t<T>>((T)v.x, (T)v.y);
}
template <typename T>
__global__ __launch_bounds__(256) void k_unpack_aos(Geom g, const c_t<T> *__restrict__ internal,
                                                    double2 *__restrict__ canon, int ncomp) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)g.V * ncomp) return;
  const uint32_t s = (uint32_t)(e / ncomp);
  const int c = (int)(e - (size_t)s * ncomp);
  const Coords k = decode(g, s);
  const uint32_t i = canon_index(g, k);
  const size_t vec = (size_t)blockIdx.y * g.V * ncomp;
  const c_t<T> v = internal[vec + e];
  canon[vec + (size_t)i * ncomp + c] = make_double2((double)v.x, (double)v.y);
}
template <typename T>
hipError_t pack_aos(const Geom &g, const double2 *canon, c_t<T> *internal, int ncomp, int nvec, hipStream_t st) {
  if (nvec <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pack_aos<T>, dim3(div_up((long)g.V * ncomp, 256), nvec), dim3(256), 0, st, g, canon,
                     internal, ncomp);
  return hipGetLastError();
}
template <typename T>
hipError_t unpack_aos(const Geom &g, const c_t<T> *internal, double2 *canon, int ncomp, int nvec, hipStream_t st) {
  if (nvec <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_unpack_aos<T>, dim3(div_up((long)g.V * ncomp, 256), nvec), dim3(256), 0, st, g, internal,
                     canon, ncomp);
  return hipGetLastError();
}
template hipError_t pack_aos<double>(const Geom &, const double2 *, double2 *, int, int, hipStream_t);
template hipError_t pack_aos<float>(const Geom &, const double2 *, float2 *, int, int, hipStream_t);
template hipError_t unpack_aos<double>(const Geom &, const double2 *, double2 *, int, int, hipStream_t);
template hipError_t unpack_aos<float>(const Geom &, const float2 *, double2 *, int, int, hipStream_t);

// Aggregate maps in canonical (lexicographic) terms, computed with the same
// site decoding and neighbour arithmetic the kernels use.
__global__ void k_maps_fine(Geom g, int32_t *f2c, int32_t *f2l, int32_t *face) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= g.V) return;
  const Coords k = decode(g, s);
  const uint32_t i = canon_index(g, k);
  f2c[i] = (int32_t)k.B;
  f2l[i] = (int32_t)k.l;
  int f = 0;
  for (int mu = 0; mu < 4; ++mu) {
    if (k.o[mu] == g.b[mu] - 1) f |= 1 << (2 * mu);
    if (k.o[mu] == 0) f |= 1 << (2 * mu + 1);
  }
  face[i] = f;
}
__global__ void k_maps_coarse(Geom gc, int32_t *cnbr) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= gc.V) return;
  const Coords k = decode(gc, s);
  const uint32_t i = canon_index(gc, k);
  for (int mu = 0; mu < 4; ++mu) {
    for (int d = 0; d < 2; ++d) {
      const uint32_t t = d == 0 ? nbr_fwd(gc, s, k, mu) : nbr_bwd(gc, s, k, mu);
      cnbr[(size_t)i * 8 + 2 * mu + d] = (int32_t)canon_index(gc, decode(gc, t));
    }
  }
}
hipError_t export_maps_k(const Geom &g, const Geom &gc, int32_t *f2c, int32_t *f2l, int32_t *face, int32_t *cnbr,
                         hipStream_t st) {
  hipLaunchKernelGGL(k_maps_fine, dim3(div_up(g.V, 256)), dim3(256), 0, st, g, f2c, f2l, face);
  hipLaunchKernelGGL(k_maps_coarse, dim3(div_up(gc.V, 256)), dim3(256), 0, st, gc, cnbr);
  return hipGetLastError();
}

template hipError_t pack_field<double>(const Geom &, const double2 *, double2 *, int, hipStream_t);
template hipError_t pack_field<float>(const Geom &, const double2 *, float2 *, int, hipStream_t);
template hipError_t unpack_field<double>(const Geom &, const double2 *, double2 *, int, hipStream_t);
template hipError_t unpack_field<float>(const Geom &, const float2 *, double2 *, int, hipStream_t);

}  // namespace mg
