// C ABI: the stateless fine operator wilson_apply (and its variant that
// allocates nothing, wilson_apply_noalloc) and mg_last_error.
#include <cstdio>
#include <mutex>

#include "kernels.h"

namespace mg {
const char *last_error_cstr();

int check_lattice(const mg_lattice_t *lat) {
  if (!lat) { set_error("lattice is NULL"); return MG_EINVAL; }
  uint64_t V = 1;
  for (int mu = 0; mu < 4; ++mu) {
    if (lat->L[mu] <= 0) { set_error("lattice extent must be positive"); return MG_EINVAL; }
    V *= (uint64_t)lat->L[mu];
  }
  if (V > (1ull << 28)) { set_error("lattice volume above 2^28 sites"); return MG_EINVAL; }
  return MG_OK;
}

// Whether the nrhs output spinors share memory with the links or the input
// (the stencil reads neighbours that the output would have replaced).
static bool out_overlaps(size_t V, const void *U, const void *in, const void *out, int nrhs) {
  const uintptr_t o = (uintptr_t)out, no = 192 * V * (size_t)nrhs, i = (uintptr_t)in, u = (uintptr_t)U;
  return (o < i + no && i < o + no) || (o < u + 576 * V && u < o + no);
}
static size_t volume(const mg_lattice_t *lat) {
  return (size_t)lat->L[0] * lat->L[1] * lat->L[2] * lat->L[3];
}

// out = D in; an output that shares memory with an input is formed in tmp
// (when it is given) or in a buffer of its own and copied.
static int wilson_apply_on(const mg_lattice_t *lat, const void *U, double mass, const void *in, void *out, int nrhs,
                           mg_prec_t prec, void *tmp, hipStream_t st, const char *who) {
  const size_t V = volume(lat);
  const bool via = out_overlaps(V, U, in, out, nrhs);
  double2 *y = (double2 *)(via ? tmp : out);
  hipError_t e = hipSuccess;
  if (!y) e = hipMallocAsync((void **)&y, 192 * V * nrhs, st);
  if (e == hipSuccess)
    e = dslash_canon(lat->L, lat->t_antiperiodic ? 1 : 0, (const double2 *)U, mass, (const double2 *)in, y, nrhs, prec,
                     st);
  if (e == hipSuccess && via) e = hipMemcpyAsync(out, y, 192 * V * nrhs, hipMemcpyDeviceToDevice, st);
  if (via && !tmp && y) (void)hipFreeAsync(y, st);
  if (e != hipSuccess) {
    set_error(hip_error_string(e, who));
    return MG_EHIP;
  }
  return MG_OK;
}

// ---------------------------------------------------------------- no-alloc
// Scratch of wilson_apply_noalloc, for an output that shares memory with an
// input: a file-scope device array that each GPU the library runs on holds
// until the process ends.  Host code never uses the array's name as an
// address: it takes the per-device address from hipGetSymbolAddress once per
// device (on the first call with that device current) and passes that.
static __device__ __align__(256) unsigned char scratch[MG_NOALLOC_BYTES];

constexpr int NOALLOC_MAX_DEVICES = 64;
static std::mutex noalloc_mu;
static void *noalloc_ptr[NOALLOC_MAX_DEVICES] = {};

static int noalloc_scratch(unsigned char **out) {
  int dev = 0;
  MG_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) {
    set_error("wilson_apply_noalloc: device ordinal out of range");
    return MG_EINVAL;
  }
  std::lock_guard<std::mutex> lk(noalloc_mu);
  if (!noalloc_ptr[dev]) {
    void *p = nullptr;
    MG_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    noalloc_ptr[dev] = p;
  }
  *out = static_cast<unsigned char *>(noalloc_ptr[dev]);
  return MG_OK;
}

static int wilson_apply_noalloc_on(const mg_lattice_t *lat, const void *U, double mass, const void *in, void *out,
                                   int nrhs, mg_prec_t prec, hipStream_t st) {
  // the entry point's documented limit: links, input and output in the
  // arithmetic type, the volume rounded up to whole 64-site tiles
  const size_t Vp = (volume(lat) + 63) / 64 * 64;
  const size_t need = (prec == MG_F64 ? 16 : 8) * (36 + 24 * (size_t)nrhs) * Vp;
  if (need > (size_t)MG_NOALLOC_BYTES) {
    char buf[256];
    std::snprintf(buf, sizeof(buf),
                  "wilson_apply_noalloc: this lattice and nrhs need %zu bytes of scratch, above the %zu-byte limit",
                  need, (size_t)MG_NOALLOC_BYTES);
    set_error(buf);
    return MG_ENOMEM;
  }
  unsigned char *base = nullptr;
  MG_TRY(noalloc_scratch(&base));
  return wilson_apply_on(lat, U, mass, in, out, nrhs, prec, base, st, "wilson_apply_noalloc");
}

}  // namespace mg

using namespace mg;

extern "C" int wilson_apply_noalloc(const mg_lattice_t *lat, const void *U, double mass, const void *in, void *out,
                                    int nrhs, mg_prec_t prec, hipStream_t stream) {
  set_error("");
  MG_TRY(check_lattice(lat));
  if (!U || !in || !out) { set_error("wilson_apply_noalloc: NULL buffer"); return MG_EINVAL; }
  if (in == out) { set_error("wilson_apply_noalloc: in and out alias"); return MG_EINVAL; }
  if (nrhs < 1 || nrhs > 65535) { set_error("wilson_apply_noalloc: nrhs out of range"); return MG_EINVAL; }
  if (prec == MG_F64 || prec == MG_F32) return wilson_apply_noalloc_on(lat, U, mass, in, out, nrhs, prec, stream);
  set_error("wilson_apply_noalloc: precision must be MG_F64 or MG_F32");
  return MG_ENOTSUP;
}

extern "C" int wilson_apply(const mg_lattice_t *lat, const void *U, double mass, const void *in, void *out,
                            int nrhs, mg_prec_t prec, hipStream_t stream) {
  set_error("");
  MG_TRY(check_lattice(lat));
  if (!U || !in || !out) { set_error("wilson_apply: NULL buffer"); return MG_EINVAL; }
  if (in == out) { set_error("wilson_apply: in and out alias"); return MG_EINVAL; }
  if (nrhs < 1 || nrhs > 65535) { set_error("wilson_apply: nrhs out of range"); return MG_EINVAL; }
  if (prec == MG_F64 || prec == MG_F32 || prec == MG_F16)
    return wilson_apply_on(lat, U, mass, in, out, nrhs, prec, nullptr, stream, "wilson_apply");
  set_error("wilson_apply: precision must be MG_F64, MG_F32 or MG_F16");
  return MG_ENOTSUP;
}

extern "C" const char *mg_last_error(void) { return last_error_cstr(); }
