// ppm_noalloc.cpp -- ppm_step_cfl_noalloc: a step of up to
// PPM_NOALLOC_MAX_PATCHES patches that allocates nothing.
//
// A plan owns device memory for its patch table, launch maps, event
// counters and per-level CFL maxima.  This entry point keeps the same four
// in `scratch`, a static device array of PPM_NOALLOC_SCRATCH_BYTES bytes that
// every device the library runs on holds until the process ends: the host
// computes the table and the maps on the stack, writes them into the array
// with small kernels that take them as arguments (no staging copy, no
// memset), and launches the plan's own sweep, CFL and fill kernels on
// pointers into it.  The array's device address is taken once per device
// (hipGetSymbolAddress, with that device current) and kept; the name
// `scratch` itself is a host-side stand-in and is never passed anywhere.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <mutex>

#include "ppm.h"
#include "ppm_kernels.hpp"
#include "ppm_plan.hpp"

using ppm_detail::fail;
using ppm_detail::hip_fail;

namespace {

constexpr int kMaxPatches = PPM_NOALLOC_MAX_PATCHES;
constexpr int kMaxLevels = PPM_NOALLOC_MAX_PATCHES;
constexpr int kMaxDevices = 64;
// The maps a call can need: of the sweep's twelve (axis, extent) kinds the three
// of its sweep order, then the CFL map.
constexpr int kMaps = 4;
constexpr int kCflCells = 4096;

// Layout of the scratch array for a call's patches: event counters, per-level
// maxima, patch table, maps.  Packed, so that a call uploads only what its own
// patches take (one patch: 46 words, one launch where the full layout took five).
struct Layout {
  size_t count, smax, patch, chunk, bytes;
};
constexpr Layout layout(int npatch, int nlevels) {
  Layout l{};
  l.count = 0;
  l.smax = l.count + 2 * sizeof(unsigned long long);
  l.patch = l.smax + nlevels * sizeof(unsigned long long);
  l.chunk = l.patch + npatch * sizeof(PatchDev);
  l.bytes = l.chunk + sizeof(int32_t) * kMaps * (npatch + 1);
  return l;
}
constexpr size_t kMostBytes = layout(kMaxPatches, kMaxLevels).bytes;
static_assert(kMostBytes <= PPM_NOALLOC_SCRATCH_BYTES, "scratch layout exceeds its size");
static_assert(sizeof(PatchDev) % 8 == 0, "alignment");

const int kOrders[6][3] = {{0, 1, 2}, {2, 1, 0}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}};

}  // namespace

static __device__ __align__(256) unsigned char scratch[PPM_NOALLOC_SCRATCH_BYTES];

namespace {

std::mutex g_scratch_mu;
unsigned char *g_scratch[kMaxDevices] = {};

// Device address of `scratch` on the current device (taken once per device).
ppm_status scratch_address(unsigned char **out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices)
    return fail(PPM_EUNSUPPORTED, "device %d: at most %d devices are supported", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    g_scratch[dev] = static_cast<unsigned char *>(p);
  }
  *out = g_scratch[dev];
  return PPM_OK;
}

inline int tmask_of(int axis, int mask) {
  const int t1 = axis == 0 ? 1 : 0, t2 = axis == 2 ? 1 : 2;
  return ((mask >> t1) & 1) | (((mask >> t2) & 1) << 1);
}

// Launch shapes of the call's three sweeps, in its order: the axes swept
// lane-parallel and the runs of a plan over the same patches with the default
// tile configuration; the other axes marched without what needs memory of its
// own (no grouped maps, each block belongs to one patch, and no marching by
// halves).
struct Shape {
  int32_t axis, mask;
  bool lanes;
  int32_t segs, nblocks;
  int32_t tail_pencil0, tail_main, tail_blocks;
};

template <class Prec>
hipError_t sweep(const Shape &sh, int32_t block, int32_t lanes_block, const PatchDev *patches,
                 const int32_t *chunks, int npatch, const double *dt, const ppm::Params &P,
                 unsigned long long *counters, unsigned long long *smax, hipStream_t s) {
  if (sh.nblocks == 0) return hipSuccess;
  if (sh.lanes)
    return ppm::launch_sweep_lanes<Prec>(patches, chunks, npatch, sh.nblocks, lanes_block, sh.axis,
                                         sh.mask, sh.segs, dt, P, counters, smax, s);
  if (sh.tail_blocks > 0) {
    hipError_t e = ppm::launch_sweep<Prec>(patches, chunks, npatch, sh.tail_main, block, sh.axis,
                                           sh.mask, dt, P, counters, smax, nullptr, 0, s);
    if (e != hipSuccess) return e;
    return ppm::launch_sweep_tail<Prec>(patches, chunks, sh.tail_blocks, lanes_block, sh.axis,
                                        sh.mask, sh.tail_pencil0, dt, P, counters, smax, s);
  }
  return ppm::launch_sweep<Prec>(patches, chunks, npatch, sh.nblocks, block, sh.axis, sh.mask, dt,
                                 P, counters, smax, nullptr, 0, s);
}

template <class Prec>
hipError_t run(const Shape (&shapes)[3], int32_t block, int32_t lanes_block, const PatchDev *host,
               const int32_t *bc, unsigned char *base, int npatch, int nlevels,
               const ppm::Params &P, double *dt, uint32_t parts, int32_t cfl_blocks,
               hipStream_t s) {
  const Layout l = layout(npatch, nlevels);
  const PatchDev *patches = reinterpret_cast<const PatchDev *>(base + l.patch);
  const int32_t *chunks = reinterpret_cast<const int32_t *>(base + l.chunk);
  unsigned long long *counters = reinterpret_cast<unsigned long long *>(base + l.count);
  unsigned long long *smax = reinterpret_cast<unsigned long long *>(base + l.smax);
  const int stride = npatch + 1;
  hipError_t e = hipSuccess;
  if (parts & PPM_NOALLOC_FILL)
    for (int i = 0; i < npatch && e == hipSuccess; ++i)
      if (bc[i] == PPM_BC_PERIODIC) e = ppm::launch_fill<Prec>(host[i], s);
  if (e == hipSuccess && (parts & PPM_NOALLOC_CFL))
    e = ppm::launch_cfl<Prec>(patches, chunks + 3 * stride, npatch, cfl_blocks, kCflCells,
                              nlevels, P, smax, dt, s);
  for (int k = 0; k < 3 && e == hipSuccess; ++k)
    e = sweep<Prec>(shapes[k], block, lanes_block, patches, chunks + k * stride, npatch, dt, P,
                    counters, k == 2 ? smax : nullptr, s);
  if (e == hipSuccess) e = ppm::launch_cfl_finalize(nlevels, P.cfl, nullptr, smax, dt, s);
  return e;
}

}  // namespace

extern "C" ppm_status ppm_step_cfl_noalloc(const ppm_patch *patches, int32_t npatch,
                                           int32_t nlevels, ppm_precision prec,
                                           const ppm_params *params, double *dt_dev,
                                           int32_t sweep_order, uint32_t parts, int64_t *events,
                                           void *hip_stream) {
  if (!patches) return fail(PPM_EINVAL, "patches is NULL");
  if (npatch < 1 || npatch > kMaxPatches)
    return fail(PPM_EINVAL, "npatch must be in 1..%d (the static scratch holds %d patches)",
                kMaxPatches, kMaxPatches);
  if (nlevels < 1 || nlevels > kMaxLevels)
    return fail(PPM_EINVAL, "nlevels must be in 1..%d (the static scratch holds %d levels)",
                kMaxLevels, kMaxLevels);
  if (prec != PPM_FP64 && prec != PPM_MIXED) return fail(PPM_EINVAL, "unknown precision %d", int(prec));
  if (!dt_dev) return fail(PPM_EINVAL, "dt_dev is NULL");
  if (sweep_order < 0 || sweep_order > 5) return fail(PPM_EINVAL, "sweep_order must be in 0..5");
  if (parts & ~uint32_t(PPM_NOALLOC_FILL | PPM_NOALLOC_CFL))
    return fail(PPM_EINVAL, "unknown parts bits 0x%x", parts);
  ppm_status st = ppm_detail::check_params(params);
  if (st != PPM_OK) return st;
  if ((st = ppm_detail::check_mixed_floors(prec, params)) != PPM_OK) return st;
  for (int i = 0; i < npatch; ++i)
    if ((st = ppm_detail::check_patch(patches[i], i, nlevels)) != PPM_OK) return st;
  ppm::Params P = ppm_detail::device_params(prec, params);

  // patch table
  PatchDev host[kMaxPatches];
  int32_t bc[kMaxPatches] = {};
  std::memset(host, 0, sizeof host);
  for (int i = 0; i < npatch; ++i) {
    const ppm_patch &q = patches[i];
    PatchDev &d = host[i];
    d.n[0] = q.nx; d.n[1] = q.ny; d.n[2] = q.nz;
    d.ghost = q.ghost; d.level = q.level; d.pad = 0;
    bc[i] = q.bc;
    d.dx[0] = q.dx; d.dx[1] = q.dy; d.dx[2] = q.dz;
    d.rho = q.rho; d.vel[0] = q.vx; d.vel[1] = q.vy; d.vel[2] = q.vz;
    d.etot = q.etot; d.eint = q.eint; d.flux_reg = q.flux_reg;
    d.acc[0] = q.gx; d.acc[1] = q.gy; d.acc[2] = q.gz;
    if (q.gx) P.flags |= ppm::kAnyGravity;
  }
  if ((parts & PPM_NOALLOC_FILL))
    for (int i = 0; i < npatch; ++i)
      if (patches[i].bc != PPM_BC_PERIODIC)
        return fail(PPM_EINVAL, "patch %d: PPM_NOALLOC_FILL needs PPM_BC_PERIODIC patches", i);

  // launch maps (prefix arrays of work chunks of the three sweeps, then the
  // CFL map) and shapes; one patch marched: whole rounds of one marching block
  // per compute unit and the pencils left over, if at most an eighth of a round,
  // to the lane-parallel tail launch.  (A plan's choice, which also weighs two
  // threads to a pencil, with tails alone: 272^3 FP64 3.92 -> 3.40 ms, 400^3 10.3 ->
  // 10.0, but mixed 300^3 3.31 -> 3.81, 320^3 3.65 -> 4.2.)
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus = 0;
  const int32_t block = npatch == 1 ? 256 : 64, lanes_block = block;
  const int32_t lanes_mask = ppm_detail::default_lanes(host, npatch, prec, cus);
  const int stride = npatch + 1;
  Shape shapes[3];
  std::memset(shapes, 0, sizeof shapes);
  int32_t chunks[kMaps * (kMaxPatches + 1)];
  std::memset(chunks, 0, sizeof chunks);
  int mask = 0;
  for (int k = 0; k < 3; ++k) {
    Shape &sh = shapes[k];
    const int axis = kOrders[sweep_order][k], tm = tmask_of(axis, mask);
    sh.axis = axis;
    sh.mask = mask;
    sh.lanes = (lanes_mask >> axis) & 1;
    if (sh.lanes) sh.segs = ppm_detail::choose_run_segments(host, npatch, prec, axis, tm, cus);
    int64_t acc = 0;
    for (int i = 0; i < npatch; ++i) {
      const PatchDev &d = host[i];
      int64_t items = ppm_detail::sweep_pencils(d, axis, tm), per_block = block;
      if (sh.lanes) {
        const int64_t rpw = ppm::rows_per_wave(d.n[axis] + 2 * d.ghost, sh.segs);
        items = (items + rpw - 1) / rpw;
        per_block = lanes_block / 64;
      }
      chunks[k * stride + i] = int32_t(acc);
      acc += (items + per_block - 1) / per_block;
      if (acc > INT32_MAX / 2) return fail(PPM_EINVAL, "too many pencils for one launch");
    }
    chunks[k * stride + npatch] = int32_t(acc);
    sh.nblocks = int32_t(acc);
    if (npatch == 1 && cus > 0 && !sh.lanes) {
      const int64_t cap = int64_t(cus) * block;
      const int64_t np = ppm_detail::sweep_pencils(host[0], axis, tm), rest = np % cap;
      if (np >= cap && rest != 0 && rest * 8 <= cap) {
        sh.tail_pencil0 = int32_t(np - rest);
        sh.tail_main = int32_t((np - rest) / block);
        sh.tail_blocks = int32_t((rest + lanes_block / 64 - 1) / (lanes_block / 64));
      }
    }
    mask |= 1 << axis;
  }
  int32_t cfl_blocks = 0;
  {
    int64_t acc = 0;
    for (int i = 0; i < npatch; ++i) {
      const PatchDev &d = host[i];
      chunks[3 * stride + i] = int32_t(acc);
      acc += (int64_t(d.n[0]) * d.n[1] * d.n[2] + kCflCells - 1) / kCflCells;
      if (acc > INT32_MAX / 2) return fail(PPM_EINVAL, "too many cells for one CFL launch");
    }
    chunks[3 * stride + npatch] = int32_t(acc);
    cfl_blocks = int32_t(acc);
  }

  unsigned char *base = nullptr;
  if ((st = scratch_address(&base)) != PPM_OK) return st;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  // zeroed counters and maxima, the table and the maps (whatever a previous call
  // left there is replaced as far as this call reads)
  const Layout l = layout(npatch, nlevels);
  uint32_t words[kMostBytes / 4];
  std::memset(words, 0, l.patch);
  unsigned char *bytes = reinterpret_cast<unsigned char *>(words);
  std::memcpy(bytes + l.patch, host, sizeof(PatchDev) * size_t(npatch));
  std::memcpy(bytes + l.chunk, chunks, sizeof(int32_t) * size_t(kMaps) * size_t(stride));
  hipError_t e = ppm::launch_write_words(reinterpret_cast<uint32_t *>(base), words,
                                         int64_t(l.bytes / 4), s);
  if (e != hipSuccess) return hip_fail(e, "scratch upload");
  e = prec == PPM_FP64 ? run<ppm::PrecF64>(shapes, block, lanes_block, host, bc, base, npatch,
                                           nlevels, P, dt_dev, parts, cfl_blocks, s)
                       : run<ppm::PrecMixed>(shapes, block, lanes_block, host, bc, base, npatch,
                                             nlevels, P, dt_dev, parts, cfl_blocks, s);
  if (e != hipSuccess) return hip_fail(e, "ppm_step_cfl_noalloc launch");
  if (events) {
    unsigned long long h[2] = {0, 0};
    e = hipMemcpyAsync(h, base + l.count, sizeof h, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "event counter read");
    events[0] = int64_t(h[0]);
    events[1] = int64_t(h[1]);
  }
  return PPM_OK;
}
