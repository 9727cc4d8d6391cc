// ppm_sweep.hpp -- the streaming 1-D PPM sweep of one pencil (device).
//
// One thread owns one pencil and walks it from its first to its last cell
// once.  Every quantity a later stage needs is kept in a short sliding window
// of registers, so each input cell is read from HBM once and each updated cell
// written once, with no LDS staging and no second pass.  With the head of the
// walk at cell k:
//   * cell k is loaded and its pressure evaluated;
//   * the limited slope of cell k-2 and the interface value between k-3 and
//     k-2 are formed, and the flattening indicator of cell k-2;
//   * the parabola of cell r = k-3 is completed (steepening, flattening,
//     monotonicity) and traced to both of its edges;
//   * the Riemann problem at face (r-1)+1/2 is solved, giving the provisional
//     update of cell r-1;
//   * cell r-2 is finalised and written.  Holding the write back by one cell
//     lets the HLL fallback (Sec. "Riemann Solvers and Fallback") re-solve
//     both faces of a cell whose provisional update went non-positive and
//     redo its neighbours before anything reaches memory.  The traced states
//     the HLL solver needs are parked in LDS (one private slot pair per
//     thread) since they are read only when a fallback actually happens.
#pragma once

#include "ppm_math.hpp"

namespace ppm {

// Storage and compute types of a precision.  S: storage of rho and the
// velocity; T: reconstruction and tracing.  Energies are stored in double,
// and the pressure selection, Riemann iteration and updates run in double.
struct PrecF64 {
  using S = double;
  using T = double;
};
struct PrecMixed {
  using S = float;
  using T = float;
};

// A pointer to device memory held in a table: in device code of the global
// address space, since a generic pointer compiles to flat accesses, which count
// as LDS operations too, so that every wait for LDS also waits for the loads in
// flight.
#if defined(__HIP_DEVICE_COMPILE__) && defined(PPM_KERNEL_SOURCE)
template <class T> using Dev = __attribute__((address_space(1))) T *;
#else
template <class T> using Dev = T *;
#endif
template <class T, class V> __device__ __forceinline__ Dev<T> dev(Dev<V> p) { return (Dev<T>)p; }

// Device copy of one patch.
struct PatchDev {
  int32_t n[3];      // active cells per axis
  int32_t ghost;
  int32_t level;
  int32_t pad;
  double dx[3];
  Dev<void> rho, vel[3];
  Dev<double> etot, eint;
  Dev<double> flux_reg;
  Dev<const void> acc[3];  // nullable: gravitational acceleration per axis (storage type)
};

// One pencil as the marcher sees it: fields in pencil order (normal velocity
// first), the offset of its cell 0 and the element stride along it.
template <class S> struct PencilRef {
  Dev<S> rho, u, v1, v2;
  Dev<double> E, e;
  int64_t base, stride;
  int n, g;
  double dx;
  Dev<double> reg;          // nullable: register slot of its low face; the high face's follows
  int64_t reg_stride;       // six fields later, reg_stride apart
  int lab[6];               // lab field index of each pencil-order flux slot
  Dev<const S> acc;         // nullable: acceleration along the pencil
};

// LDS of a marching thread, in doubles: two slots of the traced L and R states
// of a face (for the fallback), the final flux of the face behind the cell
// about to be written (read only by the fallback) and that cell's provisional
// update.  Each wave holds its threads' in one piece, a lane apart, so that
// every slot is a constant offset from the thread's first (a block-sized stride
// kept thirteen addresses in registers and added up the others in every
// iteration).  After all waves', in the sweeps that take the next timestep,
// come the waves' signal maxima (64 levels for 64 threads).
constexpr int kSlotDoubles = 10;
constexpr int kLdsFluxA = 2 * kSlotDoubles;
constexpr int kLdsProvA = kLdsFluxA + 7;
constexpr int kLdsMarch = kLdsProvA + 6;
constexpr int kLdsCfl = kLdsMarch;

// Lane-parallel sweep: halo lanes at each end of a 64-lane segment, cells a
// segment writes, and the pencils of n cells a wave streams in one run of at
// most `segs` segments (but always one pencil).  The ends of a run need no
// halo, so s segments hold 54 s + 10 cells.
constexpr int kLaneHalo = 5;
constexpr int kLaneOut = 64 - 2 * kLaneHalo;
constexpr int kMaxRunSegments = 32;
__host__ __device__ __forceinline__ int rows_per_wave(int n, int segs) {
  const int r = (segs * kLaneOut + 2 * kLaneHalo) / n;
  return r > 1 ? r : 1;
}
// A patch's pencils go to its waves in groups of at most kDealWaves waves, a
// group's in turn: wave w of G takes pencils w, w + G, ... of the group's.
constexpr int kDealWaves = 128;
__host__ __device__ __forceinline__ int run_segments(int cells) {
  return cells <= 64 ? 1 : (cells - 2 * kLaneHalo + kLaneOut - 1) / kLaneOut;
}

// Select one of three values by a (wave-uniform) axis index without
// indexing a private array, which would live in scratch memory.
template <class V> __device__ __forceinline__ V pick3(int i, V a, V b, V c) {
  return i == 0 ? a : (i == 1 ? b : c);
}

// Offset of the block of face (2*axis + hi) in a patch's flux register.
__device__ __forceinline__ int64_t reg_face_offset(int64_t nx, int64_t ny, int64_t nz, int axis,
                                                   int hi) {
  const int64_t ax = ny * nz, ay = nx * nz, az = nx * ny;
  const int64_t before = axis == 0 ? 0 : (axis == 1 ? 2 * ax : 2 * (ax + ay));
  return 6 * (before + (hi ? pick3<int64_t>(axis, ax, ay, az) : 0));
}

// Where the boundary flux of the pencil (i1, i2) goes in the patch's flux
// register (face 2 axis + hi), and the stride between the six register fields
// there; null for a pencil outside the transverse active range.
__device__ __forceinline__ Dev<double> register_slot(const PatchDev &pd, int axis, int i1, int i2,
                                                     int hi, int64_t &stride) {
  const int t1 = axis == 0 ? 1 : 0, t2 = axis == 2 ? 1 : 2;
  const int g = pd.ghost;
  const int Nt1 = pick3(t1, pd.n[0], pd.n[1], pd.n[2]);
  const int Nt2 = pick3(t2, pd.n[0], pd.n[1], pd.n[2]);
  stride = int64_t(Nt1) * Nt2;
  if (!pd.flux_reg || i1 < g || i1 >= g + Nt1 || i2 < g || i2 >= g + Nt2) return nullptr;
  return pd.flux_reg + reg_face_offset(pd.n[0], pd.n[1], pd.n[2], axis, hi) +
         int64_t(i2 - g) * Nt1 + (i1 - g);
}

// The pencil (i1, i2) of a sweep along `axis` of one patch.
template <class S>
__device__ __forceinline__ PencilRef<S> make_pencil(const PatchDev &pd, int axis, int i1, int i2) {
  const int t1 = axis == 0 ? 1 : 0, t2 = axis == 2 ? 1 : 2;
  const int g = pd.ghost;
  const int N0 = pd.n[0], N1 = pd.n[1], N2 = pd.n[2];
  const int nf0 = N0 + 2 * g, nf1 = N1 + 2 * g;
  const int Na = pick3(axis, N0, N1, N2);
  const int64_t sx = 1, sy = nf0, sz = int64_t(nf0) * nf1;
  PencilRef<S> pc;
  pc.rho = dev<S>(pd.rho);
  pc.u = dev<S>(pick3(axis, pd.vel[0], pd.vel[1], pd.vel[2]));
  pc.v1 = dev<S>(pick3(t1, pd.vel[0], pd.vel[1], pd.vel[2]));
  pc.v2 = dev<S>(pick3(t2, pd.vel[0], pd.vel[1], pd.vel[2]));
  pc.E = pd.etot;
  pc.e = pd.eint;
  pc.base = i1 * pick3(t1, sx, sy, sz) + i2 * pick3(t2, sx, sy, sz);
  pc.stride = pick3(axis, sx, sy, sz);
  pc.n = Na + 2 * g;
  pc.g = g;
  pc.dx = pick3(axis, pd.dx[0], pd.dx[1], pd.dx[2]);
  pc.lab[0] = 0; pc.lab[1] = 1 + axis; pc.lab[2] = 1 + t1; pc.lab[3] = 1 + t2;
  pc.lab[4] = 4; pc.lab[5] = 5;
  pc.acc = dev<const S>(pick3(axis, pd.acc[0], pd.acc[1], pd.acc[2]));
  pc.reg = register_slot(pd, axis, i1, i2, 0, pc.reg_stride);
  return pc;
}

// Number of pencils of a sweep along `axis` of one patch: transverse axes
// restricted to their active range where `mask` says so.
__device__ __forceinline__ int pencil_count(const PatchDev &pd, int axis, int mask) {
  const int t1 = axis == 0 ? 1 : 0, t2 = axis == 2 ? 1 : 2;
  const int g = pd.ghost;
  const int Nt1 = pick3(t1, pd.n[0], pd.n[1], pd.n[2]);
  const int Nt2 = pick3(t2, pd.n[0], pd.n[1], pd.n[2]);
  const int w1 = ((mask >> t1) & 1) ? Nt1 : Nt1 + 2 * g;
  const int w2 = ((mask >> t2) & 1) ? Nt2 : Nt2 + 2 * g;
  return w1 * w2;
}

// Pencil `idx` of the sweep's pencil set in one patch: transverse axes
// restricted to their active range where `mask` says so.  False if idx is
// past the end.
__device__ __forceinline__ bool pencil_index(const PatchDev &pd, int axis, int mask, int idx,
                                             int &i1, int &i2) {
  const int t1 = axis == 0 ? 1 : 0, t2 = axis == 2 ? 1 : 2;
  const int g = pd.ghost;
  const int Nt1 = pick3(t1, pd.n[0], pd.n[1], pd.n[2]);
  const int Nt2 = pick3(t2, pd.n[0], pd.n[1], pd.n[2]);
  const bool r1 = (mask >> t1) & 1, r2 = (mask >> t2) & 1;
  const int lo1 = r1 ? g : 0, w1 = r1 ? Nt1 : Nt1 + 2 * g;
  const int lo2 = r2 ? g : 0, w2 = r2 ? Nt2 : Nt2 + 2 * g;
  if (idx >= w1 * w2) return false;
  i1 = lo1 + idx % w1;
  i2 = lo2 + idx / w1;
  return true;
}

// Hydro CFL signal speed of one cell (Sec. "Timestepping", the harmonic
// multi-D form): sum over the axes of (c_s + |v_d|) / dx_d, with c_s from the
// dual-energy pressure.  Takes the cell as stored (rho and the velocity in
// storage precision) and its velocity in pencil order (u along `axis`, then
// the two transverse components), and evaluates everything in lab axis order,
// so the CFL reduction and the last sweep of a step that accumulates the next
// step's timestep give the same value bit for bit.
template <class S>
__device__ __forceinline__ double cell_signal(const Params &P, int axis, const double (&dx)[3],
                                              S r, S u, S v1, S v2, double E, double e) {
  const double uu = double(u), a = double(v1), b = double(v2);
  const double vx = axis == 0 ? uu : a;
  const double vy = axis == 1 ? uu : (axis == 0 ? a : b);
  const double vz = axis == 2 ? uu : b;
  double p, c;
  eos(P, double(r), vx, vy, vz, E, e, p, c);
  return ddiv(c + fabs(vx), dx[0]) + ddiv(c + fabs(vy), dx[1]) + ddiv(c + fabs(vz), dx[2]);
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// Maximum signal speed over the cells a sweep writes, for a sweep that also
// yields the next step's timestep.  Only a cell that raises its level's
// maximum matters, so most cells are dismissed by an upper bound of their
// signal in float (signal_bound) against the largest value the wave knows of,
// and the exact signal is evaluated for the few others.  That value, one word
// of LDS per wave and level (`wave`), starts from the device-wide maximum
// (`global`, the bit pattern of a non-negative double, which orders like the
// value); what a wave found goes there once, at its end, and only if it is
// more than the word holds by then.  (A wave of a 512^3 z sweep evaluated 1.5 %
// of its instructions for it, one of the 4096-patch batch 15 %: 2.09 -> 1.78 ms.)
struct CflAcc {
  int axis;
  const PatchDev *pd;
  float inv[3];  // 1/dx along the sweep and the two transverse axes
  unsigned long long *global, *wave;
};

__device__ __forceinline__ unsigned long long read_now(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The wave's own word: relaxed atomics of wavefront scope, which compile to
// plain LDS instructions.
__device__ __forceinline__ unsigned long long wave_now(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void wave_raise(unsigned long long *p, unsigned long long v) {
  __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// An upper bound of a cell's signal speed, velocities in pencil order, for
// every state, gamma and cell width the interface takes; infinity or NaN where
// float arithmetic gives none (the caller dismisses a cell only below a finite
// bound).  Each float rounding is below 1e-7: E - ke, which may cancel, is raised
// by 1e-6 of its terms (t), the whole by 1e-5.  What lies near or below the
// smallest normal float is covered by absolute terms: 1e-38 on the internal
// energy, 1e-36 on the squared sound speed, 1e-35 on the sum.  t enters the
// squared sound speed once more, since with t infinite E - ke can be NaN, which
// a maximum would drop.  gamma (gamma - 1) and gamma p_floor come from the host,
// rounded up (formed here from a float gamma, the difference from one would be
// lost for gamma near one: at 1.0005 the bound was 2.6e-5 low).
__device__ __forceinline__ float signal_bound(const Params &P, const float (&inv)[3], float r,
                                              float u, float v1, float v2, float E, float e) {
  const float ke = 0.5f * __builtin_fmaf(u, u, __builtin_fmaf(v1, v1, v2 * v2));
  const float t = fabsf(E) + ke;
  const float eps = nmax(__builtin_fmaf(1e-6f, t, E - ke), e) + 1e-38f;
  const float c2 = nmax(P.gg1_up * eps, P.gpf_up * __builtin_amdgcn_rcpf(r));
  const float c = __builtin_amdgcn_sqrtf(c2 + __builtin_fmaf(1e-30f, t, 1e-36f));
  const float s = __builtin_fmaf(c + fabsf(u), inv[0],
                                 __builtin_fmaf(c + fabsf(v1), inv[1], (c + fabsf(v2)) * inv[2]));
  // (a reciprocal density outside these limits may round to zero or overflow)
  return r > 1e-30f && r < 1e30f ? __builtin_fmaf(s, 1.00001f, 1e-35f) : __builtin_inff();
}

// 1/dx for signal_bound; infinity, which gives no finite bound, for a width
// whose reciprocal float arithmetic cannot hold to 1e-6.
__device__ __forceinline__ float bound_inverse(double dx) {
  return dx > 1e-30 && dx < 1e30 ? 1.0f / float(dx) : __builtin_inff();
}

__device__ __forceinline__ CflAcc cfl_acc(const PatchDev *pd, int axis,
                                          unsigned long long *global, unsigned long long *wave) {
  const int t1 = axis == 0 ? 1 : 0, t2 = axis == 2 ? 1 : 2;
  *wave = read_now(global);
  return CflAcc{axis, pd,
                {bound_inverse(pick3(axis, pd->dx[0], pd->dx[1], pd->dx[2])),
                 bound_inverse(pick3(t1, pd->dx[0], pd->dx[1], pd->dx[2])),
                 bound_inverse(pick3(t2, pd->dx[0], pd->dx[1], pd->dx[2]))},
                global, wave};
}

template <class S>
__device__ __forceinline__ void cfl_take(const Params &P, const CflAcc &a, S r, S u, S v1, S v2,
                                         double E, double e) {
  const double top = __longlong_as_double((long long)wave_now(a.wave));
  if (signal_bound(P, a.inv, float(r), float(u), float(v1), float(v2), float(E), float(e)) <
      float(top))
    return;
  const double dx[3] = {a.pd->dx[0], a.pd->dx[1], a.pd->dx[2]};
  const double s = cell_signal<S>(P, a.axis, dx, r, u, v1, v2, E, e);
  if (!(s > top)) return;
  const unsigned long long bits = (unsigned long long)__double_as_longlong(s);
  wave_raise(a.wave, bits);
}
// At the end of a wave's sweep: its maximum of each level among its lanes (all
// that still run), written by the level's first lane.
__device__ __forceinline__ void cfl_publish(const CflAcc &a, int level) {
  const int lane = threadIdx.x & 63;
  unsigned long long pending = __ballot(true);
  while (pending) {
    const int first = __ffsll((long long)pending) - 1;
    if (lane == first) {
      const unsigned long long top = wave_now(a.wave);
      if (top > read_now(a.global)) atomicMax(a.global, top);
    }
    pending &= ~__ballot(level == __builtin_amdgcn_readlane(level, first));
  }
}

// The part of a pencil that one thread marches when two threads share a
// pencil.  The head walks cells begin .. last; the rules of the pencil's
// start (stages that need more cells than have been read yet are skipped,
// the flattening indicator of the first cells is zero, the first g cells are
// treated as ghosts) apply relative to `begin`, those of its end to the real
// end.  A thread that starts inside the pencil thereby computes its first
// cells differently from the whole march, but no cell it writes depends on
// them: a cell's update reaches five cells either side (the flattening of its
// neighbours' parabolas three, the HLL fallback of a neighbouring face two
// more), and `own_lo` is at least begin + 5, and begin + g + 1: the cell before it
// has to be one this march updates (not one of its g ghosts), since the face
// between them takes the fallback's flux where that cell goes bad.  Cells own_lo ..
// own_hi are written (the faces between them, and below own_lo when own_lo is
// the pencil's first active cell, are counted); cells defer_lo .. defer_lo +
// kDeferCells - 1 go to `defer` (6 doubles per cell) instead, for the caller
// to store after the march: the other thread of the pencil reads them as
// input late in its own march.
constexpr int kDeferCells = 5;
struct MarchSpan {
  int begin, last, own_lo, own_hi, defer_lo;
  double *defer;
};

// One thread marches one pencil (or the part of it `span` gives).  kCFL: also
// take the signal speed of every cell written (the sweep must then be the
// last of its step).
// The marching loop holds kUnroll iterations: two spare half the moves that
// carry the window on (512^3 y sweep mixed 4.74 -> 4.52 ms, FP64 7.37 -> 7.26,
// 256^3 last sweep by halves 988 -> 942 us); over several patches, where
// pencils are short, one is as fast or faster (4096-patch batch, mixed y sweep
// 1335 us, 1370 with two).
// a: the level's expansion factor (1 for the static equations).  kGrav: the
// general build, with the gravity source terms (applied where the pencil has
// an acceleration field) and the optional diffusive flux.
template <class Prec, bool kCFL, bool kUseHLLC, bool kGrav, int kUnroll>
__device__ void march_pencil(const Params &P, const PencilRef<typename Prec::S> &pc, double dt,
                             double a, double *lds_slots, int slot_stride, uint32_t &n_fallback,
                             uint32_t &n_floor, const CflAcc &cfl,
                             const MarchSpan *span = nullptr) {
  using S = typename Prec::S;
  using T = typename Prec::T;
  // with T = double the window already holds the exact pressure
  constexpr bool kExactP = sizeof(T) == sizeof(double);
  const int n = pc.n, g = pc.g;
  const int a0 = g, a1 = n - g - 1;
  // the march's own start (cell begin is its first, begin + g its first
  // active cell) and what it writes
  const bool spanned = span != nullptr;  // known where the call is inlined
  const int begin = spanned ? span->begin : 0;
  const int kend = spanned ? span->last : n - g + 4;  // the iteration that finalises its last cell
  const int b0 = begin + g;
  const int own_lo = spanned ? span->own_lo : a0, own_hi = spanned ? span->own_hi : a1;
  const int face_lo = own_lo == a0 ? a0 - 1 : own_lo;
  const bool deferring = spanned && span->defer != nullptr;
  const int defer_lo = deferring ? span->defer_lo : 0;
  auto owned = [&](int c) { return !spanned || (c >= own_lo && c <= own_hi); };
  const double lam = dt / (a * pc.dx);
  const T tlam = T(lam);
  const bool grav = kGrav && pc.acc != nullptr;
  const double hgdt = 0.5 * dt / a;
  const bool diffuse = kGrav && (P.flags & kDiffusion) != 0;
  // the diffusive flux of the face between cells jl and jl+1 (their stored
  // sweep-input values, still in memory: a cell is written two iterations
  // after its right face is final)
  auto diffuse_face = [&](FluxT<T> &F, int jl) {
    const int64_t ol = pc.base + int64_t(jl) * pc.stride, orr = ol + pc.stride;
    add_diffusion(F, double(pc.rho[ol]), double(pc.u[ol]), double(pc.v1[ol]), double(pc.v2[ol]),
                  pc.E[ol], pc.e[ol], double(pc.rho[orr]), double(pc.u[orr]),
                  double(pc.v1[orr]), double(pc.v2[orr]), pc.E[orr], pc.e[orr]);
  };
  const double gam = P.gamma;
  const bool steepen = (P.flags & kSteepen) != 0;
  const bool flatten = (P.flags & kFlatten) != 0;
  const bool fallback = (P.flags & kFallbackHLL) != 0;
  const T rho_floor = T(P.rho_floor), p_floor = T(P.p_floor);

  // Sliding windows; index 0 is the oldest cell.
  T q[5][5];       // cells k-4..k: rho, u, v1, v2, p
  double pd[5];    // cells k-4..k: pressure in double (update source term)
  double rE[3];    // cells k-2..k: rho*E of the sweep input
  double m3[5];    // cells k-5..k-1: max of rho*E over the cell and its neighbours
  T dm[3][5];      // cells k-4..k-2: twice the limited slopes
  T d2[3];         // cells k-4..k-2: density second differences
  T ft[3];         // cells k-4..k-2: flattening indicators
  T fc[2][5];      // faces (k-4)+1/2 and (k-3)+1/2: interface values
  State<T> lcarry; // left state of face r+1/2 from the previous iteration
  State<T> rstate; // right state of face (r-1)+1/2
  FluxT<T> ft_b;   // two-shock flux at face (r-2)+1/2
  FluxT<T> ft_c;   // and at face (r-1)+1/2
  // provisional update of cell B = r-1, and its energies (and acceleration)
  // as read ahead.  Like ft_c and rstate they keep their last value on the
  // iterations that do not form them, none of which reads it (a reset would
  // cost a move per value on every iteration).
  double prov_b[6], EB, eB, gB;
  // final flux at face (r-3)+1/2 and provisional update of cell A = r-2 live
  // in LDS (written every step; the flux is read only by the fallback)
  double *ff_a = lds_slots + kLdsFluxA * slot_stride;
  double *prov_a = lds_slots + kLdsProvA * slot_stride;
  bool hll_a = false;
  bool bad_a = false;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
#pragma unroll
    for (int j = 0; j < 5; ++j) q[i][j] = T(0);
    pd[i] = 0.0;
    m3[i] = 0.0;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int j = 0; j < 5; ++j) dm[i][j] = T(0);
    d2[i] = T(0);
    ft[i] = T(0);
    rE[i] = 0.0;
  }
#pragma unroll
  for (int j = 0; j < 5; ++j) fc[0][j] = fc[1][j] = T(0);
  lcarry = rstate = State<T>{T(0), T(0), T(0), T(0), T(0)};
  ft_b = ft_c = zero_flux<T>();
#pragma unroll
  for (int j = 0; j < 6; ++j) prov_b[j] = 0.0;
  EB = eB = gB = 0.0;
#pragma unroll
  for (int j = 0; j < 7; ++j) ff_a[j * slot_stride] = 0.0;
#pragma unroll
  for (int j = 0; j < 6; ++j) prov_a[j * slot_stride] = 0.0;

  // prefetch of the head cell
  S nr = S(0), nu = S(0), nv1 = S(0), nv2 = S(0);
  double nE = 0.0, ne = 0.0;
  if (begin < n) {
    const int64_t o = pc.base + int64_t(begin) * pc.stride;
    nr = pc.rho[o]; nu = pc.u[o]; nv1 = pc.v1[o]; nv2 = pc.v2[o]; nE = pc.E[o]; ne = pc.e[o];
  }

  // The last round of two may hold one iteration too many.  Marching by halves it
  // is run (256^3 y sweep 983 -> 965 us, mixed 700 -> 686): it reads cells of the
  // patch only, and neither counts nor writes, the cell it would finish not
  // being an owned one.  The FP64 build that takes the timestep would spill more,
  // and leaves the loop instead (942 us against 1008), as the whole march does (the
  // same).
  for (int kk = begin; kk <= kend; kk += kUnroll)
#pragma unroll
  for (int step = 0; step < kUnroll; ++step) {
    const int k = kk + step;
    if (step > 0 && k > kend && !(spanned && (!kCFL || !kExactP))) break;
    const int t = k - begin;  // cells read so far, less one
    // energies of cell B = k-4 (updated below), fetched early to hide latency
    if (k - 4 >= b0 && k - 4 <= a1) {
      const int64_t o = pc.base + int64_t(k - 4) * pc.stride;
      EB = pc.E[o];
      eB = pc.e[o];
      if (grav) gB = double(pc.acc[o]);
    }
    // ---- 1. head cell: load and equation of state
    if (k < n) {
      const double r = double(nr), u = double(nu), v1 = double(nv1), v2 = double(nv2);
      const double E = nE, e = ne;
      if (k + 1 < n && (!spanned || k + 1 <= kend)) {
        const int64_t o = pc.base + int64_t(k + 1) * pc.stride;
        nr = pc.rho[o]; nu = pc.u[o]; nv1 = pc.v1[o]; nv2 = pc.v2[o]; nE = pc.E[o]; ne = pc.e[o];
      }
      const double p = eos_pressure(P, r, u, v1, v2, E, e);
      q[4][0] = T(r); q[4][1] = T(u); q[4][2] = T(v1); q[4][3] = T(v2); q[4][4] = T(p);
      if (!kExactP) pd[4] = p;
      rE[2] = r * E;
      m3[4] = vmax<double>(vmax<double>(rE[0], rE[1]), rE[2]);  // of cell k-1
    }
    // ---- 2. slope and second difference of cell k-2, 3. interface value
    // between cells k-3 and k-2 (as late as the parabola of cell k-3 allows:
    // what is carried from one iteration to the next costs a move)
    if (t >= 3 && k <= n) {
#pragma unroll
      for (int j = 0; j < 5; ++j) dm[2][j] = limited_slope2<T>(q[1][j], q[2][j], q[3][j]);
      d2[2] = second_diff<T>(q[1][0], q[2][0], q[3][0]);
#pragma unroll
      for (int j = 0; j < 5; ++j) fc[1][j] = interface_value(q[1][j], q[2][j], dm[1][j], dm[2][j]);
    }
    // ---- 4. flattening indicator of cell k-2 (zero where its stencil leaves the pencil)
    ft[2] = T(0);
    if (flatten && t >= 4 && k <= n - 1)
      ft[2] = flatten_indicator<T>(q[0][4], q[1][4], q[3][4], q[4][4], q[1][1], q[3][1]);

    // ---- 5. parabola of cell r = k-3, traced to both edges
    const int r = k - 3;
    State<T> lnew = lcarry;
    // rstate: right state of face (r-1)+1/2 (used for r >= b0); lnew: left
    // state of face r+1/2 (used for r <= a1)
    if (r >= b0 - 1 && r <= a1 + 1) {
      T l[5], rr[5], dq[5], q6[5];
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        l[j] = fc[0][j];   // face (r-1)+1/2
        rr[j] = fc[1][j];  // face r+1/2
      }
      if (steepen) {
        T eta = steepen_eta<T>(T(P.steep_gk), q[0][0], q[2][0], q[0][4], q[2][4], d2[0], d2[2]);
        if (eta != T(0)) {
          l[0] = mad<T>(l[0], T(1) - eta, xfma(T(0.25), dm[0][0], q[0][0]) * eta);
          rr[0] = mad<T>(rr[0], T(1) - eta, xfma(T(-0.25), dm[2][0], q[2][0]) * eta);
        }
      }
      if (flatten) {
        T fn = (q[2][4] - q[0][4] > T(0)) ? ft[0] : ft[2];
        T f = vmax<T>(ft[1], fn);
        if (f != T(0)) {
#pragma unroll
          for (int j = 0; j < 5; ++j) {
            l[j] = mad<T>(f, q[1][j], (T(1) - f) * l[j]);
            rr[j] = mad<T>(f, q[1][j], (T(1) - f) * rr[j]);
          }
        }
      }
#pragma unroll
      for (int j = 0; j < 5; ++j) monotonize<T>(q[1][j], l[j], rr[j], dq[j], q6[j]);
      trace_edges<T>(gam, l, rr, dq, q6, q[1][1], sound_speed(gam, q[1][4], q[1][0]), tlam,
                     rho_floor, p_floor, rstate, lnew);
    }

    // ---- 6. Riemann problem at face fc = (r-1)+1/2
    double *slot_c = lds_slots + (t & 1) * kSlotDoubles * slot_stride;
    if (r - 1 >= b0 - 1 && r - 1 <= a1) {
      ft_c = face_flux<kUseHLLC, T>(P, lcarry, rstate);
      if (diffuse) diffuse_face(ft_c, r - 1);
      if (fallback) {
        slot_c[0 * slot_stride] = double(lcarry.r);
        slot_c[1 * slot_stride] = double(lcarry.u);
        slot_c[2 * slot_stride] = double(lcarry.v1);
        slot_c[3 * slot_stride] = double(lcarry.v2);
        slot_c[4 * slot_stride] = double(lcarry.p);
        slot_c[5 * slot_stride] = double(rstate.r);
        slot_c[6 * slot_stride] = double(rstate.u);
        slot_c[7 * slot_stride] = double(rstate.v1);
        slot_c[8 * slot_stride] = double(rstate.v2);
        slot_c[9 * slot_stride] = double(rstate.p);
      }
    }

    // ---- 7. provisional update of cell B = r-1 with the two-shock fluxes
    const int B = r - 1;
    bool bad_b = false;
    if (B >= b0 && B <= a1) {
      CellInT<T> cin;
      cin.rho = q[0][0]; cin.u = q[0][1];
      cin.v1 = q[0][2]; cin.v2 = q[0][3];
      cin.E = EB; cin.e = eB;
      cin.p = kExactP ? double(q[0][4]) : pd[0];
      cin.rhoEmax = m3[1];
      bad_b = update_cell(P, lam, cin, ft_b, ft_c, prov_b, grav, hgdt * gB);
    }

    // ---- 8. face fb = (r-2)+1/2 becomes final: HLL if a neighbour went bad
    const int A = r - 2;
    const int fb = r - 2;  // face index: fb+1/2 lies between cells A and B
    FluxT<T> ff_b = ft_b;
    bool hll_b = false;
    if (fb >= b0 - 1 && fb <= a1) {
      hll_b = fallback && (bad_a || bad_b);
      if (hll_b) {
        const double *slot_b = lds_slots + ((t - 1) & 1) * kSlotDoubles * slot_stride;
        double sl[5], sr[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
          sl[j] = slot_b[j * slot_stride];
          sr[j] = slot_b[(5 + j) * slot_stride];
        }
        ff_b = narrow_flux<T>(hll_flux(P, sl, sr));
        if (diffuse) diffuse_face(ff_b, fb);
        if (!spanned || (fb >= face_lo && fb <= own_hi)) ++n_fallback;
      }
      if ((fb == a0 - 1 || fb == a1) && pc.reg) {
        // (opaque: the twelve addresses, formed ahead of the loop, took 24
        // registers and spilled what every iteration reads; without them and the
        // constants in Params the FP64 march has no spill: 256^3 z sweep 1070 ->
        // 955 us, last sweep 1126 -> 950)
        const Dev<double> reg = opaque(pc.reg + (fb == a1 ? 6 * pc.reg_stride : 0));
#pragma unroll
        for (int j = 0; j < 6; ++j) reg[pc.lab[j] * pc.reg_stride] = dt * ff_b.get(j);
      }
    }

    // ---- 9. finalise and write cell A = r-2
    if (A >= b0 && A <= a1) {
      const int64_t o = pc.base + int64_t(A) * pc.stride;
      double out[6];
#pragma unroll
      for (int j = 0; j < 6; ++j) out[j] = prov_a[j * slot_stride];
      bool bad = bad_a;
      if (hll_a || hll_b) {
        // redo the update with the final fluxes (input of A is still in memory)
        CellInT<T> cin;
        cin.rho = T(pc.rho[o]); cin.u = T(pc.u[o]);
        cin.v1 = T(pc.v1[o]); cin.v2 = T(pc.v2[o]);
        cin.E = pc.E[o]; cin.e = pc.e[o];
        double pp, cc;
        eos(P, double(cin.rho), double(cin.u), double(cin.v1), double(cin.v2), cin.E, cin.e, pp,
            cc);
        cin.p = pp;
        cin.rhoEmax = m3[0];
        FluxT<T> fa;
#pragma unroll
        for (int j = 0; j < 7; ++j) fa.set(j, ff_a[j * slot_stride]);
        bad = update_cell(P, lam, cin, fa, ff_b, out, grav,
                          grav ? hgdt * double(pc.acc[o]) : 0.0);
      }
      if (bad) {
        CellInT<T> cin;
        cin.rho = T(pc.rho[o]); cin.u = T(pc.u[o]);
        cin.v1 = T(pc.v1[o]); cin.v2 = T(pc.v2[o]);
        cin.E = pc.E[o]; cin.e = pc.e[o]; cin.p = 0.0; cin.rhoEmax = 0.0;
        floor_cell(P, cin, out);
        if (owned(A)) ++n_floor;
      }
      if (owned(A)) {
        if (deferring && A >= defer_lo && A < defer_lo + kDeferCells) {
          double *d = span->defer + (A - defer_lo) * 6;
#pragma unroll
          for (int j = 0; j < 4; ++j) d[j] = double(S(out[j]));
          d[4] = out[4];
          d[5] = out[5];
        } else {
          pc.rho[o] = S(out[0]);
          pc.u[o] = S(out[1]);
          pc.v1[o] = S(out[2]);
          pc.v2[o] = S(out[3]);
          pc.E[o] = out[4];
          pc.e[o] = out[5];
        }
        if (kCFL)
          cfl_take<S>(P, cfl, S(out[0]), S(out[1]), S(out[2]), S(out[3]), out[4], out[5]);
      }
    }

    // ---- 10. carry the face and cell state one step
#pragma unroll
    for (int j = 0; j < 7; ++j) ff_a[j * slot_stride] = ff_b.get(j);
    hll_a = hll_b;
    ft_b = ft_c;
#pragma unroll
    for (int j = 0; j < 6; ++j) prov_a[j * slot_stride] = prov_b[j];
    bad_a = bad_b;
    lcarry = lnew;

    // ---- 11. shift the windows
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int j = 0; j < 5; ++j) q[i][j] = q[i + 1][j];
      if (!kExactP) pd[i] = pd[i + 1];
      m3[i] = m3[i + 1];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int j = 0; j < 5; ++j) dm[i][j] = dm[i + 1][j];
      d2[i] = d2[i + 1];
      ft[i] = ft[i + 1];
      rE[i] = rE[i + 1];
    }
#pragma unroll
    for (int j = 0; j < 5; ++j) fc[0][j] = fc[1][j];
  }
}

}  // namespace ppm
