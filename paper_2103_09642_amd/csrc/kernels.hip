// HIP kernels of the PIC/MCC time step for gfx950.
//
// One step s of a case (section 2.1; Algorithms 2-6) is one launch per
// species (ions only on steps with s % N_SUB == 0: ion subcycling).  Every
// workgroup of k_particles first solves the field of step s from the
// fixed-point densities into its own LDS (steps 1-2: rho, the discrete
// Poisson equation, E on the nodes) and then streams its share of the
// particles: gather E, leapfrog push, wall absorption, the collision test,
// the colliders' scattering and the ionization births, and the deposit of
// the new position for step s+1 -- fused, so each particle's state is
// streamed from HBM once per step and no launch sits between two steps'
// particle passes.
//
// Deposits are int64 fixed point (2^32 units per particle), privatised in
// LDS per workgroup and flushed with one global atomic per touched node;
// integer addition makes the result independent of the order of particles,
// workgroups and atomics.  Densities use three rotating buffers so that a
// buffer is read at step s, cleared during step s+1 and refilled during step
// s+2 without any extra synchronisation.
//
// Every FP64 expression of the push and the collision kinematics is written
// in the same operation order as its definition, and the library is built
// with -ffp-contract=off, so no multiply-add is fused (but in div_by, whose
// fused steps give the correctly rounded quotient).
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "impl.hpp"

namespace edp {

// ---------------------------------------------------------------------------
// Random numbers: Philox4x32-10 (Salmon et al., SC'11), counter
// (uid_lo, uid_hi, step, species<<24 | purpose<<8 | call), key (seed_lo,
// seed_hi); each pair of output words gives a uniform in [0,1) with 53 bits.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    // one 32x32->64 multiply each (v_mad_u64_u32) gives both halves
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    c = make_uint4((uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1,
                   (uint32_t)p0);
  }
  return c;
}

// The first output word alone: the upper half of the first uniform's 64 bits
// (the last round needs one of its two products only).
__device__ __forceinline__ uint32_t philox_w0(uint64_t seed, uint64_t uid, uint32_t step, uint32_t t) {
  return philox(make_uint4((uint32_t)uid, (uint32_t)(uid >> 32), step, t), (uint32_t)seed, (uint32_t)(seed >> 32)).x;
}

__device__ __forceinline__ uint32_t tag(uint32_t species, uint32_t purpose, uint32_t call) {
  return (species << 24) | (purpose << 8) | call;
}

__device__ __forceinline__ void uniform2(uint64_t seed, uint64_t uid, uint32_t step, uint32_t t,
                                         double& u0, double& u1) {
  const uint4 w = philox(make_uint4((uint32_t)uid, (uint32_t)(uid >> 32), step, t),
                         (uint32_t)seed, (uint32_t)(seed >> 32));
  const uint64_t a = ((uint64_t)w.x << 32) | w.y;
  const uint64_t b = ((uint64_t)w.z << 32) | w.w;
  u0 = (double)(a >> 11) * (1.0 / 9007199254740992.0);
  u1 = (double)(b >> 11) * (1.0 / 9007199254740992.0);
}

// Box-Muller: two standard normals from two uniforms (log argument in (0,1]).
__device__ __forceinline__ void box_muller(double u0, double u1, double& z0, double& z1) {
  const double r = sqrt(-2.0 * log(1.0 - u0));
  // sincos: one argument reduction for both (the same values as separate
  // sin and cos calls)
  double sn, cs;
  sincos(kTwoPi * u1, &sn, &cs);
  z0 = r * cs;
  z1 = r * sn;
}

// Three normals from calls first_call and first_call+1.
__device__ __forceinline__ void normals3(uint64_t seed, uint64_t uid, uint32_t step,
                                         uint32_t species, uint32_t purpose, uint32_t first_call,
                                         double& z0, double& z1, double& z2) {
  double u0, u1, z3;
  uniform2(seed, uid, step, tag(species, purpose, first_call), u0, u1);
  box_muller(u0, u1, z0, z1);
  uniform2(seed, uid, step, tag(species, purpose, first_call + 1), u0, u1);
  box_muller(u0, u1, z2, z3);
}

// splitmix64 finaliser (Steele, Lea & Flood, OOPSLA 2014).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Identity of a particle born in an ionization: hash of (parent, step, kind),
// kind 1 = ejected electron, 2 = new ion; independent of the order of births.
__device__ __forceinline__ uint64_t child_uid(uint64_t parent, int64_t step, uint64_t kind) {
  return mix64(mix64(parent) ^ ((uint64_t)step * 0x9E3779B97F4A7C15ull) ^ kind);
}

// a / b from y = 1/b correctly rounded: the quotient's estimate a y corrected
// twice by its exact remainder, which makes it the correctly rounded quotient
// (Markstein's theorem on division by fused multiply-adds; it excepts a b
// whose significand is all ones, for which the host sets y to NaN).  Five
// operations instead of the division's dozen, several slow ones among them.
// For quotients, and remainders, in the normal range or zero, or not finite.
__device__ __forceinline__ double div_by(double a, double b, double y) {
  const double q0 = a * y;
  double q = __builtin_fma(__builtin_fma(-q0, b, a), y, q0);
  q = __builtin_fma(__builtin_fma(-q, b, a), y, q);
  return y == y ? (__builtin_isfinite(q0) ? q : q0) : a / b;
}

// Cross-section table row of a kinetic energy: the nearest of the tabulated
// energies i * de (section 3.2), every energy past the end in the last row.
__device__ __forceinline__ int energy_bin(double e_ev, double de, double inv_de, int nbins) {
  const double rows = div_by(e_ev, de, inv_de) + 0.5;
  return rows >= (double)(nbins - 1) ? nbins - 1 : (int)rows;
}

// Post-collision velocity w + f2 g' R(theta,phi)(cos chi, sin chi cos eta,
// sin chi sin eta) with the Euler angles of g from its components (phi = 0
// when g is along x); the components follow the final velocity equation of
// section 2.1.6 term by term.
struct Frame {
  double cos_theta, sin_theta, cos_phi, sin_phi;
};
__device__ __forceinline__ Frame frame_of(double gx, double gy, double gz, double gmag) {
  Frame F;
  if (gmag > 0.0) {
    const double gyz = sqrt(gy * gy + gz * gz);
    F.cos_theta = gx / gmag;
    F.sin_theta = gyz / gmag;
    if (gyz > 0.0) {
      F.cos_phi = gy / gyz;
      F.sin_phi = gz / gyz;
    } else {
      F.cos_phi = 1.0;
      F.sin_phi = 0.0;
    }
  } else {
    F.cos_theta = 1.0;
    F.sin_theta = 0.0;
    F.cos_phi = 1.0;
    F.sin_phi = 0.0;
  }
  return F;
}
__device__ __forceinline__ void rotate(const Frame& F, double gnew, double f2, double cos_chi, double sin_chi,
                                       double cos_eta, double sin_eta, double wx, double wy, double wz, double& ox,
                                       double& oy, double& oz) {
  const double a = f2 * gnew;
  ox = wx + a * (F.cos_theta * cos_chi - F.sin_theta * sin_chi * cos_eta);
  oy = wy + a * (F.sin_theta * F.cos_phi * cos_chi + F.cos_theta * F.cos_phi * sin_chi * cos_eta -
                 F.sin_phi * sin_chi * sin_eta);
  oz = wz + a * (F.sin_theta * F.sin_phi * cos_chi + F.cos_theta * F.sin_phi * sin_chi * cos_eta +
                 F.cos_phi * sin_chi * sin_eta);
}
__device__ __forceinline__ void scatter(double gx, double gy, double gz, double gmag, double gnew,
                                        double f2, double cos_chi, double sin_chi, double eta,
                                        double wx, double wy, double wz, double& ox, double& oy,
                                        double& oz) {
  const Frame F = frame_of(gx, gy, gz, gmag);
  double cos_eta, sin_eta;
  sincos(eta, &sin_eta, &cos_eta);
  rotate(F, gnew, f2, cos_chi, sin_chi, cos_eta, sin_eta, wx, wy, wz, ox, oy, oz);
}

// Fixed-point split of one particle between nodes p and p+1 (charge
// assignment equations): in cell units xi = x/dx, p = int(xi) clamped to
// N_g-2, the share of node p+1 (xi - p) 2^32 truncated, capped at 2^32.
__device__ __forceinline__ int deposit_split(double x, double inv_dx, int ng, long long& r) {
  const double xi = x * inv_dx;
  int p = (int)xi;
  p = p > ng - 2 ? ng - 2 : (p < 0 ? 0 : p);
  const double f = (xi - (double)p) * kTwo32;
  // below 2^32 a 32-bit conversion is the truncation (f is never negative:
  // p <= xi for x >= 0)
  const bool all = f >= kTwo32;
  r = (long long)(((uint64_t)(all ? 1u : 0u) << 32) | (all ? 0u : (uint32_t)f));
  return p;
}

// Slots in use, never beyond the capacity (alloc may pass it on overflow).
__device__ __forceinline__ int64_t slots(const CaseDev* C, int sp) {
  const int64_t a = C->alloc[sp];
  return a < C->sp[sp].cap ? a : C->sp[sp].cap;
}

// Lanes of the wave with b set (the compare's own mask, no second compare).
__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

__device__ __forceinline__ void lds_add(unsigned long long* a, long long v) {
  atomicAdd(a, (unsigned long long)v);
}

// Arrays reached through the CaseDev block are global memory, but the
// compiler cannot prove it for pointers loaded from memory and would emit
// FLAT instructions, which count against the LDS wait counter too: every LDS
// access would then wait for the in-flight HBM traffic.  G() states the
// address space so loads, stores and atomics are global_* instructions.
#define EDP_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ EDP_GLOBAL T* G(T* p) {
  return (EDP_GLOBAL T*)p;
}
// A case's constants (and the counters no thread of the running kernel
// writes) are read through the constant address space: uniform reads then
// become scalar loads and stay in scalar registers.  Every write goes
// through the ordinary pointer.
#define EDP_CONST __attribute__((address_space(4)))
template <class T>
__device__ __forceinline__ const EDP_CONST T* KC(const T* p) {
  return (const EDP_CONST T*)p;
}
__device__ __forceinline__ void gl_add(int64_t* a, long long v) {
  __hip_atomic_fetch_add(G((unsigned long long*)a), (unsigned long long)v, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long gl_fetch_add(int64_t* a, unsigned long long v) {
  return __hip_atomic_fetch_add(G((unsigned long long*)a), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// *a += v where no other thread adds to *a in the launch: the sum of a plain
// read, add and write, bit for bit, without waiting for the read.
__device__ __forceinline__ void gl_sum(EDP_GLOBAL double* a, double v) {
  (void)__builtin_amdgcn_global_atomic_fadd_f64((__attribute__((address_space(1))) double*)a, v);
}

// A uniform value in vector registers from here on (the scalar ones are
// short, and the compiler would read the value again at every use).
__device__ __forceinline__ double pin_v(double v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Exclusive scan of one integer per thread across the workgroup; *total
// gets the sum.  scratch: 64 int64 of LDS.
template <class T>
__device__ __forceinline__ T block_exclusive_scan_t(T x, int64_t* scratch, T* total) {
  T* sW = (T*)scratch;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  T inc = x;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const T y = __shfl_up(inc, off, 64);
    if (lane >= off) inc += y;
  }
  if (lane == 63) sW[wv] = inc;
  __syncthreads();
  T before = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    const T v = sW[w];
    if (w < wv) before += v;
    tot += v;
  }
  *total = tot;
  __syncthreads();
  return before + inc - x;
}

// ---------------------------------------------------------------------------
// Steps 1-2: density -> rho -> potential -> field.  MODE 0 (default)
// solves the discrete Poisson equation through the fluxes between nodes, in
// parallel (two workgroup scans instead of 2 N_g dependent steps); it agrees
// with an 80-bit solution to ~1e-15 of the field scale, closer than the
// sequential sweep.  MODE 1 runs the Thomas algorithm itself in one thread,
// operation for operation as the sequential definition (bit-reproducible,
// slow).
// ---------------------------------------------------------------------------
constexpr int kWave = 64;

// Fold the per-step particle sums of one node (ring slot `fold`, the step
// before the one about to run) into the time sums and, with the xt arrays,
// into time-bin row `row_prev`; the power density j E takes the field that
// step used, still in efield[] (the caller overwrites it after a barrier).
// All its reads go out together and the sums are added without being read
// (gl_sum): one wait instead of one per sum, on the path of the one workgroup
// per case that the whole launch waits for (a step of 5e4 electrons with every
// measurement 19.0 -> 17.0 us).
__device__ __forceinline__ void fold_particle_sums(const EDP_CONST CaseDev* __restrict__ C, int p,
                                                   int64_t fold, size_t row_prev, size_t plane) {
  const uint32_t fl = C->flags;
  const bool xt = (fl & kDiagXT) != 0;
  EDP_GLOBAL int64_t* aJe = G(C->acc_je) + fold + p;
  EDP_GLOBAL int64_t* aJi = G(C->acc_ji) + fold + p;
  EDP_GLOBAL int64_t* aW = G(C->acc_w) + fold + p;
  EDP_GLOBAL int64_t* aE = G(C->acc_e) + fold + p;
  EDP_GLOBAL int64_t* aWi = G(C->acc_wi) + fold + p;
  EDP_GLOBAL int64_t* aEi = G(C->acc_ei) + fold + p;
  EDP_GLOBAL int64_t* aIz = G(C->acc_iz) + fold + p;
  const int64_t je = *aJe, ji = *aJi, w = *aW, e = *aE;
  int64_t wi = 0, ei = 0, iz = 0;
  double eo = 0.0;
  if (xt) {
    wi = *aWi;
    ei = *aEi;
    iz = *aIz;
    eo = G(C->efield)[p];
  }
  if (fl & kDiagCurrent) {
    gl_sum(G(C->sum_je) + p, (double)je);
    gl_sum(G(C->sum_ji) + p, (double)ji);
  }
  if (fl & kDiagMeanE) {
    gl_sum(G(C->sum_w) + p, (double)w);
    gl_sum(G(C->sum_e) + p, (double)e);
  }
  *aJe = 0;
  *aJi = 0;
  *aW = 0;
  *aE = 0;
  if (xt) {
    EDP_GLOBAL double* __restrict__ X = G(C->xt) + row_prev + p;
    gl_sum(X + kXtJe * plane, (double)je);
    gl_sum(X + kXtPe * plane, (double)je * eo);
    gl_sum(X + kXtJi * plane, (double)ji);
    gl_sum(X + kXtPi * plane, (double)ji * eo);
    gl_sum(X + kXtWe * plane, (double)w);
    gl_sum(X + kXtEe * plane, (double)e);
    gl_sum(X + kXtWi * plane, (double)wi);
    gl_sum(X + kXtEi * plane, (double)ei);
    gl_sum(X + kXtIz * plane, (double)iz);
    *aWi = 0;
    *aEi = 0;
    *aIz = 0;
  }
}

// Duties of a step's writer (one workgroup per case and step), in loops of
// their own: inside the solve's code they would be fetched by every
// workgroup that skips them.
struct FieldWriter {
  const EDP_CONST CaseDev* C;
  int s3, k3;  // step % 3, ion step index % 3
  int ng;
  bool ion_step, xt, rings;
  size_t plane, row, row_prev;
  // node p before the solve: rho for reads, the time sums of the densities,
  // the deposit rings the next steps refill cleared, the particle sums of step
  // s-1 folded with the field that step used (still in efield[]), the xt rows
  // of the densities
  __device__ __forceinline__ void node(int p, double ne, double ni, double rho) const {
    const uint32_t fl = C->flags;
    G(C->rho)[p] = rho;
    if (fl & kDiagDensity) {
      gl_sum(G(C->sum_ne) + p, ne);
      gl_sum(G(C->sum_ni) + p, ni);
    }
    const int prev3 = s3 == 0 ? 2 : s3 - 1;
    if (rings) G(C->cnt_e)[prev3 * ng + p] = 0;
    if (rings && ion_step) G(C->cnt_i)[(k3 == 0 ? 2 : k3 - 1) * ng + p] = 0;
    if (fl & (kDiagCurrent | kDiagMeanE | kDiagXT)) fold_particle_sums(C, p, prev3 * ng, row_prev, plane);
    if (xt) {
      EDP_GLOBAL double* __restrict__ X = G(C->xt);
      gl_sum(X + kXtNe * plane + row + p, ne);
      gl_sum(X + kXtNi * plane + row + p, ni);
    }
  }
  // flux p of the solve (the last slot keeps V, for phi on demand)
  __device__ __forceinline__ void flux(int p, double f) const {
    G(C->flux)[p] = f;
    if (xt) gl_sum(G(C->xt) + kXtFlux * plane + row + p, f);
  }
  // node p after the solve
  __device__ __forceinline__ void field(int p, double e) const {
    G(C->efield)[p] = e;
    if (xt) gl_sum(G(C->xt) + kXtEf * plane + row + p, e);
  }
};

// Step s in ion steps: k = s / nsub, the step within it, and the rings' places
// s % 3 and k % 3.  32-bit division up to 2^31 steps (a 64-bit one is some 150
// dependent instructions at the start of every launch).
struct StepIndex {
  int64_t k;
  int sub, s3, k3;
  __device__ __forceinline__ StepIndex(int64_t s, int nsub) {
    if (s < (int64_t)1 << 31) {
      const uint32_t q = (uint32_t)s / (uint32_t)nsub;
      k = q;
      sub = (int)((uint32_t)s - q * (uint32_t)nsub);
      s3 = (int)((uint32_t)s % 3u);
      k3 = (int)(q % 3u);
    } else {
      k = s / nsub;
      sub = (int)(s - k * nsub);
      s3 = (int)(s % 3);
      k3 = (int)(k % 3);
    }
  }
  // of the next step
  __device__ __forceinline__ void next(int nsub) {
    s3 = s3 == 2 ? 0 : s3 + 1;
    if (++sub == nsub) {
      sub = 0;
      ++k;
      k3 = k3 == 2 ? 0 : k3 + 1;
    }
  }
};

// The constants of a field solve.
struct SolveIn {
  double scale, kpois, dx, inv_dx, inv_2dx, inv_cells;
  __device__ __forceinline__ explicit SolveIn(const EDP_CONST CaseDev* C)
      : scale(C->dens_scale), kpois(C->kpois), dx(C->dx), inv_dx(C->inv_dx_q), inv_2dx(C->inv_2dx), inv_cells(C->inv_cells) {
    asm volatile("" : "+s"(scale), "+s"(kpois), "+s"(dx), "+s"(inv_dx), "+s"(inv_2dx), "+s"(inv_cells));
  }
};

// The deposit rings a field solve reads, on their way from global memory: a
// thread's nodes t, t + NB, ... of both species (the first kRingRegs of them;
// those beyond are loaded when they are staged), and V(t) of the step.
constexpr int kRingRegs = 4;
template <int NB>
struct RingNodes {
  static constexpr bool kOwn = false;
  const EDP_GLOBAL int64_t *gE, *gI;
  int64_t e[kRingRegs], i[kRingRegs];
  double V;
  __device__ __forceinline__ RingNodes(const int64_t* cnt_e, const int64_t* cnt_i, const double* volt, int64_t s, int s3,
                                       int k3, int ng) {
    gE = G(cnt_e) + s3 * ng;
    gI = G(cnt_i) + k3 * ng;
#pragma unroll
    for (int q = 0; q < kRingRegs; ++q) {
      const int p = (int)threadIdx.x + q * NB;
      const int pc = p < ng ? p : ng - 1;  // no branch around the loads
      e[q] = gE[pc];
      i[q] = gI[pc];
    }
    V = G(volt)[s % kVoltChunk];
  }
  __device__ __forceinline__ void stage(int64_t* nE, int64_t* nI, int ng) const {
#pragma unroll
    for (int q = 0; q < kRingRegs; ++q) {
      const int p = (int)threadIdx.x + q * NB;
      if (p < ng) {
        nE[p] = e[q];
        nI[p] = i[q];
      }
    }
    for (int p = (int)threadIdx.x + kRingRegs * NB; p < ng; p += NB) {
      nE[p] = gE[p];
      nI[p] = gI[p];
    }
  }
};

// The densities of a small case whose workgroup keeps them in LDS.
struct OwnNodes {
  static constexpr bool kOwn = true;
  int64_t *e, *i;
  double V;
};

// Steps 1-2 of step s, computed by every workgroup that needs E (each
// particle workgroup of a lockstep launch, the small-case workgroup): the
// densities of the deposit rings read at step s, rho, the potential and E on
// the nodes into sE (LDS); sF: ng doubles of LDS, zero on return.  The ring and V(t)
// pointers come with the workgroup's role.  The results depend only on the
// deposit, so every workgroup gets the same bits.  The writer (one workgroup
// per case and step) also does its duties and counts the step.
//
// Bound by latency, and in a launch that starts with cold caches by the
// fetching of its code: the two rings are staged through LDS in one round of
// coalesced loads, and the rows of a thread are worked in a loop, not
// unrolled to the largest grid with the writer's code in each copy (the
// electron kernel's code 64 -> 42 KB; a step of 1e3 electrons on 400 nodes
// 13.5 -> 12.4 us).
template <int MODE, int NB, class Nodes>
__device__ __forceinline__ void solve_field(CaseDev* __restrict__ Cw, const int ng, const int64_t s,
                                            const StepIndex& I, double* sE, double* sF, const bool writer,
                                            const Nodes& N, const SolveIn& S) {
  // the flux solve is always worked by the first 256 threads (its sums then
  // have the same order, and the same bits, whatever the workgroup)
  constexpr int NS = 256;
  static_assert(NB >= NS && NB % kWave == 0, "threads of the field solve");
  __shared__ double sWave[2][NS / kWave];
  const EDP_CONST CaseDev* __restrict__ C = KC(Cw);
  const bool ion_step = I.sub == 0;
  const int t = (int)threadIdx.x;
  const int lane = t % kWave, wv = __builtin_amdgcn_readfirstlane(t / kWave);
  // the rings, staged where E and the scratch go (or kept elsewhere)
  int64_t *nE, *nI;
  if constexpr (Nodes::kOwn) {
    nE = N.e;
    nI = N.i;
  } else {
    nE = (int64_t*)sF;
    nI = (int64_t*)sE;
    N.stage(nE, nI, ng);
  }
  const double V = N.V;
  const double scale = S.scale, kp = S.kpois, dx = S.dx;
  FieldWriter W;
  W.C = C;
  W.s3 = I.s3;
  W.k3 = I.k3;
  W.ng = ng;
  W.ion_step = ion_step;
  W.rings = !Nodes::kOwn;
  W.xt = writer && (C->flags & kDiagXT) != 0;
  W.plane = W.row = W.row_prev = 0;
  uint32_t bin = 0;
  if (W.xt) {
    const uint32_t nt = (uint32_t)C->nt, nxb = (uint32_t)C->n_xt_bin;
    const uint32_t tp = s < (int64_t)1 << 31 ? (uint32_t)s % nt : (uint32_t)(s % nt);  // step within the period
    bin = tp / nxb;
    W.plane = (size_t)C->n_xt * (size_t)ng;
    W.row = (size_t)bin * (size_t)ng;
    W.row_prev = (size_t)((tp == 0 ? nt - 1 : tp - 1) / nxb) * (size_t)ng;
  }
  // densities (the electrodes' half cells count twice) and rho of node p
  auto dens = [&](int p, double& ne, double& ni) {
    ne = (double)nE[p] * scale;
    ni = (double)nI[p] * scale;
    if (p == 0 || p == ng - 1) {
      ne *= 2.0;
      ni *= 2.0;
    }
    return kECharge * (ni - ne);
  };
  double ne, ni;
  if constexpr (Nodes::kOwn) {
    // the waves that do not solve take the writer's nodes meanwhile
    static_assert(NB > NS, "waves beside the solving ones");
#pragma unroll 1
    for (int p = t - NS; p < ng; p += NB - NS) {
      if (p < 0) break;
      const double rho = dens(p, ne, ni);
      W.node(p, ne, ni, rho);
    }
  } else {
    __syncthreads();
    if (writer) {
#pragma unroll 1
      for (int p = t; p < ng; p += NB) {
        const double rho = dens(p, ne, ni);
        W.node(p, ne, ni, rho);
      }
      __syncthreads();  // the staged ions are overwritten below
    }
  }
  if (MODE == 1) {
    // node p = t + q NB: rho and the right-hand side d_p = rho_p dx^2/eps0
#pragma unroll 1
    for (int p = t; p < ng; p += NB) {
      const double rho = dens(p, ne, ni);
      sE[p] = rho;
      sF[p] = rho * kp;
    }
    __syncthreads();
    const double rho0 = sE[0], rhoN = sE[ng - 1];
    if (t == 0) {
      // Thomas algorithm: forward sweep y_p = (d_p + y_{p-1}) r_p, back
      // substitution phi_p = y_p + r_p phi_{p+1}, with the reciprocals r_p
      // precomputed on the host
      const EDP_GLOBAL double* __restrict__ rd = G(C->rden);
      const int m = ng - 2;
      // (eight rows' reads in flight together, whichever kernel this is part of:
      // one row at a time waits 77 ns for each, so 27)
      double prev = 0.0;
#pragma unroll 8
      for (int p = 1; p <= m; ++p) {
        double d = sF[p];
        if (p == 1) d = d + V;
        prev = (d + prev) * rd[p];
        sF[p] = prev;
      }
#pragma unroll 8
      for (int p = m - 1; p >= 1; --p) sF[p] = sF[p] + rd[p] * sF[p + 1];
      sF[0] = V;
      sF[ng - 1] = 0.0;
    }
    __syncthreads();
#pragma unroll 1
    for (int p = t; p < ng; p += NB) {
      double e;
      if (p == 0)
        e = (sF[0] - sF[1]) / dx - rho0 * dx / (2.0 * kEps0);
      else if (p == ng - 1)
        e = (sF[ng - 2] - sF[ng - 1]) / dx + rhoN * dx / (2.0 * kEps0);
      else
        e = (sF[p - 1] - sF[p + 1]) / (2.0 * dx);
      sE[p] = e;
      if (writer) {
        G(C->phi)[p] = sF[p];
        if (W.xt) gl_sum(G(C->xt) + kXtFlux * W.plane + W.row + p, p < ng - 1 ? sF[p] - sF[p + 1] : V);
      }
    }
    __syncthreads();
    for (int p = t; p < ng; p += NB) sF[p] = 0.0;
  } else {
    // The flux form of the same tridiagonal system: with F_q = phi_q -
    // phi_{q+1}, row p of the Poisson equation says F_p - F_{p-1} = d_p, so
    // F_p = F_0 + S_p with S the prefix sum of d over the interior nodes; the
    // fluxes add up to phi_0 - phi_{N-1} = V, which fixes
    // F_0 = (V - sum_q S_q)/(N_g - 1), and sum_q S_q = sum_r (m - r) d_r over
    // the m = N_g - 2 interior rows.  Thread t owns the contiguous rows
    // q0 <= q < q0 + nq (row q is node q + 1): it forms its prefix (kept in
    // sE) and its share of the weighted sum, and one workgroup pass (wave
    // scans, one exchange of the wave totals) gives every thread the rows
    // before its own and the weighted total.  E of its nodes then follows:
    // E_p = (F_{p-1} + F_p)/(2 dx) inside, the boundary forms (Gauss's law
    // over the half cell) at the electrodes.
    const int m = ng - 2;
    const int R = (m + NS - 1) / NS;
    const int q0 = t * R;
    const bool solver = NB == NS || wv < NS / kWave;
    // the owner of the last row also takes node N_g-1 (thread 0 when there
    // are no interior rows)
    const bool last = q0 < m ? q0 + R >= m : (t == 0 && m == 0);
    // kGroup rows at a time, so that their LDS reads are in flight together
    constexpr int kGroup = 4;
    double inc = 0.0, rho0 = 0.0, rhoN = 0.0, acc = 0.0;
    if (solver) {
      rho0 = t == 0 ? dens(0, ne, ni) : 0.0;
      rhoN = last ? dens(ng - 1, ne, ni) : 0.0;
      double wsum = 0.0, weight = (double)(m - q0);
#pragma unroll 1
      for (int r0 = 0; r0 < R; r0 += kGroup) {
        int64_t ce[kGroup], ci[kGroup];
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
          const int p = q0 + 1 + r0 + r;
          const int pc = p < ng ? p : ng - 1;
          ce[r] = nE[pc];
          ci[r] = nI[pc];
        }
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
          if (r0 + r < R && q0 + r0 + r < m) {
            const double d = kECharge * ((double)ci[r] * scale - (double)ce[r] * scale) * kp;
            acc += d;
            wsum += d * weight;
            sE[q0 + 1 + r0 + r] = acc;  // prefix within the thread
          }
          weight -= 1.0;
        }
      }
      // the workgroup pass: inclusive scan of acc and sum of wsum per wave
      inc = acc;
      const int lane4 = lane * 4;
      auto permute = [&](int from4, double v) {
        const uint64_t u = (uint64_t)__double_as_longlong(v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(from4, (int)(uint32_t)u);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(from4, (int)(u >> 32));
        return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
      };
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        const int off = 1 << u, xo = kWave / 2 >> u;
        const double y = permute(lane4 + 4 * (kWave - off), inc);  // from lane - off
        const double z = permute(lane4 ^ (4 * xo), wsum);
        inc = lane >= off ? inc + y : inc;
        wsum += z;
      }
      if (lane == kWave - 1) {
        sWave[0][wv] = inc;
        sWave[1][wv] = wsum;
      }
    }
    __syncthreads();
    for (int p = t; p < ng; p += NB) sF[p] = 0.0;
    if (solver) {
      double before = inc - acc, sum_s = 0.0;
#pragma unroll
      for (int u = 0; u < NS / kWave; ++u) {
        if (u < wv) before += sWave[0][u];
        sum_s += sWave[1][u];
      }
      const double F0 = div_by(V - sum_s, (double)(ng - 1), S.inv_cells);
      double f_prev = F0 + before;  // F_{q0}: F0 plus the rows before this thread's
#pragma unroll 1
      for (int r0 = 0; r0 < R; r0 += kGroup) {
        double v[kGroup];
#pragma unroll
        for (int r = 0; r < kGroup; ++r) {
          const int p = q0 + 1 + r0 + r;
          v[r] = sE[p < ng ? p : ng - 1];
        }
#pragma unroll
        for (int r = 0; r < kGroup; ++r)
          if (r0 + r < R && q0 + r0 + r < m) {
            const int p = q0 + 1 + r0 + r;
            const double f = F0 + (before + v[r]);  // F_{q+1} = F_p
            sE[p] = div_by(f_prev + f, 2.0 * dx, S.inv_2dx);
            if (writer) W.flux(p, f);
            f_prev = f;
          }
      }
      if (t == 0) {
        sE[0] = div_by(F0, dx, S.inv_dx) - div_by(rho0 * dx, 2.0 * kEps0, 1.0 / (2.0 * kEps0));
        if (writer) W.flux(0, F0);
      }
      if (last) {
        sE[ng - 1] = div_by(f_prev, dx, S.inv_dx) + div_by(rhoN * dx, 2.0 * kEps0, 1.0 / (2.0 * kEps0));
        if (writer) W.flux(ng - 1, V);
      }
    }
  }
  if (writer && t == 0) {
    if (W.xt) {
      gl_add(C->xt_cnt + bin, 1);
      if (ion_step) gl_add(C->xt_cnt + C->n_xt + bin, 1);
    }
    Cw->phi_valid = MODE == 1;
    gl_add(&Cw->diag_steps, 1);
    if (ion_step) gl_add(&Cw->diag_ion_steps, 1);
  }
  __syncthreads();  // sE and the zeroed sF complete
  if (writer) {
#pragma unroll 1
    for (int p = t; p < ng; p += NB) W.field(p, sE[p]);
  }
}

// ---------------------------------------------------------------------------
// Collisions (step 6): the particle kernels test every particle, pick the
// process of those that collide (partition of [0,1) into sigma_k/sigma_tot),
// and apply it at once -- COM kinematics, scattering angles, Euler rotation,
// the ionization energy split and the newborns -- in dense passes over the
// colliders (see species_pass).
// ---------------------------------------------------------------------------

// Arrays the scattering code touches, loaded once per workgroup.
struct ScatterPtrs {
  EDP_GLOBAL double *ex, *evx, *evy, *evz, *ix, *ivx, *ivy, *ivz;
  EDP_GLOBAL float* evp2;
  EDP_GLOBAL uint64_t *euid, *iuid;
  int64_t* anomaly;
};

// The arrays of species sp's buffer set `cur`, read where they are needed
// (the other species' arrays, by the few workgroups with a newborn).
__device__ __forceinline__ void read_scatter_ptrs(ScatterPtrs& P, const EDP_CONST CaseDev* __restrict__ C, int sp, int cur) {
  const EDP_CONST SpeciesDev& S = C->sp[sp];
  if (sp == 0) {
    P.ex = G(S.x[cur]);
    P.evx = G(S.vx[cur]);
    P.evy = G(S.vy[cur]);
    P.evz = G(S.vz[cur]);
    P.evp2 = G(S.vp2[cur]);
    P.euid = G(S.uid[cur]);
  } else {
    P.ix = G(S.x[cur]);
    P.ivx = G(S.vx[cur]);
    P.ivy = G(S.vy[cur]);
    P.ivz = G(S.vz[cur]);
    P.iuid = G(S.uid[cur]);
  }
}

// Electron-Ar collisions, from the colliding electron's state after the push
// (velocity, identity; position for an ionization).  The post-collision
// velocity is w + f2 g' R(theta,phi)(cos chi, sin chi cos eta, sin chi sin
// eta) about the centre-of-mass velocity w, with the frame of g from its
// components and the azimuth eta = 2 pi R_eta; an ionization shares the
// energy above its threshold between the scattered and the ejected
// electron, which leaves at the azimuth eta + pi, and creates an ion with a
// thermal gas velocity.  The three parts are separate functions that
// recompute what they share from the same inputs (same operations, same
// bits), so that the scattering code after a particle loop keeps few values
// alive at once.

// The energy share of an ionization: the COM energy above the threshold
// [eV] (clamped at 0, counted as an anomaly) and the ejected electron's part
// e_ej = w tan(R atan(E/(2w))).
__device__ __forceinline__ void ionization_share(const EDP_CONST CaseDev* __restrict__ C, const ScatterPtrs& P,
                                                 double v2, uint64_t uid, uint32_t st, double& e_ev, double& e_ej) {
  double r_share, r_unused;
  uniform2(C->seed, uid, st, tag(0, 0, 2), r_share, r_unused);
  e_ev = 0.5 * kMuEAr * v2 / kEvToJ - C->thr_ion;
  if (e_ev < 0.0) e_ev = 0.0;
  const double w_ion = C->w_ion;
  e_ej = w_ion * tan(r_share * atan(e_ev / (2.0 * w_ion)));
}

// Scattering angle of one of the two electrons of an ionization from its
// energy e and the shared energy e_ev: cos chi = sqrt(e / e_ev) (or, with the
// literal reading, chi itself).
__device__ __forceinline__ void ionization_angle(const EDP_CONST CaseDev* __restrict__ C, double e, double e_ev,
                                                 double& cs, double& sn) {
  if (C->flags & kIonizLiteral) {
    const double chi = e_ev > 0.0 ? sqrt(e / e_ev) : 0.0;
    sincos(chi, &sn, &cs);
  } else {
    cs = e_ev > 0.0 ? sqrt(e / e_ev) : 1.0;
    sn = sqrt(1.0 - cs * cs);
  }
}

// An outgoing electron of a collision: the colliding electron itself
// (process proc: 0 elastic, 1 excitation, 2 ionization) or, with `eject`,
// the electron its ionization ejects (proc 2), from the parent's pushed
// velocity and identity, with the draws r_chi and r_eta of the parent's
// counter.  Both take the frame of g; the ejected one leaves with the other share of the
// energy at the azimuth eta + pi.  Returns the new velocity.
__device__ __forceinline__ void electron_outgoing(const EDP_CONST CaseDev* __restrict__ C, const ScatterPtrs& P,
                                                  bool eject, int proc, int64_t s, double vxn, double vy,
                                                  double vz, uint64_t uid, double r_chi, double r_eta, double& ox,
                                                  double& oy, double& oz) {
  const uint32_t st = (uint32_t)s;
  // squared speed, the squares summed from x to z as the collision test does
  const double v2 = vxn * vxn + vy * vy + vz * vz;
  const double v = sqrt(v2);
  double gnew = v, cos_chi, sin_chi;
  if (proc < 2) {
    if (proc == 1) {
      double ec = 0.5 * kMuEAr * v2 - C->thr_exc * kEvToJ;
      if (ec < 0.0) {
        ec = 0.0;
        gl_add(P.anomaly, 1);
      }
      gnew = sqrt(2.0 * ec / kMuEAr);
    }
    cos_chi = 1.0 - 2.0 * r_chi;
    sin_chi = sqrt(1.0 - cos_chi * cos_chi);
  } else {
    double e_ev, e_ej;
    ionization_share(C, P, v2, uid, st, e_ev, e_ej);
    if (!eject && 0.5 * kMuEAr * v2 / kEvToJ - C->thr_ion < 0.0) gl_add(P.anomaly, 1);
    const double e_out = eject ? e_ej : e_ev - e_ej;
    gnew = sqrt(2.0 * e_out * kEvToJ / kMuEAr);
    ionization_angle(C, e_out, e_ev, cos_chi, sin_chi);
  }
  const double f1 = kEMass / (kEMass + kArMass);
  const double f2 = kArMass / (kEMass + kArMass);
  const Frame F = frame_of(vxn, vy, vz, v);
  double cos_eta, sin_eta;
  const double eta = kTwoPi * r_eta;
  sincos(eject ? eta + kPi : eta, &sin_eta, &cos_eta);
  rotate(F, gnew, f2, cos_chi, sin_chi, cos_eta, sin_eta, f1 * vxn, f1 * vy, f1 * vz, ox, oy, oz);
}

// Stores of an electron's velocity (and the float bound of vy^2 + vz^2).
__device__ __forceinline__ void store_electron_v(const ScatterPtrs& P, int64_t i, double ox, double oy, double oz) {
  P.evx[i] = ox;
  P.evy[i] = oy;
  P.evz[i] = oz;
  P.evp2[i] = float_above(oy * oy + oz * oz);
}

// The ion an ionization creates, at slot bi at the parent's position: a
// thermal gas velocity from the newborn's own counter.
__device__ __forceinline__ void ion_birth_at(const EDP_CONST CaseDev* __restrict__ C, const ScatterPtrs& P,
                                             int64_t bi, int64_t s, uint64_t uid, double x) {
  const uint64_t cu = child_uid(uid, s, 2);
  double z0, z1, z2;
  normals3(C->seed, cu, (uint32_t)s, 1u, 2u, 1u, z0, z1, z2);
  const double sa = C->sigma_a;
  P.ix[bi] = x;
  P.ivx[bi] = sa * z0;
  P.ivy[bi] = sa * z1;
  P.ivz[bi] = sa * z2;
  P.iuid[bi] = cu;
}

// Ar+ + Ar scattering of colliding ion i (proc 0 isotropic, 1 backward) with the
// thermal target of its test (redrawn from the same counter: the same atom).
__device__ __forceinline__ void ion_scatter_at(const EDP_CONST CaseDev* __restrict__ C, const ScatterPtrs& P, int64_t i,
                                               int proc, int64_t s, double vxn, double vy, double vz, uint64_t uid) {
  const uint64_t seed = C->seed;
  const uint32_t st = (uint32_t)s;
  double z0, z1, z2;
  normals3(seed, uid, st, 1u, 0u, 0u, z0, z1, z2);
  const double sa = C->sigma_a;
  const double vax = sa * z0, vay = sa * z1, vaz = sa * z2;
  const double gx = vxn - vax, gy = vy - vay, gz = vz - vaz;
  const double g = sqrt(gx * gx + gy * gy + gz * gz);
  double r_chi, r_eta;
  uniform2(seed, uid, st, tag(1, 0, 3), r_chi, r_eta);
  const double wx = 0.5 * (vxn + vax), wy = 0.5 * (vy + vay), wz = 0.5 * (vz + vaz);
  double cos_chi, sin_chi;
  if (proc == 0) {
    cos_chi = 1.0 - 2.0 * r_chi;
    sin_chi = sqrt(1.0 - cos_chi * cos_chi);
  } else {
    cos_chi = -1.0;
    sin_chi = 0.0;
  }
  double ox, oy, oz;
  scatter(gx, gy, gz, g, g, 0.5, cos_chi, sin_chi, kTwoPi * r_eta, wx, wy, wz, ox, oy, oz);
  P.ivx[i] = ox;
  P.ivy[i] = oy;
  P.ivz[i] = oz;
}
// Secondary electron of ion i, absorbed at electrode `side` (0 at
// x = 0, 1 at x = L): it starts on the surface with the velocity of a thermal
// flux at T_see -- a Rayleigh normal component into the gap and two normal
// tangential ones (Box-Muller) -- from purpose 3 of the ion's counter; its
// identity is the ion's child of kind 3.  be < 0: dropped at capacity.
__device__ __forceinline__ void see_emit_at(const EDP_CONST CaseDev* __restrict__ C, const ScatterPtrs& P,
                                            uint64_t uid, int side, int64_t be, int64_t s) {
  if (be < 0) return;
  const uint32_t st = (uint32_t)s;
  double a0, a1, b0, b1;
  uniform2(C->seed, uid, st, tag(1, 3, 1), a0, a1);
  uniform2(C->seed, uid, st, tag(1, 3, 2), b0, b1);
  const double sig = C->see_sigma;
  const double vn = sig * sqrt(-2.0 * log(1.0 - a0));
  const double vt = sig * sqrt(-2.0 * log(1.0 - a1));
  P.ex[be] = side == 0 ? 0.0 : C->L;
  P.evx[be] = side == 0 ? vn : -vn;
  double sn, cs;
  sincos(kTwoPi * b0, &sn, &cs);
  const double vy = vt * cs, vz = vt * sn;
  P.evy[be] = vy;
  P.evz[be] = vz;
  P.evp2[be] = float_above(vy * vy + vz * vz);
  P.euid[be] = child_uid(uid, s, 3);
}
// ---------------------------------------------------------------------------
// Steps 3-6 for one species plus the deposit for step s+1.
//
// A case's particle slots are cut into chunks of NB slots (the workgroup
// size).  In the lockstep kernels a case gets a fixed number of workgroups
// (its share, by expected particle count, of the resident slots the batch
// uses); each takes a contiguous range of the step's chunks by the share
// its role gives it (the later a workgroup is dispatched, the smaller its
// share, when the host weights them so), so the launch shape never depends
// on the count.  The small-case kernel runs every chunk of its case
// in one workgroup.  Inside a workgroup the range is worked in slices of 64
// slots, one per lane: wave w takes slices w, w + W, w + 2W, ... of its
// workgroup's W waves.
//
// Every particle: gather E from LDS, leapfrog, wall test, deposit the new x
// into the workgroup's LDS histogram, store x and v_x, and one Philox call
// for its collision uniform R.  Only R below a bound of the collision
// probability over the tables (the null-collision P*, with a relative
// margin for the direct test), or a speed beyond the range that bound
// covers, can give a collision; such candidates (a few percent) go to the
// wave's LDS segment and everyone else is done.  The candidates get the
// exact test -- energy bin, table lookups, exp, for ions the thermal target
// first -- and the colliders their scattering, in dense passes after the
// loop: each wave its own segment, then the workgroup's overflow list (the
// segments that filled during the loop), 64 entries per pass from an LDS
// counter.  So the table work and the transcendentals run on full waves
// instead of on every wave with one candidate lane.  An ionization takes
// slots for its newborns from the step's birth counters, writes them, and
// adds their charge (the electron a second share at the parent's x, the ion
// to the next ion step's density).
//
// Dynamic LDS: E[ng] double, then the region of H[ng] deposit (also the field
// solve's scratch); with particle diagnostics also J[ng], W[ng], En[ng]
// (int64) and EEPF[n_eepf] (uint32).  Static: the candidate segments (ions
// 4 KiB of slots; electrons 10 KiB of slots, v^2 and uids) and a few
// counters.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_rank(uint64_t mask) {
  // set bits of mask below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Candidate segment entries per wave: ions keep the slot only (their exact
// test reloads the state); electrons keep the slot, the pushed v_x and the
// uid, so that their exact test reads only v_y and v_z back.
constexpr int kSegI = 256;
constexpr int kSegE = 128;
template <int SP>
constexpr int seg_len() { return SP == 0 ? kSegE : kSegI; }

// Birth slots of one step: a species' newborns take consecutive slots after
// its slot count at the step's start, from a counter of the step's births
// (LDS in the small-case kernel, born[sp][s % 3] in global memory in the
// lockstep kernels); a slot at or beyond the capacity drops the birth.
template <bool SMALL>
struct Births {
  int64_t base[2], cap[2];
  int* lds;           // SMALL: this step's counters per species
  int64_t* glob[2];   // lockstep: this step's counters per species
  // Slot of this lane's newborn of species sp (mine), -1 if none or dropped;
  // every lane of the wave calls it.  placed / dropped count the wave's.
  __device__ __forceinline__ int64_t take(int sp, bool mine, int lane, int& placed, int& dropped) const {
    const uint64_t m = ballot(mine);
    if (m == 0) return -1;
    long long b = 0;
    if (lane == 0) {
      const int c = (int)__popcll(m);
      if (SMALL)
        b = atomicAdd(&lds[sp], c);
      else
        b = (long long)gl_fetch_add(glob[sp], (unsigned long long)c);
    }
    b = __shfl(b, 0);
    const int64_t slot = base[sp] + (int64_t)b + lane_rank(m);
    const bool ok = slot < cap[sp];
    placed += (int)__popcll(ballot(mine && ok));
    dropped += (int)__popcll(ballot(mine && !ok));
    return mine && ok ? slot : -1;
  }
  // Slots of the newborn pairs (an electron and an ion) of the wave's `cnt`
  // ionizations: issue() takes them from both counters (lane 0; the
  // atomics go out together and their values are needed only by
  // first_slots()), newborn r of the wave then has slot first + r.
  __device__ __forceinline__ void issue_pair(int cnt, int lane, long long& a_e, long long& a_i) const {
    a_e = a_i = 0;
    if (lane == 0) {
      if (SMALL) {
        a_e = atomicAdd(&lds[0], cnt);
        a_i = atomicAdd(&lds[1], cnt);
      } else {
        a_e = (long long)gl_fetch_add(glob[0], (unsigned long long)cnt);
        a_i = (long long)gl_fetch_add(glob[1], (unsigned long long)cnt);
      }
    }
  }
  __device__ __forceinline__ void first_slots(long long a_e, long long a_i, int64_t& f_e, int64_t& f_i) const {
    f_e = base[0] + (int64_t)__shfl(a_e, 0);
    f_i = base[1] + (int64_t)__shfl(a_i, 0);
  }
};

// Every line of the case block is asked for at a launch's start, where the
// scalar cache is cold: what a later phase reads is then there, instead of a
// wait of about 500 cycles at the first touch of each line.
__device__ __forceinline__ void touch_case(const EDP_CONST CaseDev* C) {
  constexpr int kLines = (int)((sizeof(CaseDev) + 63) / 64);
  static_assert(kLines <= 20, "lines of the case block");
  uint32_t d[20];
#pragma unroll
  for (int k = 0; k < 20; ++k) d[k] = ((const EDP_CONST uint32_t*)C)[16 * (k < kLines ? k : 0)];
  asm volatile("" ::"s"(d[0]), "s"(d[1]), "s"(d[2]), "s"(d[3]), "s"(d[4]), "s"(d[5]), "s"(d[6]), "s"(d[7]), "s"(d[8]),
               "s"(d[9]), "s"(d[10]), "s"(d[11]), "s"(d[12]), "s"(d[13]), "s"(d[14]), "s"(d[15]), "s"(d[16]), "s"(d[17]),
               "s"(d[18]), "s"(d[19]));
}

// What a pass over a species needs before its loop, read in one go: left
// where they are used, the reads are a dozen scalar loads one after another,
// each a wait of a few hundred cycles (more in a launch, whose caches start
// cold).  Both buffer sets' pointers are read, so that no read waits for the
// index of the current one.
template <int SP>
struct PassIn {
  double *x[2], *vx[2], *vy[2], *vz[2];
  uint64_t* uid[2];
  float* vp2[2];
  const uint32_t* pbound;
  int64_t *cnt_e, *cnt_i;
  double inv_dx, L, dt, kick, p_cand, v2_cand, blocks_per_v2, block_half, block_last;
  uint64_t seed;
  uint32_t flags, r_cand;
  int pb_n, surf_on;
  __device__ __forceinline__ explicit PassIn(const EDP_CONST CaseDev* C) {
    const EDP_CONST SpeciesDev& S = C->sp[SP];
    for (int c = 0; c < 2; ++c) {
      x[c] = S.x[c];
      vx[c] = S.vx[c];
      vy[c] = S.vy[c];
      vz[c] = S.vz[c];
      uid[c] = S.uid[c];
      vp2[c] = S.vp2[c];
    }
    pbound = C->pbound[SP];
    cnt_e = C->cnt_e;
    cnt_i = C->cnt_i;
    inv_dx = C->inv_dx;
    L = C->L;
    dt = SP == 0 ? C->dt_e : C->dt_i;
    kick = SP == 0 ? C->factor_e : C->factor_i;
    p_cand = C->p_cand[SP];
    v2_cand = C->v2_cand[SP];
    blocks_per_v2 = C->blocks_per_v2[SP];
    block_half = C->block_half;
    block_last = C->block_last;
    r_cand = C->r_cand[SP];
    seed = C->seed;
    flags = C->flags;
    pb_n = C->pb_n;
    surf_on = SP == 0 ? C->refl_on : C->see_on;
    // one point that needs them all
    asm volatile(""
                 : "+s"(x[0]), "+s"(x[1]), "+s"(vx[0]), "+s"(vx[1]), "+s"(vy[0]), "+s"(vy[1]), "+s"(vz[0]), "+s"(vz[1]),
                   "+s"(uid[0]), "+s"(uid[1]), "+s"(vp2[0]), "+s"(vp2[1]), "+s"(pbound), "+s"(inv_dx), "+s"(L), "+s"(dt),
                   "+s"(kick), "+s"(p_cand), "+s"(v2_cand), "+s"(blocks_per_v2), "+s"(seed), "+s"(flags), "+s"(r_cand),
                   "+s"(block_half), "+s"(block_last), "+s"(pb_n), "+s"(surf_on), "+s"(cnt_e), "+s"(cnt_i));
  }
};

// A wave's totals of one species' step (kRec fields): field f in lane f.
struct SpTot {
  int field;
};

// Steps 3-6 of species SP at step s over chunks [c_lo, c_hi) of slots [0, n)
// of buffer set `cur` (the other species' current set `cur_o`), E in sE,
// `reg` the LDS region for the deposit histogram (and the particle
// diagnostics), B the step's birth counters.  `solve` fills sE (and leaves
// the histogram zero) and ends with a barrier; it runs after the pass has
// read its constants and sent the loads of its first slice on their way, so
// that neither is waited for again: a launch starts with cold caches, and
// with the constants read where they are used the loop began a dozen
// dependent scalar loads after the solve.
template <int SP, bool SMALL, int NB, class Solve>
__device__ __forceinline__ SpTot species_pass(CaseDev* __restrict__ Cw, const double* sE, double* reg,
                                              const int64_t s, const StepIndex& I, const int64_t n, const int64_t c_lo,
                                              const int64_t c_hi, const int cur, const int cur_o,
                                              const Births<SMALL>& B, const int pretest, const PassIn<SP>& A,
                                              const Solve& solve, unsigned long long* own_e = nullptr,
                                              unsigned long long* own_i = nullptr) {
  const EDP_CONST CaseDev* __restrict__ C = KC(Cw);
  constexpr int kSeg = seg_len<SP>();
  // a small case's workgroup that keeps the deposits in LDS (own_e, own_i:
  // of the next step and of the next ion step)
  constexpr bool OWN = SMALL && NB > kBlock;
  constexpr bool ZEROED = !(SMALL && SP == 1);  // the solve left the histogram zero
  constexpr int kPay = SP == 0 ? NB / kWave : 1;
  __shared__ int32_t sSeg[NB / kWave][kSeg];
  __shared__ double sVx[kPay][SP == 0 ? kSeg : 1];
  __shared__ uint64_t sUid[kPay][SP == 0 ? kSeg : 1];
  // entries of the overflow list, next pass over it
  __shared__ int sOvf, sFin;
  // the pre-test's bound of P by energy block (direct collision test), as
  // candidate_limit gives it
  __shared__ uint32_t sPB[kMaxPb];
  // lanes of a pass's ionizing colliders by rank (electrons)
  __shared__ int sIon[SP == 0 ? NB / kWave : 1][SP == 0 ? kWave : 1];
  const int ng = C->ng;
  const uint32_t fl = A.flags;
  const bool pdiag = (fl & kDiagParticle) != 0;
  const bool xt = (fl & kDiagXT) != 0;
  const int n_eepf = C->n_eepf;
  const int n_ifed = C->n_ifed;
  // histogram: the EEPF for electrons, the IFEDF of both electrodes for ions
  const int n_hist = SP == 0 ? ((fl & kDiagEepf) ? n_eepf : 0) : ((fl & kDiagIfed) ? 2 * (n_ifed + 1) : 0);
  unsigned long long* sH = OWN ? (SP == 0 ? own_e : own_i) : (unsigned long long*)reg;
  unsigned long long* sJ = (unsigned long long*)reg + (OWN ? 0 : ng);
  unsigned long long* sW = sJ + ng;
  unsigned long long* sEn = sW + ng;
  unsigned long long* sIz = sEn + ng;  // electrons with the xt arrays only
  unsigned int* sF = (unsigned int*)(sIz + (SP == 0 && xt ? ng : 0));
  if (pdiag || (!ZEROED && !OWN)) {
    for (int p = threadIdx.x; p < ng; p += NB) {
      if (!ZEROED && !OWN) sH[p] = 0;
      if (!pdiag) continue;
      sJ[p] = 0;
      sW[p] = 0;
      sEn[p] = 0;
      if (SP == 0 && xt) sIz[p] = 0;
    }
  }
  for (int b = threadIdx.x; b < n_hist; b += NB) sF[b] = 0;
  constexpr int kWaves = NB / kWave;
  // candidate pre-test: R below a bound of P, or a speed beyond the bound's
  // range.  The direct test's bound is P* (with its margin), or, when a
  // wave's slots would give enough candidates by it, the
  // bound by energy: the block of the table row of an upper bound of the
  // particle's (relative) energy -- from g2u, a bound of its squared speed,
  // times (1 + 1e-12) against the rounding of the exact test's own v^2 and
  // energy -- in sPB.  The lookup costs every particle a few instructions
  // and an LDS load, so it is taken when P* would give a wave more than a
  // quarter round of candidates (measured: 2% slower on the large case with
  // 8 per wave, 4-12% faster on the batched sets with 20-400).
  const bool null_coll = (fl & kNullCollision) != 0;
  const double p_cand = A.p_cand;
  const bool by_energy =
      !null_coll && (pretest == 2 || (pretest == 0 && (double)(c_hi - c_lo) * kWave * p_cand > (double)(kWave / 4)));
  if (by_energy) {
    const int pb_n = A.pb_n;
    const EDP_GLOBAL uint32_t* __restrict__ pbg = G(A.pbound);
    for (int b = threadIdx.x; b < pb_n; b += blockDim.x) sPB[b] = pbg[b];
  }
  if (threadIdx.x == 0) {
    sOvf = 0;
    sFin = 0;
  }
  EDP_GLOBAL double* X = G(cur ? A.x[1] : A.x[0]);
  // this workgroup's overflow list of candidates: its chunk range of the
  // species' list (as many entries as the range has slots)
  EDP_GLOBAL int64_t* __restrict__ CL = G(C->clist[SP]) + c_lo * NB;
  EDP_GLOBAL double* VX = G(cur ? A.vx[1] : A.vx[0]);
  EDP_GLOBAL double* VY = G(cur ? A.vy[1] : A.vy[0]);
  EDP_GLOBAL double* VZ = G(cur ? A.vz[1] : A.vz[0]);
  EDP_GLOBAL uint64_t* UID = G(cur ? A.uid[1] : A.uid[0]);
  // electrons: a float bound of vy*vy + vz*vz per slot, read in place of vy
  // and vz for the pre-test (those only by the candidates' exact test and the
  // measurement sums)
  EDP_GLOBAL float* VP2 = G(cur ? A.vp2[1] : A.vp2[0]);
  ScatterPtrs P;
  P.anomaly = &Cw->ctr[kAnomaly];
  if (SP == 0) {
    P.ex = X;
    P.evx = VX;
    P.evy = VY;
    P.evz = VZ;
    P.evp2 = VP2;
    P.euid = UID;
  } else {
    P.ix = X;
    P.ivx = VX;
    P.ivy = VY;
    P.ivz = VZ;
    P.iuid = UID;
  }
  // the loop's constants, in vector registers (the scalar ones are short)
  const double inv_dx = pin_v(A.inv_dx), L_gap = pin_v(A.L), dt = pin_v(A.dt), kick = pin_v(A.kick);
  const EDP_GLOBAL double* __restrict__ nsig = G(SP == 0 ? C->nsig_e : C->nsig_i);
  const EDP_GLOBAL double* __restrict__ sig0 = G(SP == 0 ? C->sig_el : C->sig_iso);
  const EDP_GLOBAL double* __restrict__ sig1 = G(SP == 0 ? C->sig_exc : C->sig_back);
  const EDP_GLOBAL double* __restrict__ sig2 = G(C->sig_ion);
  // the deposits of the next step and of the next ion step
  int64_t* const cnt_e_next = A.cnt_e + (I.s3 == 2 ? 0 : I.s3 + 1) * ng;
  int64_t* const cnt_i_next = A.cnt_i + (I.k3 == 2 ? 0 : I.k3 + 1) * ng;
  int64_t* const dst = SP == 0 ? cnt_e_next : cnt_i_next;
  const double de_cs = C->de_cs, inv_de_cs = C->inv_de_cs;
  const int nbins = C->nbins;
  const uint64_t seed = A.seed;
  const uint32_t st = (uint32_t)s;
  const double x_lo = C->x_lo, x_hi = C->x_hi, de_eepf = C->de_eepf, de_ifed = C->de_ifed;
  const double sa = C->sigma_a;
  // surface processes of this species' electrode hits
  const bool surf_on = A.surf_on != 0;
  const double p_surf0 = SP == 0 ? C->eta_refl[0] : C->gamma_see[0];
  const double p_surf1 = SP == 0 ? C->eta_refl[1] : C->gamma_see[1];
  const double n_gas = C->n_gas;
  const double nu_star = SP == 0 ? C->nu_star_e : C->nu_star_i;
  const uint32_t r_cand = A.r_cand;
  const double v2_cand = pin_v(A.v2_cand);
  const double blocks_per_g2 = A.blocks_per_v2, block_half = A.block_half, block_last = A.block_last;
  const double a2_i = C->a2_i;
  const uint32_t r_tag = SP == 0 ? tag(0, 0, 0) : tag(1, 0, 2);
  // the wave's index in a scalar register: what depends on it (the slices, the
  // loop, the addresses' bases, the segment) then is scalar too
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = (int)threadIdx.x % kWave;
  // this wave's totals (uniform over the wave)
  int t_coll = 0, t_ioniz = 0, t_pow = 0, t_gnd = 0, t_live = 0, t_be = 0, t_bi = 0, t_drop = 0;
  int ncw = 0;  // entries in this wave's candidate segment

  // Step 6 for candidates.  exact_test: the exact test of one candidate
  // (direct: P = 1 - exp(-n sigma_tot g dt), collide iff R < P, process by
  // sigma_k / sigma_tot; null collision: process by R nu* against the
  // cumulative nu_k, the rest null) from its pushed v_x, v_y, v_z and uid;
  // returns the process or -1.  The table entries are asked for before the
  // random numbers are formed, so that those (for electrons also the
  // scattering angles' r_chi and r_eta) are formed while they come.
  auto exact_test = [&](const double vxn, const double vy, const double vz, const uint64_t uid, double& r_chi,
                        double& r_eta) -> int {
    double g2, energy;
    if (SP == 0) {
      // squared speed summed from x to z (Algorithm 6)
      g2 = vxn * vxn + vy * vy + vz * vz;
      energy = div_by(0.5 * kEMass * g2, kEvToJ, 1.0 / kEvToJ);
    } else {
      double z0, z1, z2;
      normals3(seed, uid, st, 1u, 0u, 0u, z0, z1, z2);
      const double gx = vxn - sa * z0, gy = vy - sa * z1, gz = vz - sa * z2;
      g2 = gx * gx + gy * gy + gz * gz;
      energy = div_by(0.5 * kMuArAr * g2, kEvToJ, 1.0 / kEvToJ);
    }
    // a valid row whatever the outcome
    const int idx = energy_bin(energy, de_cs, inv_de_cs, nbins);
    const double s_a = sig0[idx], s_b = sig1[idx], s_c = SP == 0 ? sig2[idx] : 0.0, s_n = nsig[idx];
    double r_coll, r_proc;
    uniform2(seed, uid, st, r_tag, r_coll, r_proc);
    if (SP == 0) uniform2(seed, uid, st, tag(0, 0, 1), r_chi, r_eta);
    const double g = sqrt(g2);
    if (null_coll) {
      const double c1 = (n_gas * s_a) * g;
      const double c2 = c1 + (n_gas * s_b) * g;
      const double c3 = SP == 0 ? c2 + (n_gas * s_c) * g : c2;
      // the loop's test lets R up to 2^-32 above P* through
      if (!(r_coll < p_cand)) return -1;
      if (c3 > nu_star) gl_add(&Cw->ctr[kAnomaly], 1);
      const double t = r_proc * nu_star;
      return t < c1 ? 0 : (t < c2 ? 1 : (SP == 0 && t < c3 ? 2 : -1));
    }
    const double nu = s_n * g;
    const double p_coll = 1.0 - exp(-nu * dt);
    if (!(r_coll < p_coll)) return -1;
    if (SP == 0) {
      const double s_tot = s_a + s_b + s_c;
      if (!(s_tot > 0.0) || r_proc < s_a / s_tot) return 0;
      return r_proc < (s_a + s_b) / s_tot ? 1 : 2;
    }
    return (!(s_a + s_b > 0.0) || r_proc < s_a / (s_a + s_b)) ? 0 : 1;
  };

  // A wave's full segment inside the streaming loop goes to the
  // workgroup's overflow list (entries taken from an LDS counter; the
  // workgroup's candidates are at most its slots) and is tested after the
  // loop: the loop holds no table or transcendental code, so it keeps few
  // registers.
  auto spill_segment = [&](const int count) {
    int off = 0;
    if (lane == 0) off = atomicAdd(&sOvf, count);
    off = __builtin_amdgcn_readfirstlane(__shfl(off, 0));
    for (int k = lane; k < count; k += kWave) CL[off + k] = sSeg[w][k];
  };

  // After the loop, in rounds of 64 entries: each
  // wave what is left in its segment, then rounds of the workgroup's
  // overflow list (state reloaded) from an LDS counter, until none is left.
  // Each round runs the exact test, moves the round's
  // colliders with their state to the low lanes (one push permutation), and
  // gives each its scattering; an ionization also gets its newborns (slots
  // from the step's counters, charge at the parent's new position: the
  // electron a second share of this step's deposit, the ion the next ion
  // step's density).  No workgroup barrier: waves finish at their own pace.
  // An entry of the wave's segment with what its exact test needs (v_y and v_z
  // are not changed by the push).
  struct Entry {
    int64_t i;
    double vxn, vy, vz;
    uint64_t uid;
  };
  auto own_entry = [&](const int k) {
    Entry c{};
    if (k >= ncw) return c;
    c.i = sSeg[w][k];
    c.vy = VY[c.i];
    c.vz = VZ[c.i];
    if (SP == 0) {
      // the pushed v_x and the uid from the segment
      c.vxn = sVx[SP == 0 ? w : 0][SP == 0 ? k : 0];
      c.uid = sUid[SP == 0 ? w : 0][SP == 0 ? k : 0];
    } else {
      c.vxn = VX[c.i];
      c.uid = UID[c.i];
    }
    return c;
  };
  auto finish = [&](const Entry& first) {
    const int npool = sOvf;  // written before the barrier after the loop
    const int own = (ncw + kWave - 1) / kWave;
#pragma unroll 1
    for (int round = 0;; ++round) {
      Entry c = first;
      bool have = lane < ncw;
      if (round > 0 || own == 0) {
        c = Entry{};
        if (round < own) {
          have = round * kWave + lane < ncw;
          c = own_entry(round * kWave + lane);
        } else {
          int g = 0;
          if (lane == 0) g = atomicAdd(&sFin, 1);
          const int b0 = __builtin_amdgcn_readfirstlane(g) * kWave;
          if (b0 >= npool) break;
          have = b0 + lane < npool;
          if (have) {
            c.i = CL[b0 + lane];
            c.vxn = VX[c.i];
            c.uid = UID[c.i];
            c.vy = VY[c.i];
            c.vz = VZ[c.i];
          }
        }
      }
      const int64_t i = c.i;
      const double vxn = c.vxn, vy = c.vy, vz = c.vz;
      const uint64_t uid = c.uid;
      double r_chi = 0.0, r_eta = 0.0;
      const int proc = have ? exact_test(vxn, vy, vz, uid, r_chi, r_eta) : -1;
      const bool hit = proc >= 0;
      const uint64_t mc = ballot(hit);
      const int ncol = (int)__popcll(mc);
      t_coll += ncol;
      if (ncol == 0) continue;
      if (SP == 1) {
        if (hit) ion_scatter_at(C, P, i, proc, s, vxn, vy, vz, uid);
        continue;
      }
      // The colliders' outgoing electrons and the electrons their ionizations
      // eject, the latter on the lanes without a collider, in rank order
      // (more passes if they do not fit); the new ions on their parents'
      // lanes after that.  The parent's new position and the newborns' slots
      // are loaded and taken first and used only at the stores.  One copy of
      // the scattering code for rounds with and without ionizations: its
      // fetching is a good part of its time.
      const bool ioniz = proc == 2;
      const uint64_t mi = ballot(ioniz);
      const int ni = (int)__popcll(mi);
      const int ri = lane_rank(mi);
      double xb = 0.0;
      long long a_e = 0, a_i = 0;
      if (ni) {
        t_ioniz += ni;
        read_scatter_ptrs(P, C, 1, cur_o);
        if (ioniz) {
          xb = X[i];
          sIon[SP == 0 ? w : 0][SP == 0 ? ri : 0] = lane;
        }
        B.issue_pair(ni, lane, a_e, a_i);
      }
      int64_t f_e = 0, f_i = 0;
#pragma unroll 1
      for (int e0 = 0, pass = 0; pass == 0 || e0 < ni; ++pass) {
        // the ejected electron of this lane, by rank
        const int e = pass == 0 ? lane_rank(~mc) : e0 + lane;
        const bool ej = (pass > 0 || !hit) && e < ni;
        const bool par = pass == 0 && hit;
        int src = lane;
        double tvx = vxn, tvy = vy, tvz = vz, t_eta = r_eta;
        uint64_t tuid = uid;
        if (ni) {
          if (ej) src = sIon[SP == 0 ? w : 0][SP == 0 ? e : 0];
          tvx = __shfl(vxn, src);
          tvy = __shfl(vy, src);
          tvz = __shfl(vz, src);
          t_eta = __shfl(r_eta, src);
          tuid = (uint64_t)__shfl((long long)uid, src);
        }
        double ox = 0.0, oy = 0.0, oz = 0.0;
        if (par || ej) electron_outgoing(C, P, ej, ej ? 2 : proc, s, tvx, tvy, tvz, tuid, r_chi, t_eta, ox, oy, oz);
        if (par) store_electron_v(P, i, ox, oy, oz);
        if (ni) {
          if (pass == 0) B.first_slots(a_e, a_i, f_e, f_i);
          const double tx = __shfl(xb, src);
          const int64_t be = f_e + e;
          if (ej && be < B.cap[0]) {
            P.ex[be] = tx;
            store_electron_v(P, be, ox, oy, oz);
            P.euid[be] = child_uid(tuid, s, 1);
          }
        }
        e0 += pass == 0 ? kWave - ncol : kWave;
      }
      if (ni) {
        const bool ok_e = f_e + ri < B.cap[0], ok_i = f_i + ri < B.cap[1];
        t_be += (int)__popcll(ballot(ioniz && ok_e));
        t_bi += (int)__popcll(ballot(ioniz && ok_i));
        t_drop += (int)__popcll(ballot(ioniz && !ok_e)) + (int)__popcll(ballot(ioniz && !ok_i));
        if (ioniz) {
          long long r;
          const int q = deposit_split(xb, inv_dx, ng, r);
          if constexpr (OWN) {
            lds_add(&own_e[q], 4294967296LL - r);
            lds_add(&own_e[q + 1], r);
            lds_add(&own_i[q], 4294967296LL - r);
            lds_add(&own_i[q + 1], r);
          } else {
            gl_add(&dst[q], 4294967296LL - r);
            gl_add(&dst[q + 1], r);
            gl_add(&cnt_i_next[q], 4294967296LL - r);
            gl_add(&cnt_i_next[q + 1], r);
          }
          if (ok_i) ion_birth_at(C, P, f_i + ri, s, uid, xb);
        }
      }
    }
  };

  // The streaming loop.  The state of a wave's next slice is loaded before its
  // current one is worked on.  A slice's loads and its two stores are
  // unconditional, whatever its particles do: the wave's memory counter
  // counts both in order, and only a fixed number of stores behind the loads
  // lets the next slice wait for its loads without waiting for this one's
  // stores.
  const int q_lo = (int)(c_lo * kWaves);
  const int q_end = (int)((n + kWave - 1) / kWave);
  const int q_hi = (int)(c_hi * kWaves < q_end ? c_hi * kWaves : q_end);
  struct Slice {
    double x, vx, vy, vz;
    float vp2;
    uint64_t uid;
  };
  // the slots up to the next multiple of 64 are within the capacity (and a
  // wave without a slice loads the first one, unused)
  auto fetch = [&](Slice& a, const int q) {
    const int64_t i0 = (int64_t)q * kWave;
    a.x = (X + i0)[lane];
    a.vx = (VX + i0)[lane];
    if (SP == 0) a.vp2 = (VP2 + i0)[lane];
    a.uid = (UID + i0)[lane];
    if (SP == 1) {
      a.vy = (VY + i0)[lane];
      a.vz = (VZ + i0)[lane];
    }
  };
  auto fetch_vyz = [&](Slice& a, const int q) {
    const int64_t i0 = (int64_t)q * kWave;
    a.vy = (VY + i0)[lane];
    a.vz = (VZ + i0)[lane];
  };
  const int q_first = q_lo + w;
  Slice next;
  fetch(next, q_first < q_hi ? q_first : 0);
  if (SP == 0) {
    // v_y and v_z of the first slice for the measurements; without them a
    // second read of the same x, so that these loads need no branch either
    const int64_t i0 = (int64_t)(q_first < q_hi ? q_first : 0) * kWave;
    next.vy = ((pdiag ? VY : X) + i0)[lane];
    next.vz = ((pdiag ? VZ : X) + i0)[lane];
  }
  solve();
  auto stream = [&](auto diag) {
    constexpr bool DIAG = decltype(diag)::value;  // some particle measurement is on
    int q = q_first;
    if (q >= q_hi) return;
    for (;;) {
      const Slice a = next;
      const int qn = q + kWaves;
      const bool more = qn < q_hi;
      fetch(next, more ? qn : q);
      if (SP == 0 && DIAG) fetch_vyz(next, more ? qn : q);
      const int i0 = q * kWave;
      const double vy = SP == 1 || DIAG ? a.vy : 0.0, vz = SP == 1 || DIAG ? a.vz : 0.0;
      const uint64_t uid = a.uid;
      double x = a.x, vx = a.vx, vp2 = SP == 0 ? (double)a.vp2 : 0.0;
      bool live = x == x;  // not absorbed earlier (tombstone)
      if (i0 + kWave > n) {  // the last slice: slots from n on hold nothing
        if (lane >= (int)(n - i0)) {
          live = false;
          vx = vp2 = 0.0;
        }
      }
      x = live ? x : 0.0;
      t_live += (int)__popcll(ballot(live));
      bool surf = false, cand = false;
      // Steps 3-4: linear interpolation of the nodal field (section 2.1.3)
      // from cell coordinate xi = x/dx, then the leapfrog equations of
      // section 2.1.4, the kick being e dt/m per unit field (subtracted for
      // the electron's negative charge).
      const double xi = x * inv_dx;
      int cell = (int)xi;
      cell = cell > ng - 2 ? ng - 2 : (cell < 0 ? 0 : cell);
      const double w_lo = (double)(cell + 1) - xi;  // weight of node `cell`
      const double w_hi = xi - (double)cell;        // weight of node `cell + 1`
      const double e_here = sE[cell] * w_lo + sE[cell + 1] * w_hi;
      double vxn = SP == 0 ? vx - e_here * kick : vx + e_here * kick;
      double xn = x + vxn * dt;
      // Step 6 pre-test.  A particle can collide only if its R is below the
      // bound of 1 - exp(-nu dt) over the tables (P* for null collisions), or
      // if it is faster than the range that bound covers; the upper word of R
      // decides that but for R within 2^-32 of the bound, which the exact
      // test settles like every candidate.  The bound by energy is looked up
      // first, so that the LDS load is in flight beside the rest (a
      // reflection below keeps |v|).
      const double v2 = SP == 0 ? vxn * vxn + vp2 : vxn * vxn + vy * vy + vz * vz;
      const double g2u = SP == 0 ? v2 : 2.0 * (v2 + a2_i);
      uint32_t r_lim = r_cand;
      if (by_energy) r_lim = sPB[(int)fmin(g2u * blocks_per_g2 + block_half, block_last)];
      if (DIAG && live) {
        // measurement at integer time: old position, mean of the half-step
        // velocities; the ionization rate as the expected n sigma_ion |v|
        const double vbar = 0.5 * (vx + vxn);
        if (fl & (kDiagCurrent | kDiagXT)) {
          lds_add(&sJ[cell], (long long)(w_lo * vbar * kDiagJS));
          lds_add(&sJ[cell + 1], (long long)(w_hi * vbar * kDiagJS));
        }
        if (SP == 1) {
          if (xt) {
            const double en = div_by(0.5 * kArMass * (vbar * vbar + vy * vy + vz * vz), kEvToJ, 1.0 / kEvToJ);
            lds_add(&sW[cell], (long long)(w_lo * kDiagWS));
            lds_add(&sW[cell + 1], (long long)(w_hi * kDiagWS));
            lds_add(&sEn[cell], (long long)(w_lo * en * kDiagES));
            lds_add(&sEn[cell + 1], (long long)(w_hi * en * kDiagES));
          }
        } else if (fl & (kDiagMeanE | kDiagEepf | kDiagXT)) {
          const double en = div_by(0.5 * kEMass * (vbar * vbar + vy * vy + vz * vz), kEvToJ, 1.0 / kEvToJ);
          if (xt) {
            const double vmag = sqrt(vbar * vbar + vy * vy + vz * vz);
            const double pdt = (n_gas * sig2[energy_bin(en, de_cs, inv_de_cs, nbins)]) * vmag * dt;
            lds_add(&sIz[cell], (long long)(w_lo * pdt * kDiagIZS));
            lds_add(&sIz[cell + 1], (long long)(w_hi * pdt * kDiagIZS));
          }
          if (fl & (kDiagMeanE | kDiagXT)) {
            lds_add(&sW[cell], (long long)(w_lo * kDiagWS));
            lds_add(&sW[cell + 1], (long long)(w_hi * kDiagWS));
            lds_add(&sEn[cell], (long long)(w_lo * en * kDiagES));
            lds_add(&sEn[cell + 1], (long long)(w_hi * en * kDiagES));
          }
          if ((fl & kDiagEepf) && x >= x_lo && x <= x_hi) {
            const double t = div_by(en, de_eepf, C->inv_de_eepf);
            if (t < (double)n_eepf) atomicAdd(&sF[(int)t], 1u);
          }
        }
      }
      const uint32_t r_word = philox_w0(seed, uid, st, r_tag);
      // Step 5: absorbing electrodes; an absorbed ion adds its impact energy
      // to its electrode's IFEDF (bin n_ifed: beyond the range).  Surface
      // processes (purpose 3 of the particle's counter): an electron is
      // reflected specularly with the electrode's probability eta (unless
      // its mirror image lies outside the gap); an absorbed ion emits an
      // electron with probability gamma, whose charge goes on the electrode
      // node of the next step's deposit now and which takes its slot from
      // the step's electron births below.
      bool abs_pow = live && xn < 0.0;
      bool abs_gnd = live && xn > L_gap;
      if (surf_on && (abs_pow || abs_gnd)) {
        double r_surf, r_unused;
        uniform2(seed, uid, st, tag(SP, 3, 0), r_surf, r_unused);
        if (r_surf < (abs_pow ? p_surf0 : p_surf1)) {
          if (SP == 0) {
            const double xm = abs_pow ? -xn : 2.0 * L_gap - xn;
            if (xm >= 0.0 && xm <= L_gap) {
              xn = xm;
              vxn = -vxn;
              abs_pow = abs_gnd = false;
              surf = true;
            }
          } else {
            surf = true;
            long long r;
            const int p = deposit_split(abs_pow ? 0.0 : L_gap, inv_dx, ng, r);
            if constexpr (OWN) {
              lds_add(&own_e[p], 4294967296LL - r);
              if (r) lds_add(&own_e[p + 1], r);
            } else {
              gl_add(&cnt_e_next[p], 4294967296LL - r);
              if (r) gl_add(&cnt_e_next[p + 1], r);
            }
          }
        }
      }
      const bool in = live && !(abs_pow || abs_gnd);
      if (DIAG && SP == 1 && (fl & kDiagIfed) && live && !in) {
        const double en = 0.5 * kArMass * (vxn * vxn + vy * vy + vz * vz) / kEvToJ;
        const double t = en / de_ifed;
        const int b = t < (double)n_ifed ? (int)t : n_ifed;
        atomicAdd(&sF[(abs_gnd ? n_ifed + 1 : 0) + b], 1u);
      }
      // Step 7 for step s+1: deposit the new position
      if (in) {
        long long r;
        const int p = deposit_split(xn, inv_dx, ng, r);
        lds_add(&sH[p], 4294967296LL - r);
        lds_add(&sH[p + 1], r);
        cand = r_word <= r_lim || g2u > v2_cand;
      }
      double x_out = in ? xn : __longlong_as_double(0x7FF8000000000000LL), v_out = vxn;
      unsigned at = (unsigned)lane;
      if (i0 + kWave > n) {
        // a lane without a slot stores what lane 0 stores (slots from n on
        // may be a newborn's already)
        const double x_0 = __shfl(x_out, 0), v_0 = __shfl(v_out, 0);
        const bool none = lane >= (int)(n - i0);
        x_out = none ? x_0 : x_out;
        v_out = none ? v_0 : v_out;
        at = none ? 0 : at;
      }
      (X + (int64_t)i0)[at] = x_out;
      (VX + (int64_t)i0)[at] = v_out;
      if (surf_on) {
        // reflections (electrons) or emissions per electrode (ions); an ion's
        // secondary electron takes its slot after this step's births so far
        const uint64_t m_s0 = ballot(surf && (SP == 0 || abs_pow));
        const uint64_t m_s1 = SP == 1 ? ballot(surf && abs_gnd) : 0ull;
        if (lane == 0 && m_s0) gl_add(&Cw->ctr[SP == 0 ? kRefl : kSeePow], (long long)__popcll(m_s0));
        if (lane == 0 && m_s1) gl_add(&Cw->ctr[kSeeGnd], (long long)__popcll(m_s1));
        if (SP == 1 && (m_s0 | m_s1)) {
          read_scatter_ptrs(P, C, 0, cur_o);
          const int64_t be = B.take(0, surf, lane, t_be, t_drop);
          if (surf) see_emit_at(C, P, uid, abs_pow ? 0 : 1, be, s);
        }
      }
      const uint64_t m_c = ballot(cand);
      if (m_c) {
        if (cand) {
          const int k = ncw + lane_rank(m_c);
          sSeg[w][k] = i0 + lane;
          if (SP == 0) {
            sVx[SP == 0 ? w : 0][SP == 0 ? k : 0] = vxn;
            sUid[SP == 0 ? w : 0][SP == 0 ? k : 0] = uid;
          }
        }
        ncw += (int)__popcll(m_c);
        if (ncw > kSeg - kWave) {
          spill_segment(ncw);
          ncw = 0;
        }
      }
      t_pow += (int)__popcll(ballot(abs_pow));
      t_gnd += (int)__popcll(ballot(abs_gnd));
      if (!more) break;
      q = qn;
    }
  };
  if (pdiag)
    stream(std::true_type{});
  else
    stream(std::false_type{});
  // the first round's v_y and v_z are on their way during the barrier
  const Entry first = own_entry(lane);
  __syncthreads();
  // this wave's segment, then the workgroup's overflow list
  finish(first);
  // then the flush (deposit for step s+1 and diagnostics of step s), last: a
  // wave's memory operations return in order, and behind the flush's atomics
  // every load of the candidates' rounds waited for those too (a step of 1.3e5
  // electrons on 641 nodes 16.4 -> 16.1 us).  A thread's first nodes without a
  // loop: before one, the compiler waits for whatever is on its way.
  if constexpr (!OWN) {
    unsigned long long h[kRingRegs];
#pragma unroll
    for (int u = 0; u < kRingRegs; ++u) {
      const int q = (int)threadIdx.x + u * NB;
      h[u] = q < ng ? sH[q] : 0;
    }
#pragma unroll
    for (int u = 0; u < kRingRegs; ++u)
      if (h[u]) gl_add(&dst[(int)threadIdx.x + u * NB], (long long)h[u]);
  }
  if (!OWN && ng > kRingRegs * NB)
    for (int q = (int)threadIdx.x + kRingRegs * NB; q < ng; q += NB)
      if (const unsigned long long h = sH[q]) gl_add(&dst[q], (long long)h);
  if (pdiag)
    for (int q = threadIdx.x; q < ng; q += NB) {
      const int64_t off3 = (int64_t)I.s3 * ng + q;
      const unsigned long long a = sJ[q], b = sW[q], c = sEn[q], d = SP == 0 && xt ? sIz[q] : 0;
      if (a) gl_add(&(SP == 0 ? C->acc_je : C->acc_ji)[off3], (long long)a);
      if (b) gl_add(&(SP == 0 ? C->acc_w : C->acc_wi)[off3], (long long)b);
      if (c) gl_add(&(SP == 0 ? C->acc_e : C->acc_ei)[off3], (long long)c);
      if (d) gl_add(&C->acc_iz[off3], (long long)d);
    }
  int64_t* hist = SP == 0 ? C->eepf : C->ifed;
  if (n_hist)
    for (int b = threadIdx.x; b < n_hist; b += NB)
      if (sF[b]) gl_add(&hist[b], (long long)sF[b]);
  const int v[kRec] = {t_coll, t_ioniz, t_pow, t_gnd, t_live, t_be, t_bi, t_drop};
  SpTot T;
  // lane f has field f
  T.field = 0;
#pragma unroll
  for (int f = 0; f < kRec; ++f) T.field = lane == f ? v[f] : T.field;
  if (SMALL) __syncthreads();  // the segments and the histograms are free again
  return T;
}

// Slot count of species sp at the start of a step inside a window (s3: the
// step mod 3).
__device__ __forceinline__ int64_t step_slots(const EDP_CONST CaseDev* __restrict__ C, int sp, int s3) {
  const int r = s3 == 0 ? 2 : s3 - 1;
  const int64_t a = C->nbase[sp][r] + C->born[sp][r];
  return a < C->sp[sp].cap ? a : C->sp[sp].cap;
}

// Steps 1-7 of one species for every case of a lockstep group, at step
// step0 + dstep of each case.  At most 128 VGPRs (16 waves per CU):
// the streaming loop needs about 100; the scattering code after the loop
// would take twice that if left alone, and spills there instead (colliders
// are a few percent of the particles).  Every workgroup solves its case's field into
// LDS, then takes its chunk range.  The electron launch's workgroup 0 of
// each case is the writer of the step (field outputs, ring clearing,
// measurement sums) and publishes the step's slot counts.  Each workgroup
// adds its totals to its shard of the case's counters.  NB threads: see
// particle_block in the host code.
template <int SP, int MODE, int NB>
__global__ void __launch_bounds__(NB) __attribute__((amdgpu_waves_per_eu(4)))
k_particles(const BlockRole* __restrict__ R, int dstep, int pretest) {
  extern __shared__ double psm[];
  const EDP_CONST BlockRole* r = KC(R) + blockIdx.x;
  CaseDev* Cw = r->c;
  const int ng = r->ng, nsub = r->nsub, j = r->j;
  const uint32_t f_lo = r->f_lo, f_hi = r->f_hi;
  const int64_t s = r->step0 + dstep;
  const StepIndex I(s, nsub);
  if (SP == 1 && I.sub != 0) return;  // ions move on ion steps only
  double* sE = psm;
  double* reg = psm + ng;
  const bool writer = SP == 0 && j == 0;
  const EDP_CONST CaseDev* __restrict__ C = KC(Cw);
  const RingNodes<NB> N(r->cnt_e, r->cnt_i, r->volt, s, I.s3, I.k3, ng);
  // the slot counts and the current buffer sets, with what the pass needs;
  // every line of the case block is touched now, so that what is read later
  // comes from the scalar cache (cold at a launch's start, and each first
  // touch a wait of its own)
  touch_case(C);
  const int64_t n_e = step_slots(C, 0, I.s3), n_i = step_slots(C, 1, I.s3);
  const int cur = C->cur[SP], cur_o = C->cur[1 - SP];
  Births<false> B;
  B.cap[0] = C->sp[0].cap;
  B.cap[1] = C->sp[1].cap;
  const PassIn<SP> A(C);
  const SolveIn SI(C);
  const int64_t n = SP == 0 ? n_e : n_i;
  const uint32_t nch = (uint32_t)((n + NB - 1) / NB);
  const int64_t c_lo = (int64_t)(((uint64_t)nch * f_lo) >> 31);
  const int64_t c_hi = (int64_t)(((uint64_t)nch * f_hi) >> 31);
  if (c_lo >= c_hi && !writer) return;  // whole workgroup: nothing to do this step
  auto solve = [&]() __attribute__((always_inline)) {
    solve_field<MODE, NB>(Cw, ng, s, I, sE, reg, writer, N, SI);
    if (writer && threadIdx.x == 0) {
      for (int sp = 0; sp < 2; ++sp) {
        Cw->nbase[sp][I.s3] = sp == 0 ? n_e : n_i;
        Cw->born[sp][I.s3 == 2 ? 0 : I.s3 + 1] = 0;
      }
    }
  };
  B.base[0] = n_e;
  B.base[1] = n_i;
  B.lds = nullptr;
  B.glob[0] = &Cw->born[0][I.s3];
  B.glob[1] = &Cw->born[1][I.s3];
  const SpTot T = species_pass<SP, false, NB>(Cw, sE, reg, s, I, n, c_lo, c_hi, cur, cur_o, B, pretest, A, solve);
  // every wave adds its own totals (spread over the shards): no wave waits
  // for the others at the end
  const int t = (int)threadIdx.x, f = t % kWave;
  int64_t* sh = C->shard + ((int64_t)SP * kShards + (j * (NB / kWave) + t / kWave) % kShards) * kRec;
  if (T.field) gl_add(&sh[f], T.field);  // lanes beyond the fields have 0
  if (f == kRecDropped && T.field) Cw->error = 1;
}

// First kernel of a lockstep window: every role's step0 from its case, and
// each case's slot-count rings from its slot counts (so that any host-side
// change of a case between windows is picked up).  Workgroups [0, ncase)
// take the cases of `cases`, the others the roles.
__global__ void __launch_bounds__(kBlock) k_window_begin(BlockRole* __restrict__ roles, int nroles,
                                                         const BlockRole* __restrict__ cases, int ncase) {
  const int b = (int)blockIdx.x;
  if (b < ncase) {
    if (threadIdx.x == 0) {
      CaseDev* C = cases[b].c;
      const int64_t s = C->step;
      for (int sp = 0; sp < 2; ++sp) {
        C->nbase[sp][(s + 2) % 3] = C->n[sp];
        C->born[sp][(s + 2) % 3] = 0;
        C->born[sp][s % 3] = 0;
      }
    }
    return;
  }
  const int i = (b - ncase) * kBlock + (int)threadIdx.x;
  if (i < nroles) roles[i].step0 = roles[i].c->step;
}

// Last kernel of a lockstep window of `steps` steps, one workgroup per case:
// the case's step, its slot counts, and the workgroups' shards folded into
// the counters (then cleared).
__global__ void __launch_bounds__(kBlock) k_window_end(const BlockRole* __restrict__ cases, int steps) {
  __shared__ int64_t sSum[kBlock / kWave][2 * kRec];
  CaseDev* Cw = (KC(cases) + blockIdx.x)->c;
  const EDP_CONST CaseDev* __restrict__ C = KC(Cw);
  // thread t sums field t % (2 kRec) of every shard of both species
  constexpr int kF = 2 * kRec;
  const int t = (int)threadIdx.x;
  static_assert(kBlock == 4 * kWave && kWave == 4 * kF, "shard fold layout");
  int64_t acc = 0;
  EDP_GLOBAL int64_t* sh = G(C->shard);
  {
    const int f = t % kF, sp = f / kRec, fld = f % kRec;
    for (int k = t / kF; k < kShards; k += kBlock / kF) {
      EDP_GLOBAL int64_t* a = sh + ((int64_t)sp * kShards + k) * kRec + fld;
      acc += *a;
      *a = 0;
    }
  }
  const int lane = t % kWave, wv = t / kWave;
  // lanes l and l + 16, l + 32, l + 48 hold the same field (64 = 4 * kF)
  acc += __shfl_xor(acc, 16, kWave);
  acc += __shfl_xor(acc, 32, kWave);
  if (lane < kF) sSum[wv][lane] = acc;
  __syncthreads();
  if (t == 0) {
    int64_t v[kF];
    for (int f = 0; f < kF; ++f) v[f] = sSum[0][f] + sSum[1][f] + sSum[2][f] + sSum[3][f];
    const int64_t* e = v;
    const int64_t* ii = v + kRec;
    int64_t* ctr = Cw->ctr;
    ctr[kCollE] += e[kRecColl];
    ctr[kIoniz] += e[kRecIoniz];
    ctr[kAbsEPow] += e[kRecAbsPow];
    ctr[kAbsEGnd] += e[kRecAbsGnd];
    ctr[kPstepE] += e[kRecLive];
    ctr[kCollI] += ii[kRecColl];
    ctr[kAbsIPow] += ii[kRecAbsPow];
    ctr[kAbsIGnd] += ii[kRecAbsGnd];
    ctr[kPstepI] += ii[kRecLive];
    ctr[kLiveE] += e[kRecBornE] + ii[kRecBornE] - e[kRecAbsPow] - e[kRecAbsGnd];
    ctr[kLiveI] += e[kRecBornI] + ii[kRecBornI] - ii[kRecAbsPow] - ii[kRecAbsGnd];
    ctr[kDropped] += e[kRecDropped] + ii[kRecDropped];
    const int64_t s = Cw->step + steps;
    Cw->step = s;
    for (int sp = 0; sp < 2; ++sp) {
      const int r = (int)((s + 2) % 3);
      const int64_t a = Cw->nbase[sp][r] + Cw->born[sp][r];
      const int64_t cap = C->sp[sp].cap;
      Cw->n[sp] = Cw->alloc[sp] = a < cap ? a : cap;
    }
  }
}

// Cell of a position (the deposit's node p, clamped to N_g - 2).
__device__ __forceinline__ int cell_of(double x, double inv_dx, int ng) {
  int p = (int)(x * inv_dx);
  return p > ng - 2 ? ng - 2 : (p < 0 ? 0 : p);
}

// ---------------------------------------------------------------------------
// Persistent small cases: one workgroup advances one case through a whole
// window of steps inside one launch, and every case of the launch runs at its
// own pace -- no lockstep with the other cases, no launch between two steps,
// no wait between workgroups.  Each step is the same method as the lockstep
// path's and gives the same results bit for bit: the field solve into LDS
// (steps 1-2), then per species the push, walls, collision test, the
// colliders' scattering and the newborns (steps 3-6) and the deposit for the
// next step, then the step's bookkeeping; compaction and cell sort every
// `sort_every` steps as in the lockstep path.  Meant for cases of a few
// thousand particles, whose steps are latency-bound: one workgroup per case
// keeps the chip's other CUs for the other cases.
//
// The workgroup owns the case for the launch: the step, the slot counts and
// the buffer sets live in LDS and are written back at the end.
// ---------------------------------------------------------------------------

// Compaction + counting sort by cell of species sp in one workgroup: the
// live slots of [0, n) of set `cur` go to the other set, cell by cell (order
// within a cell arbitrary); returns the live count.  sC: LDS for ng counters.
template <int NB>
__device__ __forceinline__ int64_t small_sort(CaseDev* __restrict__ Cw, int sp, int cur, int64_t n, unsigned int* sC) {
  __shared__ int64_t sRed[64];
  const EDP_CONST CaseDev* __restrict__ C = KC(Cw);
  const int ng = C->ng;
  const double inv_dx = C->inv_dx;
  const EDP_CONST SpeciesDev& S = C->sp[sp];
  const EDP_GLOBAL double* __restrict__ X = G(S.x[cur]);
  for (int p = threadIdx.x; p < ng; p += blockDim.x) sC[p] = 0;
  __syncthreads();
  for (int64_t i = threadIdx.x; i < n; i += NB) {
    const double x = X[i];
    if (x == x) atomicAdd(&sC[cell_of(x, inv_dx, ng)], 1u);
  }
  __syncthreads();
  // exclusive scan of the ng - 1 cell counts, a contiguous range per thread
  const int m = ng - 1;
  const int per = (m + NB - 1) / NB;
  const int lo = (int)threadIdx.x * per < m ? (int)threadIdx.x * per : m;
  const int hi = lo + per < m ? lo + per : m;
  int64_t acc = 0;
  for (int p = lo; p < hi; ++p) acc += sC[p];
  int64_t total;
  int64_t run = block_exclusive_scan_t<int64_t>(acc, sRed, &total);
  for (int p = lo; p < hi; ++p) {
    const unsigned int v = sC[p];
    sC[p] = (unsigned int)run;
    run += v;
  }
  __syncthreads();
  const int nxt = cur ^ 1;
  const EDP_GLOBAL double* __restrict__ VX = G(S.vx[cur]);
  const EDP_GLOBAL double* __restrict__ VY = G(S.vy[cur]);
  const EDP_GLOBAL double* __restrict__ VZ = G(S.vz[cur]);
  const EDP_GLOBAL uint64_t* __restrict__ UID = G(S.uid[cur]);
  EDP_GLOBAL double* __restrict__ X2 = G(S.x[nxt]);
  EDP_GLOBAL double* __restrict__ VX2 = G(S.vx[nxt]);
  EDP_GLOBAL double* __restrict__ VY2 = G(S.vy[nxt]);
  EDP_GLOBAL double* __restrict__ VZ2 = G(S.vz[nxt]);
  EDP_GLOBAL uint64_t* __restrict__ UID2 = G(S.uid[nxt]);
  EDP_GLOBAL float* __restrict__ VP22 = sp == 0 ? G(S.vp2[nxt]) : nullptr;
  for (int64_t i = threadIdx.x; i < n; i += NB) {
    const double x = X[i];
    if (!(x == x)) continue;
    const double vx = VX[i], vy = VY[i], vz = VZ[i];
    const uint64_t uid = UID[i];
    const int64_t d = atomicAdd(&sC[cell_of(x, inv_dx, ng)], 1u);
    X2[d] = x;
    VX2[d] = vx;
    VY2[d] = vy;
    VZ2[d] = vz;
    UID2[d] = uid;
    if (sp == 0) VP22[d] = float_above(vy * vy + vz * vz);
  }
  __syncthreads();
  return total;
}

// Window of steps of the small cases: workgroup b advances the case of role
// b by role.j steps.  Bound by the latency of a step's phases, one after
// another.  With 512 threads a case of 1e3 particles is one to three slices a
// wave; the densities and the deposits of the next step stay in LDS (no flush,
// no rings in between; the window's end writes them back), and the waves that
// do not solve the field do the writer's duties meanwhile.  256 threads where
// a case's grid and measurements ask for the LDS: deposits through the
// rings.  Every wave keeps the step's indices, the slot counts and its totals
// until the end.  Measured, us a step with 256 threads and totals every step,
// with 512, with the deposits in LDS: 1e3 electrons on 400 nodes 12.3, 11.2,
// 9.6, 5e3 on 641 nodes 31.5, 26.8, 25.2.
//
// Dynamic LDS: E (also the sort's counters), then for 512 threads the
// densities and deposits of both species and the larger of the two
// species' measurement arrays, for 256 the larger particle region (also the
// field solve's scratch).
template <int MODE, int NB>
__global__ void __launch_bounds__(NB) k_small(const BlockRole* __restrict__ R, int sort_every, int pretest) {
  extern __shared__ double ssm2[];
  // births of the steps t, t - 1 (read) and t + 1 (cleared) mod 3
  __shared__ int sBirth[3][2];
  const EDP_CONST BlockRole* r = KC(R) + blockIdx.x;
  CaseDev* Cw = r->c;
  const int steps = r->j;
  const EDP_CONST CaseDev* __restrict__ C = KC(Cw);
  const int ng = C->ng;
  const int nsub = C->nsub;
  constexpr bool OWN = NB > kBlock;
  double* sE = ssm2;
  // the electrons' density of the step and deposit for the next, the ions'
  // density and deposit for the next ion step
  int64_t* A0 = (int64_t*)(ssm2 + ng);
  int64_t* A1 = A0 + ng;
  int64_t* I0 = A1 + ng;
  int64_t* I1 = I0 + ng;
  double* reg = ssm2 + (OWN ? 5 : 1) * ng;
  int64_t s = C->step;
  int64_t n_e = C->n[0], n_i = C->n[1];
  int cur_e = C->cur[0], cur_i = C->cur[1];
  // read once: the kernel writes them at its end
  asm volatile("" : "+s"(s), "+s"(n_e), "+s"(n_i), "+s"(cur_e), "+s"(cur_i));
  const int64_t cap_e = C->sp[0].cap, cap_i = C->sp[1].cap;
  StepIndex I(s, nsub);
  // steps to the next compaction + cell sort, on the lockstep path's schedule
  const int64_t every_i = (int64_t)sort_every * nsub;
  int64_t to_e = (sort_every - s % sort_every) % sort_every, to_i = (every_i - s % every_i) % every_i;
  int64_t tot[2] = {0, 0};  // lane f: this wave's total of field f, per species
  if (threadIdx.x < 6) sBirth[threadIdx.x / 2][threadIdx.x % 2] = 0;
  if constexpr (OWN) {
    const EDP_GLOBAL int64_t *gE = G(C->cnt_e), *gI = G(C->cnt_i);
    for (int p = threadIdx.x; p < ng; p += NB) {
      // (an ion step takes I1 as its density first)
      const int64_t now = gI[I.k3 * ng + p], next = gI[(I.k3 == 2 ? 0 : I.k3 + 1) * ng + p];
      A0[p] = gE[I.s3 * ng + p];
      I0[p] = now;
      I1[p] = I.sub == 0 ? now : next;
    }
  }
  __syncthreads();
  int b3 = 0;  // t mod 3
#pragma unroll 1
  for (int t = 0; t < steps; ++t) {
    const bool ion_step = I.sub == 0;
    const int b_next = b3 == 2 ? 0 : b3 + 1, b_last = b3 == 0 ? 2 : b3 - 1;
    n_e = n_e + sBirth[b_last][0] < cap_e ? n_e + sBirth[b_last][0] : cap_e;
    n_i = n_i + sBirth[b_last][1] < cap_i ? n_i + sBirth[b_last][1] : cap_i;
    if (threadIdx.x < 2) sBirth[b_next][threadIdx.x] = 0;
    if (to_e == 0) {
      n_e = small_sort<NB>(Cw, 0, cur_e, n_e, (unsigned int*)ssm2);
      cur_e ^= 1;
      to_e = sort_every;
    }
    if (to_i == 0) {
      n_i = small_sort<NB>(Cw, 1, cur_i, n_i, (unsigned int*)ssm2);
      cur_i ^= 1;
      to_i = every_i;
    }
    --to_e;
    --to_i;
    // steps 1-2
    if constexpr (OWN) {
      if (ion_step) {
        int64_t* const a = I0;
        I0 = I1;
        I1 = a;
        for (int p = threadIdx.x; p < ng; p += NB) I1[p] = 0;
      }
    }
    auto solve = [&]() __attribute__((always_inline)) {
      if constexpr (OWN) {
        const OwnNodes N{A0, I0, G(C->volt)[s % kVoltChunk]};
        solve_field<MODE, NB>(Cw, ng, s, I, sE, (double*)A1, true, N, SolveIn(C));
      } else {
        const RingNodes<NB> N(C->cnt_e, C->cnt_i, C->volt, s, I.s3, I.k3, ng);
        solve_field<MODE, NB>(Cw, ng, s, I, sE, reg, true, N, SolveIn(C));
      }
    };
    Births<true> B;
    B.base[0] = n_e;
    B.base[1] = n_i;
    B.cap[0] = cap_e;
    B.cap[1] = cap_i;
    B.lds = sBirth[b3];
    B.glob[0] = B.glob[1] = nullptr;
    const int64_t nch_e = (n_e + NB - 1) / NB, nch_i = (n_i + NB - 1) / NB;
    tot[0] += species_pass<0, true, NB>(Cw, sE, reg, s, I, n_e, 0, nch_e, cur_e, cur_i, B, pretest, PassIn<0>(C), solve,
                                          (unsigned long long*)A1, (unsigned long long*)I1).field;
    if (ion_step)
      tot[1] += species_pass<1, true, NB>(Cw, sE, reg, s, I, n_i, 0, nch_i, cur_i, cur_e, B, pretest, PassIn<1>(C),
                                          [] { __syncthreads(); }, (unsigned long long*)A1, (unsigned long long*)I1).field;
    if constexpr (OWN) {
      int64_t* const a = A0;
      A0 = A1;
      A1 = a;
    }
    ++s;
    I.next(nsub);
    b3 = b_next;
  }
  if constexpr (OWN) {
    // the rings as the next step reads and fills them (kl: the last ion step's)
    const int kl = I.sub == 0 ? (I.k3 + 2) % 3 : I.k3;
    EDP_GLOBAL int64_t *gE = G(C->cnt_e), *gI = G(C->cnt_i);
    for (int p = threadIdx.x; p < ng; p += NB) {
      gE[I.s3 * ng + p] = A0[p];
      gE[(I.s3 + 1) % 3 * ng + p] = 0;
      gE[(I.s3 + 2) % 3 * ng + p] = 0;
      gI[kl * ng + p] = I0[p];
      gI[(kl + 1) % 3 * ng + p] = I1[p];
      gI[(kl + 2) % 3 * ng + p] = 0;
    }
  }
  // the counters of each wave's totals
  const int f = (int)threadIdx.x % kWave;
  constexpr int kTo[2][kRec] = {{kCollE, kIoniz, kAbsEPow, kAbsEGnd, kPstepE, kLiveE, kLiveI, kDropped},
                                {kCollI, -1, kAbsIPow, kAbsIGnd, kPstepI, kLiveE, kLiveI, kDropped}};
#pragma unroll
  for (int sp = 0; sp < 2; ++sp) {
    int to = -1;
#pragma unroll
    for (int q = 0; q < kRec; ++q) to = f == q ? kTo[sp][q] : to;
    if (to >= 0 && tot[sp]) {
      gl_add(&Cw->ctr[to], tot[sp]);
      if (f == kRecAbsPow || f == kRecAbsGnd) gl_add(&Cw->ctr[sp == 0 ? kLiveE : kLiveI], -tot[sp]);
      if (f == kRecDropped) Cw->error = 1;
    }
  }
  if (threadIdx.x == 0) {
    const int b_last = b3 == 0 ? 2 : b3 - 1;
    n_e = n_e + sBirth[b_last][0] < cap_e ? n_e + sBirth[b_last][0] : cap_e;
    n_i = n_i + sBirth[b_last][1] < cap_i ? n_i + sBirth[b_last][1] : cap_i;
    Cw->step = s;
    Cw->n[0] = Cw->alloc[0] = n_e;
    Cw->n[1] = Cw->alloc[1] = n_i;
    Cw->cur[0] = cur_e;
    Cw->cur[1] = cur_i;
  }
}

__global__ void k_seed(CaseDev* __restrict__ C, int sp, int64_t n, double sigma) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int cur = C->cur[sp];
  double u0, u1, z0, z1, z2;
  uniform2(C->seed, (uint64_t)i, 0u, tag((uint32_t)sp, 1u, 0u), u0, u1);
  normals3(C->seed, (uint64_t)i, 0u, (uint32_t)sp, 1u, 1u, z0, z1, z2);
  G(C->sp[sp].x[cur])[i] = C->L * u0;
  const double vy = sigma * z1, vz = sigma * z2;
  G(C->sp[sp].vx[cur])[i] = sigma * z0;
  G(C->sp[sp].vy[cur])[i] = vy;
  G(C->sp[sp].vz[cur])[i] = vz;
  if (sp == 0) G(C->sp[0].vp2[cur])[i] = float_above(vy * vy + vz * vz);
  G(C->sp[sp].uid[cur])[i] = (uint64_t)i;
}

// Deposit the live particles [0, alloc) of a species into one or two buffers.
__global__ void __launch_bounds__(256) k_deposit(CaseDev* __restrict__ C, int sp, int64_t* dst1,
                                                 int64_t* dst2) {
  extern __shared__ double dsm[];
  unsigned long long* sH = (unsigned long long*)dsm;
  const int ng = C->ng;
  for (int p = threadIdx.x; p < ng; p += blockDim.x) sH[p] = 0;
  __syncthreads();
  const int cur = C->cur[sp];
  const EDP_GLOBAL double* __restrict__ X = G(C->sp[sp].x[cur]);
  const int64_t n = slots(C, sp);
  const double inv_dx = C->inv_dx;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double x = X[i];
    if (!(x == x)) continue;
    long long r;
    const int q = deposit_split(x, inv_dx, ng, r);
    lds_add(&sH[q], 4294967296LL - r);
    lds_add(&sH[q + 1], r);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < ng; q += blockDim.x) {
    const unsigned long long h = sH[q];
    if (!h) continue;
    gl_add(&dst1[q], (long long)h);
    if (dst2) gl_add(&dst2[q], (long long)h);
  }
}

// ---------------------------------------------------------------------------
// Compaction + counting sort by cell: drops tombstones, merges births and
// restores spatial locality (contiguous particle ranges then touch few nodes,
// so the per-workgroup deposit flush stays small).  Order within a cell is
// arbitrary; results do not depend on it.
// ---------------------------------------------------------------------------



// The sort kernels serve a batch: one role per workgroup (a case's sort
// workgroups, or one per case for the scan and the finish).  A case sorts its
// electrons at steps that are multiples of `every` and its ions at multiples
// of every * N_SUB; the workgroups of a case that is not due return at once,
// so the host launches the four kernels only at steps where some case is due.
constexpr int kSortUnroll = 4;

// Step of a sort launch of a window for role r, and whether species sp of
// its case is due at that step.
__device__ __forceinline__ bool sort_due(const EDP_CONST BlockRole* r, int sp, int every, int dstep, int64_t& s) {
  s = r->step0 + dstep;
  const int64_t per = sp == 0 ? (int64_t)every : (int64_t)every * r->nsub;
  return s % per == 0;
}

__global__ void __launch_bounds__(256) k_sort_hist(const BlockRole* __restrict__ R, int sp, int every, int dstep) {
  extern __shared__ double hsm[];
  const EDP_CONST BlockRole* r = KC(R) + blockIdx.x;
  CaseDev* C = r->c;
  int64_t s;
  if (!sort_due(r, sp, every, dstep, s)) return;
  unsigned int* sC = (unsigned int*)hsm;
  const int ng = C->ng;
  for (int p = threadIdx.x; p < ng; p += blockDim.x) sC[p] = 0;
  __syncthreads();
  const int cur = C->cur[sp];
  const EDP_GLOBAL double* __restrict__ X = G(C->sp[sp].x[cur]);
  const int64_t n = step_slots(KC(C), sp, (int)(s % 3));
  const int64_t nb = r->n, per = (n + nb - 1) / nb;
  const int64_t lo = (int64_t)r->j * per, hi = lo + per < n ? lo + per : n;
  const double inv_dx = C->inv_dx;
  // kSortUnroll particles per thread and round: their loads are in flight
  // together
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += kSortUnroll * kBlock) {
    double x[kSortUnroll];
#pragma unroll
    for (int u = 0; u < kSortUnroll; ++u) {
      const int64_t i = i0 + u * kBlock;
      x[u] = i < hi ? X[i] : __longlong_as_double(0x7FF8000000000000LL);
    }
#pragma unroll
    for (int u = 0; u < kSortUnroll; ++u)
      if (x[u] == x[u]) atomicAdd(&sC[cell_of(x[u], inv_dx, ng)], 1u);
  }
  __syncthreads();
  for (int p = threadIdx.x; p < ng - 1; p += blockDim.x)
    if (sC[p]) gl_add(&C->sort_cnt[p], (long long)sC[p]);
}

// Exclusive scan of the ng-1 cell counts (one workgroup); total -> sort_cnt[ng].
__global__ void __launch_bounds__(1024) k_sort_scan(const BlockRole* __restrict__ R, int sp, int every, int dstep) {
  __shared__ int64_t sRed[64];
  const EDP_CONST BlockRole* r = KC(R) + blockIdx.x;
  CaseDev* C = r->c;
  int64_t s;
  if (!sort_due(r, sp, every, dstep, s)) return;
  const int m = C->ng - 1;
  const int t = threadIdx.x, T = blockDim.x;
  const int per = (m + T - 1) / T;
  const int lo = t * per < m ? t * per : m, hi = lo + per < m ? lo + per : m;
  int64_t acc = 0;
  for (int p = lo; p < hi; ++p) acc += C->sort_cnt[p];
  int64_t total;
  int64_t run = block_exclusive_scan_t<int64_t>(acc, sRed, &total);
  if (t == 0) C->sort_cnt[C->ng] = total;
  for (int p = lo; p < hi; ++p) {
    const int64_t v = C->sort_cnt[p];
    C->sort_cnt[p] = run;
    run += v;
  }
}

__global__ void __launch_bounds__(256) k_sort_scatter(const BlockRole* __restrict__ R, int sp, int every,
                                                      int dstep) {
  extern __shared__ double ssm[];
  const EDP_CONST BlockRole* r = KC(R) + blockIdx.x;
  CaseDev* C = r->c;
  int64_t s;
  if (!sort_due(r, sp, every, dstep, s)) return;
  unsigned int* sC = (unsigned int*)ssm;
  unsigned long long* sB = (unsigned long long*)(ssm + (C->ng + 1) / 2);
  const int ng = C->ng;
  for (int p = threadIdx.x; p < ng; p += blockDim.x) sC[p] = 0;
  __syncthreads();
  const int cur = C->cur[sp], nxt = cur ^ 1;
  const SpeciesDev& S = C->sp[sp];
  const EDP_GLOBAL double* __restrict__ X = G(S.x[cur]);
  const int64_t n = step_slots(KC(C), sp, (int)(s % 3));
  const int64_t nb = r->n, per = (n + nb - 1) / nb;
  const int64_t lo = (int64_t)r->j * per, hi = lo + per < n ? lo + per : n;
  const double inv_dx = C->inv_dx;
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += kSortUnroll * kBlock) {
    double x[kSortUnroll];
#pragma unroll
    for (int u = 0; u < kSortUnroll; ++u) {
      const int64_t i = i0 + u * kBlock;
      x[u] = i < hi ? X[i] : __longlong_as_double(0x7FF8000000000000LL);
    }
#pragma unroll
    for (int u = 0; u < kSortUnroll; ++u)
      if (x[u] == x[u]) atomicAdd(&sC[cell_of(x[u], inv_dx, ng)], 1u);
  }
  __syncthreads();
  for (int p = threadIdx.x; p < ng - 1; p += blockDim.x) {
    const unsigned int c = sC[p];
    sB[p] = c ? gl_fetch_add(&C->sort_cnt[p], (unsigned long long)c) : 0ull;
    sC[p] = 0;
  }
  __syncthreads();
  const EDP_GLOBAL double* __restrict__ VX = G(S.vx[cur]);
  const EDP_GLOBAL double* __restrict__ VY = G(S.vy[cur]);
  const EDP_GLOBAL double* __restrict__ VZ = G(S.vz[cur]);
  const EDP_GLOBAL uint64_t* __restrict__ UID = G(S.uid[cur]);
  EDP_GLOBAL double* __restrict__ X2 = G(S.x[nxt]);
  EDP_GLOBAL double* __restrict__ VX2 = G(S.vx[nxt]);
  EDP_GLOBAL double* __restrict__ VY2 = G(S.vy[nxt]);
  EDP_GLOBAL double* __restrict__ VZ2 = G(S.vz[nxt]);
  EDP_GLOBAL uint64_t* __restrict__ UID2 = G(S.uid[nxt]);
  // electrons also carry vy*vy + vz*vz: formed again from the moved vy and
  // vz, as every writer forms it, rather than read
  const bool p2 = sp == 0;
  EDP_GLOBAL float* __restrict__ VP22 = G(S.vp2[nxt]);
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += kSortUnroll * kBlock) {
    double x[kSortUnroll], vx[kSortUnroll], vy[kSortUnroll], vz[kSortUnroll];
    uint64_t uid[kSortUnroll];
#pragma unroll
    for (int u = 0; u < kSortUnroll; ++u) {
      const int64_t i = i0 + u * kBlock;
      x[u] = __longlong_as_double(0x7FF8000000000000LL);
      if (i < hi) {
        x[u] = X[i];
        vx[u] = VX[i];
        vy[u] = VY[i];
        vz[u] = VZ[i];
        uid[u] = UID[i];
      }
    }
#pragma unroll
    for (int u = 0; u < kSortUnroll; ++u) {
      if (!(x[u] == x[u])) continue;
      const int c = cell_of(x[u], inv_dx, ng);
      const int64_t d = (int64_t)sB[c] + atomicAdd(&sC[c], 1u);
      X2[d] = x[u];
      VX2[d] = vx[u];
      VY2[d] = vy[u];
      VZ2[d] = vz[u];
      UID2[d] = uid[u];
      if (p2) VP22[d] = float_above(vy[u] * vy[u] + vz[u] * vz[u]);
    }
  }
}

__global__ void k_sort_finish(const BlockRole* __restrict__ R, int sp, int every, int dstep) {
  const EDP_CONST BlockRole* r = KC(R) + blockIdx.x;
  CaseDev* C = r->c;
  int64_t s;
  if (!sort_due(r, sp, every, dstep, s)) return;
  const int ng = C->ng;
  if (threadIdx.x == 0) {
    // the step's slot count: the live particles, now in the other set
    C->nbase[sp][(s + 2) % 3] = C->sort_cnt[ng];
    C->born[sp][(s + 2) % 3] = 0;
    C->cur[sp] ^= 1;
  }
  __syncthreads();
  for (int p = threadIdx.x; p <= ng; p += blockDim.x) C->sort_cnt[p] = 0;
}

// Fold the pending per-step diagnostic sums of the last completed step.
__global__ void k_fold_diag(CaseDev* __restrict__ Cw) {
  const EDP_CONST CaseDev* __restrict__ C = KC(Cw);
  const int ng = C->ng;
  const int64_t s = Cw->step;  // next step to run; the pending sums are those of s-1
  const int64_t off = ((s + 2) % 3) * ng;
  if (!(C->flags & (kDiagCurrent | kDiagMeanE | kDiagXT))) return;
  const int64_t nt = C->nt, nxb = C->n_xt_bin;
  const size_t plane = (size_t)C->n_xt * (size_t)ng;
  const size_t row_prev = (C->flags & kDiagXT) ? (size_t)(((s + nt - 1) % nt) / nxb) * (size_t)ng : 0;
  for (int p = threadIdx.x; p < ng; p += blockDim.x) fold_particle_sums(C, p, off, row_prev, plane);
}

__global__ void k_zero(int64_t* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// Workgroups (b, *) copy part b (see GatherPart).  One side is host memory: a
// result of a few KiB leaves in one launch and one wait, where a copy of each
// part took about 15 us.
__global__ void __launch_bounds__(kBlock) k_gather(const CaseDev* __restrict__ C, GatherParts P) {
  const GatherPart& q = P.p[blockIdx.x];
  const int64_t s = C->step;
  const int64_t row = q.sel == 0 ? 0 : (q.sel == 1 ? s : s / C->nsub) % 3;
  const int64_t* __restrict__ src = q.src + row * q.n;
  for (int i = (int)(blockIdx.y * kBlock + threadIdx.x); i < q.n; i += (int)gridDim.y * kBlock) q.dst[i] = src[i];
}

// Before a window of the small-case kernel: workgroup b takes V(t) of role
// b's role.j steps from the host's copy into the case's ring.
__global__ void __launch_bounds__(kBlock) k_small_volt(const BlockRole* __restrict__ R) {
  const BlockRole& r = R[blockIdx.x];
  const double* __restrict__ src = r.c->volt_host;
  double* dst = const_cast<double*>(r.c->volt);
  const int64_t s0 = r.c->step;
  for (int i = threadIdx.x; i < r.j; i += kBlock) dst[(s0 + i) % kVoltChunk] = src[(s0 + i) % kVoltChunk];
}

// After a case's last window: its slot counts and counters for the host's
// launch sizes.
__global__ void __launch_bounds__(kWave) k_small_end(const BlockRole* __restrict__ R) {
  constexpr int n = (int)((offsetof(CaseDev, ctr) - offsetof(CaseDev, alloc)) / 8) + kNumCtr;
  const CaseDev* C = R[blockIdx.x].c;
  for (int i = threadIdx.x; i < n; i += kWave) C->est_host[i] = ((const int64_t*)C->alloc)[i];
}

// ---------------------------------------------------------------------------
// Host-side launchers (same translation unit as the kernels).
// ---------------------------------------------------------------------------
// Static LDS of a species' particle kernel: the candidate segments with
// their payload and the ionizing lanes, the pre-test's bound, plus a bound on
// the counters and the field scan's scratch.
size_t particle_static_lds(int sp, int nb) {
  const size_t waves = (size_t)nb / kWave;
  return (sp == 0 ? waves * (kSegE * (4 + 8 + 8) + kWave * 4) : waves * kSegI * 4) + kMaxPb * 4 + 1024;
}

size_t particle_lds_bytes(int ng, uint32_t flags, int n_eepf, int n_ifed, int sp) {
  size_t doubles = (size_t)2 * ng;
  if (flags & kDiagParticle) {
    doubles += (size_t)3 * ng + (sp == 0 && (flags & kDiagXT) ? (size_t)ng : 0);
    const size_t hist = sp == 0 ? ((flags & kDiagEepf) ? (size_t)n_eepf : 0)
                                : ((flags & kDiagIfed) ? 2 * (size_t)(n_ifed + 1) : 0);
    doubles += (hist + 1) / 2;
  }
  return doubles * 8;
}

// One species of a window step of a batch: `blocks` workgroups with their
// roles and nb threads each; `lds` = the largest per-case need; mode 1: the Thomas solve.  With
// ev0/ev1 the launch records its own start and end (the dispatch's
// timestamps, not those of separate event packets around it).
template <int SP, int MODE, int NB>
void launch_particles_t(const BlockRole* roles, int blocks, size_t lds, int dstep, int pretest, hipStream_t st, hipEvent_t ev0,
                        hipEvent_t ev1) {
  if (ev0)
    hipExtLaunchKernelGGL((k_particles<SP, MODE, NB>), dim3(blocks), dim3(NB), lds, st, ev0, ev1, 0, roles, dstep, pretest);
  else
    hipLaunchKernelGGL((k_particles<SP, MODE, NB>), dim3(blocks), dim3(NB), lds, st, roles, dstep, pretest);
}

template <int NB>
void launch_particles_nb(const BlockRole* roles, int sp, int blocks, size_t lds, int mode, int dstep, int pretest,
                         hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  switch (sp * 2 + (mode == 1)) {
    case 0: launch_particles_t<0, 0, NB>(roles, blocks, lds, dstep, pretest, st, ev0, ev1); break;
    case 1: launch_particles_t<0, 1, NB>(roles, blocks, lds, dstep, pretest, st, ev0, ev1); break;
    case 2: launch_particles_t<1, 0, NB>(roles, blocks, lds, dstep, pretest, st, ev0, ev1); break;
    default: launch_particles_t<1, 1, NB>(roles, blocks, lds, dstep, pretest, st, ev0, ev1); break;
  }
}

hipError_t launch_particles(const BlockRole* roles, int sp, int blocks, int nb, size_t lds, int mode, int dstep,
                            int pretest, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (nb == 512)
    launch_particles_nb<512>(roles, sp, blocks, lds, mode, dstep, pretest, st, ev0, ev1);
  else
    launch_particles_nb<256>(roles, sp, blocks, lds, mode, dstep, pretest, st, ev0, ev1);
  return hipGetLastError();
}

// The first and last kernels of a lockstep window (see k_window_begin and
// k_window_end): `roles` the group's nroles roles, `cases` its ncase case
// roles.
hipError_t launch_window_begin(BlockRole* roles, int nroles, const BlockRole* cases, int ncase, hipStream_t st) {
  const int blocks = ncase + (nroles + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(k_window_begin, dim3(blocks), dim3(kBlock), 0, st, roles, nroles, cases, ncase);
  return hipGetLastError();
}

hipError_t launch_window_end(const BlockRole* cases, int ncase, int steps, hipStream_t st) {
  hipLaunchKernelGGL(k_window_end, dim3(ncase), dim3(kBlock), 0, st, cases, steps);
  return hipGetLastError();
}

// Resident workgroups (of nb threads) per CU of a species' particle kernel with `lds` bytes
// of dynamic LDS.  A CU gives its 160 KiB out in granules of 1280 bytes, which
// the runtime's answer does not count: with every measurement on 696 to 713
// nodes it says three, two fit, and a launch of three a CU took 47.5 us a step
// (1e6 electrons) where two take 36.
template <int SP, int NB>
int particle_occupancy_t(size_t lds) {
  constexpr size_t kLds = 160 << 10, kGranule = 1280;
  int n = 0;
  hipFuncAttributes a;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_particles<SP, 0, NB>, NB, lds) != hipSuccess || n < 1 ||
      hipFuncGetAttributes(&a, (const void*)k_particles<SP, 0, NB>) != hipSuccess)
    return 1;
  const size_t granules = (lds + a.sharedSizeBytes + kGranule - 1) / kGranule;
  const size_t fit = kLds / (std::max<size_t>(1, granules) * kGranule);
  return std::max(1, std::min(n, (int)fit));
}
int particle_occupancy(int sp, int nb, size_t lds) {
  if (nb == 512) return sp == 0 ? particle_occupancy_t<0, 512>(lds) : particle_occupancy_t<1, 512>(lds);
  return sp == 0 ? particle_occupancy_t<0, 256>(lds) : particle_occupancy_t<1, 256>(lds);
}

// Dynamic LDS of the small-case kernel with nb threads for a case (see k_small).
size_t small_lds_bytes(int nb, int ng, uint32_t flags, int n_eepf, int n_ifed) {
  size_t sums = 0;  // of either species beyond E and the deposit
  for (int sp = 0; sp < 2; ++sp) {
    const size_t r = particle_lds_bytes(ng, flags, n_eepf, n_ifed, sp) / 8 - 2 * (size_t)ng;
    sums = sums > r ? sums : r;
  }
  return ((size_t)(nb == 512 ? 5 : 2) * ng + sums) * 8;
}

size_t small_static_lds(int nb) {
  const size_t waves = (size_t)nb / kWave;
  return waves * (kSegE * (4 + 8 + 8) + kWave * 4 + kSegI * 4) + 2 * kMaxPb * 4 + 2048;
}

// One window of the small cases: workgroup b runs the case of roles[b] for
// roles[b].j steps.
hipError_t launch_small(const BlockRole* roles, int ncase, int nb, size_t lds, int mode, int sort_every, int pretest,
                        hipStream_t st) {
  if (nb == 512) {
    if (mode == 1)
      hipLaunchKernelGGL((k_small<1, 512>), dim3(ncase), dim3(512), lds, st, roles, sort_every, pretest);
    else
      hipLaunchKernelGGL((k_small<0, 512>), dim3(ncase), dim3(512), lds, st, roles, sort_every, pretest);
  } else if (mode == 1) {
    hipLaunchKernelGGL((k_small<1, 256>), dim3(ncase), dim3(256), lds, st, roles, sort_every, pretest);
  } else {
    hipLaunchKernelGGL((k_small<0, 256>), dim3(ncase), dim3(256), lds, st, roles, sort_every, pretest);
  }
  return hipGetLastError();
}

hipError_t launch_gather(const CaseDev* c, const GatherParts& P, int n, int blocks, hipStream_t st) {
  hipLaunchKernelGGL(k_gather, dim3(n, blocks), dim3(kBlock), 0, st, c, P);
  return hipGetLastError();
}

hipError_t launch_small_volt(const BlockRole* roles, int ncase, hipStream_t st) {
  hipLaunchKernelGGL(k_small_volt, dim3(ncase), dim3(kBlock), 0, st, roles);
  return hipGetLastError();
}

hipError_t launch_small_end(const BlockRole* roles, int ncase, hipStream_t st) {
  hipLaunchKernelGGL(k_small_end, dim3(ncase), dim3(kWave), 0, st, roles);
  return hipGetLastError();
}

hipError_t launch_zero(void* p, int64_t bytes, hipStream_t st) {
  const int64_t n = bytes / 8;
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(256), 0, st, (int64_t*)p, n);
  return hipGetLastError();
}

hipError_t launch_seed(CaseDev* d, int sp, int64_t n, double sigma, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(k_seed, dim3((unsigned)blocks), dim3(256), 0, st, d, sp, n, sigma);
  return hipGetLastError();
}

hipError_t launch_deposit(CaseDev* d, int sp, int64_t* dst1, int64_t* dst2, int ng, int blocks,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_deposit, dim3(blocks), dim3(256), (size_t)ng * 8, st, d, sp, dst1, dst2);
  return hipGetLastError();
}

// Compaction + cell sort of species sp for every case of a batch that is due
// (see sort_due): `blocks` workgroups with roles `roles` for the histogram
// and the scatter, one per case (`case_roles`, ncase of them) for the scan
// and the finish; `max_ng` sizes the LDS.
hipError_t launch_sort(const BlockRole* roles, const BlockRole* case_roles, int sp, int blocks, int ncase, int max_ng,
                       int every, int dstep, hipStream_t st) {
  hipLaunchKernelGGL(k_sort_hist, dim3(blocks), dim3(256), (size_t)max_ng * 4, st, roles, sp, every, dstep);
  hipLaunchKernelGGL(k_sort_scan, dim3(ncase), dim3(1024), 0, st, case_roles, sp, every, dstep);
  const size_t lds = (size_t)((max_ng + 1) / 2) * 8 + (size_t)max_ng * 8;
  hipLaunchKernelGGL(k_sort_scatter, dim3(blocks), dim3(256), lds, st, roles, sp, every, dstep);
  hipLaunchKernelGGL(k_sort_finish, dim3(ncase), dim3(1024), 0, st, case_roles, sp, every, dstep);
  return hipGetLastError();
}

hipError_t launch_fold(CaseDev* d, hipStream_t st) {
  hipLaunchKernelGGL(k_fold_diag, dim3(1), dim3(1024), 0, st, d);
  return hipGetLastError();
}

}  // namespace edp
