// Fused space-time solver: a team of G workgroups owns one sample at a time
// and runs its whole nonlinear space-time solve without leaving the kernel.
//
// Method (Sec. 3.3 eq. mono_disc, Sec. 3.5): the backward-Euler space-time
// system is block lower bidiagonal, so Newton's method on it can be carried
// out slab by slab in time order (block forward substitution, eq. system_C):
// slab k is iterated with Newton steps A_k delta = -R_k until its correction is
// below tolerance, given the converged slab k-1.  On one grid a step is a defect
// correction, delta = P(A_k) (-R_k) with P the Chebyshev iteration on the
// spectrum of D^-1 A_k: the residual is evaluated anyway before the next step,
// so a Krylov space would only repeat its work (per slab about 45 sweeps in 2D and
// 80 in 3D, in three corrections, take the place of 60-70 and 100-120 inside GMRES
// with its products, dots and updates: with the passes of that time 33^2 x 64 steps
// 20.5 -> 8.9 ms, 129^2 x 64 x 32 samples 52.4 -> 25.5 ms, 65x65x17 x 32 x 16
// 98 -> 59 ms; with those of now 5.2, 14.2 and 37).
// Where it does not contract, and with a V-cycle, the linear step is GMRES,
// right-preconditioned by one geometric-multigrid V-cycle with weighted-Jacobi
// smoothing on the slab operator A_k = M/dt + K - M diag f'(u_k) (with one
// grid the V-cycle reduces to its smoothing sweeps).  The Jacobi weights are
// either fixed or the reciprocal Chebyshev roots of an interval
// [lmax/ratio, lmax] of D^-1 A, lmax estimated by power iteration once per
// sample.  The initial iterate of slab k takes the time increment of a
// previous solution (u_{k-1} + W_k - W_{k-1}; the paper initialises Newton
// from already computed samples) or, without one, u_{k-1}.  The activation
// map is updated as each slab is accepted.
//
// Teams: with G = 1 a workgroup owns the sample.  With G > 1 (levels without
// coarse V-cycle grids) member r owns a box of the grid (Team::set_box): a band
// of node rows, in 3D of one group of planes;
// passes end with a team barrier (agent-scope release/acquire around an
// atomic counter, bounded wait) and reductions sum the members' partials in
// rank order, so every member takes identical control-flow decisions.  Such
// launches are cooperative: co-residency is guaranteed or the launch fails.
//
// Memory: stencil passes stage tiles of their nodal fields and element
// conductivities into LDS with batched loads, compute each element's vertex
// contributions once (sum factorisation) and gather them per node, on the
// level's grid and on every coarse V-cycle grid alike; restriction and
// prolongation between grids are plain loops over global memory.
//
// Precision: the residual R_k, the update u += delta, the activation
// interpolation and every stored solution are float64.  The Krylov and
// multigrid vectors use TI (double, or float for iterative refinement).
#include "stm_device.h"
#include "q1_stencil.h"
#include "stm_launch.h"

namespace stm {

// A node as a pass hands it to its body: a uniform base and the thread's number
// from there, which together are the node's index.  node_ref forms the address
// from a uniform pointer and a 32-bit offset.
struct NodeAt {
  int base;
  unsigned q;
  __device__ __forceinline__ operator int() const { return base + (int)q; }
};

// Optional per-phase timers (development builds with -DSTM_PHASE_TIMERS):
// thread 0 accumulates wall-clock ticks of each solver phase.
#ifdef STM_PHASE_TIMERS
#define STM_T0(v) long long v = wall_clock64()
#define STM_T1(v, slot) \
  if (threadIdx.x == 0) ph_acc[slot] += wall_clock64() - v
#define STM_T1P(v, slot) \
  if (threadIdx.x == 0) ph[slot] += wall_clock64() - v
#else
#define STM_T0(v)
#define STM_T1(v, slot)
#define STM_T1P(v, slot)
#endif

// A wave-uniform float64 value moved to scalar registers: uniform solver state
// (tolerances, norms, step sizes) then stays out of the vector register file,
// which the stencil passes need.
__device__ __forceinline__ double uni(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffff));
  const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// |v| for a maximum: fmax drops a NaN, so a value that is not finite counts as infinite.
__device__ __forceinline__ double abs_or_inf(double v) {
  const double a = fabs(v);
  return a < HUGE_VAL ? a : HUGE_VAL;
}

// Global-memory views of generic pointers.  An access through a generic
// pointer that the compiler cannot place compiles to a flat instruction, and
// flat instructions count against the LDS wait counter as well: every LDS wait
// of a pass would then also wait for the pass's global loads and stores in
// flight.  Device arrays are global; these views make their accesses global
// (cmem: read-only tables, loaded through the scalar cache when uniform).
#define STM_GLOBAL __attribute__((address_space(1)))
#define STM_CONST __attribute__((address_space(4)))
template <typename T>
__device__ __forceinline__ STM_GLOBAL T* gmem(T* p) {
  return (STM_GLOBAL T*)p;
}
template <typename T>
__device__ __forceinline__ const STM_GLOBAL T* gmem(const T* p) {
  return (const STM_GLOBAL T*)p;
}
template <typename T>
__device__ __forceinline__ const STM_CONST T* cmem(const T* p) {
  return (const STM_CONST T*)p;
}

template <typename T>
__device__ __forceinline__ STM_GLOBAL T& node_ref(T* p, NodeAt at) {
  return gmem(p + at.base)[at.q];
}

// A uniform pointer as of here: what a pass derives from it is not computed
// ahead of the loops around the pass.  Without this every pass's tile sizes and
// addresses stay live over the whole solve, and their spills (SGPRs to VGPR
// lanes, 60-100 v_readlane per z-step) cost the passes.
template <typename P>
__device__ __forceinline__ P* here(P* p) {
  asm volatile("" : "+s"(p));
  return p;
}

// The stiffness argument c * v of a pass (kval(v, .) = c v).  The 3D pass
// folds c into the element's conductivity factors instead of scaling the
// eight vertex values; for c a power of two (the theta of backward Euler and
// Crank-Nicolson, 1 - theta) both give the same floating-point result.
template <typename T>
struct KScale {
  T c;
  __device__ __forceinline__ T operator()(T a, T) const { return c * a; }
};
template <typename F>
struct IsKScale {
  static constexpr bool value = false;
};
template <typename T>
struct IsKScale<KScale<T>> {
  static constexpr bool value = true;
};

// Storage type of the element conductivities a 3D pass in T reads.
template <typename T>
struct SigmaOf {
  using type = double;
};
template <>
struct SigmaOf<float> {
  using type = float;
};

constexpr int kWaitVm = 0x0f70;       // s_waitcnt operand: vector memory operations only
constexpr int kDeviceScope = 16;       // cache policy of a load: device scope (sc1)
constexpr int kPartStride = 16;       // doubles per member in the partials buffer
constexpr double kMinStep = 1.0 / 64;  // smallest damped fraction of a Newton step
constexpr unsigned kSpinLimit = 1u << 25;
// Defect corrections by Chebyshev sweeps.  A slab keeps to them while each
// contracts the residual by kContract; after more than kMaxFallbacks slabs in a
// row that did not, the sample gives them up for GMRES.
constexpr double kContract = 0.1;
constexpr int kMaxFallbacks = 2;
constexpr int kMaxCorrections = 16;  // per slab
// A correction's degree follows from the error reduction wanted of it, in bits
// (log2): kFirstBits of a slab's first one, whose remainder Newton's own exceeds
// soon (10 bits in 2D, where a correction costs as much as 25 sweeps, 6.5 in 3D,
// where it costs 5: 32 samples of 129x129 nodes 9.7 ms, 10.9 with 7), at least
// kLeastBits, well inside kContract, and with float32 sweeps at most kFloatBits.
// A slab is accepted with an error of kLeft newton_tol.  Drawn solves are then 8e-14 off
// in the median, 5e-13 at most, with newton_tol 1e-10; kLeft 1e-5 makes it 9e-16
// and 2e-15 for 1.11 of the time.
// Corrections are for spectra up to kWidest: 48 sweeps give 7 bits there.  7x33 nodes
// x 10 steps, 5 samples, lmax about 100 times the smallest eigenvalue, mixed: 7.5 ms,
// 16.9 by GMRES alone (float32 sweeps lose too much to rounding on the widest
// spectra; such slabs end in GMRES).
constexpr double kWidest = 300.0;
constexpr int kMaxDegree = 48;
constexpr float kFirstBits2 = 10.0f, kFirstBits3 = 6.5f, kLeastBits = 5.0f, kFloatBits = 20.0f;
constexpr double kLeft = 1e-3;
constexpr double kRounding = 1e-15;  // u is O(1)

template <int DIM>
__device__ __forceinline__ void decode(const GridDev& g, int idx, int& i, int& j, int& k) {
  const int r = fdiv(idx, g.mnx);
  i = idx - r * g.nx;
  if constexpr (DIM == 2) {
    j = r;
    k = 0;
  } else {
    k = fdiv(r, g.mny);
    j = r - k * g.ny;
  }
}

template <typename T, int DIM>
struct TensorOf;
template <typename T>
struct TensorOf<T, 2> { using type = Tensor2<T>; };
template <typename T>
struct TensorOf<T, 3> { using type = Tensor3<T>; };

// Element tensor from the fibre conductivity s and the fibre-table row f
// (kFibStride entries; the layout is described with kFibStride); zr is uniform.
template <typename T, int DIM>
__device__ __forceinline__ typename TensorOf<T, DIM>::type tensor_from(double s, const double* __restrict__ f,
                                                                       double tau, double zr) {
  const double c2 = f[0], s2 = f[1], cs = f[2];
  if constexpr (DIM == 2) {
    return Tensor2<T>{T(s * c2 + tau * s2), T(s * s2 + tau * c2), T((s - tau) * cs)};
  } else {
    return Tensor3<T>{T(s * c2 + tau * s2), T(s * s2 + tau * c2), T(fma(s, zr, tau)), T((s - tau) * cs)};
  }
}

template <typename T, int DIM>
__device__ __forceinline__ typename TensorOf<T, DIM>::type tensor_stored(const T* __restrict__ D,
                                                                         const GridDev& g, int ex, int ey,
                                                                         int ez) {
  const int e = (DIM == 2) ? (ey * g.ex + ex) : ((ez * g.ey + ey) * g.ex + ex);
  if constexpr (DIM == 2) {
    return Tensor2<T>{D[4 * e], D[4 * e + 1], D[4 * e + 3]};
  } else {
    return Tensor3<T>{D[4 * e], D[4 * e + 1], D[4 * e + 2], D[4 * e + 3]};
  }
}

// y = M fm + K fk at node (i, j, k); accessors take coordinates.
template <typename T, int DIM, typename FM, typename FK, typename FD>
__device__ __forceinline__ T apply_at(const GridDev& g, int i, int j, int k, FM fm, FK fk, FD fd, T wself,
                                      T* diag) {
  if constexpr (DIM == 2) {
    return q1_apply_2d<T>(g, i, j, [&](int a, int b) { return fm(a, b, 0); },
                          [&](int a, int b) { return fk(a, b, 0); }, [&](int ex, int ey) { return fd(ex, ey, 0); },
                          wself, diag);
  } else {
    return q1_apply_3d<T>(g, i, j, k, fm, fk, fd, wself, diag);
  }
}

__device__ __forceinline__ double react(double u, double kr, double ar) { return kr * u * (u - ar) * (1.0 - u); }
__device__ __forceinline__ double react_d(double u, double kr, double ar) {
  return kr * (-3.0 * u * u + 2.0 * (1.0 + ar) * u - ar);
}

// Weights 1 / xi_s, xi_s the roots of the degree-K Chebyshev polynomial
// shifted to [a, b], ordered to alternate large and small roots: every `stride`-th
// from s0 on.
__device__ inline void chebyshev_weights(double a, double b, int K, double* w, int s0 = 0, int stride = 1) {
  const double th = 0.5 * (b + a), de = 0.5 * (b - a);
  const double PI = 3.14159265358979323846;
  for (int s = s0; s < K; s += stride) {
    const int r = (s % 2 == 0) ? s / 2 : K - 1 - s / 2;
    const double xi = th + de * cos(PI * (2 * r + 1) / (2.0 * K));
    w[s] = 1.0 / xi;
  }
}

// What the steps of a solve take and give (dmax and resid also carry the two ends
// of the spectrum).
struct StepIO {
  double *u, *uprev, *dlt;
  double beta, eta, krylov_words;
  double model_bytes;
  double dmax;         // max-norm of the step
  double resid;        // residual norm reached (residual step: its square)
  int jdim;            // Krylov iterations
  int x1, nc;          // the correction's first sweep is the residual step's; its sweeps
};

// MG: the launch contains a level with a multigrid hierarchy.  Without one the
// V-cycle is the Chebyshev-weighted sweeps on the level's grid and no
// coarse-grid code is compiled into the kernel (it would cost registers).
template <typename TI, int DIM, int BLOCK, bool MG>
struct Team {
  const LevelDev* L;
  SolverParams prm;
  const double* sigma;
  TI *V, *Z;
  int64_t vstride;
  unsigned char* work;
  unsigned char* smem;   // dynamic LDS staging area
  double* kdiag0;        // diagonal of the stiffness matrix on grid 0 (per sample)
  TI* dinv;              // inverse diagonal of the slab operator on grid 0 (per Newton step)
  TI* w0;                // reaction weights 1/dt - f'(u) of the slab operator on grid 0
  double* omega;         // shared: per grid, the sweep weights [kMaxMG][kMaxSweeps]
  double* red;           // shared: block reduction scratch
  // team membership
  int rank, G;
  int jb0, jb1;          // owned node rows of grid 0
  int kb0, kb1;          // owned node planes of grid 0 (3D; 0, 1 in 2D)
  unsigned* bar;
  double* part;
  int* fault;
  mutable unsigned gen;  // barriers passed
  mutable unsigned hgen;  // halo barriers passed
  int gy, gz;            // the team's members along y and z (rank = iy gz + iz)
  mutable unsigned rslot;  // reductions done (partials double buffer)
  mutable bool broken;   // a barrier wait timed out: stop waiting
  // Algorithmic bytes of the passes run so far: every array a pass reads or
  // writes counted once per pass (neighbour and halo re-reads are cache/LDS
  // traffic, not counted).  Uniform across the team; rank 0 reports it.
  mutable double bytes;
#ifdef STM_PHASE_TIMERS
  long long* ph;         // shared per-phase tick accumulators
#endif

  __device__ __forceinline__ double dbytes(int l) const { return 8.0 * L->g[l].ne; }
  __device__ __forceinline__ TI* mgX(int l) const {
    return l == 0 ? nullptr : reinterpret_cast<TI*>(work + L->off_mgX[l]);
  }
  __device__ __forceinline__ TI* mgT(int l) const { return reinterpret_cast<TI*>(work + L->off_mgT[l]); }
  __device__ __forceinline__ TI* mgB(int l) const { return reinterpret_cast<TI*>(work + L->off_mgB[l]); }
  __device__ __forceinline__ TI* mgW(int l) const {
    return l == 0 ? w0 : reinterpret_cast<TI*>(work + L->off_mgW[l]);
  }
  // inverse slab diagonal, conductivities and stiffness diagonal of grid l
  __device__ __forceinline__ TI* mgI(int l) const {
    return l == 0 ? dinv : reinterpret_cast<TI*>(work + L->off_mgI[l]);
  }
  __device__ __forceinline__ const double* mgS(int l) const {
    return l == 0 ? sigma : reinterpret_cast<const double*>(work + L->off_mgS[l]);
  }
  // conductivities of grid l in the precision of a 3D pass in T (float32:
  // the copy made once per sample)
  template <typename T>
  __device__ __forceinline__ const typename SigmaOf<T>::type* mgST(int l) const {
    if constexpr (sizeof(T) == 4)
      return reinterpret_cast<const float*>(work + L->off_mgS32[l]);
    else
      return mgS(l);
  }
  __device__ __forceinline__ double* mgK(int l) const {
    return l == 0 ? kdiag0 : reinterpret_cast<double*>(work + L->off_mgK[l]);
  }

  // ---- team synchronisation and reductions --------------------------------
  // Every wave first waits until its own global stores have completed (a
  // workgroup barrier alone does not wait for them); thread 0 then releases
  // the block's writes at agent scope (write-back of the L2), arrives, waits
  // for the other members and acquires, which invalidates the CU's caches for
  // every wave of the block.
  __device__ __forceinline__ void team_barrier() const {
    if (G > 1) __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (G > 1) {
      if (threadIdx.x == 0) {
        gen += 1;
        if (!broken) {
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
          __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const unsigned target = gen * (unsigned)G;
          unsigned spins = 0;
          while (__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins > kSpinLimit) {
              broken = true;
              __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              break;
            }
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
      }
      __syncthreads();
    }
  }
  // Barrier between two sweeps of a correction.  A sweep reads of the other
  // members only the adjacent ones' boundary values of x, and x is exchanged
  // past the caches: stored and loaded with agent-scope accesses (coh_store,
  // the coherent loads of the passes), which need no write-back and no
  // invalidation.  So every member waits for its neighbours' flags only, the L2
  // keeps the fields that a sweep only reads, and a member that is late delays
  // its neighbours and not the team.  A neighbour's flag also says that it has
  // read what the member overwrites next.
  __device__ __forceinline__ unsigned* halo_flag(int r) const {
    return reinterpret_cast<unsigned*>(part + r * kPartStride + kPartStride - 1);  // a word the partials leave free
  }
  __device__ __forceinline__ void halo_barrier() const {
    if (G == 1) {
      __syncthreads();
      return;
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    hgen += 1;
    if (threadIdx.x < kWave) {
      const int lane = threadIdx.x;
      if (lane == 0) __hip_atomic_store(halo_flag(rank), hgen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int iy = rank / gz + lane / 3 - 1, iz = rank % gz + lane % 3 - 1;
      const bool adjacent = lane < 9 && lane != 4 && iy >= 0 && iy < gy && iz >= 0 && iz < gz;
      const unsigned* f = halo_flag(adjacent ? iy * gz + iz : rank);
      unsigned spins = 0;
      while (!broken) {
        const bool there = !adjacent || (int)(__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - hgen) >= 0;
        if (__all(there)) break;
        __builtin_amdgcn_s_sleep(1);
        if (++spins > kSpinLimit) {
          broken = true;
          if (lane == 0) __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    __syncthreads();
  }
  // x of a sweep: past the caches when other members read it
  __device__ __forceinline__ void coh_store(STM_GLOBAL TI* p, TI v) const {
    if (G > 1)
      __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      *p = v;
  }
  // End of a pass whose results other members read.
  __device__ __forceinline__ void sync() const { team_barrier(); }

  template <int NV>
  __device__ __forceinline__ void tsum(double (&v)[NV]) const {
    block_sum<BLOCK, NV>(v, red);
    if (G == 1) return;
    double* slot = part + (size_t)(rslot & 1) * G * kPartStride;
    rslot += 1;
    if (threadIdx.x == 0)
      for (int i = 0; i < NV; ++i)
        __hip_atomic_store(slot + rank * kPartStride + i, v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    team_barrier();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      double s = 0.0;
      for (int r = 0; r < G; ++r)
        s += __hip_atomic_load(slot + r * kPartStride + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      v[i] = s;
    }
  }
  __device__ __forceinline__ double tmax(double v) const {
    v = block_max<BLOCK>(v, red);
    if (G == 1) return v;
    double* slot = part + (size_t)(rslot & 1) * G * kPartStride;
    rslot += 1;
    if (threadIdx.x == 0)
      __hip_atomic_store(slot + rank * kPartStride, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    team_barrier();
    double s = 0.0;
    for (int r = 0; r < G; ++r)
      s = fmax(s, __hip_atomic_load(slot + r * kPartStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return s;
  }

  // ---- owned nodes of grid 0 ----------------------------------------------
  static constexpr int kCE = march_columns(BLOCK), kCB = kCE;
  template <typename LP>
  __device__ __forceinline__ int zrows_max(LP Lp, int l, int fbytes) const {
    const auto& g = Lp->g[l];
    return march_rows(g.nx, g.ex, Lp->tile_y[l][fbytes == 8 ? 0 : 1][0], BLOCK);
  }
  // A member owns node rows [jb0, jb1) of planes [kb0, kb1) (3D), q-th in
  // plane-major order.
  __device__ __forceinline__ int nband() const {
    const GridDev& g = L->g[0];
    return (jb1 - jb0) * g.nx * ((DIM == 3) ? (kb1 - kb0) : 1);
  }
  __device__ __forceinline__ int bidx(int q) const {
    const GridDev& g = L->g[0];
    if constexpr (DIM == 2) {
      return jb0 * g.nx + q;
    } else {
      if (G == 1) return q;
      const int w = (jb1 - jb0) * g.nx;
      const int kk = q / w;
      return ((kb0 + kk) * g.ny + jb0) * g.nx + (q - kk * w);
    }
  }
  // The member's box of grid 0 (team_groups; the host launches only team sizes
  // that it divides).
  __device__ __forceinline__ void set_box() {
    const GridDev& g = L->g[0];
    int Gz = 1;
    if constexpr (DIM == 3) {
      int cost;
      Gz = max(1, team_groups(3, g.nx, g.ny, g.nz, zrows_max(L, 0, sizeof(TI)), G, &cost));
    }
    const int Gy = G / Gz, ry = rank / Gz, rz = rank - ry * Gz;
    gy = Gy;
    gz = Gz;
    jb0 = (int)((long long)ry * g.ny / Gy);
    jb1 = (int)((long long)(ry + 1) * g.ny / Gy);
    // the groups share the z-steps evenly, nz planes and Gz - 1 steps below a group
    const int steps = g.nz + Gz - 1;
    kb0 = (DIM == 3) ? (int)((long long)rz * steps / Gz) - max(rz - 1, 0) : 0;
    kb1 = (DIM == 3) ? (int)((long long)(rz + 1) * steps / Gz) - rz : 1;
  }

  // ---- staged pass on grid 0 ----------------------------------------------
  // For each tile of the owned rows: stage nodal fields f0, f1 (with a
  // one-node halo), f2, f3 (optional, may be null), the tile's element
  // conductivities and fibre rows into LDS, every thread issuing all of its
  // loads before using any; compute every element's vertex contributions of
  // M mval + K kval once (phase A, kval/mval from the raw f0, f1 values); sum
  // the adjacent elements' contributions per node (phase B) and call
  // body(idx, i, j, k, y, o0, o1, o2, o3) with o* the staged values at the
  // node.  Phases A and B read LDS only; every LDS array is laid out so that
  // consecutive lanes touch consecutive words.  Index decoding uses exact
  // multiply-high division.
  // Grid l >= 1 (a coarse V-cycle grid, one-workgroup teams) is staged the
  // same way, with its own conductivities, fibre rows and tiles, every row
  // owned.
  // NF: how many of f2, f3 there are.  publish = false leaves the closing team
  // barrier to the reduction that the caller starts right after the pass.
  // COH: f0 is read with agent-scope loads (3D; see halo_barrier).
  template <typename T, int NF, bool COH = false, typename KV, typename MV, typename Body>
  __device__ __forceinline__ void staged(int l, const T* __restrict__ f0, const T* __restrict__ f1, const T* __restrict__ f2,
                         const T* __restrict__ f3, KV kval, MV mval, Body body, bool publish = true) const {
    if constexpr (DIM == 3) {
      zmarch<T, NF, COH>(l, f0, f1, f2, f3, kval, mval, body);
    } else {
      staged_tiles<T>(l, f0, f1, f2, f3, kval, mval, body);
    }
    if (G > 1 && publish) team_barrier();
  }

  // ---- z-marching pass (3D) -------------------------------------------------
  // The owned rows of grid l are cut into y-tiles of Ry rows over the whole x
  // extent, and each tile marches through the owned planes [kb0, kb1), with
  // one step on the layer below kb0 first (its top-face contributions) when
  // kb0 > 0.  A thread keeps up to kCE element columns (q = thread + n BLOCK)
  // and kCB output columns for the whole march.  LDS holds a ring of three
  // planes of f0, f1 over the tile's rows plus a one-row halo and four partial
  // sums per element of one element layer with a border of zeros (one element
  // each side in x and y).  Step k:
  //   * loads to registers of the conductivities of layer k+1 and of f2, f3 on
  //     plane k, direct-to-LDS loads of plane k+2 of f0, f1 into the free slot;
  //   * phase A: the element operator of layer k in the basis of sums and
  //     differences along each axis, where mass is diagonal and stiffness
  //     nearly (q1_stencil.h).  The x-y transform of a face is formed once and
  //     kept in registers for the layer above, as is the layer's top half; its
  //     bottom half plus the kept one of layer k-1, transformed back, are the
  //     four sums the element gives plane k (to LDS);
  //   * an LDS-only barrier (the loads stay in flight);
  //   * phase B: every output node of plane k adds the sums of the four
  //     elements around it in its plane (the zero border stands for elements
  //     outside the grid) and calls body;
  //   * a wait for the step's loads before the first store of body, and an
  //     LDS-only barrier at the end (the stores stay in flight).
  // f0 and f1 are read from memory once per tile (plus the halo rows), f2, f3
  // and the conductivities once.  A stiffness argument kval = KScale{c} is
  // folded into the element factors.
  template <typename T, int NF, bool COH, typename KV, typename MV, typename Body>
  __device__ __forceinline__ void zmarch(int l, const T* __restrict__ f0, const T* __restrict__ f1,
                                         const T* __restrict__ f2, const T* __restrict__ f3, KV kval, MV mval,
                                         Body body) const {
    const STM_CONST LevelDev* __restrict__ Lp = cmem(here(L));
    const STM_CONST GridDev& g = Lp->g[l];
    const int nx = g.nx, ny = g.ny, nz = g.nz, EX = g.ex, EY = g.ey, EZ = g.ez;
    const unsigned mnx = g.mnx, mex = g.mex;
    const int plane = ny * nx, eplane = EY * EX;
    const int EXP = EX + 2;  // padded element row
    // tile rows: the LDS budget (set on the host) and the per-thread counts
    const int jb0 = l == 0 ? this->jb0 : 0, jb1 = l == 0 ? this->jb1 : ny;
    const int kb0 = l == 0 ? this->kb0 : 0, kb1 = l == 0 ? this->kb1 : nz;
    const int ks = max(kb0 - 1, 0);  // first step: the layer below the first owned plane
    const int Rmax = zrows_max(Lp, l, sizeof(T));
    // as few tiles as Rmax allows, of equal height
    const int ntl = (jb1 - jb0 + Rmax - 1) / Rmax;
    const int Ry = (jb1 - jb0 + ntl - 1) / max(ntl, 1);
    using TS = typename SigmaOf<T>::type;
    const STM_GLOBAL TS* __restrict__ sg = gmem(mgST<T>(l));
    const STM_CONST double* __restrict__ fib = cmem(Lp->fib[l]);
    const STM_GLOBAL T* __restrict__ g0 = gmem(f0);
    const STM_GLOBAL T* __restrict__ g1 = gmem(f1);
    const STM_GLOBAL T* __restrict__ g2 = gmem(f2);
    const STM_GLOBAL T* __restrict__ g3 = gmem(f3);
    const double tau = prm.tau, zr = prm.zr;
    const T hx = T(g.hx), hy = T(g.hy), hz = T(g.hz);
    // the stiffness scale of a KScale argument goes into the element factors
    T ksc = T(1);
    if constexpr (IsKScale<KV>::value) ksc = kval.c;
    const T cxx = ksc * (hy * hz / (T(48) * hx)), cyy = ksc * (hx * hz / (T(48) * hy));
    const T czz = ksc * (hx * hy / (T(48) * hz)), cxy = ksc * (hz / T(48));
    const T kz1 = T(zr) * czz, kz0 = T(tau) * czz, tauT = T(tau);
    const T c1 = hx * hy * hz / T(1728), c3 = T(3) * c1, c9 = T(9) * c1;
    const int tid = threadIdx.x;
    // the wave's first thread: a wave without an n-th column skips it
    const int wfirst = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
    constexpr int WT = sizeof(T) / 4;  // dwords per value
    for (int j0 = jb0; j0 < jb1; j0 += Ry) {
      const int je = min(j0 + Ry, jb1);          // output rows [j0, je)
      const int jr0 = max(j0 - 1, 0);            // staged node rows [jr0, jr1]; element rows start there too
      const int jr1 = min(je, ny - 1);
      const int ey1 = min(je - 1, EY - 1);       // element rows [jr0, ey1]
      const int lay = (jr1 - jr0 + 1) * nx;      // staged nodes per plane
      const int layp = (lay + 3) & ~3;           // slots of whole 16-byte words
      const int erows = ey1 - jr0 + 1;
      const int elay = erows * EX;               // elements per layer
      const int slay = (erows + 2) * EXP;        // padded sums per vertex slot
      const int nc = (je - j0) * nx;             // output nodes per plane
      const int gn0 = jr0 * nx, ge0 = jr0 * EX, go0 = j0 * nx;
      T* __restrict__ P = reinterpret_cast<T*>(smem);  // [3 slots][2][layp] f0, f1
      T* __restrict__ S = P + 6 * layp;                // [4][slay] sums for plane k
      auto load_plane = [&](int kp, int sl) {
        const size_t base = (size_t)kp * plane + gn0;
        if (COH && G > 1)
          dma_words<kDeviceScope>(reinterpret_cast<const STM_GLOBAL unsigned*>(g0 + base), P + (2 * sl) * layp,
                                  WT * lay, wfirst);
        else
          dma_words(reinterpret_cast<const STM_GLOBAL unsigned*>(g0 + base), P + (2 * sl) * layp, WT * lay, wfirst);
        dma_words(reinterpret_cast<const STM_GLOBAL unsigned*>(g1 + base), P + (2 * sl + 1) * layp, WT * lay, wfirst);
      };
      // prologue: planes ks and ks + 1, conductivities of layer ks, a zero
      // border around the sums, the thread's columns
      load_plane(ks, 0);
      load_plane(ks + 1, 1);
      int eo[kCE];                 // staged node of the element's vertex (0, 0)
      int es[kCE];                 // its sum slot
      unsigned qe[kCE], qn[kCB];   // the columns' numbers in the tile's layer and plane
      TS sc[kCE];
      T kb[kCE][4], mb[kCE][4];    // x-y transforms of the layer's bottom face
      T ac[kCE][4];                // top half of the layer below
#pragma unroll
      for (int n = 0; n < kCE; ++n) {
        // columns past the tile read column 0's values and write nothing
        const int q = tid + n * BLOCK, qq = q < elay ? q : 0;
        const int r = (int)fdiv(qq, mex);
        qe[n] = qq;
        eo[n] = qq + r;
        es[n] = eo[n] + r + EXP + 1;
        sc[n] = sg[(size_t)ks * eplane + ge0 + qq];
#pragma unroll
        for (int v = 0; v < 4; ++v) ac[n][v] = T(0);
      }
      int no[kCB], ns[kCB];        // staged node and lower left sum slot of the output nodes
#pragma unroll
      for (int n = 0; n < kCB; ++n) {
        const int q = tid + n * BLOCK, qq = q < nc ? q : 0;
        const int r = (int)fdiv(qq, mnx);
        qn[n] = qq;
        no[n] = (j0 - jr0) * nx + qq;
        ns[n] = (j0 - jr0 + r) * EXP + (qq - r * nx);
      }
      for (int q = tid; q < 4 * (2 * EXP + 2 * erows); q += BLOCK) {
        const int v = q & 3, b = q >> 2;
        const int at = b < EXP ? b
                       : b < 2 * EXP ? (erows + 1) * EXP + (b - EXP)
                                     : (1 + ((b - 2 * EXP) >> 1)) * EXP + (((b - 2 * EXP) & 1) ? EXP - 1 : 0);
        S[v * slay + at] = T(0);
      }
      auto corners = [&](const T* __restrict__ a, int o, T (&x)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = a[o + (v & 1) + (v >> 1) * nx];
      };
      auto face = [&](const T (&x0)[4], const T (&x1)[4], T (&kf)[4], T (&mf)[4]) {
        T kv[4], mv[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if constexpr (IsKScale<KV>::value)
            kv[v] = x0[v];
          else
            kv[v] = kval(x0[v], x1[v]);
          mv[v] = mval(x0[v], x1[v]);
        }
        face_transform<T>(kv, kf);
        face_transform<T>(mv, mf);
      };
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
#pragma unroll
      for (int n = 0; n < kCE; ++n) {
        if (wfirst + n * BLOCK >= elay) continue;
        T x0[4], x1[4];
        corners(P, eo[n], x0);
        corners(P + layp, eo[n], x1);
        face(x0, x1, kb[n], mb[n]);
      }
      // the layer's fibre row (uniform: scalar loads, a step ahead of their use)
      // folded with the element constants; each factor is affine in the conductivity
      double fc2 = fib[kFibStride * ks], fs2 = fib[kFibStride * ks + 1], fcs = fib[kFibStride * ks + 2];
      int s0 = 0;  // ring slot of plane k
      for (int k = ks; k < kb1; ++k) {
        const int s1 = s0 == 2 ? 0 : s0 + 1;
        const int s2 = s1 == 2 ? 0 : s1 + 1;
        STM_T0(t_za);
        // ---- loads: conductivities of layer k+1 when that layer is computed
        // (it adds to plane k+1 < kb1), f2, f3 of plane k, plane k+2 ----
        // (a uniform address plus the column's number, which takes no vector
        // arithmetic; a wave without an n-th column leaves its values undefined)
        TS sn[kCE];
        const int kn = k + 1 < min(kb1, EZ) ? k + 1 : min(k, EZ - 1);
        const STM_GLOBAL TS* __restrict__ sgk = sg + ((size_t)kn * eplane + ge0);
#pragma unroll
        for (int n = 0; n < kCE; ++n)
          if (wfirst + n * BLOCK < elay) sn[n] = sgk[qe[n]];
        T v2[kCB], v3[kCB];
        const size_t pk = (size_t)k * plane + go0;
        if (k >= kb0) {
#pragma unroll
          for (int n = 0; n < kCB; ++n) {
            if (wfirst + n * BLOCK < nc) {
              if constexpr (NF > 0) v2[n] = g2[pk + qn[n]];
              if constexpr (NF > 1) v3[n] = g3[pk + qn[n]];
            }
          }
        }
        if (k + 2 <= min(kb1, nz - 1)) load_plane(k + 2, s2);
        const T kx1 = T(fc2) * cxx, kx0 = T(tau * fs2) * cxx;
        const T ky1 = T(fs2) * cyy, ky0 = T(tau * fc2) * cyy;
        const T kxy = T(fcs) * cxy;
        fc2 = fib[kFibStride * kn];
        fs2 = fib[kFibStride * kn + 1];
        fcs = fib[kFibStride * kn + 2];
        // ---- phase A: element layer k ----
        auto sums = [&](int n, const T (&pl)[4]) {
          if (tid + n * BLOCK < elay) {
            const T lo = pl[0] - pl[2], hi = pl[0] + pl[2], dl = pl[1] - pl[3], dh = pl[1] + pl[3];
            S[es[n]] = lo - dl;
            S[slay + es[n]] = lo + dl;
            S[2 * slay + es[n]] = hi - dh;
            S[3 * slay + es[n]] = hi + dh;
          }
        };
        if (k < EZ) {
#pragma unroll
          for (int n = 0; n < kCE; ++n) {
            if (wfirst + n * BLOCK < elay) {
              T x0[4], x1[4], kt[4], mt[4], pl[4];
              corners(P + (2 * s1) * layp, eo[n], x0);
              corners(P + (2 * s1 + 1) * layp, eo[n], x1);
              face(x0, x1, kt, mt);
              const T sT = T(sc[n]);
              layer_apply<T>(kb[n], kt, mb[n], mt, sT * kx1 + kx0, sT * ky1 + ky0, sT * kz1 + kz0, (sT - tauT) * kxy,
                             c1, c3, c9, ac[n], pl);
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                kb[n][v] = kt[v];
                mb[n][v] = mt[v];
              }
              sums(n, pl);
            }
          }
        } else {
#pragma unroll
          for (int n = 0; n < kCE; ++n)
            if (wfirst + n * BLOCK < elay) sums(n, ac[n]);
        }
        STM_T1P(t_za, 6);
        STM_T0(t_zb);
        lds_barrier();
        // ---- phase B: output nodes of plane k (an owned plane) ----
        T y[kCB], o0[kCB], o1[kCB];
#pragma unroll
        for (int n = 0; n < kCB; ++n) {
          if (k >= kb0 && wfirst + n * BLOCK < nc) {
            // element (i - 1 + a, j - 1 + b) gives vertex (1 - a) + 2 (1 - b)
            const int e = ns[n];
            y[n] = (S[3 * slay + e] + S[2 * slay + e + 1]) + (S[slay + e + EXP] + S[e + EXP + 1]);
            o0[n] = P[(2 * s0) * layp + no[n]];
            o1[n] = P[(2 * s0 + 1) * layp + no[n]];
          }
        }
        // the step's loads, all before the first store: stores then stay in
        // flight over the next step
        __builtin_amdgcn_s_waitcnt(kWaitVm);
#pragma unroll
        for (int n = 0; n < kCE; ++n)
          if (wfirst + n * BLOCK < elay) sc[n] = sn[n];
#pragma unroll
        for (int n = 0; n < kCB; ++n) {
          const int q = tid + n * BLOCK;
          if (k >= kb0 && q < nc) {
            const int r = (int)fdiv(q, mnx);
            body(NodeAt{(int)pk, (unsigned)q}, q - r * nx, j0 + r, k, y[n], o0[n], o1[n], v2[n], v3[n]);
          }
        }
        lds_barrier();
        STM_T1P(t_zb, 7);
        s0 = s1;
      }
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
    }
  }

  // n dwords from global memory to LDS by direct-to-LDS loads of 16 bytes a
  // lane (the last n % 4 dwords one a lane): lane i of the wave whose first
  // thread is w writes 16-byte word w + i + c BLOCK of the range (the LDS
  // address of a wave's load is uniform; lanes past the end do not load).  dst
  // is 16-byte aligned, src 4-byte.  Complete for every wave after a barrier
  // before which each has waited for its vector memory operations.
  template <int AUX = 0>
  __device__ __forceinline__ void dma_words(const STM_GLOBAL unsigned* __restrict__ src, void* dst, int n,
                                            int wfirst) const {
    const unsigned lane4 = 4 * threadIdx.x;
    unsigned* d = reinterpret_cast<unsigned*>(dst);
    const int n4 = n >> 2;
    for (int c0 = 0; c0 + wfirst < n4; c0 += BLOCK) {
      if (c0 + (int)threadIdx.x < n4)
        __builtin_amdgcn_global_load_lds(src + 4 * c0 + lane4,
                                         (__attribute__((address_space(3))) void*)(d + 4 * (c0 + wfirst)), 16, 0, AUX);
    }
    if (wfirst == 0 && (int)threadIdx.x < (n & 3))
      __builtin_amdgcn_global_load_lds(src + 4 * n4 + (unsigned)threadIdx.x,
                                       (__attribute__((address_space(3))) void*)(d + 4 * n4), 4, 0, AUX);
  }
  // Workgroup barrier ordering LDS accesses only: vector memory operations in
  // flight stay in flight (a fence would wait for them).
  __device__ __forceinline__ void lds_barrier() const { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

  // ---- tiled pass (2D) --------------------------------------------------------
  template <typename T, typename KV, typename MV, typename Body>
  __device__ __forceinline__ void staged_tiles(int l, const T* __restrict__ f0, const T* __restrict__ f1,
                                               const T* __restrict__ f2, const T* __restrict__ f3, KV kval, MV mval,
                                               Body body) const {
    static_assert(DIM == 2, "the tiled pass is 2D");
    constexpr int NV = 4;
    constexpr int U = 4;   // batched loads per thread in the staging loop
    constexpr int UA = 2;  // independent elements per thread in phase A
    const STM_CONST LevelDev* __restrict__ Lp = cmem(here(L));
    const STM_CONST GridDev& g = Lp->g[l];
    const int nx = g.nx, EX = g.ex;
    const unsigned mnx = g.mnx, mex = g.mex;
    const int nf = 2 + (f2 ? 1 : 0) + (f3 ? 1 : 0);
    const int Ry = Lp->tile_y[l][sizeof(T) == 8 ? 0 : 1][nf - 2];
    const int jb0 = l == 0 ? this->jb0 : 0, jb1 = l == 0 ? this->jb1 : g.ny;
    const double* __restrict__ sg = mgS(l);
    const double* __restrict__ fib = Lp->fib[l];
    const double tau = prm.tau, zr = prm.zr;
    const T hx = T(g.hx), hy = T(g.hy);
    const T cxx = hy / (T(6) * hx), cyy = hx / (T(6) * hy), cm = hx * hy / T(36);
    for (int j0 = jb0; j0 < jb1; j0 += Ry) {
      const int je = min(j0 + Ry, jb1);  // computed rows [j0, je)
      const int jr0 = max(j0 - 1, 0), jr1 = min(je, g.ny - 1);
      const int nst = (jr1 - jr0 + 1) * nx;  // staged nodes
      const int ey0 = max(j0 - 1, 0), ey1 = min(je - 1, g.ey - 1);
      const int sey = ey1 - ey0 + 1;
      const int nse = sey * EX;  // staged elements
      T* l0 = reinterpret_cast<T*>(smem);
      T* l1 = l0 + nst;
      T* l2 = l1 + nst;
      T* l3 = l2 + (f2 ? nst : 0);
      double* ls = reinterpret_cast<double*>(smem + ((nf * (size_t)nst * sizeof(T) + 15) & ~(size_t)15));
      T* lc = reinterpret_cast<T*>(ls + nse);  // [NV][nse]
      double* lf = reinterpret_cast<double*>(
          reinterpret_cast<unsigned char*>(lc) + ((NV * (size_t)nse * sizeof(T) + 15) & ~(size_t)15));
      // ---- stage: batched loads, then LDS stores ----
      STM_T0(t_st);
      const int gq0 = jr0 * nx;
      for (int qb = threadIdx.x; qb < nst; qb += BLOCK * U) {
        T r0[U], r1[U], r2[U], r3[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int q = qb + u * BLOCK;
          if (q < nst) {
            r0[u] = f0[gq0 + q];
            r1[u] = f1[gq0 + q];
            if (f2) r2[u] = f2[gq0 + q];
            if (f3) r3[u] = f3[gq0 + q];
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int q = qb + u * BLOCK;
          if (q < nst) {
            l0[q] = r0[u];
            l1[q] = r1[u];
            if (f2) l2[q] = r2[u];
            if (f3) l3[q] = r3[u];
          }
        }
      }
      {
        const int ge0 = ey0 * EX;
        for (int qb = threadIdx.x; qb < nse; qb += BLOCK * U) {
          double rs[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int q = qb + u * BLOCK;
            if (q < nse) rs[u] = sg[ge0 + q];
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int q = qb + u * BLOCK;
            if (q < nse) ls[q] = rs[u];
          }
        }
        for (int q = threadIdx.x; q < kFibStride * sey; q += BLOCK) lf[q] = fib[kFibStride * ey0 + q];
      }
      __syncthreads();
      STM_T1P(t_st, 6);
      STM_T0(t_pa);
      // ---- phase A: element contributions (UA elements per iteration) ----
      for (int qb = threadIdx.x; qb < nse; qb += UA * BLOCK) {
        T kv[UA][NV], mv[UA][NV], out[UA][NV];
        Tensor2<T> D[UA];
#pragma unroll
        for (int h = 0; h < UA; ++h) {
          const int q = qb + h * BLOCK;
          const int qq = q < nse ? q : 0;
          const int r = fdiv(qq, mex);
          D[h] = tensor_from<T, 2>(ls[qq], lf + kFibStride * r, tau, zr);
          const int base = (ey0 + r - jr0) * nx + (qq - r * EX);
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            const int o = base + ((v >> 1) & 1) * nx + (v & 1);
            const T a = l0[o], b = l1[o];
            kv[h][v] = kval(a, b);
            mv[h][v] = mval(a, b);
          }
        }
#pragma unroll
        for (int h = 0; h < UA; ++h) elem_apply_2d<T>(kv[h], mv[h], D[h], cxx, cyy, cm, out[h]);
#pragma unroll
        for (int h = 0; h < UA; ++h) {
          const int q = qb + h * BLOCK;
          if (q < nse) {
#pragma unroll
            for (int v = 0; v < NV; ++v) lc[v * nse + q] = out[h][v];
          }
        }
      }
      __syncthreads();
      STM_T1P(t_pa, 7);
      // ---- phase B: nodes of the tile ----
      const int nc = (je - j0) * nx;
      for (int q = threadIdx.x; q < nc; q += BLOCK) {
        const int r = fdiv(q, mnx);
        const int i = q - r * nx;
        const int j = j0 + r;
        T y = T(0);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int ey = j - 1 + b;
          const bool oky = ey >= 0 && ey < g.ey;
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            const int ex = i - 1 + a;
            const bool ok = oky && ex >= 0 && ex < EX;
            const int el = (ey - ey0) * EX + ex;
            const int v = (1 - a) + 2 * (1 - b);
            const T cv = lc[v * nse + (ok ? el : 0)];
            y += ok ? cv : T(0);
          }
        }
        const int o = (j - jr0) * nx + i;
        body(NodeAt{j0 * nx, (unsigned)q}, i, j, 0, y, l0[o], l1[o], f2 ? l2[o] : T(0), f3 ? l3[o] : T(0));
      }
      __syncthreads();
    }
  }

  // ---- per-sample operator data ----------------------------------------------
  // On every coarse V-cycle grid (one-workgroup teams): the conductivity of an
  // element = mean of its 2^d children, and the stiffness diagonal from it and
  // the grid's own fibre rows (rediscretisation).  On grid 0: the stiffness
  // diagonal at the owned nodes.  Ends with a team barrier.
  __device__ __forceinline__ void setup_operator() const {
    const int tid = threadIdx.x;
    const double tau = prm.tau, zr = prm.zr;
    for (int l = 1; l < (MG ? L->nmg : 1); ++l) {
      const GridDev& gc = L->g[l];
      const GridDev& gf = L->g[l - 1];
      double* Sc = const_cast<double*>(mgS(l));
      const double* Sf = mgS(l - 1);
      for (int e = tid; e < gc.ne; e += BLOCK) {
        const int E = e % gc.ex;
        const int F = (DIM == 2) ? e / gc.ex : (e / gc.ex) % gc.ey;
        const int Gz = (DIM == 2) ? 0 : e / (gc.ex * gc.ey);
        double acc = 0.0;
        const int cz = (DIM == 3) ? 2 : 1;
        for (int c = 0; c < cz; ++c)
          for (int b = 0; b < 2; ++b)
            for (int a = 0; a < 2; ++a) {
              const int fx = 2 * E + a, fy = 2 * F + b, fz = 2 * Gz + c;
              acc += Sf[(DIM == 2) ? (fy * gf.ex + fx) : ((fz * gf.ey + fy) * gf.ex + fx)];
            }
        Sc[e] = acc / (4 * cz);
        if constexpr (DIM == 3 && sizeof(TI) == 4)
          const_cast<float*>(mgST<TI>(l))[e] = float(Sc[e]);
      }
      __syncthreads();
      double* Kc = mgK(l);
      const double* fibc = L->fib[l];
      for (int idx = tid; idx < gc.n; idx += BLOCK) {
        int i, j, k;
        decode<DIM>(gc, idx, i, j, k);
        auto z = [&](int, int, int) { return 0.0; };
        double dd;
        apply_at<double, DIM>(
            gc, i, j, k, z, z,
            [&](int ex, int ey, int ez) {
              const int e = (DIM == 3) ? ((ez * gc.ey + ey) * gc.ex + ex) : (ey * gc.ex + ex);
              return tensor_from<double, DIM>(Sc[e], fibc + kFibStride * ((DIM == 3) ? ez : ey), tau, zr);
            },
            0.0, &dd);
        Kc[idx] = dd;
      }
      __syncthreads();
    }
    const GridDev& g0 = L->g[0];
    const int nb = nband();
    for (int q = tid; q < nb; q += BLOCK) {
      const int idx = bidx(q);
      int i, j, k;
      decode<DIM>(g0, idx, i, j, k);
      auto z = [&](int, int, int) { return 0.0; };
      double dd;
      apply_at<double, DIM>(
          g0, i, j, k, z, z,
          [&](int ex, int ey, int ez) {
            const int e = (DIM == 3) ? ((ez * g0.ey + ey) * g0.ex + ex) : (ey * g0.ex + ex);
            return tensor_from<double, DIM>(sigma[e], L->fib[0] + kFibStride * ((DIM == 3) ? ez : ey), tau, zr);
          },
          0.0, &dd);
      kdiag0[idx] = dd;
    }
    if constexpr (DIM == 3 && sizeof(TI) == 4) {
      // the members share the float32 conductivity copy of grid 0 out by
      // element; the closing team barrier publishes it
      float* s32 = const_cast<float*>(mgST<TI>(0));
      for (int e = rank * BLOCK + tid; e < g0.ne; e += G * BLOCK) s32[e] = float(sigma[e]);
    }
    sync();
  }

  // Reaction weights injected from grid-0 values u and the slab diagonal on
  // every coarse V-cycle grid (one-workgroup teams; no barrier).
  __device__ __forceinline__ void coarse_weights(const double* __restrict__ u, double inv_dt) const {
    const GridDev& g0 = L->g[0];
    const double kr = prm.k_react, ar = prm.a_react, th = prm.theta;
    for (int l = 1; l < (MG ? L->nmg : 1); ++l) {
      const GridDev& gc = L->g[l];
      TI* wl = mgW(l);
      TI* dl = mgI(l);
      const double* Kc = mgK(l);
      const double cmc = (DIM == 3) ? 8.0 * gc.hx * gc.hy * gc.hz / 216.0 : 4.0 * gc.hx * gc.hy / 36.0;
      const int st = 1 << l;
      for (int idx = threadIdx.x; idx < gc.n; idx += BLOCK) {
        int I, J, K;
        decode<DIM>(gc, idx, I, J, K);
        const int q = (DIM == 3) ? (((K * st) * g0.ny + J * st) * g0.nx + I * st) : ((J * st) * g0.nx + I * st);
        const double w = inv_dt - react_d(u[q], kr, ar);
        wl[idx] = TI(w);
        dl[idx] = TI(1.0 / (th * Kc[idx] + nel(l, I, J, K) * cmc * w));
      }
    }
  }

  // number of elements adjacent to node (i, j, k) of grid l
  __device__ __forceinline__ int nel(int l, int i, int j, int k) const {
    const GridDev& g = L->g[l];
    int c = ((i > 0) + (i < g.nx - 1)) * ((j > 0) + (j < g.ny - 1));
    if constexpr (DIM == 3) c *= (k > 0) + (k < g.nz - 1);
    return c;
  }
  // mass diagonal per adjacent element (times the nodal weight)
  __device__ __forceinline__ TI cmd0() const {
    const GridDev& g = L->g[0];
    return (DIM == 3) ? TI(8.0 * g.hx * g.hy * g.hz / 216.0) : TI(4.0 * g.hx * g.hy / 36.0);
  }

  // ---- smoothing -----------------------------------------------------------
  // out = x + om (b - A x) / diag on grid l;  x == null means x = 0 (out = om b / diag)
  __device__ __forceinline__ void jacobi(int l, const TI* __restrict__ b, const TI* __restrict__ x, TI* __restrict__ out,
                         TI om) const {
    const int n = L->g[l].n;
    bytes = uni(bytes + ((x ? 5.0 : 4.0) * sizeof(TI) * n + (x ? dbytes(l) : 0.0)));
    const TI* __restrict__ w = mgW(l);
    const TI* __restrict__ di = mgI(l);
    if (!x) {
      const int nb = l == 0 ? nband() : n;
      for (int qb = threadIdx.x; qb < nb; qb += BLOCK * 4) {
        TI rb[4], rd[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int q = qb + v * BLOCK;
          if (q < nb) {
            const int idx = l == 0 ? bidx(q) : q;
            rb[v] = b[idx];
            rd[v] = di[idx];
          }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int q = qb + v * BLOCK;
          if (q < nb) out[l == 0 ? bidx(q) : q] = om * rb[v] * rd[v];
        }
      }
      sync();
      return;
    }
    staged<TI, 2>(
        l, x, w, b, di, KScale<TI>{TI(prm.theta)}, [](TI a, TI ww) { return ww * a; },
        [&](int idx, int, int, int, TI y, TI xo, TI, TI bo, TI dio) { gmem(out)[idx] = xo + om * (bo - y) * dio; });
  }

  // Two Jacobi sweeps on grid 0 in one pass over the tiles (2D):
  // out = J2(J1(x)), Jq(v) = v + omq (b - A v) dinv.  A tile stages x, the
  // mass weights, b and dinv over its rows plus two halo rows each side,
  // computes the first sweep on its rows plus one row each side into LDS, and
  // the second sweep on its rows from there.  Halo rows of the first sweep take
  // the same operations in the same order as in the pass that owns them, so the
  // result equals two single sweeps.  x == null stands for the sweep from zero,
  // x = om0 b dinv, formed while staging (three sweeps in the pass).  out must
  // not alias x.  coh: x and out are exchanged past the caches (halo_barrier
  // closes the pass).  last: fin(node, value) takes every result, and the
  // closing team barrier is left to the caller's reduction.
  template <typename Fin>
  __device__ __forceinline__ void jacobi_pair(const TI* __restrict__ x, const TI* __restrict__ b, TI* __restrict__ out, TI om0,
                              TI om1, TI om2, bool coh, bool last, Fin fin) const {
    static_assert(DIM == 2, "the fused sweep pair is 2D");
    using T = TI;
    constexpr int NV = 4;
    constexpr int U = 4;
    constexpr int UA = 2;
    const GridDev& g = L->g[0];
    bytes = uni(bytes + ((x ? 5.0 : 4.0) * sizeof(TI) * g.n + dbytes(0)));
    const T* __restrict__ w = mgW(0);
    const T* __restrict__ di = dinv;
    const int nx = g.nx, EX = g.ex;
    const unsigned mnx = g.mnx, mex = g.mex;
    const int Ry = sizeof(T) == 8 ? L->tile_p8 : L->tile_p4;
    const double* __restrict__ sg = sigma;
    const double* __restrict__ fib = L->fib[0];
    const double tau = prm.tau, zr = prm.zr;
    const T hx = T(g.hx), hy = T(g.hy);
    const T cxx = hy / (T(6) * hx), cyy = hx / (T(6) * hy), cm = hx * hy / T(36);
    const T th = T(prm.theta);
    for (int j0 = jb0; j0 < jb1; j0 += Ry) {
      const int je = min(j0 + Ry, jb1);                          // second sweep: rows [j0, je)
      const int a0 = max(j0 - 1, 0), a1 = min(je + 1, g.ny);     // first sweep: rows [a0, a1)
      const int jr0 = max(j0 - 2, 0), jr1 = min(je + 1, g.ny - 1);  // staged node rows [jr0, jr1]
      const int ey0 = jr0, ey1 = min(je, g.ey - 1);              // staged element rows [ey0, ey1]
      const int nst = (jr1 - jr0 + 1) * nx;
      const int nse = (ey1 - ey0 + 1) * EX;
      T* lx0 = reinterpret_cast<T*>(smem);
      T* lw = lx0 + nst;
      T* lb = lw + nst;
      T* ld = lb + nst;
      T* lx1 = ld + nst;
      double* ls = reinterpret_cast<double*>(smem + ((5 * (size_t)nst * sizeof(T) + 15) & ~(size_t)15));
      T* lc = reinterpret_cast<T*>(ls + nse);  // [NV][nse]
      double* lf = reinterpret_cast<double*>(
          reinterpret_cast<unsigned char*>(lc) + ((NV * (size_t)nse * sizeof(T) + 15) & ~(size_t)15));
      // ---- stage ----
      const int gq0 = jr0 * nx;
      for (int qb = threadIdx.x; qb < nst; qb += BLOCK * U) {
        T r0[U], r1[U], r2[U], r3[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int q = qb + u * BLOCK;
          if (q < nst) {
            if (x) r0[u] = coh ? __hip_atomic_load(x + gq0 + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : x[gq0 + q];
            r1[u] = w[gq0 + q];
            r2[u] = b[gq0 + q];
            r3[u] = di[gq0 + q];
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int q = qb + u * BLOCK;
          if (q < nst) {
            lx0[q] = x ? r0[u] : om0 * r2[u] * r3[u];
            lw[q] = r1[u];
            lb[q] = r2[u];
            ld[q] = r3[u];
          }
        }
      }
      {
        const int ge0 = ey0 * EX;
        for (int qb = threadIdx.x; qb < nse; qb += BLOCK * U) {
          double rs[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int q = qb + u * BLOCK;
            if (q < nse) rs[u] = sg[ge0 + q];
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int q = qb + u * BLOCK;
            if (q < nse) ls[q] = rs[u];
          }
        }
        for (int q = threadIdx.x; q < kFibStride * (ey1 - ey0 + 1); q += BLOCK) lf[q] = fib[kFibStride * ey0 + q];
      }
      __syncthreads();
#pragma unroll 1
      for (int sweep = 0; sweep < 2; ++sweep) {
        // element rows [e0, e1] whose contributions this sweep gathers
        const int e0 = sweep == 0 ? ey0 : max(j0 - 1, 0);
        const int e1 = sweep == 0 ? ey1 : min(je - 1, g.ey - 1);
        const T* __restrict__ lxs = sweep == 0 ? lx0 : lx1;
        const int ne = (e1 - e0 + 1) * EX;
        // ---- phase A: element contributions of M (w v) + K (theta v) ----
        for (int qb = threadIdx.x; qb < ne; qb += UA * BLOCK) {
          T kv[UA][NV], mv[UA][NV], o4[UA][NV];
          Tensor2<T> D[UA];
          int qs[UA];
#pragma unroll
          for (int h = 0; h < UA; ++h) {
            const int q = qb + h * BLOCK;
            const int qq = q < ne ? q : 0;
            const int r = fdiv(qq, mex);
            const int ex = qq - r * EX;
            const int rr = e0 - ey0 + r;  // staged element row
            qs[h] = rr * EX + ex;
            D[h] = tensor_from<T, 2>(ls[qs[h]], lf + kFibStride * rr, tau, zr);
            const int base = rr * nx + ex;  // staged node rows start at ey0
#pragma unroll
            for (int v = 0; v < NV; ++v) {
              const int o = base + ((v >> 1) & 1) * nx + (v & 1);
              const T a = lxs[o], ww = lw[o];
              kv[h][v] = th * a;
              mv[h][v] = ww * a;
            }
          }
#pragma unroll
          for (int h = 0; h < UA; ++h) elem_apply_2d<T>(kv[h], mv[h], D[h], cxx, cyy, cm, o4[h]);
#pragma unroll
          for (int h = 0; h < UA; ++h) {
            if (qb + h * BLOCK < ne) {
#pragma unroll
              for (int v = 0; v < NV; ++v) lc[v * nse + qs[h]] = o4[h][v];
            }
          }
        }
        __syncthreads();
        // ---- phase B: nodes of rows [n0r, n1r) ----
        const int n0r = sweep == 0 ? a0 : j0, n1r = sweep == 0 ? a1 : je;
        const int nc = (n1r - n0r) * nx;
        const T om = sweep == 0 ? om1 : om2;
        for (int q = threadIdx.x; q < nc; q += BLOCK) {
          const int r = fdiv(q, mnx);
          const int i = q - r * nx;
          const int j = n0r + r;
          T y = T(0);
#pragma unroll
          for (int bb = 0; bb < 2; ++bb) {
            const int ey = j - 1 + bb;
            const bool oky = ey >= 0 && ey < g.ey;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
              const int ex = i - 1 + a;
              const bool ok = oky && ex >= 0 && ex < EX;
              const int el = (ey - ey0) * EX + ex;
              const int v = (1 - a) + 2 * (1 - bb);
              const T cv = lc[v * nse + (ok ? el : 0)];
              y += ok ? cv : T(0);
            }
          }
          const int o = (j - jr0) * nx + i;
          const T xn = lxs[o] + om * (lb[o] - y) * ld[o];
          if (sweep == 0) {
            lx1[o] = xn;
          } else {
            if (coh)
              __hip_atomic_store(out + j * nx + i, xn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else
              out[j * nx + i] = xn;
            if (last) fin(NodeAt{0, (unsigned)(j * nx + i)}, xn);
          }
        }
        __syncthreads();
      }
    }
    if (!last) {
      if (coh)
        halo_barrier();
      else if (G > 1)
        team_barrier();
    }
  }

  // Every sweep of the smoother in one pass, for a one-workgroup team whose
  // grid fits one tile (2D): the mass weights, b, dinv, sigma and the fibre
  // rows are staged once; the first sweep (from x = 0) is om b dinv, the later
  // ones alternate between two LDS vectors, and the last is written to out.
  // Each sweep takes the operations of a single sweep in the same order.  Ends
  // with a workgroup barrier.
  __device__ __forceinline__ void jacobi_resident(const TI* __restrict__ b, TI* __restrict__ out, int nc) const {
    static_assert(DIM == 2, "the resident smoother is 2D");
    using T = TI;
    constexpr int NV = 4;
    constexpr int U = 4;
    constexpr int UA = 2;
    const GridDev& g = L->g[0];
    bytes = uni(bytes + (4.0 * sizeof(TI) * g.n + dbytes(0)));
    const T* __restrict__ w = mgW(0);
    const T* __restrict__ di = dinv;
    const int nx = g.nx, EX = g.ex;
    const unsigned mnx = g.mnx, mex = g.mex;
    const double tau = prm.tau, zr = prm.zr;
    const T hx = T(g.hx), hy = T(g.hy);
    const T cxx = hy / (T(6) * hx), cyy = hx / (T(6) * hy), cm = hx * hy / T(36);
    const T th = T(prm.theta);
    const int nst = g.n, nse = g.ne;
    T* lx0 = reinterpret_cast<T*>(smem);
    T* lw = lx0 + nst;
    T* lb = lw + nst;
    T* ld = lb + nst;
    T* lx1 = ld + nst;
    double* ls = reinterpret_cast<double*>(smem + ((5 * (size_t)nst * sizeof(T) + 15) & ~(size_t)15));
    T* lc = reinterpret_cast<T*>(ls + nse);  // [NV][nse]
    double* lf = reinterpret_cast<double*>(
        reinterpret_cast<unsigned char*>(lc) + ((NV * (size_t)nse * sizeof(T) + 15) & ~(size_t)15));
    // ---- stage ----
    for (int qb = threadIdx.x; qb < nst; qb += BLOCK * U) {
      T r1[U], r2[U], r3[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = qb + u * BLOCK;
        if (q < nst) {
          r1[u] = w[q];
          r2[u] = b[q];
          r3[u] = di[q];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = qb + u * BLOCK;
        if (q < nst) {
          lw[q] = r1[u];
          lb[q] = r2[u];
          ld[q] = r3[u];
        }
      }
    }
    for (int qb = threadIdx.x; qb < nse; qb += BLOCK * U) {
      double rs[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = qb + u * BLOCK;
        if (q < nse) rs[u] = sigma[q];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = qb + u * BLOCK;
        if (q < nse) ls[q] = rs[u];
      }
    }
    for (int q = threadIdx.x; q < kFibStride * g.ey; q += BLOCK) lf[q] = L->fib[0][q];
    __syncthreads();
    // ---- sweep 1 from x = 0 ----
    {
      const T om = wgt(0, 0);
      T* dst = nc == 1 ? out : lx0;
      for (int q = threadIdx.x; q < nst; q += BLOCK) {
        dst[q] = om * lb[q] * ld[q];
      }
      __syncthreads();
    }
#pragma unroll 1
    for (int s = 2; s <= nc; ++s) {
      const T* __restrict__ cur = (s % 2 == 0) ? lx0 : lx1;
      T* nxt = (s % 2 == 0) ? lx1 : lx0;
      // ---- phase A: element contributions of M (w v) + K (theta v) ----
      for (int qb = threadIdx.x; qb < nse; qb += UA * BLOCK) {
        T kv[UA][NV], mv[UA][NV], o4[UA][NV];
        Tensor2<T> D[UA];
#pragma unroll
        for (int h = 0; h < UA; ++h) {
          const int q = qb + h * BLOCK;
          const int qq = q < nse ? q : 0;
          const int r = fdiv(qq, mex);
          const int ex = qq - r * EX;
          D[h] = tensor_from<T, 2>(ls[qq], lf + kFibStride * r, tau, zr);
          const int base = r * nx + ex;
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            const int o = base + ((v >> 1) & 1) * nx + (v & 1);
            const T a = cur[o], ww = lw[o];
            kv[h][v] = th * a;
            mv[h][v] = ww * a;
          }
        }
#pragma unroll
        for (int h = 0; h < UA; ++h) elem_apply_2d<T>(kv[h], mv[h], D[h], cxx, cyy, cm, o4[h]);
#pragma unroll
        for (int h = 0; h < UA; ++h) {
          const int q = qb + h * BLOCK;
          if (q < nse) {
#pragma unroll
            for (int v = 0; v < NV; ++v) lc[v * nse + q] = o4[h][v];
          }
        }
      }
      __syncthreads();
      // ---- phase B: every node ----
      const T om = wgt(0, s - 1);
      for (int q = threadIdx.x; q < nst; q += BLOCK) {
        const int j = fdiv(q, mnx);
        const int i = q - j * nx;
        T y = T(0);
#pragma unroll
        for (int bb = 0; bb < 2; ++bb) {
          const int ey = j - 1 + bb;
          const bool oky = ey >= 0 && ey < g.ey;
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            const int ex = i - 1 + a;
            const bool ok = oky && ex >= 0 && ex < EX;
            const int el = ey * EX + ex;
            const int v = (1 - a) + 2 * (1 - bb);
            const T cv = lc[v * nse + (ok ? el : 0)];
            y += ok ? cv : T(0);
          }
        }
        const T xn = cur[q] + om * (lb[q] - y) * ld[q];
        if (s == nc) {
          out[q] = xn;
        } else {
          nxt[q] = xn;
        }
      }
      __syncthreads();
    }
  }

  __device__ __forceinline__ void residual_inner(int l, const TI* __restrict__ b, const TI* __restrict__ x, TI* __restrict__ out) const {
    const int n = L->g[l].n;
    bytes = uni(bytes + (4.0 * sizeof(TI) * n + dbytes(l)));
    const TI* __restrict__ w = mgW(l);
    staged<TI, 1>(
        l, x, w, b, (const TI*)nullptr, KScale<TI>{TI(prm.theta)},
        [](TI a, TI ww) { return ww * a; }, [&](int idx, int, int, int, TI y, TI, TI, TI bo, TI) { gmem(out)[idx] = bo - y; });
  }

  // coarse[l+1] = P^T fine[l]  (full weighting, transpose of Q1 interpolation); G == 1 only
  __device__ __forceinline__ void restrict_to(int l, const TI* __restrict__ rf, TI* __restrict__ bc) const {
    const GridDev& gf = L->g[l];
    const GridDev& gc = L->g[l + 1];
    bytes = uni(bytes + (double(sizeof(TI)) * (gf.n + gc.n)));
    for (int idx = threadIdx.x; idx < gc.n; idx += BLOCK) {
      int I, J, K;
      decode<DIM>(gc, idx, I, J, K);
      TI acc = TI(0);
      const int kz0 = (DIM == 3) ? -1 : 0, kz1 = (DIM == 3) ? 1 : 0;
      for (int c = kz0; c <= kz1; ++c) {
        const int fk = 2 * K + c;
        if (DIM == 3 && (fk < 0 || fk >= gf.nz)) continue;
        const TI wz = (c == 0) ? TI(1) : TI(0.5);
#pragma unroll
        for (int b = -1; b <= 1; ++b) {
          const int fj = 2 * J + b;
          if (fj < 0 || fj >= gf.ny) continue;
          const TI wy = (b == 0) ? TI(1) : TI(0.5);
#pragma unroll
          for (int a = -1; a <= 1; ++a) {
            const int fi = 2 * I + a;
            if (fi < 0 || fi >= gf.nx) continue;
            const TI wx = (a == 0) ? TI(1) : TI(0.5);
            acc += wx * wy * wz * rf[(DIM == 3 ? (fk * gf.ny + fj) : fj) * gf.nx + fi];
          }
        }
      }
      bc[idx] = acc;
    }
    __syncthreads();
  }

  // fine[l] += P coarse[l+1]  (Q1 interpolation of nested grids); G == 1 only
  __device__ __forceinline__ void prolong_add(int l, const TI* __restrict__ xc, TI* __restrict__ xf) const {
    const GridDev& gf = L->g[l];
    const GridDev& gc = L->g[l + 1];
    bytes = uni(bytes + (double(sizeof(TI)) * (2.0 * gf.n + gc.n)));
    for (int idx = threadIdx.x; idx < gf.n; idx += BLOCK) {
      int i, j, k;
      decode<DIM>(gf, idx, i, j, k);
      const int I = i >> 1, J = j >> 1, K = k >> 1;
      const int oi = i & 1, oj = j & 1, ok = (DIM == 3) ? (k & 1) : 0;
      const TI w = (oi ? TI(0.5) : TI(1)) * (oj ? TI(0.5) : TI(1)) * (ok ? TI(0.5) : TI(1));
      TI acc = TI(0);
      for (int c = 0; c <= ok; ++c)
        for (int b = 0; b <= oj; ++b)
          for (int a = 0; a <= oi; ++a) {
            const int q = (DIM == 3) ? (((K + c) * gc.ny + (J + b)) * gc.nx + (I + a)) : ((J + b) * gc.nx + (I + a));
            acc += w * xc[q];
          }
      xf[idx] += acc;
    }
    __syncthreads();
  }

  // weight of sweep s (0-based) of grid l (the fixed weight fills the table at the kernel's start)
  __device__ __forceinline__ TI wgt(int l, int s) const {
    return TI(omega[l * kMaxSweeps + s]);
  }

  // out = V-cycle(b) on grid 0.  Pre- and post-smoothing sweeps alternate
  // between a level's two buffers so that buf[1] is the level's output for any
  // sweep count; the coarsest grid's sweeps start in the buffer that makes the
  // last one land in buf[1].
  __device__ __forceinline__ void vcycle(const TI* __restrict__ b0, TI* __restrict__ out0) const {
    if constexpr (!MG) {
      // sweep s (1-based) of nc writes buf[(nc - s + 1) % 2]: the last one out0
      TI* buf[2] = {mgT(0), out0};
      const int nc = L->sweeps;
      if constexpr (DIM == 3) {
        jacobi(0, b0, nullptr, buf[nc % 2], wgt(0, 0));
        for (int s = 2; s <= nc; ++s) jacobi(0, b0, buf[(nc - s + 2) % 2], buf[(nc - s + 1) % 2], wgt(0, s - 1));
      } else {
        // A one-workgroup team whose grid fits one tile runs every sweep in one
        // pass.  Otherwise the sweeps after the first run as fused pairs (one
        // pass each), and a single sweep when one is left.  Pass t (1-based) of
        // P writes buf[(P - t + 1) % 2]: the last one out0.
        if (G == 1 && (sizeof(TI) == 8 ? L->tile_p8 : L->tile_p4) >= L->g[0].ny) {
          jacobi_resident(b0, out0, nc);
          return;
        }
        // With three or more sweeps the first pass runs sweeps 1 to 3 (the sweep
        // from zero formed while staging).
        const int np = (nc - 1) / 2;
        const int P = nc - np - (nc >= 3 ? 1 : 0);
        int s, t;
        if (nc >= 3) {
          jacobi_pair(nullptr, b0, buf[P % 2], wgt(0, 0), wgt(0, 1), wgt(0, 2), false, false,
                      [](NodeAt, TI) {});
          s = 4;
        } else {
          jacobi(0, b0, nullptr, buf[P % 2], wgt(0, 0));
          s = 2;
        }
        t = 2;
        for (; s + 1 <= nc; s += 2, ++t)
          jacobi_pair(buf[(P - t + 2) % 2], b0, buf[(P - t + 1) % 2], TI(0), wgt(0, s - 1), wgt(0, s), false,
                      false, [](NodeAt, TI) {});
        for (; s <= nc; ++s, ++t) jacobi(0, b0, buf[(P - t + 2) % 2], buf[(P - t + 1) % 2], wgt(0, s - 1));
      }
      return;
    }
    const int nmg = L->nmg;
    const int nu = prm.smooth_steps;
    for (int l = 0; l < nmg - 1; ++l) {
      TI* buf[2] = {mgT(l), l == 0 ? out0 : mgX(l)};
      const TI* b = (l == 0) ? b0 : mgB(l);
      jacobi(l, b, nullptr, buf[0], wgt(l, 0));
      for (int s = 2; s <= nu; ++s) jacobi(l, b, buf[s % 2], buf[(s - 1) % 2], wgt(l, s - 1));
      residual_inner(l, b, buf[(nu - 1) % 2], buf[nu % 2]);
      restrict_to(l, buf[nu % 2], mgB(l + 1));
    }
    {
      // coarsest grid: sweep s of nc writes buf[(nc - s + 1) % 2], the last buf[1]
      const int l = nmg - 1;
      TI* buf[2] = {mgT(l), l == 0 ? out0 : mgX(l)};
      const TI* b = (l == 0) ? b0 : mgB(l);
      const int nc = L->sweeps;
      jacobi(l, b, nullptr, buf[nc % 2], wgt(l, 0));
      for (int s = 2; s <= nc; ++s) jacobi(l, b, buf[(nc - s + 2) % 2], buf[(nc - s + 1) % 2], wgt(l, s - 1));
    }
    for (int l = nmg - 2; l >= 0; --l) {
      TI* buf[2] = {mgT(l), l == 0 ? out0 : mgX(l)};
      const TI* b = (l == 0) ? b0 : mgB(l);
      prolong_add(l, mgX(l + 1), buf[(nu - 1) % 2]);
      for (int t = 1; t <= nu; ++t) jacobi(l, b, buf[(nu - 2 + t) % 2], buf[(nu - 1 + t) % 2], wgt(l, nu - t));
    }
  }

  // ---- corrections with the stencil in registers (2D) -----------------------
  static constexpr int kTriples = stencil_triples(sizeof(TI));
  // Halo depth of stencil_sweeps, 0 where the member's rows do not fit its
  // registers or the LDS (jacobi_pair then).
  __device__ __forceinline__ int stencil_halo() const {
    const STM_CONST LevelDev* __restrict__ Lp = cmem(here(L));
    const STM_CONST GridDev& g = Lp->g[0];
    return __builtin_amdgcn_readfirstlane(
        stencil_halo_depth(g.nx, g.ny, g.ex, g.ey, G, BLOCK, (int)sizeof(TI), Lp->stage_bytes));
  }
  // The sweeps of a defect correction with the scaled operator D^-1 A of every
  // node in registers: x += om (D^-1 b - D^-1 A x) takes eight products per node
  // (the diagonal is one), x lies in LDS, and a sweep is one pass with one
  // barrier, against two passes and barriers and some 60 operations per element
  // of jacobi_pair, which forms the element products anew in every sweep.  A
  // thread holds up to kTriples columns of three nodes (15 values of x from LDS
  // per column instead of 27).  On a team a member computes H - 1 rows beyond
  // its own on each side, so that x is exchanged with the neighbours once in H
  // sweeps: after the exchange the staged H rows are right, after each sweep one
  // less.  The coefficients are formed once per correction from the
  // conductivities and mass weights staged in LDS; what is left is bound by
  // latency (loads past a cold L2 after a team barrier, barriers, exchanges).
  // Per correction, before and after: 33x33 nodes on one workgroup 40 -> 16 us;
  // 129x129 on teams of 8 95 -> 40; 257x257 in float32 on teams of 16 125 -> 42 (13
  // to 15 sweeps each).  u += x; returns the member's max of |x|.
  __device__ __forceinline__ double stencil_sweeps(const TI* __restrict__ b, TI* __restrict__ out, int nc, int H,
                                                   double* __restrict__ u) const {
    static_assert(DIM == 2, "the sweeps in registers are 2D");
    using T = TI;
    const STM_CONST LevelDev* __restrict__ Lp = cmem(here(L));
    const STM_CONST GridDev& g = Lp->g[0];
    const int nx = g.nx, ny = g.ny, EX = g.ex, EY = g.ey;
    const unsigned mnx = g.mnx;
    bytes = uni(bytes + (4.0 * sizeof(TI) + 16.0) * g.n + dbytes(0));
    const int e0 = max(jb0 - (H - 1), 0), e1 = min(jb1 + (H - 1), ny);  // computed rows [e0, e1)
    const int s0 = max(jb0 - H, 0), s1 = min(jb1 + H, ny);              // staged rows [s0, s1)
    // a row and a node of zeros before the staged rows, four rows and a node after
    const int pad = nx + 1, total = pad + (s1 - s0 + 4) * nx + 1;
    const int y0 = max(e0 - 1, 0), y1 = min(e1, EY);  // element rows [y0, y1)
    T* cur = reinterpret_cast<T*>(smem);
    T* nxt = cur + total;
    double* ls = reinterpret_cast<double*>(smem + ((2 * total * sizeof(T) + 7) & ~(size_t)7));
    double* lf = ls + (y1 - y0) * EX;
    const int units = (e1 - e0 + 2) / 3 * nx;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x);  // the wave's first unit
    T c[kTriples][3][8], bd[kTriples][3];
    int o[kTriples];
    // b / diag of the thread's nodes; the mass weights (where nxt will be, with
    // its zeros around), conductivities and fibre rows to LDS
    {
      const STM_GLOBAL T* __restrict__ di = gmem(dinv);
      const STM_GLOBAL T* __restrict__ bg = gmem(b);
      T d[kTriples][3], bb[kTriples][3];
#pragma unroll
      for (int n = 0; n < kTriples; ++n) {
        const int q = min((int)threadIdx.x + n * BLOCK, units - 1);
        const int t = fdiv(q, mnx), i = q - t * nx;
        o[n] = pad + (e0 + 3 * t - s0) * nx + i;
        if (wave + n * BLOCK < units) {
#pragma unroll
          for (int r = 0; r < 3; ++r) {
            const unsigned p = min(e0 + 3 * t + r, e1 - 1) * nx + i;
            d[n][r] = di[p];
            bb[n][r] = bg[p];
          }
        }
      }
      const STM_GLOBAL T* __restrict__ w = gmem(mgW(0)) + s0 * nx;
      const STM_GLOBAL double* __restrict__ sg = gmem(sigma) + y0 * EX;
      constexpr int U = 8;
      const int nst = (s1 - s0) * nx, nse = (y1 - y0) * EX;
      for (int qb = threadIdx.x; qb < max(nst, nse); qb += U * BLOCK) {
        T rw[U];
        double rs[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (qb + u * BLOCK < nst) rw[u] = w[(unsigned)(qb + u * BLOCK)];
          if (qb + u * BLOCK < nse) rs[u] = sg[(unsigned)(qb + u * BLOCK)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (qb + u * BLOCK < nst) nxt[pad + qb + u * BLOCK] = rw[u];
          if (qb + u * BLOCK < nse) ls[qb + u * BLOCK] = rs[u];
        }
      }
      for (int q = threadIdx.x; q < kFibStride * (y1 - y0); q += BLOCK) lf[q] = cmem(Lp->fib[0])[kFibStride * y0 + q];
      for (int q = threadIdx.x; q < total; q += BLOCK) cur[q] = T(0);
      for (int q = threadIdx.x; q < total - nst; q += BLOCK) nxt[q < pad ? q : q + nst] = T(0);
#pragma unroll
      for (int n = 0; n < kTriples; ++n) {
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          const bool ok = (int)threadIdx.x + n * BLOCK < units && o[n] + r * nx < pad + (e1 - s0) * nx;
          c[n][r][0] = ok ? d[n][r] : T(0);
          bd[n][r] = ok ? d[n][r] * bb[n][r] : T(0);
        }
      }
    }
    __syncthreads();
    // the coefficients, an element row after the other: of an element the
    // stiffness couplings along x, along y and across both diagonals
    {
      const double tau = prm.tau, zr = prm.zr;
      const T th = T(prm.theta), cxx = th * T(g.hy / (6.0 * g.hx)), cyy = th * T(g.hx / (6.0 * g.hy));
      const T cxy = th * T(0.5), cm = T(g.hx * g.hy / 36.0);
#pragma unroll
      for (int n = 0; n < kTriples; ++n) {
        if (wave + n * BLOCK < units) {
          const int q = min((int)threadIdx.x + n * BLOCK, units - 1);
          const int t = fdiv(q, mnx), i = q - t * nx, j0 = e0 + 3 * t;
          const int el[2] = {max(i - 1, 0), min(i, EX - 1)};
          struct Row {
            T x[2], y[2], p[2], m[2], a[2];  // [element left, right of the node]
          };
          auto element_row = [&](int ey) {
            Row R;
            const bool in = ey >= 0 && ey < EY;
            const int yy = min(max(ey, y0), y1 - 1) - y0;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const bool ok = in && (e ? i < nx - 1 : i > 0);
              const Tensor2<T> D = tensor_from<T, 2>(ls[yy * EX + el[e]], lf + kFibStride * yy, tau, zr);
              const T ax = ok ? cxx * D.xx : T(0), ay = ok ? cyy * D.yy : T(0), xy = ok ? cxy * D.xy : T(0);
              R.x[e] = ay - T(2) * ax;
              R.y[e] = ax - T(2) * ay;
              R.p[e] = -(ax + ay) - xy;
              R.m[e] = xy - (ax + ay);
              R.a[e] = ok ? cm : T(0);
            }
            return R;
          };
          Row lo = element_row(j0 - 1);
#pragma unroll
          for (int r = 0; r < 3; ++r) {
            const Row hi = element_row(j0 + r);
            const T* __restrict__ w = nxt + o[n] + r * nx;
            const T d = c[n][r][0];
            c[n][r][0] = d * (lo.x[0] + hi.x[0] + T(2) * (lo.a[0] + hi.a[0]) * w[-1]);
            c[n][r][1] = d * (lo.x[1] + hi.x[1] + T(2) * (lo.a[1] + hi.a[1]) * w[1]);
            c[n][r][2] = d * (lo.y[0] + lo.y[1] + T(2) * (lo.a[0] + lo.a[1]) * w[-nx]);
            c[n][r][3] = d * (hi.y[0] + hi.y[1] + T(2) * (hi.a[0] + hi.a[1]) * w[nx]);
            c[n][r][4] = d * (lo.p[0] + lo.a[0] * w[-nx - 1]);
            c[n][r][5] = d * (hi.p[1] + hi.a[1] * w[nx + 1]);
            c[n][r][6] = d * (lo.m[1] + lo.a[1] * w[-nx + 1]);
            c[n][r][7] = d * (hi.m[0] + hi.a[0] * w[nx - 1]);
            lo = hi;
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
#pragma unroll
          for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int a = 0; a < 8; ++a) c[n][r][a] = T(0);
        }
      }
    }
    __syncthreads();  // the weights are read
    T* xg[2] = {mgT(0), V + vstride};  // x of the rows that the neighbours read
    int parity = 0, age = 0;
#pragma unroll 1
    for (int s = 1; s <= nc; ++s) {
      if (age == H && G > 1) {
        T* __restrict__ x = parity ? xg[1] : xg[0];
        parity ^= 1;
        age = 0;
        const int hn = H * nx;
        for (int q = threadIdx.x; q < 2 * hn; q += BLOCK) {
          const bool up = q >= hn;
          const int p = up ? (jb1 - H) * nx + q - hn : jb0 * nx + q;
          if (up ? jb1 < ny : jb0 > 0) coh_store(gmem(x) + p, cur[pad + p - s0 * nx]);
        }
        halo_barrier();
        for (int q = threadIdx.x; q < 2 * hn; q += BLOCK) {
          const bool up = q >= hn;
          const int p = up ? jb1 * nx + q - hn : (jb0 - H) * nx + q;
          if (up ? jb1 < ny && p < s1 * nx : jb0 > 0 && p >= s0 * nx)
            cur[pad + p - s0 * nx] = __hip_atomic_load(gmem(x) + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
      }
      const T om = wgt(1, s - 1);
#pragma unroll
      for (int n = 0; n < kTriples; ++n) {
        if (wave + n * BLOCK < units) {
          int on = o[n];
          asm volatile("" : "+v"(on));  // addresses formed here, not kept in registers across the sweeps
          T v[5][3];
#pragma unroll
          for (int r = 0; r < 5; ++r)
#pragma unroll
            for (int a = 0; a < 3; ++a) v[r][a] = cur[on + (r - 1) * nx + a - 1];
          const bool mine = (int)threadIdx.x + n * BLOCK < units;
          T xn[3];
#pragma unroll
          for (int r = 0; r < 3; ++r) {
            const T y0 = c[n][r][0] * v[r + 1][0] + c[n][r][1] * v[r + 1][2];
            const T y1 = c[n][r][2] * v[r][1] + c[n][r][3] * v[r + 2][1];
            const T y2 = c[n][r][4] * v[r][0] + c[n][r][5] * v[r + 2][2];
            const T y3 = c[n][r][6] * v[r][2] + c[n][r][7] * v[r + 2][0];
            xn[r] = v[r + 1][1] + om * (bd[n][r] - v[r + 1][1] - ((y0 + y1) + (y2 + y3)));
          }
          const int end = pad + (e1 - s0) * nx;
#pragma unroll
          for (int r = 0; r < 3; ++r)
            if (mine && on + r * nx < end) nxt[on + r * nx] = xn[r];
        }
      }
      ++age;
      __syncthreads();
      T* t = cur;
      cur = nxt;
      nxt = t;
    }
    // u += x, every thread's loads at once
    constexpr int U = 8;
    const int own = (jb1 - jb0) * nx;
    const T* __restrict__ x = cur + pad + (jb0 - s0) * nx;
    STM_GLOBAL double* __restrict__ ug = gmem(u) + jb0 * nx;
    STM_GLOBAL T* __restrict__ og = gmem(out) + jb0 * nx;
    double dm = 0.0;
    for (int qb = threadIdx.x; qb < own; qb += U * BLOCK) {
      double ru[U];
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (qb + k * BLOCK < own) ru[k] = ug[(unsigned)(qb + k * BLOCK)];
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (qb + k * BLOCK < own) {
          const T xn = x[qb + k * BLOCK];
          og[(unsigned)(qb + k * BLOCK)] = xn;
          ug[(unsigned)(qb + k * BLOCK)] = ru[k] + double(xn);
          dm = fmax(dm, abs_or_inf(double(xn)));
        }
    }
    return dm;
  }

  // One defect correction of the slab's Newton equation (single-grid levels):
  // nc Chebyshev-weighted sweeps from x = 0 on A x = b with the weights of
  // omega row 1, the last sweep handing every owned node's value to fin.  3D
  // (nc even): with x1 the first sweep's result is in mgT(0) already, formed by
  // the residual pass.  2D (nc odd): sweeps 1 to 3, then pairs.  Leaves the
  // closing team barrier to the caller.
  template <typename Fin>
  __device__ __forceinline__ void chebyshev(const TI* __restrict__ b0, TI* __restrict__ out0, int nc, bool x1,
                                            Fin fin) const {
    TI* buf[2] = {mgT(0), out0};
    if constexpr (DIM == 3) {
      if (!x1) jacobi(0, b0, nullptr, buf[nc % 2], wgt(1, 0));
      const TI* __restrict__ w = mgW(0);
      const int n = L->g[0].n;
#pragma unroll 1
      for (int s = 2; s <= nc; ++s) {
        const TI* x = buf[(nc - s) % 2];
        TI* out = buf[(nc - s + 1) % 2];
        const TI om = wgt(1, s - 1);
        const bool last = s == nc;
        bytes = uni(bytes + (5.0 * sizeof(TI) * n + dbytes(0)));
        staged<TI, 2, true>(
            0, x, w, b0, dinv, KScale<TI>{TI(prm.theta)}, [](TI a, TI ww) { return ww * a; },
            [&](NodeAt at, int, int, int, TI y, TI xo, TI, TI bo, TI dio) {
              const TI xn = xo + om * (bo - y) * dio;
              coh_store(&node_ref(out, at), xn);
              if (last) fin(at, xn);
            },
            false);
        if (!last) halo_barrier();
      }
    } else {
      const int P = (nc - 1) / 2;
#pragma unroll 1
      for (int t = 1; t <= P; ++t)
        jacobi_pair(t == 1 ? nullptr : buf[(P - t) % 2], b0, buf[(P - t + 1) % 2], wgt(1, 0), wgt(1, 2 * t - 1),
                    wgt(1, 2 * t), G > 1, t == P, fin);
    }
  }

  // Lower end of the spectrum of D^-1 A for the Chebyshev interval, 0 when
  // defect corrections are not for this operator.  On a uniform grid the modes
  // that alternate along some of the axes and are constant along the others
  // bound it: relative to the diagonal the Q1 mass matrix is 1/2 on such a mode
  // for each axis it alternates along and 3/2 for each other, and the stiffness
  // along axis a is twice the other axes' factors where the mode alternates along
  // a, else 0.  With r the diagonal's stiffness to mass ratio and f_a the axes'
  // shares of the stiffness, D^-1 A there is (mass + r sum f_a stiffness_a) / (1 + r);
  // the smallest over the modes and both ends of r at the nodes, with the smallest
  // share of each axis over the elements, is a lower bound for every operator
  // tried (0.54-0.99 of the smallest eigenvalue; without the modes along single
  // axes 2.4 times it on 7x7x41 nodes with a stiffness of 3 mass).
  __device__ __forceinline__ double spectrum_low() const {
    const GridDev& g = L->g[0];
    const double th = prm.theta, tau = prm.tau, zr = prm.zr;
    const TI* __restrict__ di = dinv;
    double pm = 0.0, qm = 0.0;  // largest mass and stiffness share of the diagonal
    const int nb = nband();
    for (int q = threadIdx.x; q < nb; q += BLOCK) {
      const int idx = bidx(q);
      const double s = th * kdiag0[idx] * double(di[idx]);
      qm = fmax(qm, s);
      pm = fmax(pm, 1.0 - s);
    }
    qm = tmax(qm);
    pm = tmax(pm);
    double f[DIM];  // 1 less an axis's share, largest; then the smallest share
#pragma unroll
    for (int a = 0; a < DIM; ++a) f[a] = 0.0;
    const int layer = DIM == 3 ? g.ex * g.ey : g.ex;  // elements of a fibre-table row
    for (int e = rank * BLOCK + threadIdx.x; e < g.ne; e += G * BLOCK) {
      const auto D = tensor_from<double, DIM>(sigma[e], L->fib[0] + kFibStride * (e / layer), tau, zr);
      double w[DIM], sum = 0.0;
      w[0] = D.xx / (g.hx * g.hx);
      w[1] = D.yy / (g.hy * g.hy);
      if constexpr (DIM == 3) w[2] = D.zz / (g.hz * g.hz);
#pragma unroll
      for (int a = 0; a < DIM; ++a) sum += w[a];
#pragma unroll
      for (int a = 0; a < DIM; ++a) f[a] = fmax(f[a], 1.0 - w[a] / sum);
    }
#pragma unroll
    for (int a = 0; a < DIM; ++a) f[a] = 1.0 - tmax(f[a]);
    const double r0 = fmax(0.0, 1.0 / pm - 1.0), r1 = 1.0 / fmax(1.0 - qm, 1e-300) - 1.0;
    double low = HUGE_VAL;
#pragma unroll
    for (int k = 0; k < (1 << DIM); ++k) {  // bit a: alternating along axis a
      double m = 1.0, st = 0.0;
#pragma unroll
      for (int a = 0; a < DIM; ++a) m *= (k >> a & 1) ? 0.5 : 1.5;
#pragma unroll
      for (int a = 0; a < DIM; ++a)
        if (k >> a & 1) st += f[a] * 2.0 * (m / 0.5);
      low = fmin(low, fmin((m + r0 * st) / (1.0 + r0), (m + r1 * st) / (1.0 + r1)));
    }
    return pm <= 1.0 && qm < 1.0 && low > 0.0 ? low : 0.0;
  }

  // The next degree that a correction can have: 2D odd (a first sweep and pairs),
  // 3D even (the last sweep ends in the output vector).
  __device__ __forceinline__ int odd_or_even(int n) const {
    if (n % 2 != (DIM == 2 ? 1 : 0)) n = n < kMaxDegree ? n + 1 : n - 1;
    return __builtin_amdgcn_readfirstlane(n);
  }
  // Degree of a defect correction that reduces the error by 2^-bits: 2 rho^n on
  // the interval, decay = -log2 rho.
  __device__ __forceinline__ int cheb_degree(float decay, float bits) const {
    return odd_or_even(min(max((int)ceilf((bits + 1.0f) / decay), 3), kMaxDegree));
  }
  __device__ __forceinline__ float cheb_decay(double ratio) const {
    const double rt = sqrt(ratio);
    return (float)log2((rt + 1.0) / (rt - 1.0));
  }
  // Largest reduction factor of n sweeps on [1 / ratio, 1] over [low, 1].
  __device__ __forceinline__ double cheb_reduction(double ratio, double low, int n) const {
    const double c = 1.0 + 1.0 / ratio, r = 1.0 - 1.0 / ratio;
    const double x0 = c / r, x = fmax(1.0, (c - 2.0 * low) / r);
    return cosh(n * acosh(x)) / cosh(n * acosh(x0));
  }
  // Weights of a defect correction into the omega table from row 1 on.  Between
  // two workgroup barriers.
  __device__ __forceinline__ void cheb_weights(double low, double lmax, int n) const {
    __syncthreads();
    chebyshev_weights(low, lmax, n, omega + kMaxSweeps, threadIdx.x, BLOCK);
    __syncthreads();
  }

  // lmax of D^-1 A_l by power iteration.
  // Uses buffers x0, x1 of grid l.  Returns the estimate (team-uniform).
  __device__ __forceinline__ double power_lmax(int l, TI* x0, TI* x1) const {
    const GridDev& g = L->g[l];
    const int nb = l == 0 ? nband() : g.n;  // coarse grids: one-workgroup teams own every node
    // Start: a constant plus per-node pseudo-random values in [-1/2, 1/2) (a
    // multiplicative hash of the node index, the same on every member).  When
    // the stiffness dominates A, the largest eigenvalues of D^-1 A belong to
    // modes that alternate along one axis only (Q1 in 2D and 3D); a start
    // without them, such as a checkerboard, underestimates lmax, and the
    // Chebyshev sweeps then amplify those modes.  Pseudo-random values contain
    // every mode.
    for (int q = threadIdx.x; q < nb; q += BLOCK) {
      const int idx = l == 0 ? bidx(q) : q;
      const unsigned hsh = (unsigned)idx * 2654435761u;
      x0[idx] = TI(1.0 + double(hsh >> 8) * (1.0 / 16777216.0) - 0.5);
    }
    sync();
    double lam = 0.0;
    TI scl = TI(1);
    const TI* __restrict__ w = mgW(l);
    const TI* __restrict__ di = mgI(l);
    // the iterate is scaled to norm 1 by the pass that reads it next
    for (int it = 0; it < prm.power_iters; ++it) {
      double nn[2] = {0.0, 0.0};
      staged<TI, 1>(
          l, x0, w, di, (const TI*)nullptr, KScale<TI>{TI(prm.theta)},
          [](TI a, TI ww) { return ww * a; },
          [&](int idx, int, int, int, TI ax, TI xown, TI, TI dio, TI) {
            const TI y = ax * dio * scl, xs = xown * scl;
            gmem(x1)[idx] = y;
            nn[0] += double(y) * double(y);
            nn[1] += double(xs) * double(xs);
          },
          false);
      tsum<2>(nn);
      lam = sqrt(nn[0] / nn[1]);
      scl = TI(1.0 / sqrt(nn[0]));
      TI* t = x0;
      x0 = x1;
      x1 = t;
    }
    bytes = uni(bytes + (prm.power_iters * (5.0 * sizeof(TI) * g.n + dbytes(l))));
    return lam;
  }
  // Residual of the slab (float64) -> V_0 = -R, reaction weights and inverse
  // diagonal on every grid; its squared 2-norm into io.resid.
  __device__ __forceinline__ void residual_step(StepIO& io) const {
    const GridDev& g0 = L->g[0];
    const int n0 = g0.n;
    const double th = prm.theta, inv_dt = uni(1.0 / L->dt), kr = prm.k_react, ar = prm.a_react;
    TI* V0 = V;
    TI* w0 = mgW(0);
    TI* __restrict__ di = dinv;
    TI* x1 = io.x1 ? mgT(0) : nullptr;
    const TI om1 = x1 ? wgt(1, 0) : TI(0);
    double rr[1] = {0.0};
    bytes = uni(bytes + (24.0 * n0 + 8.0 * g0.ne + (x1 ? 4.0 : 3.0) * sizeof(TI) * n0));
    for (int l = 1; l < (MG ? L->nmg : 1); ++l) bytes = uni(bytes + ((8.0 + sizeof(TI)) * L->g[l].n));
    const double cmd = (DIM == 3) ? 8.0 * g0.hx * g0.hy * g0.hz / 216.0 : 4.0 * g0.hx * g0.hy / 36.0;
    staged<double, 1>(
        0, (const double*)io.u, (const double*)io.uprev, (const double*)kdiag0, (const double*)nullptr,
        [th](double a, double b) { return th * a + (1.0 - th) * b; },
        [&](double a, double b) { return (a - b) * inv_dt - react(a, kr, ar); },
        [&](NodeAt at, int i, int j, int k, double y, double uown, double, double kd, double) {
          const double r = -y;
          const double w = inv_dt - react_d(uown, kr, ar);
          const TI dd = TI(1.0 / (th * kd + nel(0, i, j, k) * cmd * w));
          node_ref(V0, at) = TI(r);
          node_ref(w0, at) = TI(w);
          node_ref(di, at) = dd;
          if constexpr (!MG) {
            if (x1) node_ref(x1, at) = om1 * TI(r) * dd;
          }
          rr[0] += r * r;
        },
        false);
    coarse_weights(io.u, inv_dt);
    tsum<1>(rr);  // its barriers also publish the writes above
    io.resid = rr[0];
  }

  // Defect correction u += P(A) r, P the Chebyshev sweeps; max-norm into io.dmax.
  __device__ __forceinline__ void correct_step(StepIO& io) const {
    double dm = 0.0;
    double* __restrict__ u = io.u;
    bytes = uni(bytes + 16.0 * L->g[0].n);
    int H = 0;
    if constexpr (DIM == 2) {
      H = stencil_halo();
      if (H > 0) dm = stencil_sweeps(V, Z, io.nc, H, u);
    }
    if (H == 0)
      chebyshev(V, Z, io.nc, io.x1 != 0, [&](NodeAt at, TI xn) {
        const double dl = double(xn);
        node_ref(u, at) += dl;
        dm = fmax(dm, abs_or_inf(dl));
      });
    io.dmax = tmax(dm);  // its barrier also publishes u to the other members
  }

  // Newton step by GMRES(restart), right-preconditioned by the V-cycle (or the
  // sweeps), from the residual in V_0: u += delta, its max-norm and the relative
  // residual reached into io.
  __device__ __forceinline__ void gmres_step(StepIO& io) const {
    __shared__ double H[(kMaxRestart + 1) * kMaxRestart];
    __shared__ double cs_[kMaxRestart], sn_[kMaxRestart], gv[kMaxRestart + 1], sc[kMaxRestart + 1];
    __shared__ double yv[kMaxRestart], coef[kMaxRestart + 1];
    __shared__ double sh_resid;
#ifdef STM_PHASE_TIMERS
    long long* ph_acc = ph;
#endif
    double* __restrict__ u = io.u;
    double* __restrict__ dlt = io.dlt;
    const double beta = io.beta, eta = io.eta, krylov_words = io.krylov_words;
    double model_bytes = io.model_bytes;
    const int tid = threadIdx.x, n0 = L->g[0].n, nb = nband(), restart = prm.restart;
    const int64_t vs = vstride;
    // ---- GMRES(restart), right-preconditioned by the V-cycle ----
    if (tid == 0) {
      sc[0] = 1.0 / beta;
      gv[0] = beta;
    }
    __syncthreads();
    const double tol_abs = uni(eta * beta);
    int jdim = 0;
    for (int j = 0; j < restart; ++j) {
      TI* Vj = V + j * vs;
      TI* Zj = Z + j * vs;
      TI* Vn = V + (j + 1) * vs;
      model_bytes = uni(model_bytes + double(sizeof(TI)) * n0 * (krylov_words + 2.0 * j));
      STM_T0(t_vc);
      vcycle(Vj, Zj);
      STM_T1(t_vc, 1);
      STM_T0(t_pa);
      // pass A: ws = A Z_j (into V_{j+1})
      bytes = uni(bytes + (3.0 * sizeof(TI) * n0 + dbytes(0)));
      staged<TI, 0>(
          0, Zj, mgW(0), (const TI*)nullptr, (const TI*)nullptr, KScale<TI>{TI(prm.theta)},
          [](TI a, TI ww) { return ww * a; },
          [&](int idx, int, int, int, TI w, TI, TI, TI, TI) { gmem(Vn)[idx] = w; });
      STM_T1(t_pa, 2);
      // Classical Gram-Schmidt against V_0..V_j, done twice when the inner
      // vectors are float32 (CGS2: the second pass restores the orthogonality
      // the first loses to rounding); each pass adds its projections to
      // column j of H.
      double nn[1] = {0.0};
      constexpr int kPasses = sizeof(TI) == 4 ? 2 : 1;
      // dots of the next pass, accumulated by the first pass's update
      double dnext[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      bool have_dots = false;
#pragma unroll 1
      for (int pass = 0; pass < kPasses; ++pass) {
        STM_T0(t_dot);
        // dots with V_0..V_min(j,7) over the owned nodes: batched loads
        double d[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) d[q] = have_dots ? dnext[q] : 0.0;
        const int nk0 = min(j + 1, 8);
        if (!have_dots) {
          bytes = uni(bytes + ((1.0 + nk0) * sizeof(TI) * n0));
          const TI* __restrict__ Vb = V;
          const TI* __restrict__ Vr = Vn;
          for (int qb = tid; qb < nb; qb += BLOCK * 2) {
            TI wv[2], vv[2][8];
#pragma unroll
            for (int uu = 0; uu < 2; ++uu) {
              const int q = qb + uu * BLOCK;
              const int idx = q < nb ? bidx(q) : 0;
              wv[uu] = q < nb ? Vr[idx] : TI(0);
#pragma unroll
              for (int p = 0; p < 8; ++p) vv[uu][p] = (p < nk0 && q < nb) ? Vb[p * vs + idx] : TI(0);
            }
#pragma unroll
            for (int uu = 0; uu < 2; ++uu)
#pragma unroll
              for (int p = 0; p < 8; ++p) d[p] += double(vv[uu][p]) * double(wv[uu]);
          }
        }
        tsum<9>(d);
        if (tid == 0) {
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if (q < nk0) coef[q] = d[q];
        }
        for (int k0 = 8; k0 <= j; k0 += 8) {  // remaining dot chunks
          const int nk = min(j + 1 - k0, 8);
          bytes = uni(bytes + ((1.0 + nk) * sizeof(TI) * n0));
#pragma unroll
          for (int q = 0; q < 9; ++q) d[q] = 0.0;
          for (int q = tid; q < nb; q += BLOCK) {
            const int idx = bidx(q);
            const double wd = double(Vn[idx]);
#pragma unroll
            for (int p = 0; p < 8; ++p)
              if (p < nk) d[p] += double(V[(k0 + p) * vs + idx]) * wd;
          }
          tsum<9>(d);
          if (tid == 0) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
              if (q < nk) coef[k0 + q] = d[q];
          }
        }
        // projections onto the normalised basis enter H; V_q is stored with
        // norm 1/sc[q], so w loses (sc[q]^2 <V_q, w>) V_q
        if (tid == 0)
          for (int q = 0; q <= j; ++q) {
            const double hq = sc[q] * sc[j] * coef[q];
            H[q * kMaxRestart + j] = (pass ? H[q * kMaxRestart + j] : 0.0) + hq;
            coef[q] = sc[q] * sc[q] * coef[q];
          }
        __syncthreads();
        STM_T1(t_dot, 3);
        STM_T0(t_pb);
        // pass B: V_{j+1} -= sum_q coef_q V_q over the owned nodes; norm
        nn[0] = 0.0;
        bytes = uni(bytes + ((j + 3.0) * sizeof(TI) * n0));
        // The first of two passes with at most 8 basis vectors also forms
        // the second pass's dots from the values it holds: the same nodes
        // per thread, the same operations in the same order as the
        // separate loops, one read of the vectors fewer.
        const bool fuse = pass + 1 < kPasses && j < 8;
        if (fuse) {
#pragma unroll
          for (int q = 0; q < 9; ++q) dnext[q] = 0.0;
          for (int qb = tid; qb < nb; qb += BLOCK * 2) {
            double w[2];
            int ix[2];
            TI vv[2][8];
#pragma unroll
            for (int uu = 0; uu < 2; ++uu) {
              const int q = qb + uu * BLOCK;
              ix[uu] = q < nb ? bidx(q) : 0;
              w[uu] = q < nb ? double(Vn[ix[uu]]) : 0.0;
#pragma unroll
              for (int p = 0; p < 8; ++p) vv[uu][p] = (p <= j && q < nb) ? V[p * vs + ix[uu]] : TI(0);
            }
#pragma unroll
            for (int p = 0; p < 8; ++p) {
              const double cq = p <= j ? coef[p] : 0.0;
#pragma unroll
              for (int uu = 0; uu < 2; ++uu) w[uu] -= cq * double(vv[uu][p]);
            }
            TI wt[2];
#pragma unroll
            for (int uu = 0; uu < 2; ++uu) {
              wt[uu] = TI(0);
              if (qb + uu * BLOCK < nb) {
                wt[uu] = TI(w[uu]);
                Vn[ix[uu]] = wt[uu];
              }
            }
#pragma unroll
            for (int uu = 0; uu < 2; ++uu)
#pragma unroll
              for (int p = 0; p < 8; ++p) dnext[p] += double(vv[uu][p]) * double(wt[uu]);
          }
        } else {
          // vectors in chunks of 4, all loads of a chunk issued before use
          for (int qb = tid; qb < nb; qb += BLOCK * 2) {
            double w[2];
            int ix[2];
#pragma unroll
            for (int uu = 0; uu < 2; ++uu) {
              const int q = qb + uu * BLOCK;
              ix[uu] = q < nb ? bidx(q) : 0;
              w[uu] = q < nb ? double(Vn[ix[uu]]) : 0.0;
            }
            for (int q0 = 0; q0 <= j; q0 += 4) {
              TI vv[4][2];
#pragma unroll
              for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int uu = 0; uu < 2; ++uu)
                  vv[p][uu] = (q0 + p <= j) ? V[(q0 + p) * vs + ix[uu]] : TI(0);
#pragma unroll
              for (int p = 0; p < 4; ++p) {
                const double cq = (q0 + p <= j) ? coef[q0 + p] : 0.0;
#pragma unroll
                for (int uu = 0; uu < 2; ++uu) w[uu] -= cq * double(vv[p][uu]);
              }
            }
#pragma unroll
            for (int uu = 0; uu < 2; ++uu) {
              if (qb + uu * BLOCK < nb) {
                const TI wt = TI(w[uu]);
                Vn[ix[uu]] = wt;
                nn[0] += double(wt) * double(wt);
              }
            }
          }
        }
        // Only the last pass's norm is used.  A member reads V_{j+1} at
        // its own nodes only, and in the same thread-to-node order as it
        // wrote them, so the first pass ends with a workgroup barrier.
        have_dots = fuse;
        if (pass + 1 < kPasses)
          __syncthreads();
        else
          tsum<1>(nn);
        STM_T1(t_pb, 4);
      }
      const double hn = uni(sqrt(nn[0]));
      if (tid == 0) {
        const double hj1 = sc[j] * hn;
        sc[j + 1] = hn > 0.0 ? 1.0 / hn : 0.0;
        for (int q = 0; q < j; ++q) {  // previous rotations on column j
          const double a = H[q * kMaxRestart + j], b = H[(q + 1) * kMaxRestart + j];
          H[q * kMaxRestart + j] = cs_[q] * a + sn_[q] * b;
          H[(q + 1) * kMaxRestart + j] = -sn_[q] * a + cs_[q] * b;
        }
        const double a = H[j * kMaxRestart + j];
        const double r = sqrt(a * a + hj1 * hj1);
        const double c = r > 0.0 ? a / r : 1.0, sn = r > 0.0 ? hj1 / r : 0.0;
        cs_[j] = c;
        sn_[j] = sn;
        H[j * kMaxRestart + j] = r;
        H[(j + 1) * kMaxRestart + j] = 0.0;
        gv[j + 1] = -sn * gv[j];
        gv[j] = c * gv[j];
        sh_resid = fabs(gv[j + 1]);
      }
      __syncthreads();
      jdim = j + 1;
      const double resid = uni(sh_resid);
      if (!(resid > tol_abs) || !(hn > 0.0)) break;
    }
    io.jdim = jdim;
    if (tid == 0) {
      for (int q = jdim - 1; q >= 0; --q) {
        double acc = gv[q];
        for (int p = q + 1; p < jdim; ++p) acc -= H[q * kMaxRestart + p] * yv[p];
        yv[q] = acc / H[q * kMaxRestart + q];
      }
      for (int q = 0; q < jdim; ++q) coef[q] = yv[q] * sc[q];
    }
    __syncthreads();
    // ---- u += sum_q y_q z_q (float64) over the owned nodes, max-norm of the step ----
    STM_T0(t_up);
    double dm = 0.0;
    bytes = uni(bytes + (double(jdim) * sizeof(TI) * n0 + 24.0 * n0));
    for (int qb = tid; qb < nb; qb += BLOCK * 2) {
      double dl[2] = {0.0, 0.0}, uo[2];
      int ix[2];
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int q = qb + v * BLOCK;
        ix[v] = q < nb ? bidx(q) : 0;
        uo[v] = q < nb ? u[ix[v]] : 0.0;
      }
      for (int q0 = 0; q0 < jdim; q0 += 4) {
        TI zz[4][2];
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
          for (int v = 0; v < 2; ++v) zz[p][v] = (q0 + p < jdim) ? Z[(q0 + p) * vs + ix[v]] : TI(0);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const double cq = (q0 + p < jdim) ? coef[q0 + p] : 0.0;
#pragma unroll
          for (int v = 0; v < 2; ++v) dl[v] += cq * double(zz[p][v]);
        }
      }
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        if (qb + v * BLOCK < nb) {
          u[ix[v]] = uo[v] + dl[v];
          dlt[ix[v]] = dl[v];
          dm = fmax(dm, abs_or_inf(dl[v]));
        }
      }
    }
    io.dmax = uni(tmax(dm));  // its barrier also publishes u to the other members
    STM_T1(t_up, 5);
    io.model_bytes = model_bytes;
    io.resid = sh_resid;
  }

  // lmax of grid l's D^-1 A into the weights of its sweeps; returns lmax.
  __device__ __forceinline__ double sweep_weights(int l) const {
    TI* x0 = (l == 0) ? V + vstride : mgX(l);
    TI* x1 = (l == 0) ? V + 2 * vstride : mgT(l);
    const double lmax = 1.05 * power_lmax(l, x0, x1);
    const int K = (l == L->nmg - 1) ? L->sweeps : prm.smooth_steps;
    if (threadIdx.x == 0) chebyshev_weights(lmax / L->cheb_ratio, lmax, K, omega + l * kMaxSweeps);
    return lmax;
  }
};

// The steps of a 3D solve are functions, called and not inlined, so that each
// gets registers of its own: in one kernel with all of them inlined the state
// of the whole solve (every pass's tile sizes and addresses) is live in every
// pass, and the z-steps spill (780 SGPRs to VGPR lanes and 100-130 VGPRs).  The
// team's state goes through LDS, from where the callee takes it back into
// scalar registers; a call costs about 2 us.
enum { kStepSetup, kStepSpectrum, kStepResidual, kStepCorrect, kStepGmres };
#define STM_LDS __attribute__((address_space(3)))

template <typename TM>
struct CallState {
  TM tm;
  StepIO io;
};

template <typename T>
__device__ __forceinline__ T lds_uniform(const STM_LDS T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole dwords");
  unsigned w[sizeof(T) / 4];
  const STM_LDS unsigned* q = (const STM_LDS unsigned*)p;
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(q[i]);
  T r;
  __builtin_memcpy(&r, w, sizeof(T));
  return r;
}

template <int WHAT, typename TM>
__device__ __forceinline__ void run_step(const TM& tm, StepIO& io) {
  if constexpr (WHAT == kStepSetup) {
    tm.setup_operator();
  } else if constexpr (WHAT == kStepSpectrum) {
    io.dmax = tm.sweep_weights(0);
    io.resid = tm.spectrum_low();
  } else if constexpr (WHAT == kStepResidual) {
    tm.residual_step(io);
  } else if constexpr (WHAT == kStepCorrect) {
    tm.correct_step(io);
  } else {
    tm.gmres_step(io);
  }
}

template <int WHAT, typename TI, int DIM, int BLOCK>
__device__ __attribute__((noinline)) void step_function(STM_LDS CallState<Team<TI, DIM, BLOCK, false>>* st,
                                                        STM_LDS unsigned char* smem, STM_LDS double* red,
                                                        STM_LDS double* omega) {
  auto scalar = [](auto* p) { return (decltype(p))(size_t)__builtin_amdgcn_readfirstlane((int)(size_t)p); };
  st = scalar(st);
  Team<TI, DIM, BLOCK, false> tm = lds_uniform(&st->tm);
  StepIO io = lds_uniform(&st->io);
  tm.smem = (unsigned char*)scalar(smem);
  tm.red = (double*)scalar(red);
  tm.omega = (double*)scalar(omega);
  __syncthreads();  // every wave has read the state
  run_step<WHAT>(tm, io);
  __syncthreads();
  if (threadIdx.x == 0) {
    st->tm.gen = tm.gen;
    st->tm.hgen = tm.hgen;
    st->tm.rslot = tm.rslot;
    st->tm.broken = tm.broken;
    st->tm.bytes = tm.bytes;
    st->io.model_bytes = io.model_bytes;
    st->io.dmax = io.dmax;
    st->io.resid = io.resid;
    st->io.jdim = io.jdim;
  }
  __syncthreads();
}

// A step of the solve: called on single-grid 3D teams, inlined elsewhere.  st->tm
// holds the sample's team state (its counters are those of the last call).
template <int WHAT, typename TI, int DIM, int BLOCK, bool MG>
__device__ __forceinline__ void do_step(const Team<TI, DIM, BLOCK, MG>& tm, StepIO& io,
                                     CallState<Team<TI, DIM, BLOCK, MG>>* st, unsigned char* smem, double* red,
                                     double* omega) {
  if constexpr (DIM == 3 && !MG) {
    auto* s3 = (STM_LDS CallState<Team<TI, DIM, BLOCK, MG>>*)st;
    __syncthreads();
    if (threadIdx.x == 0) {
      s3->tm.gen = tm.gen;
      s3->tm.hgen = tm.hgen;
      s3->tm.rslot = tm.rslot;
      s3->tm.broken = tm.broken;
      s3->tm.bytes = tm.bytes;
      st->io = io;
    }
    __syncthreads();
    step_function<WHAT, TI, DIM, BLOCK>(s3, (STM_LDS unsigned char*)smem, (STM_LDS double*)red,
                                        (STM_LDS double*)omega);
    tm.gen = __builtin_amdgcn_readfirstlane(s3->tm.gen);
    tm.hgen = __builtin_amdgcn_readfirstlane(s3->tm.hgen);
    tm.rslot = __builtin_amdgcn_readfirstlane(s3->tm.rslot);
    tm.broken = __builtin_amdgcn_readfirstlane((int)s3->tm.broken) != 0;
    tm.bytes = uni(s3->tm.bytes);
    io.model_bytes = uni(s3->io.model_bytes);
    io.dmax = uni(s3->io.dmax);
    io.resid = uni(s3->io.resid);
    io.jdim = __builtin_amdgcn_readfirstlane(s3->io.jdim);
  } else {
    run_step<WHAT>(tm, io);
  }
}

template <typename TI, int DIM, int BLOCK, bool MG>
__global__ __launch_bounds__(BLOCK) void st_team_kernel(const LevelDev* __restrict__ levels,
                                                        const TeamTask* __restrict__ tasks, SolverParams prm) {
  constexpr int NW = BLOCK / kWave;
  extern __shared__ __align__(16) unsigned char smem_dyn[];
  __shared__ double red[NW * 9];
  __shared__ double omega_tab[kMaxMG * kMaxSweeps];
  __shared__ CallState<Team<TI, DIM, BLOCK, MG>> calls;
#ifdef STM_PHASE_TIMERS
  __shared__ long long ph_acc[8];
  if (threadIdx.x < 8) ph_acc[threadIdx.x] = 0;
  __syncthreads();
#endif

  const TeamTask task = tasks[blockIdx.x];
  const LevelDev* L = levels + task.level;
  const int tid = threadIdx.x;
  for (int q = tid; q < kMaxMG * kMaxSweeps; q += BLOCK) omega_tab[q] = prm.smooth_omega;
  __syncthreads();

  Team<TI, DIM, BLOCK, MG> tm;
  tm.L = L;
  tm.prm = prm;
  tm.work = task.work;
  tm.smem = smem_dyn;
  tm.omega = omega_tab;
  tm.red = red;
  tm.bytes = 0.0;
  tm.rank = task.rank;
  tm.G = task.G;
  tm.bar = task.bar;
  tm.part = task.part;
  tm.fault = task.fault;
  tm.gen = 0;
  tm.hgen = 0;
  tm.rslot = 0;
  tm.broken = false;
#ifdef STM_PHASE_TIMERS
  tm.ph = ph_acc;
#endif
  const GridDev g0 = L->g[0];
  tm.set_box();
  const int n0 = g0.n;
  const int nb = tm.nband();
  double* __restrict__ u = reinterpret_cast<double*>(task.work + L->off_u);
  double* __restrict__ uprev = reinterpret_cast<double*>(task.work + L->off_uprev);
  double* __restrict__ wk1 = reinterpret_cast<double*>(task.work + L->off_wk1);
  double* __restrict__ tact = reinterpret_cast<double*>(task.work + L->off_tact);
  double* __restrict__ dlt = reinterpret_cast<double*>(task.work + L->off_dlt);
  tm.V = reinterpret_cast<TI*>(task.work + L->off_V);
  tm.kdiag0 = reinterpret_cast<double*>(task.work + L->off_kd);
  tm.dinv = reinterpret_cast<TI*>(task.work + L->off_dinv);
  tm.w0 = reinterpret_cast<TI*>(task.work + L->off_mgW[0]);
  tm.Z = reinterpret_cast<TI*>(task.work + L->off_Z);
  const int64_t vs = (int64_t)((n0 + 63) & ~63);
  tm.vstride = vs;
  double* ubuf = reinterpret_cast<double*>(task.work + L->off_U);

  const int m = L->m;
  const double dt = uni(L->dt), inv_dt = uni(1.0 / L->dt);
  const double kr = uni(prm.k_react), ar = uni(prm.a_react), tau = uni(prm.tau), thr = uni(prm.threshold);
  const double zr = uni(prm.zr);
  const double th = uni(prm.theta);

  bool have_prev = false;
  const double* prevU = nullptr;
  for (int it_s = 0; it_s < task.count; ++it_s) {
    const int s = task.order ? task.order[task.first + it_s * task.stride] : task.first + it_s * task.stride;
    const long long t_start = wall_clock64();
    tm.bytes = 0.0;
    tm.sigma = task.sigma + (int64_t)s * g0.ne;
    double* Uout = task.u_out ? task.u_out + (int64_t)s * m * n0 : ubuf;
    const double* W = nullptr;
    if (task.u_guess) W = task.u_guess + (int64_t)s * m * n0;
    else if (have_prev) W = prevU;

    if (tid == 0) calls.tm = tm;
    StepIO io{};
    io.u = u;
    io.uprev = uprev;
    io.dlt = dlt;
    io.krylov_words = 7.0 + L->pc_words;
    do_step<kStepSetup>(tm, io, &calls, smem_dyn, red, omega_tab);
    // initial state, activation markers, warm-start history
    tm.bytes = uni(tm.bytes + ((24.0 + sizeof(TI) + 24.0) * n0));
    for (int q = tid; q < nb; q += BLOCK) {
      const int idx = tm.bidx(q);
      const double v = L->u0[idx];
      uprev[idx] = v;
      wk1[idx] = v;
      tact[idx] = (v >= thr) ? 0.0 : -1.0;
    }
    tm.sync();

    long long newton_total = 0, krylov_total = 0, damped = 0;
    int newton_max_slab = 0, status = 0;
    // bytes by the per-step word model: 4 float64 words per residual; per
    // Krylov iteration j, 4 (Jacobian product) + the preconditioner's words
    // (5 per sweep and per coarse-grid residual, weighted by the grid's nodes)
    // + 2j + 3 (Arnoldi step) inner words, per node
    double model_bytes = 0.0;
    double worst_final = 0.0;
    bool weights_ready = (prm.smoother == 0);
    // defect correction by Chebyshev sweeps (the default way to a Newton step
    // on single-grid levels): whether this sample takes it, the degree whose
    // weights are in the table, the level's own degree, how many slabs in a row
    // have had to fall back on GMRES, the interval with its decay per sweep, and
    // the curvature: log2 of a slab's second correction over the square of its first
    bool defect = false;
    int nc = 0, fixed = 0, fallbacks = 0;
    double lmax0 = 0.0, low0 = 0.0;
    float decay = 0.0f, curv = -3.0f;

    for (int k = 0; k < m; ++k) {
      // ---- initial iterate of slab k ----
      const double* Wk = W ? W + (int64_t)k * n0 : nullptr;
      tm.bytes = uni(tm.bytes + ((Wk ? 40.0 : 16.0) * n0));
      for (int q = tid; q < nb; q += BLOCK) {
        const int idx = tm.bidx(q);
        if (Wk) {
          const double w = Wk[idx];
          u[idx] = uprev[idx] + (w - wk1[idx]);
          wk1[idx] = w;
        } else {
          u[idx] = uprev[idx];
        }
      }
      tm.sync();

      double dprev = 0.0, eta = fmax(prm.gmres_rtol, 1e-5);
      int it = 0;
      bool conv = false;
      double dmax = 0.0;
      // damping: the residual 2-norm of the last accepted iterate and the
      // fraction of the last Newton step in u (halved while the residual grows)
      double beta_acc = 0.0, tstep = 1.0;
      // what u has had since then: a defect correction (in Z), a Newton step
      // (in dlt), or neither
      bool corrected = false, stepped = false;
      bool cheb = defect;
      int ncor = 0;  // defect corrections of the slab (not counted against newton_max)
      float ldp = 0.0f;  // log2 of the last correction, and its degree
      int ncp = 0;
      if constexpr (!MG) {
        if (cheb && !fixed) {
          const int n1 = tm.cheb_degree(decay, DIM == 2 ? kFirstBits2 : kFirstBits3);
          if (n1 != nc) tm.cheb_weights(low0, lmax0, nc = n1);
        }
      }
      for (; it - ncor < prm.newton_max; ++it) {
        // ---- residual (float64) -> V_0, Jacobian weights on every grid ----
        // 3D defect corrections start with the sweep from zero, om r / diag, there
        io.x1 = DIM == 3 && !MG && cheb;
        STM_T0(t_res);
        do_step<kStepResidual>(tm, io, &calls, smem_dyn, red, omega_tab);
        STM_T1(t_res, 0);
        model_bytes = uni(model_bytes + 32.0 * n0);
        const double beta = uni(sqrt(io.resid));
        if (!isfinite(beta) && !corrected && !(prm.damping && stepped && tstep > kMinStep)) {
          status = -5;
          break;
        }
        if (beta == 0.0) {
          conv = true;
          dmax = 0.0;
          break;
        }
        // a defect correction that did not contract the residual well (the
        // first two may owe their remainder to the reaction) leaves the rest of
        // the slab to GMRES; one that made it grow is taken back
        if (corrected && !(beta <= (ncor <= 2 ? 0.5 : kContract) * beta_acc)) {
          cheb = false;
          if (++fallbacks > kMaxFallbacks) defect = false;
          if (!(beta <= beta_acc)) {
            for (int q = tid; q < nb; q += BLOCK) {
              const int idx = tm.bidx(q);
              u[idx] = isfinite(beta) ? u[idx] - double(tm.Z[idx]) : uprev[idx];
            }
            tm.bytes = uni(tm.bytes + (16.0 + sizeof(TI)) * n0);
            beta_acc = HUGE_VAL;
            corrected = false;
            dprev = 0.0;
            ++ncor;
            tm.sync();
            continue;
          }
        }
        // the last Newton step made the residual grow (or not finite): take half of
        // it back, u -= (t/2) delta, and evaluate again (Armijo-style halving
        // down to kMinStep; the pass counts as a Newton iteration)
        if (prm.damping && stepped && !(beta <= beta_acc) && tstep > kMinStep) {
          tstep = uni(0.5 * tstep);
          for (int q = tid; q < nb; q += BLOCK) {
            const int idx = tm.bidx(q);
            u[idx] -= tstep * dlt[idx];
          }
          tm.bytes = uni(tm.bytes + 24.0 * n0);
          dmax = uni(0.5 * dmax);
          ++damped;
          tm.sync();
          continue;
        }
        beta_acc = beta;
        tstep = 1.0;
        corrected = stepped = false;
        // ---- smoother weights: once per sample, from the first slab operator ----
        if (!weights_ready) {
          if constexpr (MG) {
            for (int l = 0; l < L->nmg; ++l) tm.sweep_weights(l);
          } else {
            do_step<kStepSpectrum>(tm, io, &calls, smem_dyn, red, omega_tab);
            lmax0 = uni(io.dmax);
            low0 = uni(io.resid);
            if (low0 > 0.0 && lmax0 > low0 && lmax0 < kWidest * low0) {
              // The interval is the spectrum's and never narrower by itself:
              // corrections do not see the modes left out, and slabs would be
              // accepted with their error.  A level's own sweeps and ratio are
              // taken where they contract the whole spectrum; else they are GMRES's.
              const double own = L->own_ratio > 0.0 ? L->own_ratio : lmax0 / low0;
              fixed = 0;
              if (L->own_sweeps > 0 && tm.cheb_reduction(own, low0 / lmax0, L->own_sweeps) <= kContract) {
                low0 = lmax0 / own;
                fixed = tm.odd_or_even(max(L->own_sweeps, 3));
              }
              decay = tm.cheb_decay(lmax0 / low0);
              nc = fixed ? fixed : tm.cheb_degree(decay, DIM == 2 ? kFirstBits2 : kFirstBits3);
              tm.cheb_weights(low0, lmax0, nc);
              defect = cheb = true;
            }
          }
          __syncthreads();
          weights_ready = true;
        }

        if constexpr (!MG) {
          if (cheb) {
            // ---- defect correction: u += P(A) r, P the Chebyshev sweeps ----
            model_bytes = uni(model_bytes + double(sizeof(TI)) * n0 * 5.0 * nc);
            STM_T0(t_ch);
            io.nc = nc;
            do_step<kStepCorrect>(tm, io, &calls, smem_dyn, red, omega_tab);
            dmax = uni(io.dmax);
            corrected = true;
            STM_T1(t_ch, 1);
            ++krylov_total;
            ++ncor;
            if (!(dmax < 1e3)) {  // far out of range or not finite: GMRES from the previous slab's state
              for (int q = tid; q < nb; q += BLOCK) {
                const int idx = tm.bidx(q);
                u[idx] = uprev[idx];
              }
              defect = cheb = corrected = false;
              beta_acc = HUGE_VAL;
              dprev = 0.0;
              tm.sync();
              continue;
            }
            // The error left, as log2: what the degree leaves of it, or what is
            // seen of the contraction so far (corrections contract linearly, at
            // a rate per sweep), or Newton's own remainder, whichever is most.
            const float ld = log2f(fmaxf((float)dmax, 1e-37f));
            float shrink = 1.0f - nc * decay;
            if (sizeof(TI) == 4) shrink = fmaxf(shrink, -kFloatBits);
            if (ncor == 2) curv = ld - 2.0f * ldp;
            if (ncor >= 2) shrink = fmaxf(shrink, fminf((ld - ldp) * nc / ncp, 0.0f));
            const float left = fmaxf(ld + shrink, curv + 2.0f * ld);
            const float goal = log2f((float)fmax(kLeft * prm.newton_tol, kRounding));
            if (left <= goal && left <= log2f((float)prm.newton_tol)) {
              conv = true;
              ++it;
              break;
            }
            // the next correction's degree: down to the goal or to Newton's
            // remainder, in equal parts where that is more than one can give
            ncp = nc;
            ldp = ld;
            if (!fixed && ncor < kMaxCorrections) {
              const float bits = fmaxf(left - fmaxf(goal - 1.0f, curv + 2.0f * left), kLeastBits);
              const float most = fminf(kMaxDegree * decay - 1.0f, sizeof(TI) == 4 ? kFloatBits : 100.0f);
              const int n = tm.cheb_degree(decay, bits / ceilf(bits / most));
              if (n != nc) tm.cheb_weights(low0, lmax0, nc = n);
            }
            dprev = uni(dmax);
            eta = uni(fmax(prm.gmres_rtol, fmin(1e-4, 0.01 * dmax)));
            if (ncor >= kMaxCorrections) cheb = false;
            continue;
          }
        }

        // ---- Newton step by GMRES ----
        io.beta = beta;
        io.eta = eta;
        io.model_bytes = model_bytes;
        do_step<kStepGmres>(tm, io, &calls, smem_dyn, red, omega_tab);
        krylov_total += io.jdim;
        model_bytes = uni(io.model_bytes);
        dmax = uni(io.dmax);
        stepped = true;
        const double ach = io.resid / beta;
        if (!isfinite(dmax)) {
          status = -5;
          break;
        }
        if (dmax <= prm.newton_tol) {
          conv = true;
          ++it;
          break;
        }
        if (it >= 1) {
          const double ratio = dmax / dprev;
          const double pred = dmax * fmax(ratio * ratio, 10.0 * ach);
          if (ratio < 0.5 && pred <= 0.1 * prm.newton_tol) {
            conv = true;
            ++it;
            break;
          }
        }
        dprev = uni(dmax);
        eta = uni(fmax(prm.gmres_rtol, fmin(1e-4, 0.01 * dmax)));
      }
      if (status == -5) break;
      if (!conv && status == 0) status = -4;
      if (cheb) fallbacks = 0;
      newton_total += it;
      newton_max_slab = max(newton_max_slab, it);
      worst_final = uni(fmax(worst_final, dmax));

      // ---- accept slab k: store, activation crossing, shift history ----
      double* Uk = Uout + (int64_t)k * n0;
      const double tk = k * dt;
      tm.bytes = uni(tm.bytes + (40.0 * n0));
      for (int q = tid; q < nb; q += BLOCK) {
        const int idx = tm.bidx(q);
        const double un = u[idx], up = uprev[idx];
        Uk[idx] = un;
        if (tact[idx] < 0.0 && un >= thr) tact[idx] = tk + dt * (thr - up) / (un - up);
        uprev[idx] = un;
      }
      tm.sync();
    }

    // ---- finalize the sample ----
    double cen[1] = {0.0};
    for (int q = tid; q < nb; q += BLOCK) {
      const int idx = tm.bidx(q);
      double t = tact[idx];
      if (t < 0.0) {
        t = L->T;
        cen[0] += 1.0;
      }
      if (task.t_act) task.t_act[(int64_t)s * n0 + idx] = t;
    }
    tm.template tsum<1>(cen);
    if (tid == 0 && task.stats && task.rank == 0) {
      SampleStatsDev st;
      st.status = tm.broken ? -3 : status;
      st.newton_max_per_slab = newton_max_slab;
      st.newton_iters = newton_total;
      st.krylov_iters = krylov_total;
      st.final_step = worst_final;
      st.ticks = wall_clock64() - t_start;
      st.censored = (int)cen[0];
      st.damped = (int)damped;
      st.alg_bytes = tm.bytes;
      st.model_bytes = model_bytes;
      for (int q = 0; q < 8; ++q) st.phase_ticks[q] = 0;
#ifdef STM_PHASE_TIMERS
      for (int q = 0; q < 8; ++q) st.phase_ticks[q] = ph_acc[q];
#endif
      task.stats[s] = st;
    }
#ifdef STM_PHASE_TIMERS
    __syncthreads();
    if (threadIdx.x < 8) ph_acc[threadIdx.x] = 0;
#endif
    prevU = Uout;
    have_prev = (status == 0);
    tm.sync();
  }
}

// ---------------------------------------------------------------------------
// Global space-time solve (Sec. 3.2 eq. system_C, Sec. 3.5): Newton on the
// whole space-time system at once.  Each linear step J delta = -R is one GMRES
// over all m slabs, right-preconditioned by forward substitution in time in
// which every diagonal block is replaced by the slab preconditioner (one
// V-cycle, or the Chebyshev-weighted sweeps):
//   z_0 = P_0^-1 r_0,  z_k = P_k^-1 (r_k - B z_{k-1}),  B = -M/dt + (1 - theta) K.
// The residual and the product J x = (A_k x_k + B x_{k-1})_k treat every slab
// on its own (the parallel-in-time part of the method); the preconditioner
// sweeps the slabs in order.  The step is added in float64 and halved while
// the residual 2-norm grows, as in the slab solve; the first iterate is the
// lane's previous solution or the caller's guess, else the initial state at
// every time level.  Teams, tasks and statistics as in st_team_kernel
// (newton_max_per_slab is the number of global Newton steps).
// ---------------------------------------------------------------------------
template <typename TI, int DIM, int BLOCK, bool MG>
__global__ __launch_bounds__(BLOCK) void st_global_kernel(const LevelDev* __restrict__ levels,
                                                          const TeamTask* __restrict__ tasks, SolverParams prm) {
  constexpr int NW = BLOCK / kWave;
  extern __shared__ __align__(16) unsigned char smem_dyn[];
  __shared__ double red[NW * 9];
  __shared__ double H[(kMaxRestart + 1) * kMaxRestart];
  __shared__ double cs_[kMaxRestart], sn_[kMaxRestart], gv[kMaxRestart + 1], sc[kMaxRestart + 1];
  __shared__ double yv[kMaxRestart], coef[kMaxRestart + 1];
  __shared__ double omega_tab[kMaxMG * kMaxSweeps];
  __shared__ double sh_resid;
#ifdef STM_PHASE_TIMERS
  __shared__ long long ph_acc[8];
  if (threadIdx.x < 8) ph_acc[threadIdx.x] = 0;
  __syncthreads();
#endif

  const TeamTask task = tasks[blockIdx.x];
  const LevelDev* L = levels + task.level;
  const int tid = threadIdx.x;
  for (int q = tid; q < kMaxMG * kMaxSweeps; q += BLOCK) omega_tab[q] = prm.smooth_omega;
  __syncthreads();

  Team<TI, DIM, BLOCK, MG> tm;
  tm.L = L;
  tm.prm = prm;
  tm.work = task.work;
  tm.smem = smem_dyn;
  tm.omega = omega_tab;
  tm.red = red;
  tm.bytes = 0.0;
  tm.rank = task.rank;
  tm.G = task.G;
  tm.bar = task.bar;
  tm.part = task.part;
  tm.fault = task.fault;
  tm.gen = 0;
  tm.hgen = 0;
  tm.rslot = 0;
  tm.broken = false;
#ifdef STM_PHASE_TIMERS
  tm.ph = ph_acc;
#endif
  const GridDev g0 = L->g[0];
  tm.set_box();
  const int n0 = g0.n;
  const int nb = tm.nband();
  double* __restrict__ tact = reinterpret_cast<double*>(task.work + L->off_tact);
  tm.V = reinterpret_cast<TI*>(task.work + L->off_V);  // slab-sized scratch of the power iteration
  tm.Z = reinterpret_cast<TI*>(task.work + L->off_Z);
  tm.kdiag0 = reinterpret_cast<double*>(task.work + L->off_kd);
  tm.dinv = reinterpret_cast<TI*>(task.work + L->off_dinv);
  tm.w0 = reinterpret_cast<TI*>(task.work + L->off_mgW[0]);
  const int64_t vs = (int64_t)((n0 + 63) & ~63);
  tm.vstride = vs;
  const int m = L->m;
  const int64_t gs = (int64_t)m * vs;  // stride of space-time vectors
  TI* __restrict__ gV = reinterpret_cast<TI*>(task.work + L->off_gV);
  TI* __restrict__ gW = reinterpret_cast<TI*>(task.work + L->off_gW);
  TI* __restrict__ gD = reinterpret_cast<TI*>(task.work + L->off_gD);
  TI* __restrict__ gZ = reinterpret_cast<TI*>(task.work + L->off_gZ);
  TI* __restrict__ gT = reinterpret_cast<TI*>(task.work + L->off_gT);
  double* ubuf = reinterpret_cast<double*>(task.work + L->off_U);

  const double dt = uni(L->dt), inv_dt = uni(1.0 / L->dt);
  const double kr = uni(prm.k_react), ar = uni(prm.a_react), thr = uni(prm.threshold);
  const double th = uni(prm.theta);
  const double cmd = (DIM == 3) ? 8.0 * g0.hx * g0.hy * g0.hz / 216.0 : 4.0 * g0.hx * g0.hy / 36.0;
  const int restart = prm.restart;

  bool have_prev = false;
  const double* prevU = nullptr;

  for (int it_s = 0; it_s < task.count; ++it_s) {
    const int s = task.order ? task.order[task.first + it_s * task.stride] : task.first + it_s * task.stride;
    const long long t_start = wall_clock64();
    tm.bytes = 0.0;
    tm.sigma = task.sigma + (int64_t)s * g0.ne;
    double* __restrict__ U = task.u_out ? task.u_out + (int64_t)s * m * n0 : ubuf;
    const double* W = nullptr;
    if (task.u_guess) W = task.u_guess + (int64_t)s * m * n0;
    else if (have_prev) W = prevU;

    tm.setup_operator();
    // first iterate: the guess, else the initial state at every time level
    tm.bytes = uni(tm.bytes + 16.0 * (double)m * n0);
    for (int k = 0; k < m; ++k)
      for (int q = tid; q < nb; q += BLOCK) {
        const int idx = tm.bidx(q);
        U[(int64_t)k * n0 + idx] = W ? W[(int64_t)k * n0 + idx] : L->u0[idx];
      }
    tm.sync();

    // z = P^-1 r over the space-time vectors r, z: forward substitution in time
    auto precond = [&](const TI* __restrict__ r, TI* __restrict__ z) {
      for (int k = 0; k < m; ++k) {
        tm.w0 = gW + k * vs;
        tm.dinv = gD + k * vs;
        if (MG) tm.coarse_weights(U + (int64_t)k * n0, inv_dt);
        const TI* b = r + k * vs;
        if (k > 0) {
          tm.template staged<TI, 0>(
              0, z + (k - 1) * vs, r + k * vs, (const TI*)nullptr, (const TI*)nullptr,
              KScale<TI>{TI(1.0 - th)}, [c0 = TI(-inv_dt)](TI a, TI) { return c0 * a; },
              [&](int idx, int, int, int, TI y, TI, TI ro, TI, TI) { gmem(gT)[idx] = ro - y; });
          b = gT;
        }
        tm.vcycle(b, z + k * vs);
      }
    };
    // y = J x: slab products and the coupling to the previous slab
    auto spmv = [&](const TI* __restrict__ x, TI* __restrict__ y) {
      for (int k = 0; k < m; ++k) {
        TI* yk = y + k * vs;
        tm.template staged<TI, 0>(
            0, x + k * vs, gW + k * vs, (const TI*)nullptr, (const TI*)nullptr,
            KScale<TI>{TI(th)}, [](TI a, TI ww) { return ww * a; },
            [&](int idx, int, int, int, TI v, TI, TI, TI, TI) { gmem(yk)[idx] = v; });
        if (k > 0)
          // in place: f1 = y_k enters only the body (its own node), never the element terms
          tm.template staged<TI, 0>(
              0, x + (k - 1) * vs, yk, (const TI*)nullptr, (const TI*)nullptr,
              KScale<TI>{TI(1.0 - th)}, [c0 = TI(-inv_dt)](TI a, TI) { return c0 * a; },
              [&](int idx, int, int, int, TI v, TI, TI yo, TI, TI) { gmem(yk)[idx] = yo + v; });
      }
    };

    long long krylov_total = 0, damped = 0;
    int status = 0;
    // per-step word model: 4 float64 words per node and slab per residual; per
    // Krylov iteration j, per node and slab: 4 (slab product) + 4 (coupling) +
    // 4 (coupling in the substitution) + the slab preconditioner's words +
    // 2j + 3 (Arnoldi step) inner words
    double model_bytes = 0.0;
    const double krylov_words = 15.0 + L->pc_words;
    const double nm = (double)m * n0;
    bool weights_ready = (prm.smoother == 0);
    double dprev = 0.0, eta = fmax(prm.gmres_rtol, 1e-5), dmax = 0.0;
    double beta_acc = 0.0, tstep = 1.0;
    bool conv = false;
    int it = 0;
    for (; it < prm.newton_max; ++it) {
      // ---- residual of every slab (float64) -> V_0 = -R, weights and inverse diagonals ----
      double rr[1] = {0.0};
      tm.bytes = uni(tm.bytes + (24.0 * nm + 8.0 * g0.ne * m + 3.0 * sizeof(TI) * nm));
      for (int k = 0; k < m; ++k) {
        const double* uk = U + (int64_t)k * n0;
        const double* up = k ? U + (int64_t)(k - 1) * n0 : L->u0;
        TI* Vk = gV + k * vs;
        TI* wk = gW + k * vs;
        TI* dk = gD + k * vs;
        tm.template staged<double, 1>(
            0, uk, up, tm.kdiag0, (const double*)nullptr,
            [th](double a, double b) { return th * a + (1.0 - th) * b; },
            [&](double a, double b) { return (a - b) * inv_dt - react(a, kr, ar); },
            [&](int idx, int i, int j, int kk, double y, double uown, double, double kd, double) {
              const double r = -y;
              const double w = inv_dt - react_d(uown, kr, ar);
              gmem(Vk)[idx] = TI(r);
              gmem(wk)[idx] = TI(w);
              gmem(dk)[idx] = TI(1.0 / (th * kd + tm.nel(0, i, j, kk) * cmd * w));
              rr[0] += r * r;
            });
      }
      tm.template tsum<1>(rr);
      model_bytes = uni(model_bytes + 32.0 * nm);
      const double beta = uni(sqrt(rr[0]));
      if (!isfinite(beta) && !(prm.damping && it > 0 && tstep > kMinStep)) {
        status = -5;
        break;
      }
      if (beta == 0.0) {
        conv = true;
        dmax = 0.0;
        break;
      }
      // the last step made the residual grow: take half of it back
      if (prm.damping && it > 0 && !(beta <= beta_acc) && tstep > kMinStep) {
        tstep = uni(0.5 * tstep);
        for (int k = 0; k < m; ++k)
          for (int q = tid; q < nb; q += BLOCK) {
            const int idx = tm.bidx(q);
            U[(int64_t)k * n0 + idx] -= tstep * double(gZ[k * vs + idx]);
          }
        tm.bytes = uni(tm.bytes + (16.0 + sizeof(TI)) * nm);
        dmax = uni(0.5 * dmax);
        ++damped;
        tm.sync();
        continue;
      }
      beta_acc = beta;
      tstep = 1.0;
      // ---- smoother weights: once per sample, from the first slab operator ----
      if (!weights_ready) {
        tm.w0 = gW;
        tm.dinv = gD;
        if (MG) tm.coarse_weights(U, inv_dt);
        for (int l = 0; l < (MG ? L->nmg : 1); ++l) {
          TI* x0 = (l == 0) ? tm.V + vs : tm.mgX(l);
          TI* x1 = (l == 0) ? tm.V + 2 * vs : tm.mgT(l);
          const double lmax = 1.05 * tm.power_lmax(l, x0, x1);
          const int K = (l == L->nmg - 1) ? L->sweeps : prm.smooth_steps;
          if (tid == 0) chebyshev_weights(lmax / L->cheb_ratio, lmax, K, omega_tab + l * kMaxSweeps);
        }
        __syncthreads();
        weights_ready = true;
      }

      // ---- GMRES(restart) over the space-time vectors ----
      if (tid == 0) {
        sc[0] = 1.0 / beta;
        gv[0] = beta;
      }
      __syncthreads();
      const double tol_abs = uni(eta * beta);
      int jdim = 0;
      for (int j = 0; j < restart; ++j) {
        const TI* Vj = gV + j * gs;
        TI* Vn = gV + (j + 1) * gs;
        model_bytes = uni(model_bytes + double(sizeof(TI)) * nm * (krylov_words + 2.0 * j));
        precond(Vj, gZ);
        spmv(gZ, Vn);
        // Classical Gram-Schmidt against V_0..V_j, twice for float32 (CGS2)
        double nn[1] = {0.0};
        constexpr int kPasses = sizeof(TI) == 4 ? 2 : 1;
#pragma unroll 1
        for (int pass = 0; pass < kPasses; ++pass) {
          for (int k0 = 0; k0 <= j; k0 += 8) {
            const int nk = min(j + 1 - k0, 8);
            tm.bytes = uni(tm.bytes + ((1.0 + nk) * sizeof(TI) * nm));
            double d[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) d[q] = 0.0;
            for (int k = 0; k < m; ++k)
              for (int q = tid; q < nb; q += BLOCK) {
                const int64_t idx = k * vs + tm.bidx(q);
                const double wd = double(Vn[idx]);
#pragma unroll
                for (int p = 0; p < 8; ++p)
                  if (p < nk) d[p] += double(gV[(k0 + p) * gs + idx]) * wd;
              }
            tm.template tsum<9>(d);
            if (tid == 0) {
#pragma unroll
              for (int q = 0; q < 8; ++q)
                if (q < nk) coef[k0 + q] = d[q];
            }
          }
          // projections onto the normalised basis enter H; V_q is stored with
          // norm 1/sc[q], so w loses (sc[q]^2 <V_q, w>) V_q
          if (tid == 0)
            for (int q = 0; q <= j; ++q) {
              const double hq = sc[q] * sc[j] * coef[q];
              H[q * kMaxRestart + j] = (pass ? H[q * kMaxRestart + j] : 0.0) + hq;
              coef[q] = sc[q] * sc[q] * coef[q];
            }
          __syncthreads();
          nn[0] = 0.0;
          tm.bytes = uni(tm.bytes + ((j + 3.0) * sizeof(TI) * nm));
          for (int k = 0; k < m; ++k)
            for (int q = tid; q < nb; q += BLOCK) {
              const int64_t idx = k * vs + tm.bidx(q);
              double w = double(Vn[idx]);
              for (int p = 0; p <= j; ++p) w -= coef[p] * double(gV[p * gs + idx]);
              const TI wt = TI(w);
              Vn[idx] = wt;
              nn[0] += double(wt) * double(wt);
            }
          tm.template tsum<1>(nn);  // its barriers also publish V_{j+1}
        }
        const double hn = uni(sqrt(nn[0]));
        if (tid == 0) {
          const double hj1 = sc[j] * hn;
          sc[j + 1] = hn > 0.0 ? 1.0 / hn : 0.0;
          for (int q = 0; q < j; ++q) {  // previous rotations on column j
            const double a = H[q * kMaxRestart + j], b = H[(q + 1) * kMaxRestart + j];
            H[q * kMaxRestart + j] = cs_[q] * a + sn_[q] * b;
            H[(q + 1) * kMaxRestart + j] = -sn_[q] * a + cs_[q] * b;
          }
          const double a = H[j * kMaxRestart + j];
          const double r = sqrt(a * a + hj1 * hj1);
          const double c = r > 0.0 ? a / r : 1.0, sn = r > 0.0 ? hj1 / r : 0.0;
          cs_[j] = c;
          sn_[j] = sn;
          H[j * kMaxRestart + j] = r;
          H[(j + 1) * kMaxRestart + j] = 0.0;
          gv[j + 1] = -sn * gv[j];
          gv[j] = c * gv[j];
          sh_resid = fabs(gv[j + 1]);
        }
        __syncthreads();
        jdim = j + 1;
        const double resid = uni(sh_resid);
        if (!(resid > tol_abs) || !(hn > 0.0)) break;
      }
      krylov_total += jdim;
      if (tid == 0) {
        for (int q = jdim - 1; q >= 0; --q) {
          double acc = gv[q];
          for (int p = q + 1; p < jdim; ++p) acc -= H[q * kMaxRestart + p] * yv[p];
          yv[q] = acc / H[q * kMaxRestart + q];
        }
        for (int q = 0; q < jdim; ++q) coef[q] = yv[q] * sc[q];
      }
      __syncthreads();
      // ---- delta = P^-1 (sum_q y_q v_q); U += delta (float64), max-norm ----
      TI* t = gV + jdim * gs;  // the last basis vector is no longer needed
      tm.bytes = uni(tm.bytes + (double(jdim) + 1.0) * sizeof(TI) * nm);
      for (int k = 0; k < m; ++k)
        for (int q = tid; q < nb; q += BLOCK) {
          const int64_t idx = k * vs + tm.bidx(q);
          double acc = 0.0;
          for (int p = 0; p < jdim; ++p) acc += coef[p] * double(gV[p * gs + idx]);
          t[idx] = TI(acc);
        }
      tm.sync();
      precond(t, gZ);
      double dm = 0.0;
      tm.bytes = uni(tm.bytes + (16.0 + sizeof(TI)) * nm);
      for (int k = 0; k < m; ++k)
        for (int q = tid; q < nb; q += BLOCK) {
          const int idx = tm.bidx(q);
          const double dl = double(gZ[k * vs + idx]);
          U[(int64_t)k * n0 + idx] += dl;
          dm = fmax(dm, abs_or_inf(dl));
        }
      dmax = uni(tm.tmax(dm));  // its barrier also publishes U to the other members
      const double ach = sh_resid / beta;
      if (!isfinite(dmax)) {
        status = -5;
        break;
      }
      if (dmax <= prm.newton_tol) {
        conv = true;
        ++it;
        break;
      }
      if (it >= 1) {
        const double ratio = dmax / dprev;
        const double pred = dmax * fmax(ratio * ratio, 10.0 * ach);
        if (ratio < 0.5 && pred <= 0.1 * prm.newton_tol) {
          conv = true;
          ++it;
          break;
        }
      }
      dprev = uni(dmax);
      eta = uni(fmax(prm.gmres_rtol, fmin(1e-4, 0.01 * dmax)));
    }
    if (!conv && status == 0) status = -4;

    // ---- activation map: first up-crossing in time at every owned node ----
    double cen[1] = {0.0};
    tm.bytes = uni(tm.bytes + 8.0 * nm + 16.0 * n0);
    for (int q = tid; q < nb; q += BLOCK) {
      const int idx = tm.bidx(q);
      double up = L->u0[idx];
      double t = (up >= thr) ? 0.0 : -1.0;
      for (int k = 0; k < m; ++k) {
        const double un = U[(int64_t)k * n0 + idx];
        if (t < 0.0 && un >= thr) t = k * dt + dt * (thr - up) / (un - up);
        up = un;
      }
      if (t < 0.0) {
        t = L->T;
        cen[0] += 1.0;
      }
      tact[idx] = t;
      if (task.t_act) task.t_act[(int64_t)s * n0 + idx] = t;
    }
    tm.template tsum<1>(cen);
    if (tid == 0 && task.stats && task.rank == 0) {
      SampleStatsDev st;
      st.status = tm.broken ? -3 : status;
      st.newton_max_per_slab = it;
      st.newton_iters = it;
      st.krylov_iters = krylov_total;
      st.final_step = dmax;
      st.ticks = wall_clock64() - t_start;
      st.censored = (int)cen[0];
      st.damped = (int)damped;
      st.alg_bytes = tm.bytes;
      st.model_bytes = model_bytes;
      for (int q = 0; q < 8; ++q) st.phase_ticks[q] = 0;
#ifdef STM_PHASE_TIMERS
      for (int q = 0; q < 8; ++q) st.phase_ticks[q] = ph_acc[q];
#endif
      task.stats[s] = st;
    }
#ifdef STM_PHASE_TIMERS
    __syncthreads();
    if (threadIdx.x < 8) ph_acc[threadIdx.x] = 0;
#endif
    prevU = U;
    have_prev = (status == 0);
    tm.sync();
  }
}

// ---------------------------------------------------------------------------
// Kernels of one dimension and inner precision: this file is compiled once for
// each pair (STM_SOLVER_DIM 2 or 3, STM_SOLVER_FP32 0 or 1), side by side.
// ---------------------------------------------------------------------------
#if STM_SOLVER_FP32
using SolverInner = float;
#else
using SolverInner = double;
#endif

template <bool MG>
static const void* kernel_for_block(int block, bool global) {
  if (global) {
    switch (block) {
      case 256: return (const void*)st_global_kernel<SolverInner, STM_SOLVER_DIM, 256, MG>;
      case 512: return (const void*)st_global_kernel<SolverInner, STM_SOLVER_DIM, 512, MG>;
      default: return nullptr;
    }
  }
  switch (block) {
    case 256: return (const void*)st_team_kernel<SolverInner, STM_SOLVER_DIM, 256, MG>;
    case 512: return (const void*)st_team_kernel<SolverInner, STM_SOLVER_DIM, 512, MG>;
    case 1024: return (const void*)st_team_kernel<SolverInner, STM_SOLVER_DIM, 1024, MG>;
    default: return nullptr;
  }
}

// The multi-grid kernel variant (MG = true) serves launches with a level
// whose V-cycle has coarse grids; the others take the single-grid variant,
// which compiles none of the coarse-grid code.
template <>
const void* solver_kernel_of<STM_SOLVER_DIM, STM_SOLVER_FP32 != 0>(bool mg, int block, bool global) {
  return mg ? kernel_for_block<true>(block, global) : kernel_for_block<false>(block, global);
}

}  // namespace stm
