// Self-consistent field mode: the semi-implicit Euler-Maruyama step of the paper's
// "Final algorithm" (steps 1-5) and its field solve.
//
//   1. sigma^k = e sum_p mu_p w_p W(x - X_p^k) / dV with mu_p = mu(|E^k(X_p^k)|)
//      (eq. conductivity, electrons only; ions are immobile);
//   2. X_dagger = X^k + sqrt(2 D dt) N, regenerated from the particle's push stream;
//   3. rho_dagger = e (n+ - n- - CIC(X_dagger)) / dV, solve
//      div[(1 + sigma dt / eps0) grad phi] = -rho_dagger / eps0 (eq. poisson_simp) with
//      phi = 0 at z = 0, phi = V at z = L, homogeneous Neumann on x and y;
//   4-5. X^{k+1} = X_dagger - mu_p E^{k+1}(X^k) dt, binned by cell as in the uniform push.
//
// Discretisation: cell-centred finite volumes, 7-point stencil, face coefficients the
// harmonic mean of the two cell values, a Dirichlet face using the cell's own value
// over half a cell; E at cell centres by central differences with ghost values from
// the same conditions; CIC deposit/interpolation with tent weights about cell centres,
// clouds folded into the wall cells.
//
// Solver: geometric multigrid V(2,2) cycles with red-black Gauss-Seidel, cell-averaged
// restriction and trilinear prolongation, run in the working precision on the
// correction equation of an iterative-refinement loop whose residual and potential
// are kept in double; the loop stops at ||r||_2 <= rtol ||b||_2 (the paper's relative
// multigrid tolerance, 1e-10 by default).
#include <math.h>

#include <vector>


#include "device.hpp"
#include "itk.hpp"

namespace itk {

namespace {

constexpr double kE = 1.602176634e-19;
constexpr double kEps0 = 8.8541878128e-12;
constexpr int kMaxLevels = 12;
constexpr int kBottomMaxCells = 4096;

struct Level {
  int nx, ny, nz;
  uint32_t n;
  void* u;    // correction
  void* f;    // right-hand side (scaled by h^2)
  void* eps;  // cell coefficient 1 + sigma dt / eps0
  void* cf;   // small levels: packed face coefficients and diagonal; tiled levels in double:
              // the same as four arrays
  void* u2;   // tiled levels below the finest: the correction after post-smoothing
};

struct Coef {
  double mu_a, mu_E0, mu_b, E_floor, D;
};

template <typename T>
__device__ __forceinline__ T* tp(void* p) { return reinterpret_cast<T*>(p); }
template <typename T>
__device__ __forceinline__ const T* ctp(const void* p) { return reinterpret_cast<const T*>(p); }

// Four values of T as one 16- (float) or two 16-byte (double) accesses.
template <typename T>
struct V4 {
  T a[4];
};

template <typename T>
__device__ __forceinline__ V4<T> ld4(const T* p) {
  V4<T> v;
  if constexpr (sizeof(T) == 4) {
    const float4 x = *reinterpret_cast<const float4*>(p);
    v.a[0] = x.x; v.a[1] = x.y; v.a[2] = x.z; v.a[3] = x.w;
  } else {
    const double2 x = reinterpret_cast<const double2*>(p)[0], y = reinterpret_cast<const double2*>(p)[1];
    v.a[0] = x.x; v.a[1] = x.y; v.a[2] = y.x; v.a[3] = y.y;
  }
  return v;
}

template <typename T>
__device__ __forceinline__ void st4(T* p, const T a0, const T a1, const T a2, const T a3) {
  if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<float4*>(p) = make_float4(a0, a1, a2, a3);
  } else {
    reinterpret_cast<double2*>(p)[0] = make_double2(a0, a1);
    reinterpret_cast<double2*>(p)[1] = make_double2(a2, a3);
  }
}


constexpr int kRedBlocks = 1024;  // fixed grid of the norm kernels: one partial per block

// Block-wide sum of a double (256 threads), valid in thread 0.
__device__ __forceinline__ double block_sumd(double v) {
  __shared__ double sh[4];
  v = wave_sumd(v);
  if (lane_id() == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) s = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return s;
}

// Sum of the per-block partials in a fixed order (deterministic).
__global__ void __launch_bounds__(1024) k_sum_partials(const double* part, int n, double* out) {
  __shared__ double sh[16];
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) v += part[i];
  v = wave_sumd(v);
  if (lane_id() == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < 16; ++i) s += sh[i];
    *out = s;
  }
}

// The residual's norm as k_sum_partials computes it, also written with ||b||^2 into
// mapped host memory, followed by a sequence number (after a system-scope fence), so
// that the host can wait for it by polling instead of a copy and a stream
// synchronisation.
__global__ void __launch_bounds__(1024) k_sum_notify(const double* part, int n, double* out,
                                                     const double* bn2, double* host,
                                                     unsigned long long* seq) {
  __shared__ double sh[16];
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) v += part[i];
  v = wave_sumd(v);
  if (lane_id() == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < 16; ++i) s += sh[i];
    *out = s;
    host[0] = *bn2;
    host[1] = s;
    __threadfence_system();
    const unsigned long long q = atomicAdd(seq, 1ull) + 1ull;
    reinterpret_cast<volatile unsigned long long*>(host)[2] = q;
    __threadfence_system();
  }
}

// ---- CIC helpers ------------------------------------------------------------------

// Lower tent node and weight of the upper node along one axis for a particle in cell c
// with offset t from the cell's lower face (t may leave [0,1) for X_dagger).
template <typename T>
__device__ __forceinline__ void tent_axis(int c, T t, int n, int& i0, T& f) {
  const T s = t - (T)0.5;
  const T fl = floor(s);
  int i = c + (int)fl;
  T fr = s - fl;
  if (n == 1) { i0 = 0; f = (T)0; return; }
  if (i < 0) { i = 0; fr = (T)0; }
  if (i > n - 2) { i = n - 2; fr = (T)1; }
  i0 = i;
  f = fr;
}

// The field at a particle (CIC interpolation, section "Charge deposition &
// interpolation") from the packed (Ex, Ey, Ez, 0) array: the eight nodes' vectors are
// loaded together (node indices clamped into the grid; a node outside it has weight
// zero and is skipped), then each component is summed in node order.
// The eight node values of a CIC gather (loads only; the weights and the masks of nodes
// outside the grid or of zero weight), then their weighted sums in node order.
template <typename T>
struct CicNodes {
  V4<T> v[8];
  T wt[8];
  bool use[8];
};
template <typename T>
__device__ __forceinline__ void cic_load(const T* E4, const StepConst& K, int i0, int j0, int k0, T fx, T fy,
                                         T fz, CicNodes<T>& g) {
  const int nx = K.nx, ny = K.ny, nz = K.nz;
#pragma unroll
  for (int cc = 0; cc < 8; ++cc) {
    const int di = cc & 1, dj = (cc >> 1) & 1, dk = (cc >> 2) & 1;
    g.wt[cc] = (di ? fx : (T)1 - fx) * (dj ? fy : (T)1 - fy) * (dk ? fz : (T)1 - fz);
    const int ii = i0 + di, jj = j0 + dj, kk = k0 + dk;
    g.use[cc] = !(g.wt[cc] == (T)0 || ii >= nx || jj >= ny || kk >= nz);
    const int ic = ii < nx ? ii : nx - 1, jc = jj < ny ? jj : ny - 1, kc = kk < nz ? kk : nz - 1;
    g.v[cc] = ld4(E4 + 4 * ((size_t)ic + (size_t)nx * ((size_t)jc + (size_t)ny * kc)));
  }
}
template <typename T>
__device__ __forceinline__ void cic_sum(const CicNodes<T>& g, T out[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    T acc = (T)0;
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) acc = g.use[cc] ? acc + g.v[cc].a[a] * g.wt[cc] : acc;
    out[a] = acc;
  }
}
template <typename T>
__device__ __forceinline__ void cic_get3(const T* E4, const StepConst& K, int i0, int j0, int k0, T fx,
                                         T fy, T fz, T out[3]) {
  CicNodes<T> g;
  cic_load<T>(E4, K, i0, j0, k0, fx, fy, fz, g);
  cic_sum<T>(g, out);
}

// ---- TSC (quadratic B-spline) helpers ---------------------------------------------

// Along one axis, for a particle in cell c with offset t from the cell's lower face (t
// may leave [0,1) for X_dagger): nearest cell centre j = c + floor(t), d = t - floor(t)
// - 1/2, weights (1/2 - d)^2 / 2, 3/4 - d^2 and (1/2 + d)^2 / 2 on the centres j - 1, j
// and j + 1; a centre outside the grid hands its weight to the wall cell (the index is
// clamped), so the weights stay a convex combination that sums to one.
template <typename T>
struct Tsc {
  int ix[3], iy[3], iz[3];
  T wx[3], wy[3], wz[3];
};
template <typename T>
__device__ __forceinline__ void tsc_axis(int c, T t, int n, int idx[3], T w[3]) {
  const T fl = floor(t);
  const T d = t - fl - (T)0.5;
  const T lo = (T)0.5 - d, hi = (T)0.5 + d;
  w[0] = (T)0.5 * lo * lo;
  w[1] = (T)0.75 - d * d;
  w[2] = (T)0.5 * hi * hi;
  const int j = c + (int)fl;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int x = j - 1 + q;
    idx[q] = x < 0 ? 0 : (x > n - 1 ? n - 1 : x);
  }
}
template <typename T>
__device__ __forceinline__ Tsc<T> tsc_at(const StepConst& K, int ci, int cj, int ck, T tx, T ty, T tz) {
  Tsc<T> s;
  tsc_axis<T>(ci, tx, K.nx, s.ix, s.wx);
  tsc_axis<T>(cj, ty, K.ny, s.iy, s.wy);
  tsc_axis<T>(ck, tz, K.nz, s.iz, s.wz);
  return s;
}
// The field at a particle from the packed (Ex, Ey, Ez, 0) array: one z plane's nine
// node vectors loaded together, then each component summed in node order (z, y, x),
// weight (wx wy) wz, nodes of zero weight skipped.
template <typename T>
__device__ __forceinline__ void tsc_get3(const T* E4, const StepConst& K, const Tsc<T>& s, T out[3]) {
  const size_t nx = (size_t)K.nx, ny = (size_t)K.ny;
  T acc[3] = {(T)0, (T)0, (T)0};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    V4<T> v[9];
#pragma unroll
    for (int q = 0; q < 9; ++q)
      v[q] = ld4(E4 + 4 * ((size_t)s.ix[q % 3] + nx * ((size_t)s.iy[q / 3] + ny * (size_t)s.iz[c])));
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const T wt = (s.wx[q % 3] * s.wy[q / 3]) * s.wz[c];
#pragma unroll
      for (int a = 0; a < 3; ++a) acc[a] = wt != (T)0 ? acc[a] + v[q].a[a] * wt : acc[a];
    }
  }
  out[0] = acc[0];
  out[1] = acc[1];
  out[2] = acc[2];
}

// Ion charge (units of e) that cell (i, j, k) receives with the TSC shape: the ions are
// point charges at their cell centres, so along each axis a cell keeps 3/4 of its own
// and takes 1/8 of each neighbour's, and a wall cell also keeps the 1/8 that would fall
// outside.  Every weight is a multiple of 1/512, so the sum is formed in integers: per
// axis the weights in eighths (the cell 6, plus 1 for each wall it touches; each
// neighbour 1, or 0 past a wall), summed along x for each of the nine rows and the rows
// then weighted by y and z.  The total is exact (|total| < 2^53) and so is its scaling
// by 2^-9: the same double as the 27-term sum in any order.
__device__ __forceinline__ void tsc_ion_axis(int c, int n, int w[3], int idx[3]) {
  w[0] = c > 0 ? 1 : 0;
  w[1] = 6 + (c == 0 ? 1 : 0) + (c == n - 1 ? 1 : 0);
  w[2] = c < n - 1 ? 1 : 0;
  idx[0] = c > 0 ? c - 1 : c;  // a tap past the wall reads the cell itself, weight 0
  idx[1] = c;
  idx[2] = c < n - 1 ? c + 1 : c;
}
__device__ __forceinline__ double ion_tsc(const uint32_t* np, const uint32_t* nm, int i, int j, int k,
                                          int nx, int ny, int nz) {
  int wx[3], wy[3], wz[3], xi[3], yj[3], zk[3];
  tsc_ion_axis(i, nx, wx, xi);
  tsc_ion_axis(j, ny, wy, yj);
  tsc_ion_axis(k, nz, wz, zk);
  int64_t acc = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const size_t row = (size_t)nx * ((size_t)yj[b] + (size_t)ny * (size_t)zk[c]);
      int64_t r = 0;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const size_t q = row + (size_t)xi[a];
        r += (int64_t)wx[a] * ((int64_t)np[q] - (int64_t)nm[q]);
      }
      acc += (int64_t)(wy[b] * wz[c]) * r;
    }
  }
  return (double)acc * 0x1p-9;
}

template <typename T> struct Mob;
template <> struct Mob<double> {
  __device__ static double mu(const Coef& c, double E) {
    const double Ec = E > c.E_floor ? E : c.E_floor;
    return c.mu_a * pow(Ec / c.mu_E0, c.mu_b);
  }
};
template <> struct Mob<float> {
  // mu_a (E / E0)^b with hardware exp2/log2
  __device__ static float mu(const Coef& c, float E) {
    const float Ec = E > (float)c.E_floor ? E : (float)c.E_floor;
    return (float)c.mu_a *
           __builtin_amdgcn_exp2f((float)c.mu_b * __builtin_amdgcn_logf(Ec / (float)c.mu_E0));
  }
};

template <typename T> struct NormalsF;
template <> struct NormalsF<double> {
  __device__ __forceinline__ static void get(uint4 r, double n[3]) {
    const double two_pi = 6.283185307179586476925286766559;
    const double r0 = sqrt(-2.0 * log(u_oc(r.x)));
    const double t0 = two_pi * u_co(r.y);
    const double r1 = sqrt(-2.0 * log(u_oc(r.z)));
    const double t1 = two_pi * u_co(r.w);
    n[0] = r0 * cos(t0);
    n[1] = r0 * sin(t0);
    n[2] = r1 * cos(t1);
  }
};
template <> struct NormalsF<float> {
  __device__ __forceinline__ static void get(uint4 r, float n[3]) {
    const float m2ln2 = -1.3862943611198906f;
    const float r0 = __builtin_sqrtf(m2ln2 * __builtin_amdgcn_logf(u_ocf(r.x)));
    const float r1 = __builtin_sqrtf(m2ln2 * __builtin_amdgcn_logf(u_ocf(r.z)));
    const float a0 = (float)(r.y >> 8) * 0x1p-24f;
    const float a1 = (float)(r.w >> 8) * 0x1p-24f;
    n[0] = r0 * __builtin_amdgcn_cosf(a0);
    n[1] = r0 * __builtin_amdgcn_sinf(a0);
    n[2] = r1 * __builtin_amdgcn_cosf(a1);
  }
};

// ---- particle passes --------------------------------------------------------------

// Deposit accumulators.  In single precision the node sums are fixed-point integers
// (conductivity weight mu w in units of 2^-32, electron number in units of 2^-28,
// 64-bit), so a sum does not depend on the order of its atomic additions and the field
// of a realization is bit-reproducible.  A contribution is the product of the
// single-precision tent weight and the particle's integer weight (times the mobility
// for the conductivity), formed in double: the integer weight is not rounded to 24
// bits, so a node that receives all of a particle's charge receives it exactly (a
// quasi-neutral plasma of heavy particles would otherwise carry a spurious charge of
// 2^-24 of its density).  Ranges: 2^31 and 2^35 per node.  Double precision sums
// doubles.
template <typename T> struct DepAcc;
template <> struct DepAcc<double> {
  using S = double;
  static constexpr double kUnit[2] = {1.0, 1.0};
  __device__ static S enc(double a, bool) { return a; }
  __device__ static double dec0(S v) { return v; }
  __device__ static double dec1(S v) { return v; }
};
template <> struct DepAcc<float> {
  using S = unsigned long long;
  static constexpr double kUnit[2] = {0x1p32, 0x1p28};  // units per (mu w) and per electron
  // a in units (the scaling by a power of two is exact, so it is applied to the particle's
  // weight once), rounded to the nearest integer.  fits: a < 2^52, where adding 2^52 leaves
  // that integer in the mantissa (one addition and a mask instead of the conversion).
  __device__ static S enc(double a, bool fits) {
    if (fits) return (S)__double_as_longlong(a + 0x1p52) & 0xFFFFFFFFFFFFFull;
    return (S)rint(a);
  }
  __device__ static double dec0(S v) { return (double)v * 0x1p-32; }
  __device__ static double dec1(S v) { return (double)v * 0x1p-28; }
};

// Charge deposit for the field solve.  Mode 0 deposits the electron number at X^k only
// (initial field); mode 1 deposits the conductivity weight mu(|E^k|) w at X^k and the
// electron number at X_dagger (the position after the diffusive part of the step, with the
// normals of the push), and keeps each particle's mobility mu^k for the push, which then
// reads it instead of interpolating E^k again.
//
// A workgroup takes a chunk of kDepChunk consecutive (cell-sorted, hence spatially compact)
// particles, one per thread, and sums them in LDS before the global atomics (25e9 requests of
// a 64 B line a second, whatever they hold).  Two kernels:
//
// * k_field_deposit_lanes: every particle adds to a hash table keyed by grid node (linear
//   probing, at most kDepProbes probes, then a direct global atomic), flushed with one
//   global atomic per touched node and field: consecutive cells share most of their nodes.
//   TSC in single precision first sums over runs of equal cells (tbl_tsc_runs).
// * k_field_deposit_blocks: each run of equal cells in a wavefront, kDepRuns of them at a
//   time, has the nodes around its cell as a small dense array (CIC and the conductivity
//   3^3; TSC's displaced charge 5^3), so that a contribution is one LDS atomic at a fixed
//   offset, without a hash or a key, and neighbouring lanes of a run take its nodes in
//   different orders (64 lanes that add to one address take 128 cycles, to 8 of them in turn
//   15).  The blocks of a wavefront of at most kDepDense runs go to the table, one node per
//   lane; those of more would fill it with nodes that hardly repeat, so they go to the grid,
//   a row of a block being one request.  A particle displaced out of its block adds to the
//   table by itself; so does, with CIC in double precision, one of a wavefront of more than
//   kDepRuns runs.
//
// Blocks win where cells hold many particles, lanes where a wavefront's many runs would go
// through batches of blocks after each other.  The lines (dep_lanes), in particles and in
// particles per occupied cell; ms of lanes | blocks:
//   CIC, single: 2^21 particles (a launch of fewer is as long as one wavefront: 128^3 request
//     0.029 | 0.034) and 12 a cell (1.0e7 in 3.3e6 cells 0.97 | 1.12, 1.3e7 1.31 | 1.72; 6e6
//     in 3.2e5 0.32 | 0.29, 4.5e7 in 2.2e6 2.15 | 1.86).
//   CIC, double: 5 a cell from 2^19 particles on (1.6e6 in adjacent cells, 3 a cell 0.200 |
//     0.239, 6 a cell 0.161 | 0.172, 16 a cell 0.137 | 0.112; 2e5 of 2 a cell 0.067 | 0.058).
//   TSC, single: 5 a cell (1.6e6 in adjacent cells, 1 a cell 0.44 | 1.72, 4 a cell 0.31 |
//     0.43, 6 a cell 0.31 | 0.32, 8 a cell 0.270 | 0.271; streamers of 4.8 a cell 0.66 | 0.70,
//     of 5.2 2.73 | 1.91), below 2^19 particles 3 (2e4 of 2 a cell 0.062 | 0.065, of 4 0.056 |
//     0.036).
//   TSC, double: 2 a cell (1.6e6, 1 a cell 1.03 to 1.35 | 2.0 to 2.1, 2 a cell 1.00 to 1.67 |
//     1.11 to 1.16).
// The counts are on the device, so both kernels are launched and one returns (2-10 us: a
// workgroup's LDS is allocated all the same).
//
// The table takes the blocks of at most kDepDense runs (CIC: of 2 or 64 instead of 8 2.92 and
// 3.25 ms where 8 takes 1.88, 4.5e7 particles), with TSC in double precision none (1.6e6 of 8 a
// cell 0.46 ms, 0.80 with 8; a streamer's 2.8e6 1.28 and 1.39).  CIC blocks in single precision: 512
// entries (24 KB with the blocks) and 79 VGPRs let six workgroups of a CU overlap their
// loads; 1024 entries leave four (2.37 ms).  What bounds it is that latency: the loads, the
// field gather and the flush of a chunk follow each other.
constexpr int kDepChunk = 256;
constexpr int kDepProbes = 8;
template <int SH> constexpr int kDepRuns = SH == 0 ? 8 : 4;  // 4: 2.01 ms, 16: 2.21 (CIC)
template <typename T, int SH> constexpr int kDepDense = SH == 1 && sizeof(T) == 8 ? 0 : 8;
template <typename T> constexpr uint32_t kDepFew = sizeof(T) == 4 ? 1u << 21 : 1u << 19;  // CIC
constexpr uint32_t kEmptyKey = 0xFFFFFFFFu;
template <typename T, int SH> constexpr int kDepL2 = SH == 0 && sizeof(T) == 4 ? 9 : 10;  // the blocks' table
constexpr int kDepLanesL2 = 10;
// Nodes per axis of a run's block of the displaced charge.
template <int SH> constexpr int kDepW = SH == 0 ? 3 : 5;
template <int SH> constexpr int kDepBlock = 27 + kDepW<SH> * kDepW<SH> * kDepW<SH>;
template <typename T, int SH>
constexpr size_t dep_lds_bytes(bool lanes) {
  using S = typename DepAcc<T>::S;
  return lanes ? ((size_t)1 << kDepLanesL2) * (4 + 2 * sizeof(S))
               : ((size_t)1 << kDepL2<T, SH>) * (4 + 2 * sizeof(S)) +
                     (size_t)(kDepChunk / 64) * kDepRuns<SH> * kDepBlock<SH> * sizeof(S);
}

// True if the particles are left to the per-lane kernel (see above for the lines).
template <typename T, int SH>
__device__ __forceinline__ bool dep_lanes(uint32_t n, const Counters* ctr) {
  const uint32_t occ = ctr->n_occ;
  if constexpr (SH == 0 && sizeof(T) == 4) return n < kDepFew<T> || n / 12u < occ;
  else if constexpr (SH == 0) return n >= kDepFew<T> && n / 5u < occ;
  else return n / (sizeof(T) == 8 ? 2u : n < (1u << 19) ? 3u : 5u) < occ;
}

// Slot of a node in the table: the row hashed, x kept in order, so that a row's nodes sit
// in consecutive slots and the flush's atomics of neighbouring lanes share lines.
template <int L2>
__device__ __forceinline__ uint32_t tbl_slot(uint32_t x, uint32_t row) {
  return (x + ((row * 2654435761u) >> (32 - L2))) & ((1u << L2) - 1u);
}

// Add e to the node's sum of one field (v in the table, g in global memory).  The probes are
// unrolled: nearly every call ends at the first (as a loop 1.6e6 particles of 3 a cell take
// 193 us instead of 181).
template <typename S, int L2>
__device__ __forceinline__ void tbl_put(uint32_t* keys, S* v, uint32_t node, uint32_t h, S e, S* g) {
  if (e == (S)0) return;
  for (int probe = 0; probe < kDepProbes; ++probe) {
    uint32_t k = keys[h];
    if (k == kEmptyKey) {
      const uint32_t prev = atomicCAS(&keys[h], kEmptyKey, node);
      k = prev == kEmptyKey ? node : prev;
    }
    if (k == node) {
      atomicAdd(&v[h], e);
      return;
    }
    h = (h + 1u) & ((1u << L2) - 1u);
  }
  atomicAdd(&g[node], e);
}

// A particle's tent weights along the three axes and their node offsets (0 or 1), in the
// lane's own order: lane l starts at corner l mod 8, so that the lanes of a run, which add
// to the same nodes, do not add to one node at the same time.
template <typename T>
struct Corner {
  T w[3][2];
  int o[3][2];
};
template <typename T>
__device__ __forceinline__ Corner<T> corners(int lane, T fx, T fy, T fz) {
  Corner<T> c;
  const T f[3] = {fx, fy, fz};
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int flip = (lane >> q) & 1;
    const T g = (T)1 - f[q];
    c.w[q][0] = flip ? f[q] : g;
    c.w[q][1] = flip ? g : f[q];
    c.o[q][0] = flip;
    c.o[q][1] = 1 - flip;
  }
  return c;
}

// The 8 CIC contributions q wt of one particle to the table (q in units; fits: as enc).
template <typename T, int L2>
__device__ __forceinline__ void tbl_cic(uint32_t* keys, typename DepAcc<T>::S* v, const StepConst& K, int i0,
                                        int j0, int k0, const Corner<T>& c, double q, bool fits,
                                        typename DepAcc<T>::S* g) {
  using S = typename DepAcc<T>::S;
#pragma unroll
  for (int cc = 0; cc < 8; ++cc) {
    const int di = cc & 1, dj = (cc >> 1) & 1, dk = (cc >> 2) & 1;
    const T wt = c.w[0][di] * c.w[1][dj] * c.w[2][dk];
    const int ii = i0 + c.o[0][di], jj = j0 + c.o[1][dj], kk = k0 + c.o[2][dk];
    if (wt == (T)0 || ii >= K.nx || jj >= K.ny || kk >= K.nz) continue;
    const uint32_t row = (uint32_t)jj + (uint32_t)K.ny * (uint32_t)kk;
    tbl_put<S, L2>(keys, v, (uint32_t)ii + (uint32_t)K.nx * row, tbl_slot<L2>((uint32_t)ii, row),
                   DepAcc<T>::enc(q * (double)wt, fits), g);
  }
}

// The 27 TSC contributions of one particle (clamped wall nodes repeat and simply add).
template <typename T, int L2, int U>
__device__ __forceinline__ void tbl_tsc(uint32_t* keys, typename DepAcc<T>::S* v, const StepConst& K,
                                        const Tsc<T>& s, double q, bool fits, typename DepAcc<T>::S* g) {
  using S = typename DepAcc<T>::S;
#pragma unroll U
  for (int cb = 0; cb < 9; ++cb) {
    const int c = cb / 3, b = cb - 3 * c;
    const T wy = b == 0 ? s.wy[0] : b == 1 ? s.wy[1] : s.wy[2], wz = c == 0 ? s.wz[0] : c == 1 ? s.wz[1] : s.wz[2];
    const int iy = b == 0 ? s.iy[0] : b == 1 ? s.iy[1] : s.iy[2], iz = c == 0 ? s.iz[0] : c == 1 ? s.iz[1] : s.iz[2];
    const uint32_t row = (uint32_t)iy + (uint32_t)K.ny * (uint32_t)iz;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const T wt = (s.wx[a] * wy) * wz;
      tbl_put<S, L2>(keys, v, (uint32_t)s.ix[a] + (uint32_t)K.nx * row, tbl_slot<L2>((uint32_t)s.ix[a], row),
                     DepAcc<T>::enc(q * (double)wt, fits), g);
    }
  }
}

// The same contributions to a run's block (W nodes per axis): blk points at the particle's
// lowest node.  TSC: lane l starts at node l mod 27 (rotated along each axis).
template <typename T, int W>
__device__ __forceinline__ void blk_cic(typename DepAcc<T>::S* blk, const Corner<T>& c, double q, bool fits) {
#pragma unroll
  for (int cc = 0; cc < 8; ++cc) {
    const int di = cc & 1, dj = (cc >> 1) & 1, dk = (cc >> 2) & 1;
    const T wt = c.w[0][di] * c.w[1][dj] * c.w[2][dk];
    atomicAdd(&blk[c.o[0][di] + W * (c.o[1][dj] + W * c.o[2][dk])], DepAcc<T>::enc(q * (double)wt, fits));
  }
}
template <typename T>
__device__ __forceinline__ void rot3(int r, int stride, const T w[3], T v[3], int o[3]) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    v[q] = r == 0 ? w[q] : r == 1 ? w[(q + 1) % 3] : w[(q + 2) % 3];
    o[q] = stride * (r == 0 ? q : r == 1 ? (q + 1) % 3 : (q + 2) % 3);
  }
}
template <typename T>
__device__ __forceinline__ void blk_tsc(typename DepAcc<T>::S* blk, int W, int lane, const Tsc<T>& s, double q,
                                        bool fits) {
  T wx[3], wy[3], wz[3];
  int ox[3], oy[3], oz[3];
  rot3<T>(lane % 3, 1, s.wx, wx, ox);
  rot3<T>(lane / 3 % 3, W, s.wy, wy, oy);
  rot3<T>(lane / 9 % 3, W * W, s.wz, wz, oz);
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const T wt = (wx[a] * wy[b]) * wz[c];
        atomicAdd(&blk[ox[a] + (oy[b] + oz[c])], DepAcc<T>::enc(q * (double)wt, fits));
      }
}

// The 27 contributions in single precision, one particle per lane of a whole wavefront
// (inactive lanes contribute nothing): particles of one cell (before the walls' clamping)
// share their nodes, so each node's fixed-point contributions are summed over every run of
// equal cells j by a segmented scan and the run's last lane inserts the sum.
template <int L2>
__device__ __forceinline__ void tbl_tsc_runs(uint32_t* keys, unsigned long long* v, const StepConst& K,
                                             const Tsc<float>& s, bool active, int jx, int jy, int jz, double q,
                                             bool fits, unsigned long long* g) {
  const int lane = lane_id();
  // run key: the three cell indices, each biased into 21 bits (an index off the grid by
  // up to 2^20 cells still has a key of its own); inactive lanes all differ from it
  const uint64_t key = active ? ((uint64_t)(uint32_t)(jx + (1 << 20)) << 42) |
                                    ((uint64_t)(uint32_t)(jy + (1 << 20)) << 21) |
                                    (uint64_t)(uint32_t)(jz + (1 << 20))
                              : ~0ull;
  const uint32_t klo = (uint32_t)key, khi = (uint32_t)(key >> 32);
  const uint32_t plo = dpp_from_prev(klo, ~klo), phi = dpp_from_prev(khi, ~khi);
  const uint32_t nlo = dpp_from_next(klo, ~klo), nhi = dpp_from_next(khi, ~khi);
  const uint32_t head = (plo != klo || phi != khi) ? 1u : 0u;
  const bool tail = active && (lane == 63 || nlo != klo || nhi != khi);
  // no run of two or more in the wavefront: every lane inserts its own contributions
  const bool runs = __ballot(active && lane > 0 && head == 0u) != 0ull;
  const uint64_t zid[1] = {0ull};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const uint32_t row = (uint32_t)s.iy[b] + (uint32_t)K.ny * (uint32_t)s.iz[c];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float wt = (s.wx[a] * s.wy[b]) * s.wz[c];
        uint64_t e[1] = {active ? DepAcc<float>::enc(q * (double)wt, fits) : 0ull};
        if (runs) (void)seg_scan(e, head, zid, [](int, uint64_t u, uint64_t w) { return u + w; });
        if (tail)
          tbl_put<unsigned long long, L2>(keys, v, (uint32_t)s.ix[a] + (uint32_t)K.nx * row,
                                          tbl_slot<L2>((uint32_t)s.ix[a], row), e[0], g);
      }
    }
  }
}

// The table's flush: one global atomic per touched node and field; the table is left empty.
template <typename S, int TBL>
__device__ __forceinline__ void tbl_flush(uint32_t* keys, S* v0, S* v1, S* g0, S* g1) {
  for (int t = threadIdx.x; t < TBL; t += kDepChunk) {
    const uint32_t k = keys[t];
    if (k == kEmptyKey) continue;
    const S e0 = v0[t], e1 = v1[t];
    if (e0 != (S)0) atomicAdd(&g0[k], e0);
    if (e1 != (S)0) atomicAdd(&g1[k], e1);
    keys[t] = kEmptyKey;
    v0[t] = (S)0;
    v1[t] = (S)0;
  }
}

template <typename T, int SH>
__global__ void __launch_bounds__(256, sizeof(T) == 4 && SH == 0 ? 7 : 1)
    k_field_deposit_lanes(Bank a, const Counters* ctr, int which, StepConst K, const void* E4, Coef co, int mode,
                          typename DepAcc<T>::S* sig, typename DepAcc<T>::S* ne, T* mu_out) {
  using A = DepAcc<T>;
  using S = typename A::S;
  constexpr int L2 = kDepLanesL2, TBL = 1 << L2;
  extern __shared__ __align__(16) char smem[];
  S* v0 = reinterpret_cast<S*>(smem);
  S* v1 = v0 + TBL;
  uint32_t* keys = reinterpret_cast<uint32_t*>(v1 + TBL);
  const uint32_t n = min(ctr->n[which], K.cap);
  if (!dep_lanes<T, SH>(n, ctr)) return;
  const T diff = (T)K.diff;
  for (int t = threadIdx.x; t < TBL; t += kDepChunk) {
    keys[t] = kEmptyKey;
    v0[t] = (S)0;
    v1[t] = (S)0;
  }
  __syncthreads();
  for (uint32_t c0 = blockIdx.x * kDepChunk; c0 < n; c0 += gridDim.x * kDepChunk) {
    const uint32_t i = c0 + threadIdx.x;
    const uint32_t w = i < n ? a.w[i] : 0u;
    if constexpr (SH == 1 && sizeof(T) == 4) {
      // every lane takes part in the run sums (inactive: weight 0)
      const bool act = w != 0u;
      Tsc<T> sk{}, sd{};
      int jk[3] = {0, 0, 0}, jd[3] = {0, 0, 0};
      double qs = 0.0;
      const double qn = (double)w * A::kUnit[1];
      if (act) {
        cell_ijk(a.cell[i], K, jk[0], jk[1], jk[2]);
        const T o[3] = {tp<T>(a.ox)[i], tp<T>(a.oy)[i], tp<T>(a.oz)[i]};
        sk = tsc_at<T>(K, jk[0], jk[1], jk[2], o[0], o[1], o[2]);
        if (mode != 0) {
          T e[3];
          tsc_get3<T>(ctp<T>(E4), K, sk, e);
          const T mu = Mob<T>::mu(co, sqrt(e[0] * e[0] + e[1] * e[1] + e[2] * e[2]));
          mu_out[i] = mu;
          qs = (double)mu * (double)w * A::kUnit[0];
          const uint64_t id = a.id[i];
          const uint4 r = philox_block((uint32_t)id, (uint32_t)(id >> 32), K.step, TAG_PUSH, 0, K.key);
          T nr[3];
          NormalsF<T>::get(r, nr);
          const T t[3] = {o[0] + diff * nr[0], o[1] + diff * nr[1], o[2] + diff * nr[2]};
          sd = tsc_at<T>(K, jk[0], jk[1], jk[2], t[0], t[1], t[2]);
#pragma unroll
          for (int q = 0; q < 3; ++q) jd[q] = jk[q] + (int)floor(t[q]);
        }
      }
      const bool fits = __ballot(!(qs < 0x1p52 && qn < 0x1p52)) == 0ull;
      if (mode == 0) {
        tbl_tsc_runs<L2>(keys, v1, K, sk, act, jk[0], jk[1], jk[2], qn, fits, ne);
      } else {
        tbl_tsc_runs<L2>(keys, v0, K, sk, act, jk[0], jk[1], jk[2], qs, fits, sig);
        tbl_tsc_runs<L2>(keys, v1, K, sd, act, jd[0], jd[1], jd[2], qn, fits, ne);
      }
    } else if (w) {
      const uint32_t cell = a.cell[i];
      int ci, cj, ck;
      cell_ijk(cell, K, ci, cj, ck);
      const T o[3] = {tp<T>(a.ox)[i], tp<T>(a.oy)[i], tp<T>(a.oz)[i]};
      const double qn = (double)w * A::kUnit[1];
      // the charge at the particle's position (conductivity, or electrons of the first field)
      // and, in a step, the electrons at its displaced one
      const auto add = [&](const T t[3], double q, S* v, S* g) {
        const bool fits = __ballot(!(q < 0x1p52)) == 0ull;
        if constexpr (SH == 0) {
          int i0, j0, k0;
          T fx, fy, fz;
          tent_axis<T>(ci, t[0], K.nx, i0, fx);
          tent_axis<T>(cj, t[1], K.ny, j0, fy);
          tent_axis<T>(ck, t[2], K.nz, k0, fz);
          tbl_cic<T, L2>(keys, v, K, i0, j0, k0, corners<T>(0, fx, fy, fz), q, fits, g);
        } else {
          tbl_tsc<T, L2, 9>(keys, v, K, tsc_at<T>(K, ci, cj, ck, t[0], t[1], t[2]), q, fits, g);
        }
      };
      if (mode == 0) {
        add(o, qn, v1, ne);
      } else {
        T e[3];
        if constexpr (SH == 0) {
          int i0, j0, k0;
          T fx, fy, fz;
          tent_axis<T>(ci, o[0], K.nx, i0, fx);
          tent_axis<T>(cj, o[1], K.ny, j0, fy);
          tent_axis<T>(ck, o[2], K.nz, k0, fz);
          cic_get3<T>(ctp<T>(E4), K, i0, j0, k0, fx, fy, fz, e);
        } else {
          tsc_get3<T>(ctp<T>(E4), K, tsc_at<T>(K, ci, cj, ck, o[0], o[1], o[2]), e);
        }
        const T mu = Mob<T>::mu(co, sqrt(e[0] * e[0] + e[1] * e[1] + e[2] * e[2]));
        mu_out[i] = mu;
        add(o, (double)mu * (double)w * A::kUnit[0], v0, sig);
        const uint64_t id = a.id[i];
        const uint4 r = philox_block((uint32_t)id, (uint32_t)(id >> 32), K.step, TAG_PUSH, 0, K.key);
        T nr[3];
        NormalsF<T>::get(r, nr);
        const T t[3] = {o[0] + diff * nr[0], o[1] + diff * nr[1], o[2] + diff * nr[2]};
        add(t, qn, v1, ne);
      }
    }
    __syncthreads();
    tbl_flush<S, TBL>(keys, v0, v1, sig, ne);
    __syncthreads();
  }
}

template <typename T, int SH>
__global__ void __launch_bounds__(256, sizeof(T) == 4 ? (SH == 0 ? 6 : 4) : (SH == 0 ? 4 : 1))
    k_field_deposit_blocks(Bank a, const Counters* ctr, int which, StepConst K, const void* E4, Coef co, int mode,
                           typename DepAcc<T>::S* sig, typename DepAcc<T>::S* ne, T* mu_out) {
  using A = DepAcc<T>;
  using S = typename A::S;
  constexpr int L2 = kDepL2<T, SH>, TBL = 1 << L2, W = kDepW<SH>, B = kDepBlock<SH>;
  extern __shared__ __align__(16) char smem[];
  __shared__ uint32_t rcell[kDepChunk / 64][kDepRuns<SH>];
  S* v0 = reinterpret_cast<S*>(smem);
  S* v1 = v0 + TBL;
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  S* const blocks = v1 + TBL + (size_t)wv * kDepRuns<SH> * B;  // this wavefront's
  uint32_t* keys = reinterpret_cast<uint32_t*>(v1 + TBL + (kDepChunk / 64) * kDepRuns<SH> * B);
  const uint32_t n = min(ctr->n[which], K.cap);
  if (dep_lanes<T, SH>(n, ctr)) return;
  const T diff = (T)K.diff;
  for (int t = threadIdx.x; t < TBL; t += kDepChunk) {
    keys[t] = kEmptyKey;
    v0[t] = (S)0;
    v1[t] = (S)0;
  }
  __syncthreads();
  for (uint32_t c0 = blockIdx.x * kDepChunk; c0 < n; c0 += gridDim.x * kDepChunk) {
    const uint32_t i = c0 + threadIdx.x, il = min(i, n - 1u);
    uint32_t w = a.w[il], cell = a.cell[il];
    const T o[3] = {tp<T>(a.ox)[il], tp<T>(a.oy)[il], tp<T>(a.oz)[il]};
    const uint64_t id = mode != 0 ? a.id[il] : 0ull;
    if (i >= n) w = 0u;
    const bool act = w != 0u;
    if (!act) cell = kInvalidCell;
    const uint32_t prev = dpp_from_prev(cell, ~cell);  // lane 0: not its cell
    const uint64_t heads = __ballot(act && prev != cell);
    const int runs = __popcll(heads);
    const bool dense = runs <= kDepDense<T, SH>;  // wave-uniform
    const uint64_t upto = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
    const int run = __popcll(heads & upto) - 1;
    int ci = 0, cj = 0, ck = 0;
    if (act) cell_ijk(cell, K, ci, cj, ck);
    T pos[3] = {o[0], o[1], o[2]};
    double qs = 0.0;
    if (mode != 0 && act) {
      T e[3];
      if constexpr (SH == 0) {
        int i0, j0, k0;
        T fx, fy, fz;
        tent_axis<T>(ci, o[0], K.nx, i0, fx);
        tent_axis<T>(cj, o[1], K.ny, j0, fy);
        tent_axis<T>(ck, o[2], K.nz, k0, fz);
        cic_get3<T>(ctp<T>(E4), K, i0, j0, k0, fx, fy, fz, e);
      } else {
        tsc_get3<T>(ctp<T>(E4), K, tsc_at<T>(K, ci, cj, ck, o[0], o[1], o[2]), e);
      }
      const T Em = sqrt(e[0] * e[0] + e[1] * e[1] + e[2] * e[2]);
      const T mu = Mob<T>::mu(co, Em);
      mu_out[i] = mu;
      qs = (double)mu * (double)w * A::kUnit[0];
      const uint4 r = philox_block((uint32_t)id, (uint32_t)(id >> 32), K.step, TAG_PUSH, 0, K.key);
      T nr[3];
      NormalsF<T>::get(r, nr);
#pragma unroll
      for (int q = 0; q < 3; ++q) pos[q] = o[q] + diff * nr[q];
    }
    const double qn = (double)w * A::kUnit[1];
    // contributions small enough for the short conversion, in every lane of the wavefront
    const bool fits = __ballot(!(qs < 0x1p52 && qn < 0x1p52)) == 0ull;
    const bool single = SH == 0 && sizeof(T) == 8 && runs > kDepRuns<SH>;  // wave-uniform
#pragma unroll 1
    for (int r0 = 0; r0 < runs; r0 += single ? 64 : kDepRuns<SH>) {
      const int nr = single ? 0 : min(runs - r0, kDepRuns<SH>);
      for (int t = lane; t < nr * B; t += 64) blocks[t] = (S)0;
      wave_lds_sync();
      if (act && (single || (run >= r0 && run < r0 + kDepRuns<SH>))) {
        S* const blk = blocks + (single ? 0 : run - r0) * B;
        if (!single && (heads >> lane) & 1ull) rcell[wv][run - r0] = cell;
#pragma unroll 1
        for (int f = mode != 0 ? 0 : 1; f < 2; ++f) {  // conductivity at X^k, electrons at X_dagger
          const T t[3] = {f ? pos[0] : o[0], f ? pos[1] : o[1], f ? pos[2] : o[2]};
          const double q = f ? qn : qs;
          S* const bf = f ? blk + 27 : blk;
          if constexpr (SH == 0) {
            int i0, j0, k0;
            T fx, fy, fz;
            tent_axis<T>(ci, t[0], K.nx, i0, fx);
            tent_axis<T>(cj, t[1], K.ny, j0, fy);
            tent_axis<T>(ck, t[2], K.nz, k0, fz);
            const Corner<T> c = corners<T>(lane, fx, fy, fz);
            const unsigned dx = (unsigned)(i0 - ci + 1), dy = (unsigned)(j0 - cj + 1), dz = (unsigned)(k0 - ck + 1);
            if (!single && dx < 2u && dy < 2u && dz < 2u)
              blk_cic<T, 3>(bf + dx + 3 * (dy + 3 * dz), c, q, fits);
            else
              tbl_cic<T, L2>(keys, f ? v1 : v0, K, i0, j0, k0, c, q, fits, f ? ne : sig);
          } else {
            const int wf = f ? W : 3;
            const T reach = f ? (T)1 : (T)0;
            const Tsc<T> s = tsc_at<T>(K, ci, cj, ck, t[0], t[1], t[2]);
            const T bx = floor(t[0]), by = floor(t[1]), bz = floor(t[2]);
            if (fabs(bx) <= reach && fabs(by) <= reach && fabs(bz) <= reach)
              blk_tsc<T>(bf + ((int)bx + f) + wf * (((int)by + f) + wf * ((int)bz + f)), wf, lane, s, q, fits);
            else
              tbl_tsc<T, L2, 1>(keys, f ? v1 : v0, K, s, q, fits, f ? ne : sig);
          }
        }
      }
      wave_lds_sync();
      // the runs' blocks to the table or the grid, one node and field per lane; a node
      // outside the grid belongs to the wall cell (TSC; CIC leaves nothing there)
      for (int t = lane; t < nr * B; t += 64) {
        const S e = blocks[t];
        if (e == (S)0) continue;
        const int r = t / B, u = t - r * B;
        int ri, rj, rk;
        cell_ijk(rcell[wv][r], K, ri, rj, rk);
        const bool f = u >= 27;
        int lx, ly, lz;
        if (W == 3 || !f) {
          const int q = f ? u - 27 : u;
          lz = q / 9;
          ly = (q - 9 * lz) / 3;
          lx = q - 9 * lz - 3 * ly;
          lx -= 1; ly -= 1; lz -= 1;
        } else {
          const int q = u - 27;
          lz = q / (W * W);
          ly = (q - W * W * lz) / W;
          lx = q - W * W * lz - W * ly;
          lx -= W / 2; ly -= W / 2; lz -= W / 2;
        }
        const int x = min(max(ri + lx, 0), K.nx - 1), y = min(max(rj + ly, 0), K.ny - 1),
                  z = min(max(rk + lz, 0), K.nz - 1);
        const uint32_t row = (uint32_t)y + (uint32_t)K.ny * (uint32_t)z;
        const uint32_t node = (uint32_t)x + (uint32_t)K.nx * row;
        S* const g = f ? ne : sig;
        if (dense) tbl_put<S, L2>(keys, f ? v1 : v0, node, tbl_slot<L2>((uint32_t)x, row), e, g);
        else atomicAdd(&g[node], e);
      }
      wave_lds_sync();
    }
    __syncthreads();
    tbl_flush<S, TBL>(keys, v0, v1, sig, ne);
    __syncthreads();
  }
}

// Semi-implicit push: X^{k+1} = X^k + sqrt(2 D dt) N - mu(|E^k(X^k)|) E^{k+1}(X^k) dt,
// then binning exactly as the uniform push.
template <typename T, int SH>
__global__ void __launch_bounds__(256) k_push_field(Bank a, Counters* ctr, int which,
                                                   unsigned long long* cellacc, uint32_t* tiles,
                                                   StepConst K, const T* mu_in, const void* En4) {
  const uint32_t n = min(ctr->n[which], K.cap);
  const T diff = (T)K.diff;
  const T dtdx = (T)(K.dt / K.dx);
  uint64_t out_w = 0, pushed = 0;
  for (uint32_t base = blockIdx.x * blockDim.x; base < n; base += gridDim.x * blockDim.x) {
    const uint32_t i = base + threadIdx.x;
    uint32_t key = kInvalidCell, w = 0;
    // the particle's own words are read before its weight is tested (one round trip)
    uint32_t cell0 = 0;
    T o0[3] = {(T)0, (T)0, (T)0};
    uint64_t id0 = 0;
    T mu0 = (T)0;
    if (i < n) {
      w = a.w[i];
      cell0 = a.cell[i];
      o0[0] = tp<T>(a.ox)[i];
      o0[1] = tp<T>(a.oy)[i];
      o0[2] = tp<T>(a.oz)[i];
      id0 = a.id[i];
      mu0 = mu_in[i];
    }
    if (w > 0) {
      ++pushed;
      const uint32_t cell = cell0;
      int ci[3];
      cell_ijk(cell, K, ci[0], ci[1], ci[2]);
      T o[3] = {o0[0], o0[1], o0[2]};
      T en[3];
      if constexpr (SH == 0) {
        int i0, j0, k0;
        T fx, fy, fz;
        tent_axis<T>(ci[0], o[0], K.nx, i0, fx);
        tent_axis<T>(ci[1], o[1], K.ny, j0, fy);
        tent_axis<T>(ci[2], o[2], K.nz, k0, fz);
        CicNodes<T> gn;
        cic_load<T>(ctp<T>(En4), K, i0, j0, k0, fx, fy, fz, gn);
        __builtin_amdgcn_sched_barrier(0);  // the eight gathers in flight together
        cic_sum<T>(gn, en);
      } else {
        tsc_get3<T>(ctp<T>(En4), K, tsc_at<T>(K, ci[0], ci[1], ci[2], o[0], o[1], o[2]), en);
      }
      const T mu = mu0;  // mu(|E^k(X^k)|), kept by this step's deposit
      const uint64_t id = id0;
      const uint4 r = philox_block((uint32_t)id, (uint32_t)(id >> 32), K.step, TAG_PUSH, 0, K.key);
      T nr[3];
      NormalsF<T>::get(r, nr);
      const int lim[3] = {K.nx, K.ny, K.nz};
      bool inside = true;
#pragma unroll
      for (int ax = 0; ax < 3; ++ax) {
        T x = (o[ax] + diff * nr[ax]) + (-mu * en[ax]) * dtdx;
        T f = floor(x);
        x -= f;
        if (x >= (T)1) { x -= (T)1; f += (T)1; }
        o[ax] = x;
        ci[ax] += (int)f;
        inside = inside && ci[ax] >= 0 && ci[ax] < lim[ax];
      }
      if (inside) {
        key = (uint32_t)ci[0] + (uint32_t)K.nx * ((uint32_t)ci[1] + (uint32_t)K.ny * (uint32_t)ci[2]);
        a.cell[i] = key;
        tp<T>(a.ox)[i] = o[0];
        tp<T>(a.oy)[i] = o[1];
        tp<T>(a.oz)[i] = o[2];
      } else {
        out_w += w;
        a.w[i] = 0;
      }
    }
    const uint32_t rank = bin_add(cellacc, key, w);
    mark_tile(tiles, key, (uint64_t)rank << 32);
    if (key != kInvalidCell) a.rank[i] = rank;
  }
  out_w = wave_sum64(out_w);
  pushed = wave_sum64(pushed);
  if (lane_id() == 0) {
    tally_add(ctr, T_OUTFLOW, out_w);
    tally_add(ctr, T_PUSHED, pushed);
  }
}

// ---- grid passes ------------------------------------------------------------------

// Storage positions of a cell and of its face neighbours.  Natural order on every
// level: c = i + nx (j + ny k).  Split red-black order on the finest level (nx even):
// an x row keeps its colour-0 cells ((i + j + k) even) at positions 0 .. nx/2 - 1 and
// its colour-1 cells at nx/2 .. nx - 1, each at i / 2.  Every face neighbour has the
// other colour: at the same half-row position in the four neighbouring rows, and at
// the same or the adjacent position in the cell's own row.  A sweep of one colour
// then reads and writes whole lines of each half-row.
struct NatAt {
  ptrdiff_t c, sy, sz;
  __device__ __forceinline__ size_t operator()(int dx, int dy, int dz) const {
    return (size_t)(c + dx + dy * sy + dz * sz);
  }
};

struct SplitAt {
  ptrdiff_t own, oth, sy, sz;
  int odd;  // i & 1
  __device__ __forceinline__ size_t operator()(int dx, int dy, int dz) const {
    if ((dx | dy | dz) == 0) return (size_t)own;
    return (size_t)(oth + (dx < 0 ? odd - 1 : (dx > 0 ? odd : 0)) + dy * sy + dz * sz);
  }
};

__device__ __forceinline__ NatAt nat_at(int i, int j, int k, int nx, int ny) {
  const ptrdiff_t sy = nx, sz = (ptrdiff_t)nx * ny;
  return NatAt{(ptrdiff_t)i + sy * j + sz * k, sy, sz};
}

__device__ __forceinline__ SplitAt split_at(int i, int j, int k, int nx, int ny) {
  const ptrdiff_t sy = nx, sz = (ptrdiff_t)nx * ny;
  const ptrdiff_t row = sy * j + sz * k;
  const int h = nx >> 1, q = (i + j + k) & 1;
  return SplitAt{row + q * h + (i >> 1), row + (1 - q) * h + (i >> 1), sy, sz, i & 1};
}

template <bool kSplit>
__device__ __forceinline__ size_t pos_of(int i, int j, int k, int nx, int ny) {
  if constexpr (kSplit) return (size_t)split_at(i, j, k, nx, ny).own;
  else return (size_t)nat_at(i, j, k, nx, ny).c;
}

template <typename T>
__global__ void k_zero(T* p, uint32_t n) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = (T)0;
}

// Fine-level coefficient (at its storage position) and right-hand side
// b = dx^2 rho / eps0 (+ the lift of the anode potential on the top layer), both
// scaled by dx^2; accumulates ||b||^2.
template <typename T>
__global__ void __launch_bounds__(256) k_field_prep(StepConst K, const uint32_t* nplus,
                                                   const uint32_t* nminus,
                                                   const typename DepAcc<T>::S* ne,
                                                   const typename DepAcc<T>::S* sig,
                                                   double sig_scale, double V, int split, int tsc,
                                                   T* eps, double* b, double* partial) {
  const uint32_t n = K.ncell;
  const double dV = K.dx * K.dx * K.dx;
  const double qscale = K.dx * K.dx * kE / (kEps0 * dV);
  double acc = 0.0;
  for (uint32_t base = blockIdx.x * blockDim.x; base < n; base += gridDim.x * blockDim.x) {
    const uint32_t c = base + threadIdx.x;
    double bb = 0.0;
    if (c < n) {
      const double e = 1.0 + sig_scale * DepAcc<T>::dec0(sig[c]);
      const uint32_t row = c / (uint32_t)K.nx, k = row / (uint32_t)K.ny;
      const int i = (int)(c - row * (uint32_t)K.nx), j = (int)(row - k * (uint32_t)K.ny);
      eps[split ? pos_of<true>(i, j, (int)k, K.nx, K.ny) : (size_t)c] = (T)e;
      const double ions = tsc ? ion_tsc(nplus, nminus, i, j, (int)k, K.nx, K.ny, K.nz)
                              : (double)nplus[c] - (double)nminus[c];
      const double rho_units = ions - DepAcc<T>::dec1(ne[c]);
      bb = qscale * rho_units;
      if (k == (uint32_t)K.nz - 1) bb += 2.0 * (double)(T)e * V;
      b[c] = bb;
    }
    acc += bb * bb;
  }
  acc = block_sumd(acc);
  if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

// Mean of the eight children's coefficients of coarse cell (i, j, k).
template <typename T>
__device__ __forceinline__ T eps_child_mean(const T* ef, int fnx, int fny, int fsplit, int i, int j, int k) {
  double s = 0.0;
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    const int fi = 2 * i + (d & 1), fj = 2 * j + ((d >> 1) & 1), fk = 2 * k + (d >> 2);
    s += (double)ef[fsplit ? pos_of<true>(fi, fj, fk, fnx, fny) : pos_of<false>(fi, fj, fk, fnx, fny)];
  }
  return (T)(s * 0.125);
}

template <typename T>
__global__ void k_eps_restrict(const T* ef, int fnx, int fny, int fsplit, T* ec, int cnx, int cny, int cnz,
                               int csplit) {
  const uint32_t n = (uint32_t)cnx * cny * cnz;
  for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) {
    const int i = c % cnx, j = (c / cnx) % cny, k = c / (cnx * cny);
    ec[csplit ? pos_of<true>(i, j, k, cnx, cny) : (size_t)c] = eps_child_mean<T>(ef, fnx, fny, fsplit, i, j, k);
  }
}

// Harmonic mean for the smoother: exact in double; fast reciprocal in single precision
// (the smoother only has to reduce the error; the double residual of the refinement
// loop defines the solution).
__device__ __forceinline__ double hmean_s(double a, double b) { return 2.0 * a * b / (a + b); }
__device__ __forceinline__ float hmean_s(float a, float b) {
  return (2.0f * a * b) * __builtin_amdgcn_rcpf(a + b);  // v_rcp_f32 (1 ulp), not a full division
}
// The smoother's cell update (f + offsum) / diag, in every smoother form: a division in
// double, the hardware reciprocal in single precision.
__device__ __forceinline__ double smooth_div(double num, double d) { return num / d; }
__device__ __forceinline__ float smooth_div(float num, float d) { return num * __builtin_amdgcn_rcpf(d); }

// Operator of the scaled system at one cell (homogeneous boundary values): sum over
// faces of beta (u_c - u_nb), beta the harmonic mean of the two cells' coefficients,
// plus 2 eps_c u_c on the Dirichlet z faces; x and y faces are Neumann.  Returned as
// the diagonal and the neighbour sum, from the coefficient at the cell and the
// coefficients and values at its six face neighbours (faces ordered x-, x+, y-, y+,
// z-, z+; in[q] false for a face on the domain boundary, whose values are not used: it
// contributes nothing, or the Dirichlet term).  Every finest- and coarse-level kernel
// forms its rows through op_row (working precision) or op_row_r (double accumulation
// for the residual), so all share one arithmetic order.
template <typename T>
__device__ __forceinline__ void op_row(T ec, const T en[6], const T un[6], const bool in[6], T& diag,
                                       T& offsum) {
  T d = 0, s = 0;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const T b = hmean_s(ec, en[q]);
    d = in[q] ? d + b : (q >= 4 ? d + (T)2 * ec : d);
    s = in[q] ? s + b * un[q] : s;
  }
  diag = d;
  offsum = s;
}

// Residual row: face coefficients computed exactly as the smoother computes them
// (single-precision harmonic means in FP32 mode, exact double in FP64 mode), the
// potential and the accumulation in double.
template <typename T>
__device__ __forceinline__ void op_row_r(T ec, const T en[6], const double un[6], const bool in[6],
                                         double& diag, double& offsum) {
  double d = 0, s = 0;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const double b = (double)hmean_s(ec, en[q]);
    d = in[q] ? d + b : (q >= 4 ? d + 2.0 * (double)ec : d);
    s = in[q] ? s + b * un[q] : s;
  }
  diag = d;
  offsum = s;
}

__device__ __forceinline__ void faces_in(int i, int j, int k, int nx, int ny, int nz, bool in[6]) {
  in[0] = i > 0; in[1] = i < nx - 1; in[2] = j > 0; in[3] = j < ny - 1; in[4] = k > 0; in[5] = k < nz - 1;
}

// Operator row through value accessors a(dx, dy, dz) of the correction and of the
// coefficient at the neighbour (dx, dy, dz) of cell (i, j, k).  All thirteen values
// are read before any arithmetic (offsets clamped to the cell itself on the domain
// faces), so their loads are in flight together.
template <typename T, typename UA, typename EA>
__device__ __forceinline__ void stencil_acc(UA ua, EA ea, int nx, int ny, int nz, int i, int j, int k,
                                            T& diag, T& offsum) {
  bool in[6];
  faces_in(i, j, k, nx, ny, nz, in);
  const int ox[6] = {in[0] ? -1 : 0, in[1] ? 1 : 0, 0, 0, 0, 0};
  const int oy[6] = {0, 0, in[2] ? -1 : 0, in[3] ? 1 : 0, 0, 0};
  const int oz[6] = {0, 0, 0, 0, in[4] ? -1 : 0, in[5] ? 1 : 0};
  const T ec = ea(0, 0, 0);
  T en[6], un[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    en[q] = ea(ox[q], oy[q], oz[q]);
    un[q] = ua(ox[q], oy[q], oz[q]);
  }
  op_row<T>(ec, en, un, in, diag, offsum);
}

template <typename T, typename AT>
__device__ __forceinline__ void stencil_at(const T* u, const T* eps, AT at, int nx, int ny, int nz, int i,
                                           int j, int k, T& diag, T& offsum) {
  stencil_acc<T>([&](int dx, int dy, int dz) { return u[at(dx, dy, dz)]; },
                 [&](int dx, int dy, int dz) { return eps[at(dx, dy, dz)]; }, nx, ny, nz, i, j, k, diag,
                 offsum);
}

template <typename T>
__device__ __forceinline__ void stencil_s(const T* u, const T* eps, int nx, int ny, int nz, int i, int j,
                                          int k, size_t c, T& diag, T& offsum) {
  const ptrdiff_t sy = (ptrdiff_t)nx, sz = (ptrdiff_t)nx * ny;
  stencil_at<T>(u, eps, NatAt{(ptrdiff_t)c, sy, sz}, nx, ny, nz, i, j, k, diag, offsum);
}

// Residual operator row: the potential in natural order, the coefficient through its
// level's positions `at`.
template <typename T, typename AT>
__device__ __forceinline__ void stencil_r(const double* u, const T* eps, AT at, int nx, int ny, int nz,
                                          int i, int j, int k, size_t c, double& diag, double& offsum) {
  const ptrdiff_t sy = (ptrdiff_t)nx, sz = (ptrdiff_t)nx * ny;
  bool in[6];
  faces_in(i, j, k, nx, ny, nz, in);
  const int ox[6] = {in[0] ? -1 : 0, in[1] ? 1 : 0, 0, 0, 0, 0};
  const int oy[6] = {0, 0, in[2] ? -1 : 0, in[3] ? 1 : 0, 0, 0};
  const int oz[6] = {0, 0, 0, 0, in[4] ? -1 : 0, in[5] ? 1 : 0};
  const T ec = eps[at(0, 0, 0)];
  T en[6];
  double un[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    en[q] = eps[at(ox[q], oy[q], oz[q])];
    un[q] = u[(size_t)((ptrdiff_t)c + ox[q] + oy[q] * sy + oz[q] * sz)];
  }
  op_row_r<T>(ec, en, un, in, diag, offsum);
}

// Logical (x, y, z) block of a 3-D grid after the XCD remap.
__device__ __forceinline__ void xcd_block3(int& bx, int& by, int& bz) {
  const uint32_t nb = gridDim.x * gridDim.y * gridDim.z;
  const uint32_t lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const uint32_t l = xcd_block(lin, nb);
  bx = (int)(l % gridDim.x);
  by = (int)((l / gridDim.x) % gridDim.y);
  bz = (int)(l / (gridDim.x * gridDim.y));
}

// Gauss-Seidel update of cell (i, j, k) of a level in natural order.
template <typename T>
__device__ __forceinline__ void smooth_cell(T* u, const T* f, const T* eps, int nx, int ny, int nz, int i,
                                            int j, int k) {
  const size_t c = (size_t)i + (size_t)nx * ((size_t)j + (size_t)ny * k);
  T d, s;
  stencil_s<T>(u, eps, nx, ny, nz, i, j, k, c, d, s);
  u[c] = smooth_div(f[c] + s, d);
}

// One colour of a red-black Gauss-Seidel sweep in natural order: grid (x: half a row,
// y: j, z: k), every thread updates the one cell of the colour in its pair.  kFine
// marks the finest level's instantiation, so that kernel traces report it apart.
template <typename T, bool kFine>
__global__ void __launch_bounds__(128) k_smooth_rb(T* u, const T* f, const T* eps, int nx, int ny, int nz,
                                                  int color) {
  int bx, j, k;
  xcd_block3(bx, j, k);
  const int i = 2 * (int)(bx * blockDim.x + threadIdx.x) + ((j + k + color) & 1);
  if (i >= nx) return;
  smooth_cell<T>(u, f, eps, nx, ny, nz, i, j, k);
}

// One colour of a red-black sweep on the finest level in split order: grid (x: half a
// row, y: j, z: k); the thread at half-row position m updates cell
// i = 2m + ((j + k + colour) & 1), reading its own coefficient and right-hand side and
// the other colour's values, all as whole lines.  Same arithmetic as k_smooth_rb.
template <typename T>
__global__ void __launch_bounds__(128) k_smooth_split(T* u, const T* f, const T* eps, int nx, int ny,
                                                     int nz, int color) {
  int bx, j, k;
  xcd_block3(bx, j, k);
  const int m = (int)(bx * blockDim.x + threadIdx.x);
  if (m >= (nx >> 1)) return;
  const int i = 2 * m + ((j + k + color) & 1);
  const SplitAt at = split_at(i, j, k, nx, ny);
  T d, s;
  stencil_at<T>(u, eps, at, nx, ny, nz, i, j, k, d, s);
  u[at.own] = smooth_div(f[at.own] + s, d);
}

// r = b - A phi in double with the true boundary values (the lift is in b) over
// 256-cell runs, a block taking every gridDim-th run (after the XCD remap); writes the
// working-precision right-hand side of the correction equation and one partial of
// ||r||^2 per block, summed over its runs in order.
constexpr int kResBlocks = 8192;

template <typename T, bool kSplit>
__global__ void __launch_bounds__(256) k_residual_rows(const double* phi, const double* b, const T* eps,
                                                      int nx, int ny, int nz, T* f0, double* partial) {
  const uint32_t n = (uint32_t)nx * ny * nz;
  const uint32_t blk = xcd_block(blockIdx.x, gridDim.x);
  const uint32_t runs = (n + 255u) / 256u;
  double acc = 0.0;
  for (uint32_t run = blk; run < runs; run += gridDim.x) {
    const uint32_t c = run * 256u + threadIdx.x;
    double rr = 0.0;
    if (c < n) {
      const int i = (int)(c % (uint32_t)nx), j = (int)((c / (uint32_t)nx) % (uint32_t)ny),
                k = (int)(c / ((uint32_t)nx * (uint32_t)ny));
      double d, s;
      size_t q;
      if constexpr (kSplit) {
        const SplitAt at = split_at(i, j, k, nx, ny);
        stencil_r<T>(phi, eps, at, nx, ny, nz, i, j, k, c, d, s);
        q = (size_t)at.own;
      } else {
        const NatAt at = nat_at(i, j, k, nx, ny);
        stencil_r<T>(phi, eps, at, nx, ny, nz, i, j, k, c, d, s);
        q = c;
      }
      rr = b[c] - (d * phi[c] - s);
      f0[q] = (T)rr;
    }
    acc += block_sumd(rr * rr);
  }
  if (threadIdx.x == 0) partial[blk] = acc;
}

// Coarse right-hand side at coarse cell (ci, cj, ck): the sum of its 8 child residuals
// / 2, in the children's order (x offset, then y, then z); zero coarse correction.  The
// fine level in split order if kSplit.
template <typename T, bool kSplit>
__device__ __forceinline__ void restrict_cell(const T* u, const T* f, const T* eps, int nx, int ny, int nz,
                                              T* fc, T* uc, int cnx, int cny, int ci, int cj, int ck) {
  T s8 = 0;
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    const int i = 2 * ci + (d & 1), j = 2 * cj + ((d >> 1) & 1), k = 2 * ck + (d >> 2);
    T dg, sm;
    size_t q;
    if constexpr (kSplit) {
      const SplitAt at = split_at(i, j, k, nx, ny);
      stencil_at<T>(u, eps, at, nx, ny, nz, i, j, k, dg, sm);
      q = (size_t)at.own;
    } else {
      const NatAt at = nat_at(i, j, k, nx, ny);
      stencil_at<T>(u, eps, at, nx, ny, nz, i, j, k, dg, sm);
      q = (size_t)at.c;
    }
    s8 += f[q] - (dg * u[q] - sm);
  }
  const size_t cc = (size_t)ci + (size_t)cnx * ((size_t)cj + (size_t)cny * ck);
  fc[cc] = s8 * (T)0.5;
  uc[cc] = (T)0;
}

// Restriction launch: grid (x: coarse row, y: cj, z: ck).
template <typename T, bool kSplit>
__global__ void __launch_bounds__(128) k_restrict3(const T* u, const T* f, const T* eps, int nx, int ny,
                                                  int nz, T* fc, T* uc, int cnx, int cny) {
  int bx, cj, ck;
  xcd_block3(bx, cj, ck);
  const int ci = bx * blockDim.x + threadIdx.x;
  if (ci >= cnx) return;
  restrict_cell<T, kSplit>(u, f, eps, nx, ny, nz, fc, uc, cnx, cny, ci, cj, ck);
}

// Trilinear prolongation of the coarse correction onto cell centres: along each axis
// the nearer coarse centre weighs 3/4 and the farther 1/4; coarse ghost values mirror
// the cell on the Neumann x and y faces and negate it on the homogeneous Dirichlet z
// faces.  (Second-order transfer: with cell-averaged restriction the transfer orders
// then exceed the order of the operator.)
template <typename T>
__device__ __forceinline__ T prolong_value(const T* uc, int cnx, int cny, int cnz, int i, int j, int k) {
  const int I = i >> 1, J = j >> 1, K = k >> 1;
  const int ia[2] = {I, (i & 1) ? I + 1 : I - 1};
  const int ja[2] = {J, (j & 1) ? J + 1 : J - 1};
  const int ka[2] = {K, (k & 1) ? K + 1 : K - 1};
  const T wt[2] = {(T)0.75, (T)0.25};
  T acc = 0;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    int a = ia[c & 1], b = ja[(c >> 1) & 1], z = ka[c >> 2];
    a = a < 0 ? 0 : (a >= cnx ? cnx - 1 : a);
    b = b < 0 ? 0 : (b >= cny ? cny - 1 : b);
    T sg = (T)1;
    if (z < 0) { z = 0; sg = (T)-1; }
    if (z >= cnz) { z = cnz - 1; sg = (T)-1; }
    acc += wt[c & 1] * wt[(c >> 1) & 1] * wt[c >> 2] * sg *
           uc[(size_t)a + (size_t)cnx * ((size_t)b + (size_t)cny * z)];
  }
  return acc;
}

template <typename T, bool kSplit>
__global__ void __launch_bounds__(128) k_prolong3(T* u, int nx, int ny, int nz, const T* uc, int cnx,
                                                 int cny, int cnz) {
  int bx, j, k;
  xcd_block3(bx, j, k);
  const int p = bx * blockDim.x + threadIdx.x;  // storage position in the row
  if (p >= nx) return;
  int i = p;
  if constexpr (kSplit) {
    const int h = nx >> 1, q = p >= h ? 1 : 0;
    i = 2 * (p - q * h) + ((j + k + q) & 1);
  }
  u[(size_t)p + (size_t)nx * ((size_t)j + (size_t)ny * k)] += prolong_value<T>(uc, cnx, cny, cnz, i, j, k);
}

// ---- small levels ---------------------------------------------------------------------
// Levels of at most kSmallLevel cells below the finest (and a single-level grid) run their
// sweeps in one workgroup with the correction in LDS.  Their face coefficients and
// diagonals do not change within a solve, so one launch per solve forms them for all of
// them (k_small_setup, level_faces: three face coefficients towards the + neighbours and
// the diagonal per cell; the harmonic mean is symmetric in its two cells, so both read the
// same value).  In the sweeps a thread owns up to NR cells of each colour and keeps their
// coefficients, diagonals and right-hand sides in registers: a colour is six LDS reads
// and the update.  Owning cells by colour keeps every lane of a wavefront at work in each
// colour.  The arithmetic and its order are op_row's and smooth_div's (a face outside the
// domain has coefficient zero and the cell itself as its neighbour, which adds zero).
// Bound by the latency of a colour (LDS, a chain of six additions, the division, a
// barrier).  16^3 in double: 33.8 -> 11.4 us per launch; 9x7x11 bottom, 60 sweeps in double:
// 180 -> 29 us; 11x9x13 bottom, 68 sweeps in single: 44 -> 28.5 us.  Three cells of a colour
// per thread have room for their state in single precision only with the neighbours' LDS
// offsets packed (a cycle of 28x36x240, whose bottom is 7x9x60: 390 us, of 64x64 in one
// plane 269; four cells unpacked, with spills: 553 and 584).
constexpr uint32_t kSmallLevel = 4096;
static_assert(kBottomMaxCells <= (int)kSmallLevel, "the coarsest level runs as a small level");

struct SmallLevels {
  int count;
  int nx[kMaxLevels], ny[kMaxLevels], nz[kMaxLevels];
  void* eps[kMaxLevels];
  void* cf[kMaxLevels];  // packed (x, y, z face coefficient, diagonal) per cell
};

// Coefficients of cell (i, j, k) of a level in natural order: its faces towards the +
// neighbours (zero on the domain boundary) and its diagonal, by op_row's arithmetic.
template <typename T>
__device__ __forceinline__ void level_faces(const T* e, int nx, int ny, int nz, int i, int j, int k, T v[4]) {
  const int sy = nx, sz = nx * ny, c = i + sy * j + sz * k;
  bool in[6];
  faces_in(i, j, k, nx, ny, nz, in);
  const int off[6] = {in[0] ? -1 : 0, in[1] ? 1 : 0, in[2] ? -sy : 0,
                      in[3] ? sy : 0, in[4] ? -sz : 0, in[5] ? sz : 0};
  const T ec = e[c];
  T d = 0;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const T b = hmean_s(ec, e[c + off[q]]);
    d = in[q] ? d + b : (q >= 4 ? d + (T)2 * ec : d);
    if (q & 1) v[q >> 1] = in[q] ? b : (T)0;
  }
  v[3] = d;
}

// Coefficients of the small levels, finest first, in one workgroup: the cell coefficient
// of each (restricted from the level above it; the first one from ef unless that is null:
// a single-level grid) and its faces.
template <typename T>
__global__ void __launch_bounds__(1024) k_small_setup(SmallLevels L, const T* ef, int fnx, int fny, int fsplit) {
  for (int l = 0; l < L.count; ++l) {
    const int nx = L.nx[l], ny = L.ny[l], nz = L.nz[l], n = nx * ny * nz, sz = nx * ny;
    T* const e = reinterpret_cast<T*>(L.eps[l]);
    T* const cf = reinterpret_cast<T*>(L.cf[l]);
    if (ef)
      for (int c = threadIdx.x; c < n; c += 1024)
        e[c] = eps_child_mean<T>(ef, fnx, fny, fsplit, c % nx, (c / nx) % ny, c / sz);
    __syncthreads();
    for (int c = threadIdx.x; c < n; c += 1024) {
      T v[4];
      level_faces<T>(e, nx, ny, nz, c % nx, (c / nx) % ny, c / sz, v);
      st4<T>(cf + 4 * (size_t)c, v[0], v[1], v[2], v[3]);
    }
    ef = e;
    fnx = nx;
    fny = ny;
    fsplit = 0;
  }
}

// One small level (see above): pre-smoothing with the restriction of the residual
// (fc_out), prolongation of the coarse correction (uc_in) with post-smoothing, or the
// coarsest level's sweeps.  LDS: the correction, and with fc_out the residual.
template <typename T, int NR, int MAXT>
__global__ void __launch_bounds__(MAXT) k_small_level(T* u, const T* f, const T* cf, int nx, int ny, int nz,
                                                      int pair, int sweeps, bool zero_u, const T* uc_in, T* fc_out,
                                                      T* uc_out, int cnx, int cny, int cnz) {
  extern __shared__ __align__(16) char smem[];
  const int n = nx * ny * nz, sy = nx, sz = nx * ny, NT = (int)blockDim.x;
  const int wx = pair == 0 ? (nx + 1) >> 1 : nx, wy = pair == 1 ? (ny + 1) >> 1 : ny;
  T* const su = reinterpret_cast<T*>(smem);
  T* const sr = su + n;
  T b[2][NR][6], dg[2][NR], fr[2][NR];
  int cell[2][NR];  // -1 past the colour's cells
  // the six neighbours' cells or, packed, their byte offsets in LDS (below 2^16), two to a
  // register
  constexpr bool kPack = NR > 2;
  uint32_t nb[2][NR][kPack ? 3 : 6];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      // the colour's cells row by row: along the axis `pair`, position m is cell 2 m + parity
      const int p = (int)threadIdx.x + r * NT, row = p / wx;
      int i = p - row * wx, k = row / wy, j = row - k * wy;
      if (pair == 0) i = 2 * i + ((j + k + q) & 1);
      else if (pair == 1) j = 2 * j + ((i + k + q) & 1);
      else k = 2 * k + ((i + j + q) & 1);
      const bool own = i < nx && j < ny && k < nz;
      const int c = own ? i + sy * j + sz * k : 0;
      cell[q][r] = own ? c : -1;
      bool in[6];
      faces_in(own ? i : 0, own ? j : 0, own ? k : 0, nx, ny, nz, in);
      const int off[6] = {in[0] ? -1 : 0, in[1] ? 1 : 0, in[2] ? -sy : 0,
                          in[3] ? sy : 0, in[4] ? -sz : 0, in[5] ? sz : 0};
#pragma unroll
      for (int a = 0; a < 6; ++a) {
        const uint32_t at = (uint32_t)(c + off[a]);
        if constexpr (!kPack) nb[q][r][a] = at;
        else if (a & 1) nb[q][r][a >> 1] |= at * (uint32_t)sizeof(T) << 16;
        else nb[q][r][a >> 1] = at * (uint32_t)sizeof(T);
        // the face below a cell is the + face of its lower neighbour
        const T v = cf[4 * (size_t)((a & 1) ? c : c + off[a]) + (a >> 1)];
        b[q][r][a] = in[a] ? v : (T)0;
      }
      dg[q][r] = cf[4 * (size_t)c + 3];
      fr[q][r] = f[c];
      T v = zero_u ? (T)0 : u[c];
      if (uc_in && own) v = v + prolong_value<T>(uc_in, cnx, cny, cnz, i, j, k);
      if (own) su[c] = v;
      if (NR > 2) __builtin_amdgcn_sched_barrier(0);  // the next cell's loads would need spills
    }
  __syncthreads();
  // `zero` is opaque to the compiler, so that the offsets stay packed outside the loop
  auto nbsum = [&](int q, int r, uint32_t zero) {
    T un[6];
#pragma unroll
    for (int a = 0; a < 6; ++a) {
      if constexpr (kPack) {
        const uint32_t w = nb[q][r][a >> 1];
        un[a] = *reinterpret_cast<const T*>(smem + ((a & 1) ? w >> (16u + zero) : w & (0xFFFFu + zero)));
      } else {
        un[a] = su[nb[q][r][a]];
      }
    }
    T acc = 0;
#pragma unroll
    for (int a = 0; a < 6; ++a) acc = acc + b[q][r][a] * un[a];
    return acc;
  };
  uint32_t zero = 0;
  for (int it = 0; it < sweeps; ++it) {
    if constexpr (kPack) asm volatile("" : "+s"(zero));
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const T v = smooth_div(fr[q][r] + nbsum(q, r, zero), dg[q][r]);
        if (cell[q][r] >= 0) su[cell[q][r]] = v;
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int c = cell[q][r];
      if (c < 0) continue;
      const T uc = su[c];
      u[c] = uc;
      if (fc_out) sr[c] = fr[q][r] - (dg[q][r] * uc - nbsum(q, r, zero));
    }
  if (fc_out) {
    __syncthreads();
    const int cn = cnx * cny * cnz;
    for (int q = threadIdx.x; q < cn; q += NT) {
      const int ci = q % cnx, cj = (q / cnx) % cny, ck = q / (cnx * cny);
      T s8 = 0;
#pragma unroll
      for (int d = 0; d < 8; ++d)
        s8 += sr[2 * ci + (d & 1) + sy * (2 * cj + ((d >> 1) & 1)) + sz * (2 * ck + (d >> 2))];
      fc_out[q] = s8 * (T)0.5;
      uc_out[q] = (T)0;
    }
  }
}

static int n_pairs(int n, bool paired) { return paired ? (n + 1) / 2 : n; }
template <typename T>
static void launch_small_level(hipStream_t s, T* u, const T* f, const T* cf, int nx, int ny, int nz, int sweeps,
                               bool zero_u, const T* uc_in, T* fc_out, T* uc_out, int cnx, int cny, int cnz) {
  // positions of one colour: pairs of cells along x, or along the longest axis where rows of
  // one or three cells would leave a half or a quarter of the positions empty.  n <= 4096
  // makes at most 2458 of them (rows of five).
  const int pair = nx != 1 && nx != 3 ? 0 : (ny > nz ? 1 : 2);
  const int pos = n_pairs(nx, pair == 0) * n_pairs(ny, pair == 1) * n_pairs(nz, pair == 2);
  const int nr = pos <= 1024 ? 1 : pos <= 2048 ? 2 : 3;
  const int nt = ((pos + nr - 1) / nr + 63) / 64 * 64;
  const size_t lds = (size_t)(fc_out ? 2 : 1) * nx * ny * nz * sizeof(T);
  const auto go = [&](auto kern) {
    kern<<<1, nt, lds, s>>>(u, f, cf, nx, ny, nz, pair, sweeps, zero_u, uc_in, fc_out, uc_out, cnx, cny, cnz);
  };
  if (nt == 64) go(k_small_level<T, 1, 64>);
  else if (nr == 1 && nt <= 512) go(k_small_level<T, 1, 512>);
  else if (nr == 1) go(k_small_level<T, 1, 1024>);
  else if (nr == 2) go(k_small_level<T, 2, 1024>);
  else go(k_small_level<T, 3, 1024>);
}

// ---- tiled levels ---------------------------------------------------------------------
// Levels of up to tile_max cells are bound by their launches, not by memory: a colour of a
// 32^3 or 64^3 level takes the 3.5 us that any launch takes.  Here one launch does a
// level's whole pre-smoothing (from the zero correction, with the restriction of the
// residual) or its post-smoothing (with the prolongation): a workgroup takes an 8^3 core
// with a halo of kHalo cells, whose colours it repeats in LDS.  A cell of the halo is
// right as long as its distance from the region's edge is at least the number of colours
// done (pre-smoothing, from known zeros outside: one less), so up to kHalo colours leave
// the core right (and, for the residual, the ring around it).  A thread owns two cells of
// each colour, with their coefficients (formed once per solve by k_tile_faces), diagonals
// and right-hand sides in registers; a cell outside the domain has zero coefficients and
// stays zero.  The arithmetic and its order are those of the one-colour launches.
// Single precision, microseconds per cycle (tiled: two launches; one colour each: eight
// sweeps, restriction, prolongation): 32^3 18 against 45, 64^3 30 against 43, 128^3 225
// against 57 (the redundant work is 8 region cells per core cell).  Double: 32^3 17 against
// 64, 64^3 37 against 62, 72x56x88 (finest: with the potential's update) 55 against 67.
constexpr int kTile = 8, kHalo = 4, kRegion = kTile + 2 * kHalo, kTileLd = kRegion + 2;
constexpr uint32_t tile_max(size_t T) { return T == 8 ? 1u << 19 : 1u << 18; }  // cells

template <typename T>
__global__ void __launch_bounds__(256) k_tile_faces(const T* e, int nx, int ny, int nz, T* cf) {
  const uint32_t n = (uint32_t)nx * ny * nz;
  for (uint32_t c = blockIdx.x * 256u + threadIdx.x; c < n; c += gridDim.x * 256u) {
    const uint32_t row = c / (uint32_t)nx, k = row / (uint32_t)ny;
    T v[4];
    level_faces<T>(e, nx, ny, nz, (int)(c - row * (uint32_t)nx), (int)(row - k * (uint32_t)ny), (int)k, v);
#pragma unroll
    for (int q = 0; q < 4; ++q) cf[(size_t)q * n + c] = v[q];
  }
}

// Two neighbouring values of T as one access.
template <typename T>
__device__ __forceinline__ void ld2(const T* p, T v[2]) {
  if constexpr (sizeof(T) == 4) {
    const float2 x = *reinterpret_cast<const float2*>(p);
    v[0] = x.x; v[1] = x.y;
  } else {
    const double2 x = *reinterpret_cast<const double2*>(p);
    v[0] = x.x; v[1] = x.y;
  }
}

// kPost: u + the prolonged coarse correction uc, then the sweeps, into `out` (another
// array than u, whose halo the neighbouring workgroups read) or, on the finest level,
// added to the potential phi.  Otherwise: the sweeps from zero into u, and the coarse
// right-hand side fc.
// A thread owns the cells (2m, 2m + 1) of a row in two planes z and z + 8: one cell of
// each colour in each pair, loaded together (the levels' rows are even, as they are
// coarsened).  Single precision forms the face coefficients from the cell coefficients
// staged in LDS (the hardware reciprocal is cheaper than the halo's traffic); double reads
// the ones k_tile_faces has formed (no division here).  A wavefront's cells lie in one
// plane: the planes that no longer matter for the core are skipped colour by colour.
template <typename T, bool kPost>
__global__ void __launch_bounds__(1024) k_tile_level(T* u, const T* f, const T* eps, const T* cf, int nx, int ny,
                                                     int nz, int sweeps, const T* uc, int cnx, int cny, int cnz,
                                                     T* out, double* phi, T* fc) {
  constexpr int kLy = kTileLd, kLz = kTileLd * kTileLd, kAll = kTileLd * kLz;
  constexpr int kC = kRegion / 2 + 2, kCy = kC, kCz = kC * kC;  // coarse cells under the region
  __shared__ T su[kAll];
  // post: the coarse correction; pre: the residual of the core
  __shared__ T sx[kPost ? kC * kCz : kTile * kTile * kTile];
  const int tx = (nx + kTile - 1) / kTile, ty = (ny + kTile - 1) / kTile;
  const int tile = (int)xcd_block(blockIdx.x, gridDim.x);
  const int bz = tile / (tx * ty), by = (tile - bz * tx * ty) / tx, bx = tile - (bz * ty + by) * tx;
  const int x0 = bx * kTile - kHalo, y0 = by * kTile - kHalo, z0 = bz * kTile - kHalo;
  const int sy = nx, sz = nx * ny;
  const int m = (int)threadIdx.x & 7, y = (int)(threadIdx.x >> 3) & 15, zb = (int)(threadIdx.x >> 7);
  const int i = x0 + 2 * m, j = y0 + y;  // the pair's first cell
  if constexpr (sizeof(T) == 4) {
    for (int t = (int)threadIdx.x; t < kAll; t += 1024) {
      const int lz = t / kLz, ly = (t - lz * kLz) / kLy, lx = t - lz * kLz - ly * kLy;
      const int ei = min(max(x0 + lx - 1, 0), nx - 1), ej = min(max(y0 + ly - 1, 0), ny - 1),
                ek = min(max(z0 + lz - 1, 0), nz - 1);
      su[t] = eps[ei + sy * ej + sz * ek];
    }
  }
  if constexpr (kPost) {
    // a coarse value past a Neumann face is its cell's, past a Dirichlet face its negative
    // (prolong_value's rules; the sign is exact)
    const int cx0 = (x0 >> 1) - 1, cy0 = (y0 >> 1) - 1, cz0 = (z0 >> 1) - 1;
    if (threadIdx.x < (unsigned)(kC * kCz)) {
      const int lz = (int)threadIdx.x / kCz, ly = ((int)threadIdx.x - lz * kCz) / kCy,
                lx = (int)threadIdx.x - lz * kCz - ly * kCy;
      const int ci = min(max(cx0 + lx, 0), cnx - 1), cj = min(max(cy0 + ly, 0), cny - 1), kk = cz0 + lz;
      const T v = uc[ci + (size_t)cnx * (cj + (size_t)cny * min(max(kk, 0), cnz - 1))];
      sx[threadIdx.x] = kk < 0 || kk >= cnz ? -v : v;
    }
  }
  T b[2][2][6], dg[2][2], fr[2][2], v0[2][2];  // [colour][plane]
  int at[2][2];                                // LDS position
  bool own[2];
  if constexpr (sizeof(T) == 4) __syncthreads();
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int z = zb + 8 * r, k = z0 + z;
    own[r] = i >= 0 && i < nx && j >= 0 && j < ny && k >= 0 && k < nz;  // the whole pair
    const int c = own[r] ? i + sy * j + sz * k : 0;
    T ff[2], uu[2] = {(T)0, (T)0}, bp[2][6], dp[2];
    ld2<T>(f + c, ff);
    if constexpr (kPost) ld2<T>(u + c, uu);
    if constexpr (sizeof(T) == 4) {
      const T* e = su + (2 * m + 1) + kLy * (y + 1) + kLz * (z + 1);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        bool in[6];
        faces_in(i + a, j, k, nx, ny, nz, in);
        const T* p = e + a;
        const T en[6] = {p[-1], p[1], p[-kLy], p[kLy], p[-kLz], p[kLz]};
        T d = 0;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
          const T w = hmean_s(p[0], en[q]);
          d = in[q] ? d + w : (q >= 4 ? d + (T)2 * p[0] : d);
          bp[a][q] = in[q] ? w : (T)0;
        }
        dp[a] = d;
      }
    } else {
      const size_t n = (size_t)sz * nz;
      const bool ym = own[r] && j > 0, zm = own[r] && k > 0;
      T fx[2], fy[2], fz[2], gy[2], gz[2];
      const T gx = cf[own[r] && i > 0 ? c - 1 : c];
      ld2<T>(cf + c, fx);
      ld2<T>(cf + n + c, fy);
      ld2<T>(cf + n + (ym ? c - sy : c), gy);
      ld2<T>(cf + 2 * n + c, fz);
      ld2<T>(cf + 2 * n + (zm ? c - sz : c), gz);
      ld2<T>(cf + 3 * n + c, dp);
      bp[0][0] = i > 0 ? gx : (T)0; bp[0][1] = fx[0];
      bp[1][0] = fx[0];             bp[1][1] = fx[1];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        bp[a][2] = ym ? gy[a] : (T)0; bp[a][3] = fy[a];
        bp[a][4] = zm ? gz[a] : (T)0; bp[a][5] = fz[a];
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      // the region's origin is even in every axis: local and global colours agree
      const int a = (y + z + q) & 1;
      at[q][r] = (2 * m + a + 1) + kLy * (y + 1) + kLz * (z + 1);
#pragma unroll
      for (int w = 0; w < 6; ++w) b[q][r][w] = own[r] ? (a ? bp[1][w] : bp[0][w]) : (T)0;
      dg[q][r] = own[r] ? (a ? dp[1] : dp[0]) : (T)1;
      fr[q][r] = own[r] ? (a ? ff[1] : ff[0]) : (T)0;
      v0[q][r] = own[r] ? (a ? uu[1] : uu[0]) : (T)0;
    }
  }
  if constexpr (sizeof(T) == 4) __syncthreads();  // the coefficients are read
  for (int t = (int)threadIdx.x; t < kAll; t += 1024) su[t] = (T)0;
  __syncthreads();
  if constexpr (kPost) {
    const T wt[2] = {(T)0.75, (T)0.25};
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int z = zb + 8 * r, x = 2 * m + ((y + z + q) & 1);
        // the nearer coarse centre and the step to the farther one, along each axis
        const T* p = sx + ((x >> 1) + 1) + kCy * ((y >> 1) + 1) + kCz * ((z >> 1) + 1);
        const int ox = (x & 1) ? 1 : -1, oy = (y & 1) ? kCy : -kCy, oz = (z & 1) ? kCz : -kCz;
        T acc = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c)
          acc += wt[c & 1] * wt[(c >> 1) & 1] * wt[c >> 2] *
                 p[((c & 1) ? ox : 0) + ((c & 2) ? oy : 0) + ((c & 4) ? oz : 0)];
        if (own[r]) su[at[q][r]] = v0[q][r] + acc;
      }
    __syncthreads();
  }
  auto nbsum = [&](int q, int r) {
    const T* p = su + at[q][r];
    const T un[6] = {p[-1], p[1], p[-kLy], p[kLy], p[-kLz], p[kLz]};
    T acc = 0;
#pragma unroll
    for (int a = 0; a < 6; ++a) acc = acc + b[q][r][a] * un[a];
    return acc;
  };
  int edge = kPost ? 1 : 0;  // planes nearer to the region's edge than this have gone wrong
  for (int it = 0; it < sweeps; ++it) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int z = zb + 8 * r;
        if (z >= edge && z < kRegion - edge) su[at[q][r]] = smooth_div(fr[q][r] + nbsum(q, r), dg[q][r]);
      }
      ++edge;
      __syncthreads();
    }
  }
  const int cx = 2 * m - kHalo, cy = y - kHalo;
  const bool core = cx >= 0 && cx < kTile && cy >= 0 && cy < kTile;
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int z = zb + 8 * r, cz = z - kHalo;
    if (!core || cz < 0 || cz >= kTile) continue;
    const size_t c = (size_t)i + (size_t)sy * j + (size_t)sz * (z0 + z);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int a = (y + z + q) & 1;
      const T v = su[at[q][r]];
      if constexpr (kPost) {
        if (own[r]) {
          if (phi) phi[c + a] += (double)v;
          else out[c + a] = v;
        }
      } else {
        if (own[r]) u[c + a] = v;
        sx[cx + a + kTile * (cy + kTile * cz)] = fr[q][r] - (dg[q][r] * v - nbsum(q, r));
      }
    }
  }
  if constexpr (!kPost) {
    __syncthreads();
    if (threadIdx.x < 64) {
      const int x = (int)threadIdx.x & 3, yy = ((int)threadIdx.x >> 2) & 3, z = (int)threadIdx.x >> 4;
      const int ci = bx * 4 + x, cj = by * 4 + yy, ck = bz * 4 + z;
      if (ci < cnx && cj < cny && ck < cnz) {
        T s8 = 0;
#pragma unroll
        for (int d = 0; d < 8; ++d)
          s8 += sx[2 * x + (d & 1) + kTile * (2 * yy + ((d >> 1) & 1) + kTile * (2 * z + (d >> 2)))];
        fc[(size_t)ci + (size_t)cnx * ((size_t)cj + (size_t)cny * ck)] = s8 * (T)0.5;
      }
    }
  }
}

static int tile_blocks(int nx, int ny, int nz) {
  return ((nx + kTile - 1) / kTile) * ((ny + kTile - 1) / kTile) * ((nz + kTile - 1) / kTile);
}

// ---- finest level over row segments ---------------------------------------------------
// With nx a multiple of 8 the finest-level kernels give each thread a segment of eight
// cells of an x row (i = 8t .. 8t+7; the smoother: four cells of one colour).  In split
// order a segment is positions 4t .. 4t+3 of both half rows, in natural order eight
// consecutive values, so every access to the level's arrays is a 16-byte vector.  The
// per-cell arithmetic is op_row / op_row_r, as in the one-cell kernels, and both orders
// run the same segment kernels (the smoother has no reduction and is order-free), so
// their results are identical.

// Cells 8t .. 8t+7 of the finest-level row starting at rb (parity par = (j + k) & 1),
// in natural order; h = nx / 2.  Cell 8t + 2r + e has colour (e + par) & 1 and sits at
// position 4t + r of that colour's half row.
template <typename T, bool kSplit>
__device__ __forceinline__ void ld_seg(const T* a, size_t rb, int h, int t, int par, T v[8]) {
  if constexpr (kSplit) {
    const V4<T> c0 = ld4(a + rb + 4 * t), c1 = ld4(a + rb + h + 4 * t);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[2 * r] = par ? c1.a[r] : c0.a[r];
      v[2 * r + 1] = par ? c0.a[r] : c1.a[r];
    }
  } else {
    const V4<T> a0 = ld4(a + rb + 8 * t), a1 = ld4(a + rb + 8 * t + 4);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = a0.a[r];
      v[4 + r] = a1.a[r];
    }
  }
}

template <typename T, bool kSplit>
__device__ __forceinline__ void st_seg(T* a, size_t rb, int h, int t, int par, const T v[8]) {
  if constexpr (kSplit) {
    const int e0 = par, e1 = 1 - par;  // the natural parity of the colour-0 and colour-1 cells
    st4<T>(a + rb + 4 * t, v[e0], v[2 + e0], v[4 + e0], v[6 + e0]);
    st4<T>(a + rb + h + 4 * t, v[e1], v[2 + e1], v[4 + e1], v[6 + e1]);
  } else {
    st4<T>(a + rb + 8 * t, v[0], v[1], v[2], v[3]);
    st4<T>(a + rb + 8 * t + 4, v[4], v[5], v[6], v[7]);
  }
}

template <typename T, bool kSplit>
__device__ __forceinline__ T ld_cell(const T* a, size_t rb, int h, int i, int par) {
  if constexpr (kSplit) return a[rb + (((i + par) & 1) ? (size_t)h : 0) + (size_t)(i >> 1)];
  else return a[rb + (size_t)i];
}

// Segment g of a level with ns segments per row: row index, t, j, k, parity.
struct Seg {
  uint32_t row;
  int t, j, k, par;
};

__device__ __forceinline__ Seg seg_of(uint32_t g, int ns, int ny) {
  Seg s;
  s.row = g / (uint32_t)ns;
  s.t = (int)(g - s.row * (uint32_t)ns);
  s.k = (int)(s.row / (uint32_t)ny);
  s.j = (int)(s.row - (uint32_t)s.k * (uint32_t)ny);
  s.par = (s.j + s.k) & 1;
  return s;
}

// The segment's row and its four neighbouring rows (each replaced by the row itself
// where there is none: those values are not used), with their parities.
struct SegRows {
  size_t rb, ym, yp, zm, zp;
  int pym, pyp, pzm, pzp;
};

__device__ __forceinline__ SegRows seg_rows(const Seg& s, int nx, int ny, int nz) {
  SegRows R;
  const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
  R.rb = (size_t)s.row * sy;
  R.ym = s.j > 0 ? R.rb - sy : R.rb;
  R.yp = s.j < ny - 1 ? R.rb + sy : R.rb;
  R.zm = s.k > 0 ? R.rb - sz : R.rb;
  R.zp = s.k < nz - 1 ? R.rb + sz : R.rb;
  R.pym = s.j > 0 ? s.par ^ 1 : s.par;
  R.pyp = s.j < ny - 1 ? s.par ^ 1 : s.par;
  R.pzm = s.k > 0 ? s.par ^ 1 : s.par;
  R.pzp = s.k < nz - 1 ? s.par ^ 1 : s.par;
  return R;
}

// A segment's values of one array: the eight cells, the cells before and after it in
// the row (clamped to the segment at the row ends), and the same eight cells of the
// four neighbouring rows.
template <typename T>
struct SegVals {
  T c[8], ym[8], yp[8], zm[8], zp[8];
  T l, r;
};

template <typename T, bool kSplit>
__device__ __forceinline__ void ld_seg_vals(const T* a, const SegRows& R, const Seg& s, int nx, SegVals<T>& v) {
  const int h = nx >> 1, i0 = 8 * s.t;
  ld_seg<T, kSplit>(a, R.rb, h, s.t, s.par, v.c);
  ld_seg<T, kSplit>(a, R.ym, h, s.t, R.pym, v.ym);
  ld_seg<T, kSplit>(a, R.yp, h, s.t, R.pyp, v.yp);
  ld_seg<T, kSplit>(a, R.zm, h, s.t, R.pzm, v.zm);
  ld_seg<T, kSplit>(a, R.zp, h, s.t, R.pzp, v.zp);
  v.l = ld_cell<T, kSplit>(a, R.rb, h, i0 > 0 ? i0 - 1 : i0, s.par);
  v.r = ld_cell<T, kSplit>(a, R.rb, h, i0 + 8 < nx ? i0 + 8 : i0 + 7, s.par);
}

// Face-neighbour values of cell r of the segment (faces ordered as in op_row).
template <typename T>
__device__ __forceinline__ void seg_faces(const SegVals<T>& v, int r, T out[6]) {
  out[0] = r > 0 ? v.c[r - 1] : v.l;
  out[1] = r < 7 ? v.c[r + 1] : v.r;
  out[2] = v.ym[r];
  out[3] = v.yp[r];
  out[4] = v.zm[r];
  out[5] = v.zp[r];
}

// Double residual over segments (as k_residual_rows: a block takes every gridDim-th run
// of 256 segments; one partial of ||r||^2 per block, each thread's eight cells summed
// in order).
template <typename T, bool kSplit>
__global__ void __launch_bounds__(256) k_residual_seg(const double* phi, const double* b, const T* eps,
                                                     int nx, int ny, int nz, T* f0, double* partial) {
  const int ns = nx >> 3, h = nx >> 1;
  const uint32_t nseg = (uint32_t)ns * ny * nz;
  const uint32_t blk = xcd_block(blockIdx.x, gridDim.x);
  const uint32_t runs = (nseg + 255u) / 256u;
  double acc = 0.0;
  for (uint32_t run = blk; run < runs; run += gridDim.x) {
    const uint32_t g = run * 256u + threadIdx.x;
    double rs = 0.0;
    if (g < nseg) {
      const Seg s = seg_of(g, ns, ny);
      const SegRows R = seg_rows(s, nx, ny, nz);
      const int i0 = 8 * s.t;
      // two rounds of loads, each issued together before its arithmetic: the segment's
      // row with its x and y neighbours (faces 0-3), then the z neighbour rows (faces
      // 4-5); the face sums continue in the operator's face order (same values), and
      // the y rows are dead before the z rows arrive (fewer registers, more waves)
      double Pc[8], Pym[8], Pyp[8], B[8];
      T Ec[8], Eym[8], Eyp[8];
      ld_seg<double, false>(phi, R.rb, h, s.t, s.par, Pc);
      ld_seg<double, false>(phi, R.ym, h, s.t, R.pym, Pym);
      ld_seg<double, false>(phi, R.yp, h, s.t, R.pyp, Pyp);
      const double Pl = ld_cell<double, false>(phi, R.rb, h, i0 > 0 ? i0 - 1 : i0, s.par);
      const double Pr = ld_cell<double, false>(phi, R.rb, h, i0 + 8 < nx ? i0 + 8 : i0 + 7, s.par);
      ld_seg<T, kSplit>(eps, R.rb, h, s.t, s.par, Ec);
      ld_seg<T, kSplit>(eps, R.ym, h, s.t, R.pym, Eym);
      ld_seg<T, kSplit>(eps, R.yp, h, s.t, R.pyp, Eyp);
      const T El = ld_cell<T, kSplit>(eps, R.rb, h, i0 > 0 ? i0 - 1 : i0, s.par);
      const T Er = ld_cell<T, kSplit>(eps, R.rb, h, i0 + 8 < nx ? i0 + 8 : i0 + 7, s.par);
      ld_seg<double, false>(b, R.rb, h, s.t, s.par, B);
      __builtin_amdgcn_sched_barrier(0);
      double d[8], sm[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        bool in[6];
        faces_in(i0 + r, s.j, s.k, nx, ny, nz, in);
        const T en[4] = {r > 0 ? Ec[r - 1] : El, r < 7 ? Ec[r + 1] : Er, Eym[r], Eyp[r]};
        const double un[4] = {r > 0 ? Pc[r - 1] : Pl, r < 7 ? Pc[r + 1] : Pr, Pym[r], Pyp[r]};
        double dd = 0, ss = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double bq = (double)hmean_s(Ec[r], en[q]);
          dd = in[q] ? dd + bq : dd;
          ss = in[q] ? ss + bq * un[q] : ss;
        }
        d[r] = dd;
        sm[r] = ss;
      }
      __builtin_amdgcn_sched_barrier(0);  // the z rows are loaded after the y rows are dead
      double Pzm[8], Pzp[8];
      T Ezm[8], Ezp[8];
      ld_seg<double, false>(phi, R.zm, h, s.t, R.pzm, Pzm);
      ld_seg<double, false>(phi, R.zp, h, s.t, R.pzp, Pzp);
      ld_seg<T, kSplit>(eps, R.zm, h, s.t, R.pzm, Ezm);
      ld_seg<T, kSplit>(eps, R.zp, h, s.t, R.pzp, Ezp);
      __builtin_amdgcn_sched_barrier(0);
      T F[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const bool in4 = s.k > 0, in5 = s.k < nz - 1;
        double dd = d[r], ss = sm[r];
        {
          const double bq = (double)hmean_s(Ec[r], Ezm[r]);
          dd = in4 ? dd + bq : dd + 2.0 * (double)Ec[r];
          ss = in4 ? ss + bq * Pzm[r] : ss;
        }
        {
          const double bq = (double)hmean_s(Ec[r], Ezp[r]);
          dd = in5 ? dd + bq : dd + 2.0 * (double)Ec[r];
          ss = in5 ? ss + bq * Pzp[r] : ss;
        }
        const double rr = B[r] - (dd * Pc[r] - ss);
        F[r] = (T)rr;
        rs += rr * rr;
      }
      st_seg<T, kSplit>(f0, R.rb, h, s.t, s.par, F);
    }
    acc += block_sumd(rs);
  }
  if (threadIdx.x == 0) partial[blk] = acc;
}

// One colour of a red-black sweep on a split segment level, four cells of the colour
// per thread (kFine marks the finest level's instantiation for kernel traces): cells i = 2m + odd for half-row positions m = 4t .. 4t+3, odd =
// (j + k + colour) & 1.  Their x neighbours have the other colour, at positions
// m - 1 + odd and m + odd.
template <typename T, bool kFine, bool kZero = false>
__global__ void __launch_bounds__(256) k_smooth_seg(T* u, const T* f, const T* eps, int nx, int ny, int nz,
                                                   int color) {
  const int ns = nx >> 3, h = nx >> 1;
  const uint32_t g = xcd_block(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  if (g >= (uint32_t)ns * ny * nz) return;
  const Seg s = seg_of(g, ns, ny);
  const int odd = (s.par + color) & 1;
  const size_t rb = (size_t)s.row * nx;
  const size_t own = rb + (color ? (size_t)h : 0) + 4 * s.t, oth = rb + (color ? 0 : (size_t)h) + 4 * s.t;
  const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
  const size_t oym = s.j > 0 ? oth - sy : oth, oyp = s.j < ny - 1 ? oth + sy : oth;
  const size_t ozm = s.k > 0 ? oth - sz : oth, ozp = s.k < nz - 1 ? oth + sz : oth;
  // the one x neighbour outside the segment's other-colour values: on the left of the
  // first cell (odd = 0) or on the right of the last (odd = 1); a single unconditional
  // load, so that it joins the others in flight
  const size_t pe = odd ? (4 * s.t + 4 < h ? oth + 4 : oth + 3) : (s.t > 0 ? oth - 1 : oth);
  const V4<T> Fo = ld4(f + own), Eo = ld4(eps + own);
  const V4<T> Ec = ld4(eps + oth);
  const V4<T> Eym = ld4(eps + oym), Eyp = ld4(eps + oyp), Ezm = ld4(eps + ozm), Ezp = ld4(eps + ozp);
  const T EX = eps[pe];
  // kZero: the first colour-0 sweep of a cycle, from u = 0 (the neighbours' values are
  // zeros, not read)
  const V4<T> zero = {{(T)0, (T)0, (T)0, (T)0}};
  const V4<T> Uc = kZero ? zero : ld4(u + oth);
  const V4<T> Uym = kZero ? zero : ld4(u + oym), Uyp = kZero ? zero : ld4(u + oyp);
  const V4<T> Uzm = kZero ? zero : ld4(u + ozm), Uzp = kZero ? zero : ld4(u + ozp);
  const T UX = kZero ? (T)0 : u[pe];
  __builtin_amdgcn_sched_barrier(0);  // all loads issued before the arithmetic
  T un_[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    bool in[6];
    faces_in(2 * (4 * s.t + r) + odd, s.j, s.k, nx, ny, nz, in);
    const T en[6] = {odd ? Ec.a[r] : (r > 0 ? Ec.a[r - 1] : EX), odd ? (r < 3 ? Ec.a[r + 1] : EX) : Ec.a[r],
                     Eym.a[r], Eyp.a[r], Ezm.a[r], Ezp.a[r]};
    const T un[6] = {odd ? Uc.a[r] : (r > 0 ? Uc.a[r - 1] : UX), odd ? (r < 3 ? Uc.a[r + 1] : UX) : Uc.a[r],
                     Uym.a[r], Uyp.a[r], Uzm.a[r], Uzp.a[r]};
    T d, sm;
    op_row<T>(Eo.a[r], en, un, in, d, sm);
    un_[r] = smooth_div(Fo.a[r] + sm, d);
  }
  st4<T>(u + own, un_[0], un_[1], un_[2], un_[3]);
}

// Restriction from a segment level: four coarse cells (coarse x 4t .. 4t+3) and their
// children, the fine segment t of four fine rows, belong to the same lane of a workgroup's
// four wavefronts.  Each forms the residuals of one row; the first adds them in the
// children's order (j offset, then k offset; x offset within a row), so each coarse sum
// adds its eight child residuals in the order of k_restrict3.  (One thread for the four
// rows after each other: 57 us at 256^3 in single precision, 44 now; 9.2 -> 7.9 at 128^3:
// a fourth of the threads, and three wavefronts a SIMD where this form has four.)  The fine
// level in split order if kSplit, the coarse one if kCSplit (coarse cells 4t, 4t+1 sit at
// half-row position 2t, 4t+2 and 4t+3 at 2t+1, one of each pair in each half).
template <typename T, bool kSplit, bool kCSplit>
__global__ void __launch_bounds__(256) k_restrict_seg(const T* u, const T* f, const T* eps, int nx, int ny,
                                                     int nz, T* fc, T* uc) {
  const int ns = nx >> 3, h = nx >> 1, cnx = nx >> 1, cny = ny >> 1, cnz = nz >> 1;
  const int dd = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t g = xcd_block(blockIdx.x, gridDim.x) * 64u + (uint32_t)lane;
  const bool in_range = g < (uint32_t)ns * cny * cnz;
  const Seg cs = seg_of(in_range ? g : 0u, ns, cny);
  __shared__ T part[3][8][64];
  T res[8];
  {
    Seg s;
    s.t = cs.t;
    s.j = 2 * cs.j + (dd & 1);
    s.k = 2 * cs.k + (dd >> 1);
    s.row = (uint32_t)s.j + (uint32_t)ny * (uint32_t)s.k;
    s.par = (s.j + s.k) & 1;
    const SegRows R = seg_rows(s, nx, ny, nz);
    SegVals<T> U, E;
    ld_seg_vals<T, kSplit>(u, R, s, nx, U);
    ld_seg_vals<T, kSplit>(eps, R, s, nx, E);
    T F[8];
    ld_seg<T, kSplit>(f, R.rb, h, s.t, s.par, F);
    __builtin_amdgcn_sched_barrier(0);  // the row's loads in flight together
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      bool in[6];
      faces_in(8 * s.t + r, s.j, s.k, nx, ny, nz, in);
      T en[6], un[6];
      seg_faces(E, r, en);
      seg_faces(U, r, un);
      T dg, sm;
      op_row<T>(E.c[r], en, un, in, dg, sm);
      res[r] = F[r] - (dg * U.c[r] - sm);
    }
  }
  if (dd > 0) {
#pragma unroll
    for (int r = 0; r < 8; ++r) part[dd - 1][r][lane] = res[r];
  }
  __syncthreads();
  if (dd > 0 || !in_range) return;
  T s8[4] = {0, 0, 0, 0};
#pragma unroll
  for (int r = 0; r < 8; ++r) s8[r >> 1] += res[r];
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int r = 0; r < 8; ++r) s8[r >> 1] += part[q][r][lane];
  const size_t cb = (size_t)cs.row * cnx;
  if constexpr (kCSplit) {
    const int ch = cnx >> 1;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ci = 4 * cs.t + r;
      const size_t q = cb + (((ci + cs.par) & 1) ? (size_t)ch : 0) + (size_t)(ci >> 1);
      fc[q] = s8[r] * (T)0.5;
      uc[q] = (T)0;
    }
  } else {
    st4<T>(fc + cb + 4 * cs.t, s8[0] * (T)0.5, s8[1] * (T)0.5, s8[2] * (T)0.5, s8[3] * (T)0.5);
    st4<T>(uc + cb + 4 * cs.t, (T)0, (T)0, (T)0, (T)0);
  }
}

// Trilinear prolongation onto the finest level over segments: the coarse values of
// the eight cells come from the coarse rows (J or its neighbour toward the cell) x
// (K or its neighbour), x from 4t-1 to 4t+4 with the clamps and Dirichlet signs of
// k_prolong3, in the same order and arithmetic.
template <typename T, bool kSplit, bool kCSplit>
__global__ void __launch_bounds__(256) k_prolong_seg(T* u, int nx, int ny, int nz, const T* uc, int cnx,
                                                    int cny, int cnz) {
  const int ns = nx >> 3, h = nx >> 1;
  const uint32_t g = xcd_block(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  if (g >= (uint32_t)ns * ny * nz) return;
  const Seg s = seg_of(g, ns, ny);
  const int J = s.j >> 1, K = s.k >> 1;
  const int jb = (s.j & 1) ? J + 1 : J - 1, kb = (s.k & 1) ? K + 1 : K - 1;
  const int jbc = jb < 0 ? 0 : (jb >= cny ? cny - 1 : jb);
  const int kbc = kb < 0 ? 0 : (kb >= cnz ? cnz - 1 : kb);
  const T sgk = (kb < 0 || kb >= cnz) ? (T)-1 : (T)1;
  T W[2][2][6];
#pragma unroll
  for (int dj = 0; dj < 2; ++dj)
#pragma unroll
    for (int dk = 0; dk < 2; ++dk) {
      const int rj = dj ? jbc : J, rk = dk ? kbc : K;
      const size_t crow = (size_t)cnx * ((size_t)rj + (size_t)cny * (size_t)rk);
      const int xl = s.t > 0 ? 4 * s.t - 1 : 0, xr = 4 * s.t + 4 < cnx ? 4 * s.t + 4 : cnx - 1;
      if constexpr (kCSplit) {
        const int ch = cnx >> 1, cp = (rj + rk) & 1;
        auto cv = [&](int x) { return uc[crow + (((x + cp) & 1) ? (size_t)ch : 0) + (size_t)(x >> 1)]; };
        W[dj][dk][0] = cv(xl);
#pragma unroll
        for (int q = 0; q < 4; ++q) W[dj][dk][1 + q] = cv(4 * s.t + q);
        W[dj][dk][5] = cv(xr);
      } else {
        const V4<T> m = ld4(uc + crow + 4 * s.t);
        W[dj][dk][0] = uc[crow + xl];
        W[dj][dk][1] = m.a[0]; W[dj][dk][2] = m.a[1]; W[dj][dk][3] = m.a[2]; W[dj][dk][4] = m.a[3];
        W[dj][dk][5] = uc[crow + xr];
      }
    }
  const size_t rb = (size_t)s.row * nx;
  T V[8];
  ld_seg<T, kSplit>(u, rb, h, s.t, s.par, V);
  const T wt[2] = {(T)0.75, (T)0.25};
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    T acc = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      // x: I = 4t + r/2 sits at window index r/2 + 1; the far neighbour is I + 1 for
      // odd i and I - 1 for even i
      const int xa = (c & 1) ? ((r & 1) ? (r >> 1) + 2 : (r >> 1)) : (r >> 1) + 1;
      const T sg = (c >> 2) ? sgk : (T)1;
      acc += wt[c & 1] * wt[(c >> 1) & 1] * wt[c >> 2] * sg * W[(c >> 1) & 1][c >> 2][xa];
    }
    V[r] += acc;
  }
  st_seg<T, kSplit>(u, rb, h, s.t, s.par, V);
}

// phi += u over the finest level, a segment per thread.
template <typename T, bool kSplit>
__global__ void __launch_bounds__(256) k_phi_update_seg(double* phi, const T* u, int nx, int ny, int nz) {
  const int ns = nx >> 3, h = nx >> 1;
  const uint32_t g = xcd_block(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  if (g >= (uint32_t)ns * ny * nz) return;
  const Seg s = seg_of(g, ns, ny);
  const size_t rb = (size_t)s.row * nx;
  T V[8];
  double P[8];
  ld_seg<T, kSplit>(u, rb, h, s.t, s.par, V);
  ld_seg<double, false>(phi, rb, h, s.t, s.par, P);
#pragma unroll
  for (int r = 0; r < 8; ++r) P[r] += (double)V[r];
  st_seg<double, false>(phi, rb, h, s.t, s.par, P);
}

// Initial guess by linear extrapolation in time: phi <- 2 phi - prev, prev <- old phi.
__global__ void k_extrapolate(double* phi, double* prev, uint32_t n, int have_prev) {
  for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) {
    const double p = phi[c];
    if (have_prev) phi[c] = 2.0 * p - prev[c];
    prev[c] = p;
  }
}

// phi += u over the finest level; grid (x: row position, y: j, z: k), u read in its
// storage order.
template <typename T, bool kSplit>
__global__ void __launch_bounds__(128) k_phi_update(double* phi, const T* u, int nx, int ny) {
  int bx, j, k;
  xcd_block3(bx, j, k);
  const int p = bx * blockDim.x + threadIdx.x;
  if (p >= nx) return;
  int i = p;
  if constexpr (kSplit) {
    const int h = nx >> 1, q = p >= h ? 1 : 0;
    i = 2 * (p - q * h) + ((j + k + q) & 1);
  }
  const size_t row = (size_t)nx * ((size_t)j + (size_t)ny * k);
  phi[row + i] += (double)u[row + p];
}

// E = -grad phi at cell centres into the packed (Ex, Ey, Ez, 0) array.
template <typename T>
__global__ void k_efield(const double* phi, int nx, int ny, int nz, double V, double inv2h, T* E4) {
  const uint32_t n = (uint32_t)nx * ny * nz;
  const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
  for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) {
    const int i = c % nx, j = (c / nx) % ny, k = c / (nx * ny);
    // neighbour indices clamped to the cell itself on the faces, so the seven loads are
    // unconditional and in flight together (the clamped value is the Neumann one)
    const double pc = phi[c];
    const double xm = phi[i > 0 ? c - 1 : c], xp = phi[i < nx - 1 ? c + 1 : c];
    const double ym = phi[j > 0 ? c - sy : c], yp = phi[j < ny - 1 ? c + sy : c];
    const double vzm = phi[k > 0 ? c - sz : c], vzp = phi[k < nz - 1 ? c + sz : c];
    __builtin_amdgcn_sched_barrier(0);
    const double zm = k > 0 ? vzm : -pc, zp = k < nz - 1 ? vzp : 2.0 * V - pc;
    st4<T>(E4 + 4 * (size_t)c, (T)(-(xp - xm) * inv2h), (T)(-(yp - ym) * inv2h), (T)(-(zp - zm) * inv2h),
           (T)0);
  }
}

// The same field over 4-cell row segments (nx a multiple of 4): a thread reads the
// potential of its four cells and of the four cells of each neighbouring row as
// 16-byte vectors, plus the cells before and after the segment, all in flight
// together, and writes four packed values; each cell's differences are those of
// k_efield (same values).
template <typename T>
__global__ void __launch_bounds__(256) k_efield_seg(const double* phi, int nx, int ny, int nz, double V,
                                                   double inv2h, T* E4) {
  const int ns = nx >> 2;
  const uint32_t nseg = (uint32_t)ns * ny * nz;
  const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
  for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < nseg; g += gridDim.x * blockDim.x) {
    const uint32_t row = g / (uint32_t)ns;
    const int t = (int)(g - row * (uint32_t)ns);
    const int j = (int)(row % (uint32_t)ny), k = (int)(row / (uint32_t)ny);
    const size_t c0 = (size_t)row * sy + 4 * (size_t)t;
    const V4<double> pc = ld4(phi + c0);
    const V4<double> ym = ld4(phi + (j > 0 ? c0 - sy : c0)), yp = ld4(phi + (j < ny - 1 ? c0 + sy : c0));
    const V4<double> zm = ld4(phi + (k > 0 ? c0 - sz : c0)), zp = ld4(phi + (k < nz - 1 ? c0 + sz : c0));
    const double pl = phi[t > 0 ? c0 - 1 : c0], pr = phi[4 * t + 4 < nx ? c0 + 4 : c0 + 3];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double xm = r > 0 ? pc.a[r - 1] : pl, xp = r < 3 ? pc.a[r + 1] : pr;
      const double vzm = k > 0 ? zm.a[r] : -pc.a[r], vzp = k < nz - 1 ? zp.a[r] : 2.0 * V - pc.a[r];
      st4<T>(E4 + 4 * (c0 + r), (T)(-(xp - xm) * inv2h), (T)(-(yp.a[r] - ym.a[r]) * inv2h),
             (T)(-(vzp - vzm) * inv2h), (T)0);
    }
  }
}

// One component of the packed field, as double.
template <typename T>
__global__ void k_component(const T* E4, int a, double* out, uint32_t n) {
  for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x)
    out[c] = (double)E4[4 * (size_t)c + a];
}

inline int blocks(uint64_t n, int max_blocks = 16384) {
  uint64_t b = (n + 255) / 256;
  if (b < 1) b = 1;
  if (b > (uint64_t)max_blocks) b = max_blocks;
  return (int)b;
}

}  // namespace

// ---- host side ------------------------------------------------------------------------

struct FieldState {
  int nlev = 0;
  Level lev[kMaxLevels];
  double* phi = nullptr;
  double* b = nullptr;
  void* E[2] = {nullptr, nullptr};  // packed (Ex, Ey, Ez, 0) per cell; E[cur] holds the latest
  int cur = 0;        // E[cur] holds the latest field
  void* sig = nullptr;
  void* ne = nullptr;
  double* norms = nullptr;   // device: ||b||^2, ||r||^2, then per-block partials
  double* host_norms = nullptr;    // mapped pinned host memory: ||b||^2, ||r||^2, sequence
  double* host_norms_dev = nullptr;  // its device address
  unsigned long long seq_expect = 0;  // notifications the host has waited for
  double* phi_prev = nullptr;  // converged potential of the previous step
  bool have_prev = false;
  bool split = false;  // finest level in split red-black order (nx even, more than one level)
  bool seg = false;    // finest-level kernels over 8-cell row segments (nx % 8 == 0, more than one level)
  // per level: split red-black order, and 8-cell row-segment kernels.  The finest level
  // as above; a coarser level (not the coarsest) with nx % 8 == 0 and more than
  // kSmallLevel cells takes both when the finest level is split.
  bool lsplit[kMaxLevels] = {};
  bool lseg[kMaxLevels] = {};
  bool ltile[kMaxLevels] = {};  // k_tile_level (natural order)
  bool graph_failed = false;
  hipGraphExec_t graph_exec = nullptr;
  // optional timing of the finest-level smoother launches: event pairs recorded around
  // each launch; while timing is on the cycle runs eagerly (not from the graph)
  static constexpr int kMaxTimed = 64;
  hipEvent_t sm_ev[2 * kMaxTimed] = {};
  int sm_n = 0;              // event pairs recorded by the cycle being enqueued
  int sm_pending = 0;        // pairs recorded by the last enqueued cycle, unread
  bool timing = false;
};

static int build_levels(const itokmc_grid_desc* d, int dims[kMaxLevels][3]) {
  int nl = 0;
  int nx = d->nx, ny = d->ny, nz = d->nz;
  for (;;) {
    dims[nl][0] = nx; dims[nl][1] = ny; dims[nl][2] = nz;
    ++nl;
    const int mn = nx < ny ? (nx < nz ? nx : nz) : (ny < nz ? ny : nz);
    if (nl == kMaxLevels || mn < 4 || (nx | ny | nz) & 1) break;
    nx /= 2; ny /= 2; nz /= 2;
  }
  return nl;
}

// Levels that run in one workgroup (k_small_level).
static bool small_level(int l, int nlev, size_t n) { return (l > 0 || nlev == 1) && n <= kSmallLevel; }
// Levels that can run in tiles (k_tile_level): every one above the coarsest that is not
// small.
static bool tile_level(int l, int nlev, size_t n, size_t T) {
  return l < nlev - 1 && !small_level(l, nlev, n) && n <= tile_max(T);
}

size_t field_bytes(const itokmc_grid_desc* d) {
  if (d->field_mode != ITOKMC_FIELD_POISSON) return 0;
  const size_t T = d->precision == ITOKMC_FP64 ? 8 : 4;
  const size_t n = (size_t)d->nx * d->ny * d->nz;
  int dims[kMaxLevels][3];
  const int nl = build_levels(d, dims);
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t npart = (size_t)kRedBlocks > (n + 255) / 256 ? (size_t)kRedBlocks : (n + 255) / 256;
  size_t total = al(n * 8) * 3 + al(n * 4 * T) * 2 + al(n * 8) * 2 + al(8 * (8 + npart));
  for (int l = 0; l < nl; ++l) {
    const size_t m = (size_t)dims[l][0] * dims[l][1] * dims[l][2];
    total += 3 * al(m * T);
    if (small_level(l, nl, m) || (T == 8 && tile_level(l, nl, m, T))) total += al(4 * m * T);
    if (tile_level(l, nl, m, T) && l > 0) total += al(m * T);
  }
  return total;
}

static FieldState* fs(itokmc_ctx* ctx) { return reinterpret_cast<FieldState*>(ctx->field_state); }

int field_init(itokmc_ctx* ctx, char* base) {
  const itokmc_grid_desc* d = &ctx->d;
  int dims[kMaxLevels][3];
  const int nl = build_levels(d, dims);
  const uint64_t bottom = (uint64_t)dims[nl - 1][0] * dims[nl - 1][1] * dims[nl - 1][2];
  if (bottom > (uint64_t)kBottomMaxCells)
    return set_error(ctx, ITOKMC_EINVAL, "grid cannot be coarsened to <= %d cells (dims must be even)",
                     kBottomMaxCells);
  FieldState* F = new FieldState();
  const size_t T = d->precision == ITOKMC_FP64 ? 8 : 4;
  const size_t n = ctx->ncell;
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  char* p = base;
  F->phi = (double*)p; p += al(n * 8);
  F->b = (double*)p; p += al(n * 8);
  F->phi_prev = (double*)p; p += al(n * 8);
  for (int s = 0; s < 2; ++s)
    { F->E[s] = p; p += al(n * 4 * T); }
  F->sig = p; p += al(n * 8);  // deposit accumulators (8 bytes in either precision)
  F->ne = p; p += al(n * 8);
  const size_t npart = (size_t)kRedBlocks > (n + 255) / 256 ? (size_t)kRedBlocks : (n + 255) / 256;
  F->norms = (double*)p; p += al(8 * (8 + npart));
  F->nlev = nl;
  F->seg = nl > 1 && d->nx % 8 == 0;
  for (int l = 0; l < nl; ++l) {
    Level& L = F->lev[l];
    L.nx = dims[l][0]; L.ny = dims[l][1]; L.nz = dims[l][2];
    L.n = (uint32_t)((size_t)L.nx * L.ny * L.nz);
    L.u = p; p += al(L.n * T);
    L.f = p; p += al(L.n * T);
    L.eps = p; p += al(L.n * T);
    L.cf = nullptr;
    L.u2 = nullptr;
    if (small_level(l, nl, L.n) || (T == 8 && tile_level(l, nl, L.n, T))) { L.cf = p; p += al(4 * (size_t)L.n * T); }
    if (tile_level(l, nl, L.n, T) && l > 0) { L.u2 = p; p += al(L.n * T); }
  }
  hipError_t e = hipHostMalloc((void**)&F->host_norms, 64, hipHostMallocMapped | hipHostMallocCoherent);
  if (e == hipSuccess) {
    for (int i = 0; i < 8; ++i) F->host_norms[i] = 0.0;
    e = hipHostGetDevicePointer((void**)&F->host_norms_dev, F->host_norms, 0);
  }
  if (e == hipSuccess) e = hipMemsetAsync(F->norms, 0, 8 * sizeof(double), ctx->s);
  if (e == hipSuccess) e = hipMemsetAsync(F->phi, 0, n * 8, ctx->s);
  for (int s = 0; s < 2 && e == hipSuccess; ++s)
    e = hipMemsetAsync(F->E[s], 0, n * 4 * T, ctx->s);
  if (e != hipSuccess) {
    delete F;
    return check_hip(ctx, e, "field init");
  }
  ctx->field_state = F;
  return ITOKMC_OK;
}

// Drop the captured cycle (its launch parameters depend on the tuning).
void field_reset_graph(itokmc_ctx* ctx) {
  FieldState* F = fs(ctx);
  if (!F) return;
  if (F->graph_exec) (void)hipGraphExecDestroy(F->graph_exec);
  F->graph_exec = nullptr;
  F->graph_failed = false;
}

// Turn timing of the finest-level smoother on or off (the cycle graph is rebuilt).
void field_set_timing(itokmc_ctx* ctx, bool on) {
  FieldState* F = fs(ctx);
  if (!F || F->timing == on) return;
  (void)hipStreamSynchronize(ctx->s);
  if (on && !F->sm_ev[0])
    for (int i = 0; i < 2 * FieldState::kMaxTimed; ++i) (void)hipEventCreate(&F->sm_ev[i]);
  F->timing = on;
  F->sm_pending = 0;
}

void field_destroy(itokmc_ctx* ctx) {
  FieldState* F = fs(ctx);
  if (!F) return;
  for (int i = 0; i < 2 * FieldState::kMaxTimed; ++i)
    if (F->sm_ev[i]) (void)hipEventDestroy(F->sm_ev[i]);
  if (F->host_norms) (void)hipHostFree(F->host_norms);
  if (F->graph_exec) (void)hipGraphExecDestroy(F->graph_exec);
  delete F;
  ctx->field_state = nullptr;
}

static Coef coef(const itokmc_ctx* ctx) {
  return Coef{ctx->c.mu_a, ctx->c.mu_E0, ctx->c.mu_b, ctx->c.E_floor, ctx->c.D};
}

// Blocks of 256 threads for one thread per 8-cell row segment of an nx x ny x nz level.
static int seg_blocks(int nx, int ny, int nz) {
  const uint64_t n = (uint64_t)(nx >> 3) * ny * nz;
  return (int)((n + 255) / 256);
}

static dim3 row_grid(int half_nx, int ny, int nz) {
  return dim3((unsigned)((half_nx + 127) / 128), (unsigned)ny, (unsigned)nz);
}

// One colour sweep at level l (the finest level in split order when F->split); the
// finest level's launches are bracketed by event pairs when timing is on.
template <typename T>
static void smooth(FieldState* F, int l, hipStream_t s, int color, bool from_zero = false) {
  Level& L = F->lev[l];
  const dim3 gs = row_grid((L.nx + 1) / 2, L.ny, L.nz);
  T* u = (T*)L.u;
  const T* f = (const T*)L.f;
  const T* ep = (const T*)L.eps;
  if (l > 0) {
    if (F->lsplit[l])
      k_smooth_seg<T, false><<<seg_blocks(L.nx, L.ny, L.nz), 256, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, color);
    else
      k_smooth_rb<T, false><<<gs, 128, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, color);
    return;
  }
  const bool timed = F->timing && F->sm_n < FieldState::kMaxTimed;  // eager cycles only
  if (timed) (void)hipEventRecord(F->sm_ev[2 * F->sm_n], s);
  if (F->split && F->seg && from_zero)
    k_smooth_seg<T, true, true><<<seg_blocks(L.nx, L.ny, L.nz), 256, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, color);
  else if (F->split && F->seg)
    k_smooth_seg<T, true><<<seg_blocks(L.nx, L.ny, L.nz), 256, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, color);
  else if (F->split)
    k_smooth_split<T><<<gs, 128, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, color);
  else
    k_smooth_rb<T, true><<<gs, 128, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, color);
  if (timed) (void)hipEventRecord(F->sm_ev[2 * F->sm_n + 1], s);
  if (timed) ++F->sm_n;
}

// from_zero: the level's correction is zero on entry and not stored (first sweeps of a
// refinement cycle on the finest level with the row-segment smoother).
template <typename T>
static void smooth_sweeps(FieldState* F, int l, hipStream_t s, int count, bool from_zero = false) {
  for (int it = 0; it < count; ++it) {
    smooth<T>(F, l, s, 0, from_zero && it == 0);
    smooth<T>(F, l, s, 1);
  }
}

static bool zero_free_start(const itokmc_ctx* ctx, const FieldState* F) {
  return F->split && F->seg && ctx->tune.mg_pre >= 1;
}

static int bottom_count(const itokmc_ctx* ctx, const Level& L) {
  int mx = L.nx > L.ny ? L.nx : L.ny;
  mx = mx > L.nz ? mx : L.nz;
  return ctx->tune.bottom_sweeps > 0 ? ctx->tune.bottom_sweeps : 4 * mx + 16;
}

// Where level l's correction is after its part of the cycle.
template <typename T>
static T* correction(FieldState* F, int l) {
  return (T*)(F->ltile[l] && l > 0 ? F->lev[l].u2 : F->lev[l].u);
}

// V-cycle from level l.
template <typename T>
static void vcycle(itokmc_ctx* ctx, FieldState* F, int l, hipStream_t s) {
  Level& L = F->lev[l];
  T* u = (T*)L.u;
  const T* f = (const T*)L.f;
  const T* ep = (const T*)L.eps;
  const T* cf = (const T*)L.cf;
  if (l == F->nlev - 1) {
    launch_small_level<T>(s, u, f, cf, L.nx, L.ny, L.nz, bottom_count(ctx, L), true, nullptr, nullptr, nullptr,
                          0, 0, 0);
    return;
  }
  Level& C = F->lev[l + 1];
  if (F->ltile[l]) {
    const int nt = tile_blocks(L.nx, L.ny, L.nz);
    k_tile_level<T, false><<<nt, 1024, 0, s>>>(u, f, ep, cf, L.nx, L.ny, L.nz, ctx->tune.mg_pre, nullptr, C.nx, C.ny,
                                               C.nz, nullptr, nullptr, (T*)C.f);
    vcycle<T>(ctx, F, l + 1, s);
    k_tile_level<T, true><<<nt, 1024, 0, s>>>(u, f, ep, cf, L.nx, L.ny, L.nz, ctx->tune.mg_post,
                                              correction<T>(F, l + 1), C.nx, C.ny, C.nz, (T*)L.u2,
                                              l == 0 ? F->phi : nullptr, nullptr);
    return;
  }
  if (small_level(l, F->nlev, L.n)) {
    // natural order (small levels are never split): smoothing from the zero
    // correction that every restriction leaves, and restriction; the coarser cycle;
    // prolongation and smoothing
    launch_small_level<T>(s, u, f, cf, L.nx, L.ny, L.nz, ctx->tune.mg_pre, true, nullptr, (T*)C.f, (T*)C.u,
                          C.nx, C.ny, C.nz);
    vcycle<T>(ctx, F, l + 1, s);
    launch_small_level<T>(s, u, f, cf, L.nx, L.ny, L.nz, ctx->tune.mg_post, false,
                          correction<T>(F, l + 1), nullptr, nullptr, C.nx, C.ny, C.nz);
    return;
  }
  smooth_sweeps<T>(F, l, s, ctx->tune.mg_pre, l == 0 && zero_free_start(ctx, F));
  const dim3 gr = row_grid(C.nx, C.ny, C.nz), gp = row_grid(L.nx, L.ny, L.nz);
  const int sb = seg_blocks(L.nx, L.ny, L.nz);
  T* fcp = (T*)C.f;
  T* ucp = (T*)C.u;
  const int rg = (int)(((uint32_t)(L.nx >> 3) * C.ny * C.nz + 63u) / 64u);
  const bool fs = F->lsplit[l], csp = F->lsplit[l + 1];
  if (F->lseg[l]) {
    if (fs && csp) k_restrict_seg<T, true, true><<<rg, 256, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, fcp, ucp);
    else if (fs) k_restrict_seg<T, true, false><<<rg, 256, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, fcp, ucp);
    else k_restrict_seg<T, false, false><<<rg, 256, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, fcp, ucp);
  } else if (fs) {
    k_restrict3<T, true><<<gr, 128, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, fcp, ucp, C.nx, C.ny);
  } else {
    k_restrict3<T, false><<<gr, 128, 0, s>>>(u, f, ep, L.nx, L.ny, L.nz, fcp, ucp, C.nx, C.ny);
  }
  vcycle<T>(ctx, F, l + 1, s);
  const T* ucc = correction<T>(F, l + 1);
  if (F->lseg[l]) {
    if (fs && csp) k_prolong_seg<T, true, true><<<sb, 256, 0, s>>>(u, L.nx, L.ny, L.nz, ucc, C.nx, C.ny, C.nz);
    else if (fs) k_prolong_seg<T, true, false><<<sb, 256, 0, s>>>(u, L.nx, L.ny, L.nz, ucc, C.nx, C.ny, C.nz);
    else k_prolong_seg<T, false, false><<<sb, 256, 0, s>>>(u, L.nx, L.ny, L.nz, ucc, C.nx, C.ny, C.nz);
  } else if (fs) {
    k_prolong3<T, true><<<gp, 128, 0, s>>>(u, L.nx, L.ny, L.nz, ucc, C.nx, C.ny, C.nz);
  } else {
    k_prolong3<T, false><<<gp, 128, 0, s>>>(u, L.nx, L.ny, L.nz, ucc, C.nx, C.ny, C.nz);
  }
  smooth_sweeps<T>(F, l, s, ctx->tune.mg_post);
}

// Wait for the next residual-norm notification (k_sum_notify) by polling the mapped
// host word; after a fraction of a second without it (a failed launch), synchronise the stream,
// which reports the error.  While the smoother is being timed the stream is
// synchronised instead (its events are read right after).
static hipError_t wait_norms(FieldState* F, hipStream_t s) {
  const unsigned long long want = ++F->seq_expect;
  if (F->timing) return hipStreamSynchronize(s);
  volatile unsigned long long* q = reinterpret_cast<volatile unsigned long long*>(F->host_norms) + 2;
  for (long spin = 0; *q < want; ++spin) {
    if (spin > (1L << 26)) {
      const hipError_t e = hipStreamSynchronize(s);
      if (e != hipSuccess) return e;
      if (*q < want) return hipErrorUnknown;
      break;
    }
  }
  return hipSuccess;
}

// Accumulate the timed finest-level smoother launches of the last cycle (the stream
// has been synchronised).
static void collect_smooth(itokmc_ctx* ctx, FieldState* F) {
  for (int i = 0; i < F->sm_pending; ++i) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, F->sm_ev[2 * i], F->sm_ev[2 * i + 1]) == hipSuccess) {
      ctx->phase_ms[PH_SMOOTH_FINE] += ms;
      ctx->phase_calls[PH_SMOOTH_FINE] += 1;
    }
  }
  F->sm_pending = 0;
}

// Double residual of the finest level into f (working precision) and ||r||^2 into
// norms[1].
template <typename T>
static void residual(FieldState* F, hipStream_t s) {
  Level& L0 = F->lev[0];
  if (F->seg) {
    const uint32_t runs = ((L0.n >> 3) + 255) / 256;
    const int rb = runs < (uint32_t)kResBlocks ? (int)runs : kResBlocks;
    if (F->split)
      k_residual_seg<T, true><<<rb, 256, 0, s>>>(F->phi, F->b, (const T*)L0.eps, L0.nx, L0.ny, L0.nz,
                                                 (T*)L0.f, F->norms + 8);
    else
      k_residual_seg<T, false><<<rb, 256, 0, s>>>(F->phi, F->b, (const T*)L0.eps, L0.nx, L0.ny, L0.nz,
                                                  (T*)L0.f, F->norms + 8);
    k_sum_notify<<<1, 1024, 0, s>>>(F->norms + 8, rb, F->norms + 1, F->norms, F->host_norms_dev,
                                    reinterpret_cast<unsigned long long*>(F->norms + 2));
    return;
  }
  const uint32_t runs = (L0.n + 255) / 256;
  const int rb = runs < (uint32_t)kResBlocks ? (int)runs : kResBlocks;
  if (F->split)
    k_residual_rows<T, true><<<rb, 256, 0, s>>>(F->phi, F->b, (const T*)L0.eps, L0.nx, L0.ny, L0.nz,
                                                (T*)L0.f, F->norms + 8);
  else
    k_residual_rows<T, false><<<rb, 256, 0, s>>>(F->phi, F->b, (const T*)L0.eps, L0.nx, L0.ny, L0.nz,
                                                 (T*)L0.f, F->norms + 8);
  k_sum_notify<<<1, 1024, 0, s>>>(F->norms + 8, rb, F->norms + 1, F->norms, F->host_norms_dev,
                                  reinterpret_cast<unsigned long long*>(F->norms + 2));
}

// One refinement cycle: correction V-cycle from zero, potential update, new double
// residual and its norm.
template <typename T>
static void refine_cycle(itokmc_ctx* ctx, FieldState* F, hipStream_t s) {
  Level& L0 = F->lev[0];
  F->sm_n = 0;
  // the correction starts at zero; the first colour-0 sweep can assume it instead (the
  // colour-1 sweep that follows writes the rest of the level before anything reads it)
  if (!F->ltile[0] && !zero_free_start(ctx, F)) k_zero<T><<<blocks(L0.n), 256, 0, s>>>((T*)L0.u, L0.n);
  vcycle<T>(ctx, F, 0, s);
  const dim3 gp = row_grid(L0.nx, L0.ny, L0.nz);
  const int sb = seg_blocks(L0.nx, L0.ny, L0.nz);
  if (F->ltile[0]) {
    // the last tiled launch has added the correction to the potential
  } else if (F->seg && F->split)
    k_phi_update_seg<T, true><<<sb, 256, 0, s>>>(F->phi, (const T*)L0.u, L0.nx, L0.ny, L0.nz);
  else if (F->seg)
    k_phi_update_seg<T, false><<<sb, 256, 0, s>>>(F->phi, (const T*)L0.u, L0.nx, L0.ny, L0.nz);
  else if (F->split) k_phi_update<T, true><<<gp, 128, 0, s>>>(F->phi, (const T*)L0.u, L0.nx, L0.ny);
  else k_phi_update<T, false><<<gp, 128, 0, s>>>(F->phi, (const T*)L0.u, L0.nx, L0.ny);
  residual<T>(F, s);
}

// Capture one refinement cycle into a HIP graph (on a private stream: the caller's
// stream may be the legacy default stream, which cannot be captured).  The graph holds
// kernel nodes only.  Returns false if capture is unavailable; the caller then runs the
// cycle eagerly.
template <typename T>
static bool capture_cycle(itokmc_ctx* ctx, FieldState* F) {
  if (F->graph_exec) return true;
  if (F->graph_failed) return false;
  hipStream_t cs = nullptr;
  if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) { F->graph_failed = true; return false; }
  hipGraph_t g = nullptr;
  bool ok = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) == hipSuccess;
  if (ok) {
    refine_cycle<T>(ctx, F, cs);
    ok = hipStreamEndCapture(cs, &g) == hipSuccess && g != nullptr;
  }
  hipGraphExec_t ex = nullptr;
  if (ok) ok = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) == hipSuccess;
  if (g) (void)hipGraphDestroy(g);
  (void)hipStreamDestroy(cs);
  (void)hipGetLastError();
  if (!ok) { F->graph_failed = true; return false; }
  F->graph_exec = ex;
  return true;
}

// Solve with the current right-hand side b and fine coefficient lev[0].eps.
template <typename T>
static int solve(itokmc_ctx* ctx, FieldState* F) {
  hipStream_t s = ctx->s;
  Level& L0 = F->lev[0];
  SmallLevels S{};
  const T* ef = nullptr;  // the coefficient above the first small level
  int above = 0;
  for (int l = 0; l < F->nlev; ++l) {
    Level& Cl = F->lev[l];
    if (small_level(l, F->nlev, Cl.n)) {
      if (S.count == 0 && l > 0) { ef = (const T*)F->lev[l - 1].eps; above = l - 1; }
      S.nx[S.count] = Cl.nx; S.ny[S.count] = Cl.ny; S.nz[S.count] = Cl.nz;
      S.eps[S.count] = Cl.eps; S.cf[S.count] = Cl.cf;
      ++S.count;
    } else if (l > 0) {
      Level& Fl = F->lev[l - 1];
      k_eps_restrict<T><<<blocks(Cl.n), 256, 0, s>>>((const T*)Fl.eps, Fl.nx, Fl.ny, F->lsplit[l - 1] ? 1 : 0,
                                                     (T*)Cl.eps, Cl.nx, Cl.ny, Cl.nz, F->lsplit[l] ? 1 : 0);
    }
  }
  for (int l = 0; l < F->nlev && sizeof(T) == 8; ++l) {
    Level& Cl = F->lev[l];
    if (F->ltile[l])
      k_tile_faces<T><<<blocks(Cl.n), 256, 0, s>>>((const T*)Cl.eps, Cl.nx, Cl.ny, Cl.nz, (T*)Cl.cf);
  }
  k_small_setup<T><<<1, 1024, 0, s>>>(S, ef, F->lev[above].nx, F->lev[above].ny, F->lsplit[above] ? 1 : 0);
  const int maxc = ctx->d.gmg_max_cycles > 0 ? ctx->d.gmg_max_cycles : 50;
  ctx->total_solves += 1;
  residual<T>(F, s);
  const bool graph = ctx->tune.use_graph && !F->timing && capture_cycle<T>(ctx, F);
  for (int cyc = 0;; ++cyc) {
    // every residual launch ends with one notification: wait for this one
    hipError_t e = wait_norms(F, s);
    if (e != hipSuccess) return check_hip(ctx, e, "solve residual");
    collect_smooth(ctx, F);
    const double bn2 = F->host_norms[0], rn2 = F->host_norms[1];
    const double bn = bn2 > 0.0 ? sqrt(bn2) : 1.0;
    ctx->last_relres = sqrt(rn2) / bn;
    ctx->last_cycles = cyc;
    if (sqrt(rn2) <= ctx->d.gmg_rtol * bn) break;
    if (cyc >= maxc)
      return set_error(ctx, ITOKMC_ENOCONV, "field solve: relres %.3e after %d cycles", ctx->last_relres, cyc);
    ctx->total_cycles += 1;
    if (graph) {
      e = hipGraphLaunch(F->graph_exec, s);
      if (e != hipSuccess) return check_hip(ctx, e, "solve graph");
      F->sm_pending = 0;
    } else {
      refine_cycle<T>(ctx, F, s);
      F->sm_pending = F->sm_n;
    }
  }
  return check_hip(ctx, hipGetLastError(), "solve");
}

// Deposit (mode 0 initial / 1 semi-implicit), right-hand side, solve, E into E[next].
template <typename T>
static int deposit_and_solve(itokmc_ctx* ctx, FieldState* F, const StepConst& K, int mode) {
  hipStream_t s = ctx->s;
  const uint32_t n = ctx->ncell;
  // levels that run in tiles (their colours have to fit the halo) keep natural order
  const bool tiled = ctx->tune.mg_pre >= 1 && 2 * ctx->tune.mg_pre <= kHalo && 2 * ctx->tune.mg_post <= kHalo;
  for (int l = 0; l < F->nlev; ++l) F->ltile[l] = tiled && tile_level(l, F->nlev, F->lev[l].n, sizeof(T));
  const bool split = ctx->tune.fine_layout == 0 && F->nlev > 1 && !F->ltile[0];
  if (split != F->split) {
    field_reset_graph(ctx);
    F->split = split;
  }
  for (int l = 0; l < F->nlev; ++l) {
    const Level& L = F->lev[l];
    if (l == 0) {
      F->lsplit[0] = F->split;
      F->lseg[0] = F->seg;
    } else {
      F->lseg[l] = F->lsplit[l] =
          F->split && l < F->nlev - 1 && L.nx % 8 == 0 && L.n > kSmallLevel && !F->ltile[l];
    }
  }
  phase_begin(ctx, PH_FIELD_PREP);
  using S = typename DepAcc<T>::S;
  k_zero<S><<<blocks(n), 256, 0, s>>>((S*)F->sig, n);
  k_zero<S><<<blocks(n), 256, 0, s>>>((S*)F->ne, n);
  phase_end(ctx, PH_FIELD_PREP);
  const void* Eo = F->E[F->cur];
  phase_begin(ctx, PH_DEPOSIT);  // the deposit kernel alone
  {
    int g = (int)((ctx->cap + kDepChunk - 1) / kDepChunk);
    g = g < 1 ? 1 : (g > 16384 ? 16384 : g);
    const auto launch = [&](auto kern, int grid, size_t lds) {
      kern<<<grid, 256, lds, s>>>(ctx->bank[ctx->cur], ctx->ctr, ctx->cur, K, Eo, coef(ctx), mode, (S*)F->sig,
                               (S*)F->ne, (T*)ctx->mu_p);
    };
    const bool many = ctx->cap >= kDepFew<T>;
    // a kernel that returns costs its workgroups: 4096 are enough for the per-lane form where
    // cells hold few particles
    const int gl = std::min(g, 4096);
    if (ctx->d.shape == ITOKMC_SHAPE_TSC) {
      launch(k_field_deposit_blocks<T, 1>, g, dep_lds_bytes<T, 1>(false));
      launch(k_field_deposit_lanes<T, 1>, gl, dep_lds_bytes<T, 1>(true));
    } else {
      if (sizeof(T) == 8 || many) launch(k_field_deposit_blocks<T, 0>, g, dep_lds_bytes<T, 0>(false));
      if (sizeof(T) == 4 || many) launch(k_field_deposit_lanes<T, 0>, sizeof(T) == 4 ? g : gl, dep_lds_bytes<T, 0>(true));
    }
  }
  phase_end(ctx, PH_DEPOSIT);
  phase_begin(ctx, PH_FIELD_PREP);
  const double sig_scale = mode == 1 ? kE * K.dt / (kEps0 * K.dx * K.dx * K.dx) : 0.0;
  if (mode == 1) {
    k_extrapolate<<<blocks(n), 256, 0, s>>>(F->phi, F->phi_prev, n,
                                           (F->have_prev && ctx->tune.extrapolate) ? 1 : 0);
    F->have_prev = true;
  } else {
    F->have_prev = false;
  }
  k_field_prep<T><<<kRedBlocks, 256, 0, s>>>(K, ctx->nplus, ctx->nminus, (const S*)F->ne,
                                             (const S*)F->sig, sig_scale, ctx->d.V_anode,
                                             F->split ? 1 : 0, ctx->d.shape == ITOKMC_SHAPE_TSC ? 1 : 0,
                                             (T*)F->lev[0].eps, F->b, F->norms + 8);
  k_sum_partials<<<1, 1024, 0, s>>>(F->norms + 8, kRedBlocks, F->norms);
  phase_end(ctx, PH_FIELD_PREP);
  phase_begin(ctx, PH_SOLVE);
  const int rc = solve<T>(ctx, F);
  const int nxt = 1 - F->cur;
  if (ctx->d.nx % 4 == 0)
    k_efield_seg<T><<<blocks(n / 4), 256, 0, s>>>(F->phi, ctx->d.nx, ctx->d.ny, ctx->d.nz, ctx->d.V_anode,
                                                  1.0 / (2.0 * ctx->d.dx), (T*)F->E[nxt]);
  else
    k_efield<T><<<blocks(n), 256, 0, s>>>(F->phi, ctx->d.nx, ctx->d.ny, ctx->d.nz, ctx->d.V_anode,
                                          1.0 / (2.0 * ctx->d.dx), (T*)F->E[nxt]);
  phase_end(ctx, PH_SOLVE);
  return rc ? rc : check_hip(ctx, hipGetLastError(), "field");
}

// Initial field: the solution for the present charge with sigma = 0 (the deposit's mode
// 0 uses neither dt nor the diffusion of K).
template <typename T>
static int ensure_field(itokmc_ctx* ctx, FieldState* F, const StepConst& K) {
  if (ctx->field_valid) return 0;
  const int rc = deposit_and_solve<T>(ctx, F, K, 0);
  if (rc) return rc;
  F->cur = 1 - F->cur;
  ctx->field_valid = true;
  return 0;
}

template <typename T>
static int transport_t(itokmc_ctx* ctx, const StepConst& K) {
  FieldState* F = fs(ctx);
  int rc = ensure_field<T>(ctx, F, K);
  if (rc) return rc;
  rc = deposit_and_solve<T>(ctx, F, K, 1);
  if (rc) return rc;
  const int nxt = 1 - F->cur;
  phase_begin(ctx, PH_FIELD_PUSH);
  // at most 4096 workgroups looping over the particles: 0.186 ms per step at 6e6 particles
  // against 0.199 with 1024 and 0.188 with 16384; 1.26 against 1.35 and 1.24 ms at 4.5e7
  if (ctx->d.shape == ITOKMC_SHAPE_TSC)
    k_push_field<T, 1><<<blocks(ctx->cap, 4096), 256, 0, ctx->s>>>(
        ctx->bank[ctx->cur], ctx->ctr, ctx->cur, ctx->cellacc, ctx->tiles, K, (const T*)ctx->mu_p, F->E[nxt]);
  else
    k_push_field<T, 0><<<blocks(ctx->cap, 4096), 256, 0, ctx->s>>>(
        ctx->bank[ctx->cur], ctx->ctr, ctx->cur, ctx->cellacc, ctx->tiles, K, (const T*)ctx->mu_p, F->E[nxt]);
  phase_end(ctx, PH_FIELD_PUSH);
  F->cur = nxt;  // E^{k+1} becomes the field of the next step
  if (mobile_ions(ctx)) {
    const hipError_t e = launch_ion_move(ctx, K, F->E[nxt]);
    if (e != hipSuccess) return check_hip(ctx, e, "ions");
  }
  return check_hip(ctx, hipGetLastError(), "field push");
}

int field_transport(itokmc_ctx* ctx, const StepConst& K) {
  return ctx->d.precision == ITOKMC_FP64 ? transport_t<double>(ctx, K) : transport_t<float>(ctx, K);
}

// Largest |E|^2 over the cell centres of the packed (Ex, Ey, Ez, 0) field: one partial
// per workgroup, squares summed in double from the stored components (exact for
// single-precision fields), then the largest partial.  Non-negative doubles order as
// their bit patterns, but plain comparisons suffice here: no atomics.
template <typename T>
__global__ void __launch_bounds__(256) k_emax_partial(const T* E4, uint32_t n, double* part) {
  __shared__ double sh[4];
  double m = 0.0;
#pragma unroll 4
  for (uint32_t c = blockIdx.x * 256u + threadIdx.x; c < n; c += gridDim.x * 256u) {
    const V4<T> e = ld4(E4 + 4 * (size_t)c);
    const double x = (double)e.a[0], y = (double)e.a[1], z = (double)e.a[2];
    m = fmax(m, x * x + y * y + z * z);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) m = fmax(m, __shfl_xor(m, d, 64));
  if (lane_id() == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

__global__ void __launch_bounds__(1024) k_max_partials(const double* part, int n, double* out) {
  __shared__ double sh[16];
  double m = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) m = fmax(m, part[i]);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) m = fmax(m, __shfl_xor(m, d, 64));
  if (lane_id() == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int i = 0; i < 16; ++i) r = fmax(r, sh[i]);
    *out = r;
  }
}

template <typename T>
static int field_max_t(itokmc_ctx* ctx, double* Emax) {
  FieldState* F = fs(ctx);
  int rc = ensure_field<T>(ctx, F, make_const(ctx, 0.0));
  if (rc) return rc;
  const uint32_t n = ctx->ncell;
  // at most 2048 workgroups (one resident round of 32 waves per CU); the partials
  // buffer holds max(kRedBlocks, blocks(n)) entries
  const int nb = (int)std::min<size_t>(2048, blocks(n));
  hipStream_t s = ctx->s;
  phase_begin(ctx, PH_EMAX);  // the per-cell pass alone
  k_emax_partial<T><<<nb, 256, 0, s>>>((const T*)F->E[F->cur], n, F->norms + 8);
  phase_end(ctx, PH_EMAX);
  k_max_partials<<<1, 1024, 0, s>>>(F->norms + 8, nb, F->norms + 3);
  double m2 = 0.0;
  hipError_t e = hipMemcpyAsync(&m2, F->norms + 3, sizeof(double), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  rc = check_hip(ctx, e, "field max");
  if (rc) return rc;
  *Emax = sqrt(m2);
  return ITOKMC_OK;
}

int field_max(itokmc_ctx* ctx, double* Emax) {
  if (!fs(ctx)) return set_error(ctx, ITOKMC_EINVAL, "no field state");
  return ctx->d.precision == ITOKMC_FP64 ? field_max_t<double>(ctx, Emax) : field_max_t<float>(ctx, Emax);
}

FieldRates field_rates(itokmc_ctx* ctx) {
  FieldState* F = fs(ctx);
  FieldRates r{};
  if (!F) return r;
  r.E4 = F->E[F->cur];
  r.is_double = ctx->d.precision == ITOKMC_FP64 ? 1 : 0;
  r.mu_a = ctx->c.mu_a; r.mu_E0 = ctx->c.mu_E0; r.mu_b = ctx->c.mu_b; r.E_floor = ctx->c.E_floor;
  r.alpha_A = ctx->c.alpha_A; r.alpha_B = ctx->c.alpha_B; r.eta = ctx->c.eta;
  r.kgamma_ratio = ctx->c.kgamma_ratio;
  r.beta_ep = ctx->c.beta_ep; r.beta_ep_b = ctx->c.beta_ep_b; r.Te_a = ctx->c.Te_a;
  r.Te_b = ctx->c.Te_b; r.beta_np = ctx->c.beta_np;
  r.dV = ctx->d.dx * ctx->d.dx * ctx->d.dx;
  return r;
}

int field_get_phi(itokmc_ctx* ctx, double* host) {
  FieldState* F = fs(ctx);
  hipError_t e = hipStreamSynchronize(ctx->s);
  if (e == hipSuccess) e = copy_on(ctx->s, host, F->phi, (size_t)ctx->ncell * 8, hipMemcpyDeviceToHost);
  return check_hip(ctx, e, "get_field");
}

int field_set_phi(itokmc_ctx* ctx, const double* host) {
  FieldState* F = fs(ctx);
  hipError_t e = hipStreamSynchronize(ctx->s);
  if (e == hipSuccess) e = copy_on(ctx->s, F->phi, host, (size_t)ctx->ncell * 8, hipMemcpyHostToDevice);
  if (e != hipSuccess) return check_hip(ctx, e, "set_field");
  F->have_prev = false;
  const uint32_t n = ctx->ncell;
  if (ctx->d.precision == ITOKMC_FP64)
    k_efield<double><<<blocks(n), 256, 0, ctx->s>>>(F->phi, ctx->d.nx, ctx->d.ny, ctx->d.nz,
                                                    ctx->d.V_anode, 1.0 / (2.0 * ctx->d.dx),
                                                    (double*)F->E[F->cur]);
  else
    k_efield<float><<<blocks(n), 256, 0, ctx->s>>>(F->phi, ctx->d.nx, ctx->d.ny, ctx->d.nz,
                                                   ctx->d.V_anode, 1.0 / (2.0 * ctx->d.dx),
                                                   (float*)F->E[F->cur]);
  ctx->field_valid = true;
  return check_hip(ctx, hipGetLastError(), "set_field");
}

int field_deposit(itokmc_ctx* ctx, int what, void* dev_out) {
  FieldState* F = fs(ctx);
  const uint32_t n = ctx->ncell;
  if (what == ITOKMC_Q_PHI)
    return check_hip(ctx, hipMemcpyAsync(dev_out, F->phi, (size_t)n * 8, hipMemcpyDeviceToDevice, ctx->s),
                     "deposit phi");
  const int a = what - ITOKMC_Q_EX;
  if (ctx->d.precision == ITOKMC_FP64)
    k_component<double><<<blocks(n), 256, 0, ctx->s>>>((const double*)F->E[F->cur], a, (double*)dev_out, n);
  else
    k_component<float><<<blocks(n), 256, 0, ctx->s>>>((const float*)F->E[F->cur], a, (double*)dev_out, n);
  return check_hip(ctx, hipGetLastError(), "deposit E");
}

// Electron density of the current particles (diagnostic query), in double.  The bank is
// cell-sorted but for what was appended, so a workgroup's 256 particles share most of
// their nodes: they are summed in an LDS hash table first (kDenTbl entries, the slots and
// probing of the field deposit) and each touched node takes one global atomic.  A
// wavefront whose particles hardly share cells (runs of equal cells cover fewer than a
// quarter of its lanes: an unsorted seed, scattered photo-electrons) would only fill the
// table with single contributions and adds to the grid directly.  5.5e7 particles in
// 7e6 cells: 13.6 -> 1.5 ms (an unsorted 2e5-particle bank stays at 0.11 ms).
namespace {
constexpr int kDenL2 = 10;
__device__ __forceinline__ void den_add(uint32_t* keys, double* v, bool table, uint32_t node, uint32_t h,
                                        double x, double* out) {
  constexpr uint32_t mask = (1u << kDenL2) - 1u;
  if (table) {
    for (int probe = 0; probe < kDepProbes; ++probe) {
      uint32_t k = keys[h];
      if (k == kEmptyKey) {
        const uint32_t prev = atomicCAS(&keys[h], kEmptyKey, node);
        k = prev == kEmptyKey ? node : prev;
      }
      if (k == node) {
        atomicAdd(&v[h], x);
        return;
      }
      h = (h + 1u) & mask;
    }
  }
  atomicAdd(&out[node], x);
}

template <typename T, int SH>
__global__ void __launch_bounds__(256) k_cic_density(Bank a, const Counters* ctr, int which, StepConst K,
                                                     double inv_dV, double* out) {
  __shared__ double v[1 << kDenL2];
  __shared__ uint32_t keys[1 << kDenL2];
  const uint32_t n = min(ctr->n[which], K.cap);
  const int lane = lane_id();
  for (uint32_t base = blockIdx.x * 256u; base < n; base += gridDim.x * 256u) {
    for (int t = threadIdx.x; t < (1 << kDenL2); t += 256) {
      keys[t] = kEmptyKey;
      v[t] = 0.0;
    }
    __syncthreads();
    const uint32_t i = base + threadIdx.x;
    const uint32_t w = i < n ? a.w[i] : 0u;
    const uint32_t cell = w ? a.cell[i] : kInvalidCell;
    const uint64_t live = __ballot(w != 0u);
    const uint64_t same = __ballot(w != 0u && lane > 0 && dpp_from_prev(cell, ~cell) == cell);
    const bool table = 4 * __popcll(same) >= __popcll(live);
    if (w) {
      int ci, cj, ck;
      cell_ijk(cell, K, ci, cj, ck);
      const double ox = (double)ctp<T>(a.ox)[i], oy = (double)ctp<T>(a.oy)[i], oz = (double)ctp<T>(a.oz)[i];
      const double q = (double)w * inv_dV;
      if constexpr (SH == 0) {
        int i0, j0, k0;
        double fx, fy, fz;
        tent_axis<double>(ci, ox, K.nx, i0, fx);
        tent_axis<double>(cj, oy, K.ny, j0, fy);
        tent_axis<double>(ck, oz, K.nz, k0, fz);
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) {
          const int di = cc & 1, dj = (cc >> 1) & 1, dk = (cc >> 2) & 1;
          const double wt = (di ? fx : 1.0 - fx) * (dj ? fy : 1.0 - fy) * (dk ? fz : 1.0 - fz);
          const int ii = i0 + di, jj = j0 + dj, kk = k0 + dk;
          if (wt == 0.0 || ii >= K.nx || jj >= K.ny || kk >= K.nz) continue;
          const uint32_t row = (uint32_t)jj + (uint32_t)K.ny * (uint32_t)kk;
          const uint32_t h = ((uint32_t)ii + ((row * 2654435761u) >> (32 - kDenL2))) & ((1u << kDenL2) - 1u);
          den_add(keys, v, table, (uint32_t)ii + (uint32_t)K.nx * row, h, q * wt, out);
        }
      } else {
        const Tsc<double> s = tsc_at<double>(K, ci, cj, ck, ox, oy, oz);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const uint32_t row = (uint32_t)s.iy[b] + (uint32_t)K.ny * (uint32_t)s.iz[c];
            const uint32_t hr = (row * 2654435761u) >> (32 - kDenL2);
#pragma unroll
            for (int aa = 0; aa < 3; ++aa) {
              const double wt = (s.wx[aa] * s.wy[b]) * s.wz[c];
              if (wt == 0.0) continue;
              den_add(keys, v, table, (uint32_t)s.ix[aa] + (uint32_t)K.nx * row,
                      ((uint32_t)s.ix[aa] + hr) & ((1u << kDenL2) - 1u), q * wt, out);
            }
          }
      }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < (1 << kDenL2); t += 256) {
      const uint32_t k = keys[t];
      if (k != kEmptyKey) atomicAdd(&out[k], v[t]);
    }
    __syncthreads();
  }
}
}  // namespace

hipError_t launch_cic_density(itokmc_ctx* ctx, double* out) {
  hipError_t e = hipMemsetAsync(out, 0, sizeof(double) * ctx->ncell, ctx->s);
  if (e != hipSuccess) return e;
  StepConst K = make_const(ctx, 0.0);
  const double inv_dV = 1.0 / (ctx->d.dx * ctx->d.dx * ctx->d.dx);
  const bool tsc = ctx->d.shape == ITOKMC_SHAPE_TSC;
  Bank b = ctx->bank[ctx->cur];
  const int g = blocks(ctx->cap, 16384);
  if (ctx->d.precision == ITOKMC_FP64) {
    if (tsc) k_cic_density<double, 1><<<g, 256, 0, ctx->s>>>(b, ctx->ctr, ctx->cur, K, inv_dV, out);
    else k_cic_density<double, 0><<<g, 256, 0, ctx->s>>>(b, ctx->ctr, ctx->cur, K, inv_dV, out);
  } else {
    if (tsc) k_cic_density<float, 1><<<g, 256, 0, ctx->s>>>(b, ctx->ctr, ctx->cur, K, inv_dV, out);
    else k_cic_density<float, 0><<<g, 256, 0, ctx->s>>>(b, ctx->ctr, ctx->cur, K, inv_dV, out);
  }
  return hipGetLastError();
}

// Space charge of the current state (deposit query): e ((n+ - n-) / dV - n_e) with n_e
// the CIC density written into out by launch_cic_density.
namespace {
__global__ void k_rho_from_density(double* out, const uint32_t* np, const uint32_t* nm, StepConst K,
                                   int tsc, double inv_dV) {
  const uint32_t n = K.ncell;
  for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) {
    double ions = (double)np[c] - (double)nm[c];
    if (tsc) {
      const uint32_t row = c / (uint32_t)K.nx, k = row / (uint32_t)K.ny;
      ions = ion_tsc(np, nm, (int)(c - row * (uint32_t)K.nx), (int)(row - k * (uint32_t)K.ny), (int)k, K.nx,
                     K.ny, K.nz);
    }
    out[c] = kE * (ions * inv_dV - out[c]);
  }
}
}  // namespace

hipError_t launch_rho(itokmc_ctx* ctx, double* out) {
  hipError_t e = launch_cic_density(ctx, out);
  if (e != hipSuccess) return e;
  const double inv_dV = 1.0 / (ctx->d.dx * ctx->d.dx * ctx->d.dx);
  const int tsc = ctx->d.shape == ITOKMC_SHAPE_TSC ? 1 : 0;
  k_rho_from_density<<<blocks(ctx->ncell), 256, 0, ctx->s>>>(out, ctx->nplus, ctx->nminus, make_const(ctx, 0.0),
                                                            tsc, inv_dV);
  return hipGetLastError();
}

}  // namespace itk
