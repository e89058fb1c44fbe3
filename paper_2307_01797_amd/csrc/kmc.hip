// Per-cell Kinetic Monte Carlo on the GPU: one lane per occupied cell, double
// precision, random numbers from the cell's sequential Philox stream (cell, step, KMC).
//
// Network (rows 1, 2 and 5 of the paper's air-chemistry table), species (e, M+, M-,
// photons), first-order propensities a_r = k_r X_e:
//   ionization  e -> 2e + M+ ; attachment e -> M- ; photo-emission e -> e + photon.
// Only attachment consumes a reactant, so it is the only reaction that can be
// critical (X_e < N_c).  The hybrid integrator follows the paper's reaction-algorithm
// outline with the SSA exception (A h <= 1) tested before the critical time is drawn
// (ordering of Cao, Gillespie and Petzold 2006); a rejected leap halves the step.
// A pure tau-leaping mode (eq. tau_leaping) is selectable.
//
// With recombination (rows 3 and 4 of the table: e + M+ and M- + M+, second order) the
// step runs the five-reaction code of kmc_device.hpp on every occupied cell, and a
// second kernel takes the cells that hold ions of both signs but no electrons, where
// only ion-ion recombination can fire.
#include <math.h>

#include "device.hpp"
#include "itk.hpp"
#include "kmc_device.hpp"
#include "poisson.hpp"

namespace itk {

namespace {

// Rates from |E| at the cell centre (local field approximation).
__device__ void rates_from_field(const FieldRates& fr, const double e[3], double k[3]) {
  const double Em = sqrt(e[0] * e[0] + e[1] * e[1] + e[2] * e[2]);
  const double Ec = Em > fr.E_floor ? Em : fr.E_floor;
  const double mu = fr.mu_a * pow(Ec / fr.mu_E0, fr.mu_b);
  const double alpha = Em > 0.0 ? fr.alpha_A * exp(-fr.alpha_B / Em) : 0.0;
  const double v = mu * Em;
  k[0] = alpha * v;
  k[1] = fr.eta * v;
  k[2] = fr.kgamma_ratio * k[0];
}

// Rates of the five-reaction network (recombination on) from |E| at the cell centre:
// the three above, k_ep = beta_ep T_e^b / dV with T_e = max(300 K, Te_a (E/E0)^Te_b),
// and k_np = beta_np / dV.
__device__ void rates5_from_field(const FieldRates& fr, const double e[3], double k[5]) {
  rates_from_field(fr, e, k);
  const double Em = sqrt(e[0] * e[0] + e[1] * e[1] + e[2] * e[2]);
  k[3] = 0.0;
  if (fr.beta_ep > 0.0) {
    const double Ec = Em > fr.E_floor ? Em : fr.E_floor;
    const double Te = fmax(300.0, fr.Te_a * pow(Ec / fr.mu_E0, fr.Te_b));
    k[3] = fr.beta_ep * pow(Te, fr.beta_ep_b) / fr.dV;
  }
  k[4] = fr.beta_np > 0.0 ? fr.beta_np / fr.dV : 0.0;
}

__device__ __forceinline__ void load_field(const FieldRates& fr, uint32_t c, double e[3]) {
  if (fr.is_double) {
    for (int a = 0; a < 3; ++a) e[a] = reinterpret_cast<const double*>(fr.E4)[4 * (size_t)c + a];
  } else {
    for (int a = 0; a < 3; ++a) e[a] = (double)reinterpret_cast<const float*>(fr.E4)[4 * (size_t)c + a];
  }
}

// Step kernels: occupied cells from the binning pass.  Each writes the per-cell
// fires, the updated ions and pending photons, the net electron change, clears the
// cell's bin accumulator, queues cells for the coupling pass and reserves the bank
// slots of their products.  The fast pass (kFast) takes every occupied cell and
// settles those whose step is a single SSA excursion with a small register footprint;
// it queues the rest, untouched, for the full pass (!kFast), which runs the complete
// method from the same state and stream (with the rates the fast pass computed).
// A thread takes kKmcPer cells between the workgroup-aggregated appends to the queues, and
// fewer where the launch has threads for that: a small launch is as long as one thread's
// chain of excursions (a 32^3 avalanche: 15.7 -> 10.9 us, 128^3: 19.1 -> 15.6 us).
constexpr int kKmcPer = 4;

template <bool kFast>
__global__ void __launch_bounds__(kFast ? 256 : 64) k_kmc_step(
    KmcParams P, StepConst K, Counters* ctr, const uint32_t* occ, unsigned long long* cellacc,
    uint32_t* nplus, uint32_t* nminus, uint32_t* ngamma, uint32_t* occ_fires, int32_t* dN,
    uint32_t* work, uint32_t* cbase, uint32_t* heavy, double* rates, FieldRates fr,
    int queue_all, int n_new, int dest) {
  if (ctr->halt) return;
  __shared__ uint32_t sh[18];
  const uint32_t n = kFast ? ctr->n_occ : ctr->n_heavy;
  const uint32_t all = gridDim.x * blockDim.x;
  const uint32_t per = n >= kKmcPer * all ? (uint32_t)kKmcPer : (n + all - 1) / all;
  const uint32_t span = blockDim.x * per;
  uint64_t t0 = 0, t1 = 0, t2 = 0;
  for (uint32_t base = blockIdx.x * span; base < n; base += gridDim.x * span) {
    uint32_t js[kKmcPer], Ms[kKmcPer], fl[kKmcPer];  // fl: 1 queue, 2 defer
    uint32_t nq = 0, nd = 0, nm = 0;
    // the words of the thread's cells are read first, all in flight together: the
    // cell indices, then each cell's counts and field (or the rates kept for it)
    // (indices past the end are clamped to the last cell, whose words are then unused,
    // so that no load is conditional)
    uint32_t cs[kKmcPer], xe0[kKmcPer], xp0[kKmcPer], xm0[kKmcPer];
    double kv[kKmcPer][3];
#pragma unroll
    for (int r = 0; r < kKmcPer; ++r) {
      const uint32_t jj = base + (uint32_t)r * blockDim.x + threadIdx.x;
      const uint32_t jc = jj < n ? jj : n - 1;
      js[r] = kFast ? jc : heavy[jc];
    }
#pragma unroll
    for (int r = 0; r < kKmcPer; ++r) cs[r] = occ[js[r]];
#pragma unroll
    for (int r = 0; r < kKmcPer; ++r) {
      xe0[r] = (uint32_t)cellacc[cs[r]];
      xp0[r] = nplus[cs[r]];
      xm0[r] = nminus[cs[r]];
    }
    if (fr.E4 && kFast && fr.is_double) {
#pragma unroll
      for (int r = 0; r < kKmcPer; ++r)
        for (int a = 0; a < 3; ++a) kv[r][a] = reinterpret_cast<const double*>(fr.E4)[4 * (size_t)cs[r] + a];
    } else if (fr.E4 && kFast) {
#pragma unroll
      for (int r = 0; r < kKmcPer; ++r)
        for (int a = 0; a < 3; ++a) kv[r][a] = (double)reinterpret_cast<const float*>(fr.E4)[4 * (size_t)cs[r] + a];
    } else if (fr.E4) {
#pragma unroll
      for (int r = 0; r < kKmcPer; ++r)
        for (int a = 0; a < 3; ++a) kv[r][a] = rates[3 * (size_t)js[r] + a];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < kKmcPer; ++r) {
      const uint32_t jj = base + (uint32_t)r * blockDim.x + threadIdx.x;
      Ms[r] = 0; fl[r] = 0;
      if (r >= (int)per || jj >= n) continue;
      const uint32_t j = js[r];
      const uint32_t c = cs[r];
      const uint32_t Xe = xe0[r];
      State X{(int64_t)Xe, (int64_t)xp0[r], (int64_t)xm0[r], 0};
      double k[3];
      if (!fr.E4) { k[0] = K.k[0]; k[1] = K.k[1]; k[2] = K.k[2]; }
      else if (kFast) rates_from_field(fr, kv[r], k);
      else { k[0] = kv[r][0]; k[1] = kv[r][1]; k[2] = kv[r][2]; }
      CellStream st;
      st.init(c, K.step, TAG_KMC, 0, K.key);
      int64_t f[3];
      if (kFast) {
        if (!advance_fast(P, X, k, K.dt, st, f)) {
          fl[r] = 2; ++nd;
          if (fr.E4) {
            rates[3 * (size_t)j] = k[0]; rates[3 * (size_t)j + 1] = k[1]; rates[3 * (size_t)j + 2] = k[2];
          }
          continue;
        }
      } else {
        advance(P, X, k, K.dt, st, f);
      }
      cellacc[c] = 0ull;
      occ_fires[3 * (size_t)j] = (uint32_t)f[0];
      occ_fires[3 * (size_t)j + 1] = (uint32_t)f[1];
      occ_fires[3 * (size_t)j + 2] = (uint32_t)f[2];
      nplus[c] = (uint32_t)X.p;
      nminus[c] = (uint32_t)X.m;
      ngamma[c] = (uint32_t)X.g;
      const int64_t d = X.e - (int64_t)Xe;
      dN[j] = (int32_t)d;
      if (queue_all || d != 0) { fl[r] = 1; ++nq; }
      if (d > 0) { Ms[r] = d < (int64_t)n_new ? (uint32_t)d : (uint32_t)n_new; nm += Ms[r]; }
      t0 += (uint64_t)f[0]; t1 += (uint64_t)f[1]; t2 += (uint64_t)f[2];
    }
    uint32_t hb = kFast ? block_append(&ctr->n_heavy, nd, sh) : 0u;
    uint32_t qb = block_append(&ctr->n_work, nq, sh);
    uint32_t mb = block_append(&ctr->n[dest], nm, sh);  // bank slots of the products
#pragma unroll
    for (int r = 0; r < kKmcPer; ++r) {
      if (fl[r] == 2) heavy[hb++] = js[r];
      if (fl[r] == 1) work[qb++] = js[r];
      if (Ms[r]) { cbase[js[r]] = mb; mb += Ms[r]; }
    }
  }
  t0 = wave_sum64(t0); t1 = wave_sum64(t1); t2 = wave_sum64(t2);
  if (lane_id() == 0) {
    tally_add(ctr, T_FIRES, t0);
    tally_add(ctr, T_FIRES + 1, t1);
    tally_add(ctr, T_FIRES + 2, t2);
    tally_add(ctr, T_EMITTED, t2);
  }
}

// The step with recombination: every occupied cell through the five-reaction code, one
// cell per lane (the ion-only cells follow in k_kmc_ions, launched before this kernel
// clears the bin accumulators it reads).
__global__ void __launch_bounds__(64) k_kmc_step_rec(
    KmcParams P, StepConst K, Counters* ctr, const uint32_t* occ, unsigned long long* cellacc,
    uint32_t* nplus, uint32_t* nminus, uint32_t* ngamma, uint32_t* occ_fires, int32_t* dN,
    uint32_t* work, uint32_t* cbase, FieldRates fr, int queue_all, int n_new, int dest) {
  if (ctr->halt) return;
  __shared__ uint32_t sh[18];
  const uint32_t n = ctr->n_occ;
  uint64_t t[5] = {0, 0, 0, 0, 0};
  for (uint32_t base = blockIdx.x * blockDim.x; base < n; base += gridDim.x * blockDim.x) {
    const uint32_t j = base + threadIdx.x;
    uint32_t M = 0;
    bool q = false;
    if (j < n) {
      const uint32_t c = occ[j];
      const uint32_t Xe = (uint32_t)cellacc[c];
      State5 X{{(int64_t)Xe, (int64_t)nplus[c], (int64_t)nminus[c], 0}};
      double k[5];
      if (!fr.E4) {
        for (int r = 0; r < 5; ++r) k[r] = K.k[r];
      } else {
        double e[3];
        load_field(fr, c, e);
        rates5_from_field(fr, e, k);
      }
      CellStream st;
      st.init(c, K.step, TAG_KMC, 0, K.key);
      int64_t f[5];
      advance5(P, X, k, K.dt, st, f);
      cellacc[c] = 0ull;
      occ_fires[3 * (size_t)j] = (uint32_t)f[0];
      occ_fires[3 * (size_t)j + 1] = (uint32_t)f[1];
      occ_fires[3 * (size_t)j + 2] = (uint32_t)f[2];
      nplus[c] = (uint32_t)X.x[1];
      nminus[c] = (uint32_t)X.x[2];
      ngamma[c] = (uint32_t)X.x[3];
      const int64_t d = X.x[0] - (int64_t)Xe;
      dN[j] = (int32_t)d;
      q = queue_all || d != 0;
      if (d > 0) M = d < (int64_t)n_new ? (uint32_t)d : (uint32_t)n_new;
      for (int r = 0; r < 5; ++r) t[r] += (uint64_t)f[r];
    }
    const uint32_t qb = block_append(&ctr->n_work, q ? 1u : 0u, sh);
    const uint32_t mb = block_append(&ctr->n[dest], M, sh);  // bank slots of the products
    if (q) work[qb] = j;
    if (M) cbase[j] = mb;
  }
  for (int r = 0; r < 5; ++r) t[r] = wave_sum64(t[r]);
  if (lane_id() == 0) {
    for (int r = 0; r < 5; ++r) tally_add(ctr, T_FIRES + r, t[r]);
    tally_add(ctr, T_EMITTED, t[2]);
  }
}

// Cells without electrons this step (bin count 0) that hold ions of both signs: ion-ion
// recombination, the only reaction that can fire there, by the same five-reaction code
// and the cell's own stream.
__global__ void __launch_bounds__(256) k_kmc_ions(KmcParams P, StepConst K, Counters* ctr,
                                                  const unsigned long long* cellacc, uint32_t* nplus,
                                                  uint32_t* nminus, FieldRates fr) {
  if (ctr->halt) return;
  uint64_t t4 = 0;
  for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < K.ncell; c += gridDim.x * blockDim.x) {
    const uint32_t p0 = nplus[c], m0 = nminus[c];
    if (p0 == 0 || m0 == 0 || (cellacc[c] >> 32) != 0) continue;
    State5 X{{0, (int64_t)p0, (int64_t)m0, 0}};
    double k[5];
    if (!fr.E4) {
      for (int r = 0; r < 5; ++r) k[r] = K.k[r];
    } else {
      double e[3];
      load_field(fr, c, e);
      rates5_from_field(fr, e, k);
    }
    CellStream st;
    st.init(c, K.step, TAG_KMC, 0, K.key);
    int64_t f[5];
    advance5(P, X, k, K.dt, st, f);
    nplus[c] = (uint32_t)X.x[1];
    nminus[c] = (uint32_t)X.x[2];
    t4 += (uint64_t)f[4];
  }
  t4 = wave_sum64(t4);
  if (lane_id() == 0) tally_add(ctr, T_FIRES + 4, t4);
}

// Independent cells (unit parity): the three-reaction code when both recombination
// rates of the cell are zero, the five-reaction code otherwise.
__global__ void __launch_bounds__(256, 2) k_kmc_cells(KmcParams P, Key key, uint64_t n, const uint32_t* ids, int64_t* Xa,
                            const double* ka, double dt, uint32_t step, int64_t* fa) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    CellStream st;
    st.init(ids[i], step, TAG_KMC, 0, key);
    if (ka[5 * i + 3] == 0.0 && ka[5 * i + 4] == 0.0) {
      State X{Xa[4 * i], Xa[4 * i + 1], Xa[4 * i + 2], Xa[4 * i + 3]};
      const double k[3] = {ka[5 * i], ka[5 * i + 1], ka[5 * i + 2]};
      int64_t f[3];
      advance(P, X, k, dt, st, f);
      Xa[4 * i] = X.e; Xa[4 * i + 1] = X.p; Xa[4 * i + 2] = X.m; Xa[4 * i + 3] = X.g;
      fa[5 * i] = f[0]; fa[5 * i + 1] = f[1]; fa[5 * i + 2] = f[2]; fa[5 * i + 3] = 0; fa[5 * i + 4] = 0;
    } else {
      State5 X{{Xa[4 * i], Xa[4 * i + 1], Xa[4 * i + 2], Xa[4 * i + 3]}};
      double k[5];
      for (int r = 0; r < 5; ++r) k[r] = ka[5 * i + r];
      int64_t f[5];
      advance5(P, X, k, dt, st, f);
      for (int a = 0; a < 4; ++a) Xa[4 * i + a] = X.x[a];
      for (int r = 0; r < 5; ++r) fa[5 * i + r] = f[r];
    }
  }
}

int blocks_for(uint64_t n, int per_block, int max_blocks) {
  uint64_t b = (n + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > (uint64_t)max_blocks) b = max_blocks;
  return (int)b;
}

// Zero-dimensional reactors: nsteps steps per reactor in one launch, each reactor with
// its own key (seed, realization) and stream cell id; X stays in registers.
//
// The steps of one reactor are a serial chain, but the first word of a step's stream
// depends only on the step, and most steps of the hybrid method are one SSA excursion
// whose first waiting time already ends beyond the step (ssa_reach): nothing changes.  A
// thread therefore draws the first words of kRunBatch steps together (independent Philox
// chains in flight), skips the quiet ones by comparing their exponents with the
// threshold of the present state, and runs the method only for the others, one at a time.
// Bound by the Philox rounds (about 110 VALU instructions per step and wavefront): 10^6
// reactors x 50 steps at 10 MV/m 1.96 -> 0.29 ms, 4096 x 275 steps 0.69 -> 0.106 ms (one
// step at a time, with a double logarithm and two divisions each, before; the compiler's
// 128-register default for unbounded launches also spilled 884 bytes a lane).
constexpr int kRunBatch = 8;

// Threshold of a quiet step from state X: the first exponent beyond it leaves the state as
// it is.  -inf if nothing can fire, +inf if the step is not one SSA excursion.
__device__ __forceinline__ float quiet_reach(const KmcParams& P, const State& X, const double k[3], double dt) {
  const double a1 = k[0] * (double)X.e, a2 = k[1] * (double)X.e, a3 = k[2] * (double)X.e;
  const double A = a1 + a2 + a3;
  if (!(A > 0.0)) return -INFINITY;
  if (P.mode != ITOKMC_KMC_HYBRID) return INFINITY;
  const bool crit2 = (a2 > 0.0) && X.e < (int64_t)P.nc;
  const double h = fmin(dt, leap_bound(P, X, a1, a2, a3, crit2));
  if (h != dt || !(A * h <= 1.0)) return INFINITY;
  return ssa_reach(A, h);
}

// One wavefront per workgroup: a few thousand reactors then spread over every CU.
__global__ void __launch_bounds__(64, 2) k_kmc_run(KmcParams P, uint32_t seed, uint32_t real0, uint64_t n,
                                                    const uint32_t* ids, const uint32_t* real,
                                                    const uint32_t* nst, int64_t* Xa, const double* ka,
                                                    double dt, uint32_t step0, uint32_t nsteps0, int64_t* fa) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const Key key{seed, real ? real[i] : real0};
    const uint32_t id = ids[i];
    const uint64_t want = nst ? nst[i] : nsteps0;
    const uint32_t nsteps = (uint32_t)(want < 0x100000000ull - step0 ? want : 0x100000000ull - step0);
    int64_t F[5] = {0, 0, 0, 0, 0};
    if (ka[5 * i + 3] == 0.0 && ka[5 * i + 4] == 0.0) {
      State X{Xa[4 * i], Xa[4 * i + 1], Xa[4 * i + 2], Xa[4 * i + 3]};
      const double k[3] = {ka[5 * i], ka[5 * i + 1], ka[5 * i + 2]};
      float reach = quiet_reach(P, X, k, dt);
      for (uint32_t s0 = 0; s0 < nsteps;) {
        float ex[kRunBatch];
#pragma unroll
        for (int q = 0; q < kRunBatch; ++q)
          ex[q] = ssa_exponent(philox_block(id, 0, step0 + s0 + (uint32_t)q, TAG_KMC, 0, key).x);
        const uint32_t left = nsteps - s0;
        const uint32_t in = left < (uint32_t)kRunBatch ? (1u << left) - 1u : (1u << kRunBatch) - 1u;
        uint32_t todo = in;  // steps of the batch not yet passed
        for (;;) {
          uint32_t loud = 0;
#pragma unroll
          for (int q = 0; q < kRunBatch; ++q) loud |= ex[q] > reach ? 0u : (1u << q);
          loud &= todo;
          if (loud == 0u) break;
          const uint32_t q = (uint32_t)__ffs((int)loud) - 1u;
          todo &= ~((2u << q) - 1u);
          CellStream st;
          st.init(id, step0 + s0 + q, TAG_KMC, 0, key);
          int64_t f[3];
          State Y = X;
          if (advance_fast(P, Y, k, dt, st, f)) {
            X = Y;
          } else {
            st.init(id, step0 + s0 + q, TAG_KMC, 0, key);
            advance(P, X, k, dt, st, f);
          }
          F[0] += f[0]; F[1] += f[1]; F[2] += f[2];
          reach = quiet_reach(P, X, k, dt);
        }
        s0 += left < (uint32_t)kRunBatch ? left : (uint32_t)kRunBatch;
      }
      Xa[4 * i] = X.e; Xa[4 * i + 1] = X.p; Xa[4 * i + 2] = X.m; Xa[4 * i + 3] = X.g;
    } else {
      State5 X{{Xa[4 * i], Xa[4 * i + 1], Xa[4 * i + 2], Xa[4 * i + 3]}};
      double k[5];
      for (int r = 0; r < 5; ++r) k[r] = ka[5 * i + r];
      for (uint32_t s = 0; s < nsteps; ++s) {
        CellStream st;
        st.init(id, step0 + s, TAG_KMC, 0, key);
        int64_t f[5];
        advance5(P, X, k, dt, st, f);
        for (int r = 0; r < 5; ++r) F[r] += f[r];
      }
      for (int a = 0; a < 4; ++a) Xa[4 * i + a] = X.x[a];
    }
    for (int r = 0; r < 5; ++r) fa[5 * i + r] = F[r];
  }
}

// Device-side stop rule of a run (itokmc_step_until): a run stops after the first step
// that began with at least stop_particles live particles (the push counts them).
static_assert(kTallyLines == 64, "one lane per tally line");
__device__ __forceinline__ unsigned long long pushed_total(const Counters* ctr) {
  return wave_sum64(ctr->tally[lane_id()].v[T_PUSHED]);
}
// One wavefront each.
__global__ void __launch_bounds__(64) k_stop_begin(Counters* ctr) {
  const unsigned long long pushed = pushed_total(ctr);
  if (lane_id()) return;
  ctr->halt = 0u;
  ctr->steps_done = 0u;
  ctr->pushed_mark = pushed;
}
__global__ void __launch_bounds__(64) k_stop_step(Counters* ctr, uint64_t stop_particles) {
  if (ctr->halt) return;
  const unsigned long long pushed = pushed_total(ctr);
  if (lane_id()) return;
  ctr->steps_done += 1u;
  const unsigned long long live = pushed - ctr->pushed_mark;
  ctr->pushed_mark = pushed;
  if (stop_particles && live >= stop_particles) ctr->halt = 1u;
}
__global__ void k_stop_end(Counters* ctr) { ctr->halt = 0u; }

KmcParams params(const itokmc_ctx* ctx) {
  return KmcParams{ctx->d.kmc_mode, ctx->d.kmc_nc, ctx->d.kmc_nssa, ctx->d.kmc_eps};
}

}  // namespace

hipError_t launch_kmc_step(itokmc_ctx* ctx, const StepConst& k, const FieldRates& fr) {
  if (recombination(ctx)) {
    const int qa = ctx->d.n_ppc > 0 ? 1 : 0, dest = 1 - ctx->cur;
    if (ctx->c.beta_np > 0.0) {
      k_kmc_ions<<<blocks_for(ctx->ncell, 256, 8192), 256, 0, ctx->s>>>(params(ctx), k, ctx->ctr, ctx->cellacc,
                                                                    ctx->nplus, ctx->nminus, fr);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    k_kmc_step_rec<<<blocks_for(ctx->ncell, 64, 8192), 64, 0, ctx->s>>>(
        params(ctx), k, ctx->ctr, ctx->occ, ctx->cellacc, ctx->nplus, ctx->nminus, ctx->ngamma,
        ctx->occ_fires, ctx->dN, ctx->work, ctx->cbase, fr, qa, ctx->d.n_new, dest);
    return hipGetLastError();
  }
  // at most 512 workgroups (two per CU), each looping over its share of the occupied
  // cells: 0.197 ms per step at 5.5e7 particles in 7e6 cells against 0.306 with 256 and
  // 0.202 with 1024; 0.215 against 0.307 and 0.219 at 4.5e7 in 3e6
  int g = (int)((ctx->ncell + 255) / 256);
  if (g > 512) g = 512;
  if (g < 1) g = 1;
  const int qa = ctx->d.n_ppc > 0 ? 1 : 0, dest = 1 - ctx->cur;
  k_kmc_step<true><<<g, 256, 0, ctx->s>>>(params(ctx), k, ctx->ctr, ctx->occ, ctx->cellacc, ctx->nplus,
                                          ctx->nminus, ctx->ngamma, ctx->occ_fires, ctx->dN, ctx->work,
                                          ctx->cbase, ctx->heavy, ctx->rates, fr, qa, ctx->d.n_new, dest);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  int gh = (int)((ctx->ncell + 63) / 64);
  if (gh > 4096) gh = 4096;
  if (gh < 1) gh = 1;
  k_kmc_step<false><<<gh, 64, 0, ctx->s>>>(params(ctx), k, ctx->ctr, ctx->occ, ctx->cellacc, ctx->nplus,
                                           ctx->nminus, ctx->ngamma, ctx->occ_fires, ctx->dN, ctx->work,
                                           ctx->cbase, ctx->heavy, ctx->rates, fr, qa, ctx->d.n_new, dest);
  return hipGetLastError();
}

hipError_t launch_stop_begin(itokmc_ctx* ctx) {
  k_stop_begin<<<1, 64, 0, ctx->s>>>(ctx->ctr);
  return hipGetLastError();
}
hipError_t launch_stop_step(itokmc_ctx* ctx, uint64_t stop_particles) {
  k_stop_step<<<1, 64, 0, ctx->s>>>(ctx->ctr, stop_particles);
  return hipGetLastError();
}
hipError_t launch_stop_end(itokmc_ctx* ctx) {
  k_stop_end<<<1, 1, 0, ctx->s>>>(ctx->ctr);
  return hipGetLastError();
}

hipError_t launch_kmc_run(itokmc_ctx* ctx, uint64_t n, const uint32_t* ids, const uint32_t* real,
                          const uint32_t* nst, int64_t* X, const double* k, double dt, uint32_t step0,
                          uint32_t nsteps, int64_t* fires) {
  k_kmc_run<<<blocks_for(n, 64, 32768), 64, 0, ctx->s>>>(params(ctx), ctx->d.seed, ctx->d.realization,
                                                         n, ids, real, nst, X, k, dt, step0, nsteps,
                                                         fires);
  return hipGetLastError();
}

hipError_t launch_kmc_cells(itokmc_ctx* ctx, uint64_t n, const uint32_t* ids, int64_t* X,
                            const double* k, double dt, uint32_t step, int64_t* fires) {
  int g = (int)((n + 255) / 256);
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  k_kmc_cells<<<g, 256, 0, ctx->s>>>(params(ctx), Key{ctx->d.seed, ctx->d.realization}, n, ids, X,
                                     k, dt, step, fires);
  return hipGetLastError();
}

}  // namespace itk
