// Counting sort of particles by cell, as a kernel-level entry point: the binning step
// that groups each cell's computational particles (the per-cell particle lists that the
// reactions and the superparticle pass of the paper's final algorithm work on).
//
//   count:   per live particle (w > 0), a run-aggregated atomic on its cell's counter
//            returns the particle's rank inside the cell;
//   scan:    exclusive prefix of the counters over all cells gives start[0 .. ncell];
//   scatter: particle i goes to start[cell] + rank (no atomics).
// Within a cell the order is that of the counting atomics (unspecified).
//
// Small sorts (kSortOneN particles, kSortOneCells cells) take one launch of one workgroup
// with the counters in LDS instead of these six.
//
// Scratch (32-bit words): the per-cell counters [ncell], the ranks [n] and the scan's
// block partials.  itokmc_sort_by_cell takes it from a caller workspace;
// itokmc_sort_by_cell_noalloc from a file-scope device array (one per GPU, resolved once
// per device with hipGetSymbolAddress), for callers that cannot allocate.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "device.hpp"
#include "itk.hpp"

namespace itk {
namespace {

constexpr int kSortBlock = 256;
constexpr int kSortPer = 8;                          // cells per thread in the scan
constexpr uint32_t kSortTile = kSortBlock * kSortPer;  // cells per scan block
constexpr int kSortTopThreads = 1024;

// Words of scratch for n particles and ncell cells.
inline uint64_t sort_words(uint64_t n, uint64_t ncell) {
  const uint64_t nblk = (ncell + kSortTile - 1) / kSortTile;
  auto al = [](uint64_t w) { return (w + 63) & ~(uint64_t)63; };  // 256-byte alignment
  return al(ncell) + al(n) + al(nblk + 2);
}

__global__ void k_sort_fill(uint32_t* p, uint32_t n) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

// Run-aggregated 32-bit atomic increment: lanes whose keys form a run (particles are
// usually grouped by cell already) take one atomic per run; each active lane gets the
// counter's value before its own increment.
__device__ __forceinline__ uint32_t run_inc(uint32_t* acc, uint32_t key) {
  const int lane = lane_id();
  const bool active = key != kInvalidCell;
  const uint32_t prev = __shfl_up(key, 1, 64);
  const bool head = lane == 0 || prev != key;
  const uint64_t heads = __ballot(head);
  const uint64_t upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
  const int seg_start = 63 - __clzll(heads & upto);
  const uint64_t after = heads & ~upto;
  const int seg_end = after ? (__ffsll((long long)after) - 2) : 63;
  uint32_t old = 0;
  if (active && lane == seg_end) old = atomicAdd(&acc[key], (uint32_t)(seg_end - seg_start + 1));
  old = __shfl(old, seg_end, 64);
  return old + (uint32_t)(lane - seg_start);
}

// A particle with w == 0 or a cell index outside [0, ncell) is dropped.
__global__ void __launch_bounds__(kSortBlock) k_sort_count(const uint32_t* cell, const uint32_t* w,
                                                          uint32_t n, uint32_t ncell, uint32_t* counts,
                                                          uint32_t* rank) {
  for (uint32_t base = blockIdx.x * blockDim.x; base < n; base += gridDim.x * blockDim.x) {
    const uint32_t i = base + threadIdx.x;
    uint32_t key = kInvalidCell;
    if (i < n && w[i] > 0) {
      const uint32_t c = cell[i];
      key = c < ncell ? c : kInvalidCell;
    }
    const uint32_t r = run_inc(counts, key);
    if (key != kInvalidCell) rank[i] = r;
  }
}

// Exclusive block scan of one value per thread (kSortBlock threads); *total gets the sum.
__device__ __forceinline__ uint32_t sort_block_scan(uint32_t v, uint32_t* sh, uint32_t* total) {
  const int lane = lane_id(), wid = threadIdx.x >> 6;
  constexpr int nw = kSortBlock / 64;
  uint32_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) sh[wid] = x;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < nw; ++k) {
    const uint32_t s = sh[k];
    off += k < wid ? s : 0u;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return off + x - v;
}

__global__ void __launch_bounds__(kSortBlock) k_sort_scan_blocks(const uint32_t* counts, uint32_t ncell,
                                                                uint32_t* part) {
  __shared__ uint32_t sh[kSortBlock / 64];
  const uint32_t nblk = (ncell + kSortTile - 1) / kSortTile;
  for (uint32_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    uint32_t v = 0;
#pragma unroll
    for (int j = 0; j < kSortPer; ++j) {
      const uint32_t c = b * kSortTile + (uint32_t)j * kSortBlock + threadIdx.x;
      v += c < ncell ? counts[c] : 0u;
    }
    uint32_t tot;
    sort_block_scan(v, sh, &tot);
    if (threadIdx.x == 0) part[b] = tot;
  }
}

// One workgroup: exclusive scan of the block partials in place; part[nblk] = total.
__global__ void __launch_bounds__(kSortTopThreads) k_sort_scan_top(uint32_t* part, uint32_t nblk,
                                                                  uint32_t* n_out) {
  __shared__ uint32_t sh[kSortTopThreads / 64];
  __shared__ uint32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  const int lane = lane_id(), wid = threadIdx.x >> 6;
  for (uint32_t b0 = 0; b0 < nblk; b0 += kSortTopThreads) {
    const uint32_t b = b0 + threadIdx.x;
    const uint32_t v = b < nblk ? part[b] : 0u;
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) sh[wid] = x;
    __syncthreads();
    uint32_t off = carry, tot = 0;
    for (int k = 0; k < kSortTopThreads / 64; ++k) {
      const uint32_t s = sh[k];
      off += k < wid ? s : 0u;
      tot += s;
    }
    if (b < nblk) part[b] = off + x - v;
    __syncthreads();
    if (threadIdx.x == 0) carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[nblk] = carry;
    *n_out = carry;
  }
}

__global__ void __launch_bounds__(kSortBlock) k_sort_scan_down(const uint32_t* counts, uint32_t ncell,
                                                              const uint32_t* part, uint32_t* start) {
  __shared__ uint32_t sh[kSortBlock / 64];
  __shared__ __align__(16) uint32_t tile[kSortTile];
  const uint32_t nblk = (ncell + kSortTile - 1) / kSortTile;
  for (uint32_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    const uint32_t cb = b * kSortTile;
    // coalesced loads through LDS, then eight consecutive cells per thread
#pragma unroll
    for (int j = 0; j < kSortPer; ++j) {
      const uint32_t i = (uint32_t)j * kSortBlock + threadIdx.x;
      tile[i] = cb + i < ncell ? counts[cb + i] : 0u;
    }
    __syncthreads();
    uint32_t v[kSortPer], s = 0;
#pragma unroll
    for (int j = 0; j < kSortPer; ++j) { v[j] = tile[threadIdx.x * kSortPer + j]; s += v[j]; }
    uint32_t tot;
    uint32_t p = sort_block_scan(s, sh, &tot) + part[b];
#pragma unroll
    for (int j = 0; j < kSortPer; ++j) {
      const uint32_t c = cb + threadIdx.x * kSortPer + (uint32_t)j;
      if (c < ncell) start[c] = p;
      p += v[j];
    }
    __syncthreads();
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) start[ncell] = part[nblk];
}

template <typename T>
__global__ void __launch_bounds__(kSortBlock) k_sort_scatter(const uint32_t* cell, const T* ox, const T* oy,
                                                            const T* oz, const uint32_t* w,
                                                            const uint64_t* id, uint32_t n, uint32_t ncell,
                                                            const uint32_t* start, const uint32_t* rank,
                                                            uint32_t* cell_o, T* ox_o, T* oy_o, T* oz_o,
                                                            uint32_t* w_o, uint64_t* id_o) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t wi = w[i];
    const uint32_t c = cell[i];
    if (wi == 0 || c >= ncell) continue;
    const uint32_t q = start[c] + rank[i];
    cell_o[q] = c;
    ox_o[q] = ox[i];
    oy_o[q] = oy[i];
    oz_o[q] = oz[i];
    w_o[q] = wi;
    id_o[q] = id[i];
  }
}

// The whole sort in one workgroup: the counters in LDS (a spare word every 32, so that the
// scan's threads, a run of consecutive cells each, start in different banks), a thread's
// particles in registers between the count and the scatter.  The six launches are bound by
// launch latency (2-5 us each for a few hundred KB of traffic); one workgroup is bound by
// the latency of its phases and what one CU can load and store.  3001 particles, 32768
// cells, double: 25.0 -> 12.1 us a call in a stream of calls, 30.1 -> 24.8 us waited for.
//
// Up to 3072 particles go straight to their slots.  In any order that costs what the six
// launches do at most (3001 in random order 18.4 us, 29.8 waited for); of more, random
// slots are a line for every store and one CU (6144 25.9 us, 41.2 waited for).  So the arrays
// of up to 6144 go through LDS one after another, which takes 1 us more of nearly sorted
// particles (6144 17.6 us, 28.9 waited for) and the same of random ones (18.0 and 29.3).  The
// lines: 8192 particles waited for 31.3 against 29.7 us, and the counters of 36864 cells are
// what LDS holds.
constexpr int kSortOnePer = 6;  // particles per thread (3 if they go straight)
constexpr uint32_t kSortOneN = 1024 * kSortOnePer;
constexpr uint32_t kSortOneStraight = kSortOneN / 2;
constexpr uint32_t kSortOneCells = 36 << 10;
__host__ __device__ constexpr uint32_t sort_one_word(uint32_t c) { return c + (c >> 5); }

template <typename T, bool kStraight>
__global__ void __launch_bounds__(1024) k_sort_one(const uint32_t* cell, const T* ox, const T* oy, const T* oz,
                                                   const uint32_t* w, const uint64_t* id, uint32_t n,
                                                   uint32_t ncell, uint32_t* cell_o, T* ox_o, T* oy_o,
                                                   T* oz_o, uint32_t* w_o, uint64_t* id_o, uint32_t* start,
                                                   uint32_t* n_out) {
  extern __shared__ __align__(16) uint32_t cnt[];
  __shared__ uint32_t sh[1024 / 64];
  constexpr int kPer = kStraight ? kSortOnePer / 2 : kSortOnePer;
  const uint32_t tid = threadIdx.x;
  uint32_t key[kPer], wi[kPer], rank[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint32_t i = tid + 1024u * q;
    wi[q] = i < n ? w[i] : 0u;
    key[q] = i < n ? cell[i] : kInvalidCell;
  }
  for (uint32_t t = tid; t <= sort_one_word(ncell - 1) / 4; t += 1024)
    reinterpret_cast<uint4*>(cnt)[t] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    if (wi[q] == 0u || key[q] >= ncell) key[q] = kInvalidCell;
    rank[q] = key[q] != kInvalidCell ? atomicAdd(&cnt[sort_one_word(key[q])], 1u) : 0u;
  }
  __syncthreads();
  const uint32_t per = (ncell + 1023u) / 1024u, c0 = tid * per, c1 = min(c0 + per, ncell);
  uint32_t s = 0;
#pragma unroll 4
  for (uint32_t c = c0; c < c1; ++c) s += cnt[sort_one_word(c)];
  uint32_t x = s;
  const int lane = lane_id(), wid = tid >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) sh[wid] = x;
  __syncthreads();
  uint32_t p = x - s, total = 0;
#pragma unroll
  for (int k = 0; k < 1024 / 64; ++k) {
    p += k < wid ? sh[k] : 0u;
    total += sh[k];
  }
  for (uint32_t c = c0; c < c1; c += 4) {
    uint32_t v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = c + j < c1 ? cnt[sort_one_word(c + j)] : 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (c + j < c1) cnt[sort_one_word(c + j)] = p;
      p += v[j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q)  // the particle's slot
    if (key[q] != kInvalidCell) rank[q] += cnt[sort_one_word(key[q])];
  if constexpr (kStraight) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (key[q] == kInvalidCell) continue;
      const uint32_t i = tid + 1024u * q, to = rank[q];
      cell_o[to] = key[q];
      ox_o[to] = ox[i];
      oy_o[to] = oy[i];
      oz_o[to] = oz[i];
      w_o[to] = wi[q];
      id_o[to] = id[i];
    }
  }
#pragma unroll 8
  for (uint32_t c = tid; c < ncell; c += 1024) start[c] = cnt[sort_one_word(c)];
  if constexpr (!kStraight) {
    // through the counters' space, once they are read
    const auto move = [&](auto* out, auto value) {
      using V = std::remove_pointer_t<decltype(out)>;
      V* const buf = reinterpret_cast<V*>(cnt);
      V v[kPer];
#pragma unroll
      for (int q = 0; q < kPer; ++q) v[q] = key[q] != kInvalidCell ? value(q) : V{};
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kPer; ++q)
        if (key[q] != kInvalidCell) buf[rank[q]] = v[q];
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const uint32_t t = tid + 1024u * q;
        if (t < total) out[t] = buf[t];
      }
    };
    move(cell_o, [&](int q) { return key[q]; });
    move(w_o, [&](int q) { return wi[q]; });
    move(ox_o, [&](int q) { return ox[tid + 1024u * q]; });
    move(oy_o, [&](int q) { return oy[tid + 1024u * q]; });
    move(oz_o, [&](int q) { return oz[tid + 1024u * q]; });
    move(id_o, [&](int q) { return id[tid + 1024u * q]; });
  }
  if (tid == 0) {
    start[ncell] = total;
    *n_out = total;
  }
}

inline int sort_grid(uint64_t n, uint32_t cap) {
  uint64_t b = (n + kSortBlock - 1) / kSortBlock;
  if (b < 1) b = 1;
  return (int)(b > cap ? cap : b);
}

// The sort on a given scratch of at least sort_words(n, ncell) words.
int sort_run(int precision, uint64_t n, uint32_t ncell, const uint32_t* cell, const void* ox,
             const void* oy, const void* oz, const uint32_t* w, const uint64_t* id, uint32_t* cell_o,
             void* ox_o, void* oy_o, void* oz_o, uint32_t* w_o, uint64_t* id_o, uint32_t* start,
             uint32_t* n_out, uint32_t* scratch, hipStream_t s) {
  auto al = [](uint64_t x) { return (x + 63) & ~(uint64_t)63; };
  uint32_t* counts = scratch;
  uint32_t* rank = counts + al(ncell);
  uint32_t* part = rank + al(n);
  const uint32_t nblk = (ncell + kSortTile - 1) / kSortTile;
  const uint32_t nn = (uint32_t)n;
  if (nn <= kSortOneN && ncell <= kSortOneCells) {
    const bool straight = nn <= kSortOneStraight;
    const size_t counters = ((size_t)sort_one_word(ncell - 1) / 4 + 1) * 16;
    const size_t lds = straight ? counters : std::max(counters, (size_t)nn * 8);
    const auto go = [&](auto kern, auto t) {
      using T = decltype(t);
      kern<<<1, 1024, lds, s>>>(cell, (const T*)ox, (const T*)oy, (const T*)oz, w, id, nn, ncell, cell_o, (T*)ox_o,
                                (T*)oy_o, (T*)oz_o, w_o, id_o, start, n_out);
    };
    if (precision == ITOKMC_FP64) {
      if (straight) go(k_sort_one<double, true>, 0.0);
      else go(k_sort_one<double, false>, 0.0);
    } else {
      if (straight) go(k_sort_one<float, true>, 0.0f);
      else go(k_sort_one<float, false>, 0.0f);
    }
    return hipGetLastError() == hipSuccess ? ITOKMC_OK : ITOKMC_EHIP;
  }
  // the counters start from zero on every call (a fill kernel, so that a captured call
  // records no memset node)
  k_sort_fill<<<sort_grid(ncell, 2048), kSortBlock, 0, s>>>(counts, ncell);
  if (nn) k_sort_count<<<sort_grid(n, 8192), kSortBlock, 0, s>>>(cell, w, nn, ncell, counts, rank);
  k_sort_scan_blocks<<<nblk < 4096 ? nblk : 4096, kSortBlock, 0, s>>>(counts, ncell, part);
  k_sort_scan_top<<<1, kSortTopThreads, 0, s>>>(part, nblk, n_out);
  k_sort_scan_down<<<nblk < 4096 ? nblk : 4096, kSortBlock, 0, s>>>(counts, ncell, part, start);
  if (nn) {
    if (precision == ITOKMC_FP64)
      k_sort_scatter<double><<<sort_grid(n, 8192), kSortBlock, 0, s>>>(
          cell, (const double*)ox, (const double*)oy, (const double*)oz, w, id, nn, ncell, start, rank, cell_o,
          (double*)ox_o, (double*)oy_o, (double*)oz_o, w_o, id_o);
    else
      k_sort_scatter<float><<<sort_grid(n, 8192), kSortBlock, 0, s>>>(
          cell, (const float*)ox, (const float*)oy, (const float*)oz, w, id, nn, ncell, start, rank, cell_o,
          (float*)ox_o, (float*)oy_o, (float*)oz_o, w_o, id_o);
  }
  return hipGetLastError() == hipSuccess ? ITOKMC_OK : ITOKMC_EHIP;
}

bool sort_args_ok(int precision, uint64_t n, uint32_t ncell, const void* const* p, int np) {
  if (precision != ITOKMC_FP32 && precision != ITOKMC_FP64) return false;
  if (ncell < 1 || ncell > (1u << 24) || n > 0x7FFFFFFFull) return false;
  for (int i = 0; i < np; ++i)
    if (!p[i] && (n > 0 || i >= np - 2)) return false;  // start and n_out always needed
  return true;
}

// ---- file-scope scratch for the no-allocation entry point --------------------------
constexpr uint64_t kNoAllocScratchBytes = 32ull << 20;
static __device__ __align__(256) uint32_t scratch[kNoAllocScratchBytes / 4];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint32_t* g_scratch_ptr[kMaxDevices] = {nullptr};

// The device address of this GPU's scratch array, resolved once per device with that
// device current (each GPU holds its own copy at its own address).
hipError_t scratch_for_current_device(uint32_t** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = (uint32_t*)p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace
}  // namespace itk

using namespace itk;

extern "C" {

size_t itokmc_sort_workspace_bytes(uint64_t n, uint32_t ncell) {
  if (ncell < 1 || ncell > (1u << 24) || n > 0x7FFFFFFFull) return 0;
  return (size_t)sort_words(n, ncell) * 4;
}

int itokmc_sort_by_cell(int precision, uint64_t n, uint32_t ncell, const uint32_t* cell, const void* ox,
                        const void* oy, const void* oz, const uint32_t* w, const uint64_t* id,
                        uint32_t* cell_out, void* ox_out, void* oy_out, void* oz_out, uint32_t* w_out,
                        uint64_t* id_out, uint32_t* start, uint32_t* n_out, void* workspace,
                        size_t workspace_bytes, void* stream) {
  const void* p[] = {cell, ox, oy, oz, w, id, cell_out, ox_out, oy_out, oz_out, w_out, id_out, start, n_out};
  if (!sort_args_ok(precision, n, ncell, p, 14) || !workspace) return ITOKMC_EINVAL;
  if (workspace_bytes < (size_t)sort_words(n, ncell) * 4) return ITOKMC_ENOMEM;
  return sort_run(precision, n, ncell, cell, ox, oy, oz, w, id, cell_out, ox_out, oy_out, oz_out, w_out,
                  id_out, start, n_out, (uint32_t*)workspace, (hipStream_t)stream);
}

int itokmc_sort_by_cell_noalloc(int precision, uint64_t n, uint32_t ncell, const uint32_t* cell,
                                const void* ox, const void* oy, const void* oz, const uint32_t* w,
                                const uint64_t* id, uint32_t* cell_out, void* ox_out, void* oy_out,
                                void* oz_out, uint32_t* w_out, uint64_t* id_out, uint32_t* start,
                                uint32_t* n_out, void* stream) {
  const void* p[] = {cell, ox, oy, oz, w, id, cell_out, ox_out, oy_out, oz_out, w_out, id_out, start, n_out};
  if (!sort_args_ok(precision, n, ncell, p, 14)) return ITOKMC_EINVAL;
  if ((uint64_t)sort_words(n, ncell) * 4 > kNoAllocScratchBytes) return ITOKMC_ECAPACITY;
  uint32_t* sp = nullptr;
  if (scratch_for_current_device(&sp) != hipSuccess) return ITOKMC_EHIP;
  return sort_run(precision, n, ncell, cell, ox, oy, oz, w, id, cell_out, ox_out, oy_out, oz_out, w_out,
                  id_out, start, n_out, sp, (hipStream_t)stream);
}

}  // extern "C"
