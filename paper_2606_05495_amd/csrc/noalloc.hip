// Vector jobs with no allocation: set_run_vector_jobs_noalloc.
//
// The same bucketed persistent computation as set_run_vector_jobs (per job
// S = sum tanh(a*x + y) over pool windows, split into work items whose size
// is chosen per size bucket floor(log2 n)), for callers that cannot allocate
// device or pinned memory: code under graph capture, tight serving loops.
// Jobs and results are caller-owned device arrays and the call is ordered on
// the caller's stream; the work-item table, the per-item partials and the
// work counter live in one static device array per GPU, whose address is
// looked up once per device.
//
// Short jobs (up to 32767 elements at the default item sizes) take one launch, a
// block to a job (k_vec_short_jobs).
// Other calls of up to kBlock jobs take two launches on the caller's stream, a tile kernel whose
// blocks each plan the call in LDS and the totals; more take three:
//   plan   (one block): validate each job, pick its item size, prefix-sum the
//          tile counts into a descriptor table and rewind the work counter;
//   tiles  (persistent grid): the batch pipeline's (job, tile) kernel;
//   totals (one wave per job): each job's tile partials in a fixed order.
// A job's result depends only on (n, its item size), as on the batch path,
// so both calls give bit-identical sums for the same jobs and tuning.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <string>

#include "kernels.hpp"

namespace setrt {
namespace {

constexpr uint32_t kNaMaxJobs = SET_NOALLOC_MAX_JOBS;
constexpr uint32_t kNaMaxItems = SET_NOALLOC_MAX_ITEMS;
constexpr int kNaPlanThreads = 1024;
constexpr int kNaMaxDevices = 64;
// Blocks of the tile kernel: twice what the device holds at once, so that the
// dispatcher hands most shares out by itself and few are claimed; or as many as
// the call can have tiles (a block without one still plans a small call: 4096
// blocks took one job 14.5 us).  Uneven jobs, us, at 1024 blocks / so: 1024 of up
// to 8192 elements 29.4 / 26.5, of up to 131072 77 / 70, 256 of up to 2^22 201 /
// 195, 2048 of up to 2^22 1550 / 1546, one of up to 8192 14.5 / 12.8.
constexpr uint32_t kNaGrid = 4096;

// Byte offsets inside the static array (each 256-byte aligned).
constexpr uint64_t kNaHdrOff = 0;        // DevSlotHdr the item kernel stamps
constexpr uint64_t kNaWorkOff = 64;      // uint32 work-item counter
constexpr uint64_t kNaTabOff = 256;      // VecBatchHdr + VecBatchDesc[kNaMaxJobs]
constexpr uint64_t kNaTabBytes = (sizeof(VecBatchHdr) + sizeof(VecBatchDesc) * (uint64_t)kNaMaxJobs + 255) / 256 * 256;
constexpr uint64_t kNaPartOff = kNaTabOff + kNaTabBytes;  // float[kNaMaxItems]
constexpr uint64_t kNaBytes = kNaPartOff + 4ull * kNaMaxItems;

}  // namespace
}  // namespace setrt

// The static work area.  In host code this name is only a stand-in for the
// symbol: the device address comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[setrt::kNaBytes];

namespace setrt {
namespace {

struct NaTotalsArgs {
  const uint8_t* tab;
  const float* partials;
  float* results;
};

// Block-wide exclusive prefix of one value per thread (kNaPlanThreads
// threads); *total receives the block's sum.
__device__ inline uint32_t block_excl_u32(uint32_t v, uint32_t* s_wave, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_u32(v);
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
  for (int k = 0; k < kNaPlanThreads / 64; ++k) {
    const uint32_t t = s_wave[k];
    if (k < wave) before += t;
    all += t;
  }
  __syncthreads();
  *total = all;
  return before + incl - v;
}

// One block, so latency and instructions count, us at 300 / 1000 / 2000 jobs: 7.9 /
// 8.2 / 11.1 with shuffles, an LDS addition a thread for the call's length and
// divisions of 64 bits; 3.2 / 4.0 / 6.0 with DPP prefixes, an addition a wave,
// 32 bits and the next round of jobs asked for early.
__global__ __launch_bounds__(kNaPlanThreads) void k_vec_noalloc_plan(VecPlanArgs a) {
  __shared__ uint32_t s_wave[kNaPlanThreads / 64];
  __shared__ unsigned long long s_elems;
  VecBatchDesc* D = reinterpret_cast<VecBatchDesc*>(a.tab + sizeof(VecBatchHdr));
  uint32_t carry = 0;
  uint32_t elems_lo = 0, elems_hi = 0;  // 16 bits and the rest of each length
  if (threadIdx.x == 0) s_elems = 0;
  set_vec_job job{};  // the round's, asked for a round ahead
  if (threadIdx.x < a.count) job = a.jobs[threadIdx.x];
  for (uint32_t base = 0; base < a.count; base += kNaPlanThreads) {
    const uint32_t j = base + threadIdx.x;
    VecBatchDesc d{};
    if (j < a.count) d = vec_plan_job(a, job);
    if (j + kNaPlanThreads < a.count) job = a.jobs[j + kNaPlanThreads];
    uint32_t chunk_total;
    const uint32_t excl = block_excl_u32(d.ntiles, s_wave, &chunk_total);
    d.tile_start = carry + excl;
    elems_lo += d.n & 0xFFFFu;
    elems_hi += d.n >> 16;
    if (j < a.count) D[j] = d;
    carry += chunk_total;
  }
  elems_lo = wave_total_u32(elems_lo);
  elems_hi = wave_total_u32(elems_hi);
  if ((threadIdx.x & 63) == 0)  // cleared before the prefix's barriers
    atomicAdd(&s_elems, ((unsigned long long)elems_hi << 16) + elems_lo);
  __syncthreads();
  if (threadIdx.x == 0) {
    VecBatchHdr* H = reinterpret_cast<VecBatchHdr*>(a.tab);
    H->count = a.count;
    H->total_tiles = carry;
    H->claim = vec_claim(s_elems, carry, a.grid);
    H->planned = kVecPlanned;
    *a.work = 0u;
  }
}

// Job j = wave j: NaN for a job the plan rejected (n == 0 in its descriptor),
// else its tiles' partials in their fixed order.
__global__ __launch_bounds__(kBlock) void k_vec_noalloc_totals(NaTotalsArgs a) {
  const VecBatchHdr* H = reinterpret_cast<const VecBatchHdr*>(a.tab);
  const VecBatchDesc* D = reinterpret_cast<const VecBatchDesc*>(a.tab + sizeof(VecBatchHdr));
  const uint32_t j = blockIdx.x * kVecFinalJobs + (threadIdx.x >> 6);
  if (j >= H->count) return;
  const float s = vec_job_total(a.partials + D[j].tile_start, D[j].ntiles, D[j].per_item);
  if ((threadIdx.x & 63) == 0) a.results[j] = D[j].n == 0 ? __builtin_nanf("") : s;
}

bool overlap(const void* a, uint64_t a_bytes, const void* b, uint64_t b_bytes) {
  const uint64_t x = reinterpret_cast<uint64_t>(a), y = reinterpret_cast<uint64_t>(b);
  return x < y + b_bytes && y < x + a_bytes;
}

std::mutex g_na_mu;
std::atomic<unsigned char*> g_na_ptr[kNaMaxDevices];

int na_fail(int code, const std::string& msg) {
  set_thread_error(msg);
  return code;
}

// Device address of `scratch` on the current device `dev`, looked up on the
// first call there.
int na_scratch(int dev, unsigned char** out) {
  unsigned char* p = g_na_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    std::lock_guard<std::mutex> g(g_na_mu);
    p = g_na_ptr[dev].load(std::memory_order_relaxed);
    if (!p) {
      void* q = nullptr;
      const hipError_t e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !q)
        return na_fail(SET_EDEVICE, std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e));
      p = static_cast<unsigned char*>(q);
      g_na_ptr[dev].store(p, std::memory_order_release);
    }
  }
  *out = p;
  return SET_OK;
}

int run_noalloc(int device, hipStream_t stream, const float* x, const float* y, uint64_t pool_len, uint64_t max_n,
                const set_vec_job* jobs, uint64_t count, float* results, const set_vec_tuning* tuning, uint32_t grid) {
  set_thread_error("");
  if (!x || !y || (count && (!jobs || !results))) return na_fail(SET_EINVAL, "null pool, jobs or results pointer");
  if (device < 0 || device >= kNaMaxDevices) return na_fail(SET_EINVAL, "device ordinal out of range");
  if (max_n < 1 || max_n > (1ull << 31)) return na_fail(SET_EINVAL, "max_n outside [1, 2^31]");
  if (count > kNaMaxJobs)
    return na_fail(SET_EINVAL, "count " + std::to_string(count) + " above the maximum of " +
                                   std::to_string(kNaMaxJobs) + " jobs per call");
  if (grid > 65535) return na_fail(SET_EINVAL, "grid above 65535");
  VecPlanArgs pa{};
  // Item size per bucket and the most items any job of length <= max_n needs.
  const int top = 63 - __builtin_clzll(max_n);
  uint64_t worst = 0, worst_units = 0;
  uint32_t longest_item = 0;
  for (int b = 0; b < 64; ++b) {
    const uint32_t te = (tuning && tuning->tile_elems[b]) ? tuning->tile_elems[b] : vec_default_tile(b);
    if (b <= top) {
      if (te == 0 || te % 1024 != 0) return na_fail(SET_EINVAL, "tile_elems must be a positive multiple of 1024");
      const uint64_t nmax = b == 63 ? max_n : std::min<uint64_t>(max_n, (2ull << b) - 1);
      worst = std::max<uint64_t>(worst, (nmax + te - 1) / te);
      longest_item = std::max(longest_item, te);
      worst_units = std::max<uint64_t>(worst_units, vec_units(nmax, te, kBlock));
    }
    pa.item_elems[b] = te;
  }
  if (count * worst > kNaMaxItems)
    return na_fail(SET_EINVAL, std::to_string(count) + " jobs of length up to max_n may need " +
                                   std::to_string(count * worst) + " work items, above the maximum of " +
                                   std::to_string(kNaMaxItems));
  if (count == 0) return SET_OK;

  int prev = -1;
  hipError_t e = hipGetDevice(&prev);
  if (e == hipSuccess && prev != device) e = hipSetDevice(device);
  if (e != hipSuccess) return na_fail(SET_EDEVICE, std::string("hipSetDevice failed: ") + hipGetErrorString(e));
  unsigned char* base = nullptr;
  int rc = na_scratch(device, &base);
  if (rc == SET_OK) {
    uint8_t* tab = base + kNaTabOff;
    uint32_t* work = reinterpret_cast<uint32_t*>(base + kNaWorkOff);
    float* partials = reinterpret_cast<float*>(base + kNaPartOff);
    pa.jobs = jobs;
    pa.count = (uint32_t)count;
    pa.max_n = max_n;
    pa.pool_len = pool_len;
    pa.tab = tab;
    pa.work = work;
    pa.split = count * worst_units <= kNaMaxItems;
    const uint64_t most_tiles = count * (pa.split ? worst_units : worst);
    pa.grid = grid ? grid : (uint32_t)std::min<uint64_t>(kNaGrid, most_tiles);
    // The one kernel of short jobs writes results while other blocks still read: where
    // they replace what it reads, the call takes the kernels that read everything first.
    const bool reused = overlap(results, 4 * count, jobs, sizeof(set_vec_job) * count) ||
                        overlap(results, 4 * count, x, 4 * pool_len) || overlap(results, 4 * count, y, 4 * pool_len);
    const bool is_short = worst <= kVecShortItems && longest_item <= kVecShortItem && grid == 0 && !reused;
    if (is_short) {
      VecShortArgs sa{pa, x, y, results};
      hipLaunchKernelGGL(k_vec_short_jobs, dim3((unsigned)count), dim3(64 * (unsigned)worst), 0, stream, sa);
    } else if (count <= (uint64_t)kBlock) {
      VecFewArgs fa{pa, x, y, partials};
      hipLaunchKernelGGL(k_vec_few_tiles, dim3(pa.grid), dim3(kBlock), 0, stream, fa);
    } else {
      hipLaunchKernelGGL(k_vec_noalloc_plan, dim3(1), dim3(kNaPlanThreads), 0, stream, pa);
      JobScalars js{};
      VecBatchArgs va{tab, x, y, partials, work, reinterpret_cast<DevSlotHdr*>(base + kNaHdrOff), js};
      hipLaunchKernelGGL(k_vec_batch_tiles<kBlock>, dim3(pa.grid), dim3(kBlock), 0, stream, va);
    }
    if (!is_short) {
      NaTotalsArgs ta{tab, partials, results};
      hipLaunchKernelGGL(k_vec_noalloc_totals, dim3((unsigned)((count + kVecFinalJobs - 1) / kVecFinalJobs)),
                         dim3(kBlock), 0, stream, ta);
    }
    e = hipGetLastError();
    if (e != hipSuccess) rc = na_fail(SET_EDEVICE, std::string("kernel launch failed: ") + hipGetErrorString(e));
  }
  if (prev >= 0 && prev != device) (void)hipSetDevice(prev);
  return rc;
}

}  // namespace
}  // namespace setrt

extern "C" int set_run_vector_jobs_noalloc(int device, void* stream, const float* dev_x_pool, const float* dev_y_pool,
                                           uint64_t pool_len, uint64_t max_n, const set_vec_job* dev_jobs,
                                           uint64_t count, float* dev_results, const set_vec_tuning* tuning,
                                           uint32_t grid) {
  return setrt::run_noalloc(device, static_cast<hipStream_t>(stream), dev_x_pool, dev_y_pool, pool_len, max_n,
                            dev_jobs, count, dev_results, tuning, grid);
}
