// Stage kernels of the job chains and their argument blocks.  Each kernel
// takes one argument struct by value, so a graph kernel node's per-job
// placeholder (Section 4.1) is a single struct that the binder rewrites.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "tiles.hpp"

namespace setrt {

// What the last stage of every chain needs to publish the output header (fixed
// when the slot is laid out; outh is rebound where it points to host memory).
struct SlotConst {
  DevSlotHdr* hdr;
  const uint64_t* tail;
  set_out_header* outh;  // in the slot; in the job's host buffer where the kernel writes the output there
  uint64_t canary_head;
  uint64_t canary_tail;
  uint64_t* word;        // completion word this kernel stores last, or null
};

// ---- argument blocks
struct BoxArgs {
  const uint8_t* in;
  uint16_t* S;
  int h, w;
  DevSlotHdr* hdr;
  JobScalars js;
};
struct BoxHistArgs {
  const uint8_t* in;
  int h, w;
  int shift;           // box_hist_shift(h, w)
  uint32_t* partials;  // [grid][256]
  DevSlotHdr* hdr;
  JobScalars js;
};
struct Div9Args {
  const uint16_t* S;
  uint8_t* Q;
  int64_t npix;
};
struct HistArgs {
  const uint8_t* Q;
  int64_t npix;
  uint32_t* partials;  // [grid][256]
};
struct HistFinalArgs {
  const uint32_t* partials;
  unsigned nblocks;
  uint32_t* H;         // output payload
  SlotConst sc;
};
struct GaussArgs {
  const float* in;
  float* out;
  int h, w;
  float g0, g1, g2;    // taps (g[-2]=g[2]=g0, g[-1]=g[1]=g1, centre g2)
  DevSlotHdr* hdr;
  JobScalars js;
};
struct SobelArgs {
  const float* blur;
  uint8_t* mask;
  int h, w;
  float thr;
  uint32_t* pcount;    // [grid]
  float* psum;         // [grid]
};
struct SobelFinalArgs {
  const uint32_t* pcount;
  const float* psum;
  unsigned nparts;     // partial pairs to combine
  uint32_t* out_count; // output payload
  float* out_sum;
  SlotConst sc;
};
struct GaussSobelArgs {
  const float* in;
  int h, w;
  float g0, g1, g2;    // taps, as in GaussArgs
  float thr;
  uint32_t* pcount;    // [grid]
  float* psum;         // [grid]
  uint32_t* arrivals;  // arrival_bytes(grid)
  uint32_t* out_count; // output payload
  float* out_sum;
  DevSlotHdr* hdr;
  SlotConst sc;
  JobScalars js;
};
struct VecArgs {
  const float* x;      // pool base
  const float* y;
  float* partials;     // [grid]
  DevSlotHdr* hdr;
  JobScalars js;       // n, a, x_off, y_off
};
struct VecFinalArgs {
  const float* partials;  // [vec_blocks(n)], n read from the slot header
  float* out_sum;
  SlotConst sc;
};
struct VecBatchArgs {
  const uint8_t* tab;  // descriptor table in the slot (VecBatchHdr + VecBatchDesc[count])
  const float* x;
  const float* y;
  float* partials;     // [total_tiles]
  uint32_t* work;      // claim counter (zero between batches)
  DevSlotHdr* hdr;
  JobScalars js;
};
// Planning of a no-allocation call: jobs to descriptors.
struct VecPlanArgs {
  const set_vec_job* jobs;
  uint32_t count;
  uint32_t grid;            // blocks of the tile kernel
  uint64_t max_n;
  uint64_t pool_len;
  uint8_t* tab;             // VecBatchHdr + VecBatchDesc[count]
  uint32_t* work;           // claim counter
  uint32_t split;           // a tile is a unit of a work item, not all of it
  uint32_t item_elems[64];  // elements per work item, per size bucket
};
struct VecFewArgs {
  VecPlanArgs plan;
  const float* x;
  const float* y;
  float* partials;
};
__global__ void k_vec_few_tiles(VecFewArgs a);
struct VecShortArgs {
  VecPlanArgs plan;
  const float* x;
  const float* y;
  float* results;
};
__global__ void k_vec_short_jobs(VecShortArgs a);
struct VecBatchFinalArgs {
  uint8_t* tab;
  const float* partials;
  uint32_t* work;
  float* results;      // output payload, one float per job
  SlotConst sc;
  uint32_t* arrivals;  // where the last block writes the output (arrival_bytes(grid)), or null
  uint32_t n;          // results it writes
};
// Scan as reduce -> spine -> downsweep, or without the first one or two where the
// downsweep's blocks add up what lies before them (scan_prefix); launched with the
// grid of the template's largest n, so a job of any length needs no grid update.
// The reduce and the downsweep take the job's n in their argument blocks; the
// one-block spine reads it from the slot header.
struct ScanReduceArgs {
  const int32_t* in;
  int64_t* tile_sum;   // [tiles]
  unsigned max_tiles;
  DevSlotHdr* hdr;
  JobScalars js;
};
struct ScanSpineArgs {
  const int64_t* tile_sum;
  int64_t* tile_excl;  // [tiles] exclusive prefix of tile sums
  SlotConst sc;
  uint64_t n;          // the job's length, rebound per job like the downsweep's
};
// The downsweep carries the job's n in its own argument block (rebound with
// the first kernel's), so its data loads need no dependent load of the slot
// header first: one memory round trip instead of two.
struct ScanDownArgs {
  const int32_t* in;
  const int64_t* tiles;  // the spine's tile_excl, or the reduce's tile_sum
  void* out;           // int64[n], or uint32[n] low words
  int low32;
  SlotConst sc;        // without the spine, block 0 publishes the header
  JobScalars js;       // n; without the reduce, block 0 writes them to the slot
};

// Host<->device copy as a kernel: a small grid of 16-byte loads/stores that
// keeps PCIe busy without occupying the whole device.
struct CopyArgs {
  const void* src;
  void* dst;
  uint64_t bytes;
};
// Output copies: k_copy_out_publish writes the header from the slot itself (the
// stages before it have ended) and copies what follows it.
struct CopyOutArgs {
  CopyArgs c;
  SlotConst sc;
};
__global__ void k_copy_out_publish(CopyOutArgs a);
__global__ void k_copy_in(CopyArgs a);   // host-to-device
// Bandwidth reference: word i of `nvec` 16-byte words copied by thread i.
struct RefCopyArgs {
  const void* src;
  void* dst;
  uint64_t nvec;
};
__global__ void k_ref_copy(RefCopyArgs a);
__global__ void k_copy_out(CopyArgs a);  // device-to-host

// Completion word: one thread stores the job's binding sequence number (from
// the slot header) into a pinned host word with a system-scope release.
struct DoneFlagArgs {
  const DevSlotHdr* hdr;
  uint64_t* word;
};
__global__ void k_done_flag(DoneFlagArgs a);

// Memory-safety stress (template options).  k_poison runs after a job's
// output copy and fills the slot's buffers (everything between the header
// and the tail canary) with 0xFF bytes, so a job that read anything a
// previous job left in its slot would read NaN / all-ones values; the one
// word the slot carries from job to job on purpose (the work counter of
// batched vector templates, rewound to zero by the job's last stage) is
// written as zero.  k_stress_delay runs before the first stage and sleeps
// until the device's constant-rate clock has advanced by `ticks`, stretching
// the window in which a slot released too early would be overwritten.
struct PoisonArgs {
  void* p;              // 16-byte aligned start of the poisoned range
  uint64_t nvec;        // 16-byte words in the range
  uint64_t zero_word;   // index (uint32 units from p) of the word written as 0, or ~0 for none
};
__global__ void k_poison(PoisonArgs a);
struct DelayArgs {
  uint64_t ticks;       // constant-clock ticks to wait
  uint64_t max_sleeps;  // bound on the sleep loop, so the wait ends whatever the clock reads
};
__global__ void k_stress_delay(DelayArgs a);

// Bracket kernels of a job whose middle stages are library code captured
// into the job graph: the first writes the job's scalars into the slot
// header, the last checks the canaries and publishes the output header.
struct JobBeginArgs {
  DevSlotHdr* hdr;
  JobScalars js;
};
struct JobEndArgs {
  SlotConst sc;
};
__global__ void k_job_begin(JobBeginArgs a);
__global__ void k_job_end(JobEndArgs a);

// The library stage of a library-call template: rocPRIM's device-wide
// inclusive scan of n int32 values into int64 sums, widening on load, on
// stream st (lib_scan.hip).  With ws == nullptr only ws_bytes is computed.
hipError_t lib_scan(void* ws, size_t& ws_bytes, const int32_t* in, int64_t* out, size_t n, hipStream_t st);

// Explicit steps of the thermal grid: tout = tin after `steps` of them (1 in
// the one-step kernels).  The first launch of a job (first != 0) also writes
// the job's scalars into the slot header.
struct HotspotArgs {
  const float* tin;
  const float* p;
  float* tout;
  int h, w;
  int first;
  int publish;         // tout is the job's output in host memory
  int steps;
  SlotConst sc;
  JobScalars js;       // in the first and the publishing launch
};
template <int HALO>
__global__ void k_hotspot_steps_f32(HotspotArgs a);
template <bool FULL>
__global__ void k_hotspot_win_f32(HotspotArgs a);
template <int R>
__global__ void k_hotspot_band_f32(HotspotArgs a);
__global__ void k_hotspot_f32(HotspotArgs a);

__global__ void k_box3_u8_u16(BoxArgs a);
__global__ void k_div9_u16_u8(Div9Args a);
__global__ void k_hist256_u8(HistArgs a);
__global__ void k_box_hist_u8(BoxHistArgs a);
__global__ void k_hist256_final(HistFinalArgs a);
__global__ void k_copy_out_hist256(HistFinalArgs a);
__global__ void k_gauss5_f32(GaussArgs a);
template <int R, bool FULL>
__global__ void k_gauss5_win_f32(GaussArgs a);
template <int R>
__global__ void k_gauss5_band_f32(GaussArgs a);
__global__ void k_sobel_thresh_f32(SobelArgs a);
template <int R, bool FULL>
__global__ void k_sobel_thresh_win_f32(SobelArgs a);
template <bool COLUMNS_FIRST>
__global__ void k_gauss_sobel_f32(GaussSobelArgs a);
__global__ void k_sobel_final(SobelFinalArgs a);
__global__ void k_copy_out_sobel(SobelFinalArgs a);
__global__ void k_saxpy_tanh_sum_f32(VecArgs a);
__global__ void k_vec_final(VecFinalArgs a);
__global__ void k_copy_out_vec(VecFinalArgs a);
#if defined(__HIPCC__)
// Sum over the wave in six DPP steps: two quad permutes, the half-row and row
// mirrors (each lane then holds its 16-lane row's sum), then row_bcast:15 into
// rows 1 and 3 and row_bcast:31 into rows 2 and 3; lane 63 ends with the total,
// which readlane returns to every lane.  Lanes of rows a broadcast leaves out
// add the old value 0.  The order of the additions is fixed.
template <int CTRL, int ROWS = 0xf, int BANKS = 0xf>
__device__ inline int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, BANKS, false);
}
__device__ inline uint32_t wave_total_u32(uint32_t v) {
  int x = (int)v;
  x += dpp_i<0xb1>(x);
  x += dpp_i<0x4e>(x);
  x += dpp_i<0x141>(x);
  x += dpp_i<0x140>(x);
  x += dpp_i<0x142, 0xa>(x);
  x += dpp_i<0x143, 0xc>(x);
  return (uint32_t)__builtin_amdgcn_readlane(x, 63);
}
// Inclusive prefix sum over the wave: the inputs 1, 2 and 3 lanes below (each lane
// then holds its 4-lane window's sum), row_shr:4 and 8 into the upper banks, the
// totals of the rows below by row_bcast.
__device__ inline uint32_t wave_inclusive_u32(uint32_t in) {
  const int x = (int)in;
  int v = x + dpp_i<0x111>(x) + dpp_i<0x112>(x) + dpp_i<0x113>(x);
  v += dpp_i<0x114, 0xf, 0xe>(v);
  v += dpp_i<0x118, 0xf, 0xc>(v);
  v += dpp_i<0x142, 0xa>(v);
  v += dpp_i<0x143, 0xc>(v);
  return (uint32_t)v;
}
__device__ inline float wave_total_f32(float v) {
  v += __int_as_float(dpp_i<0xb1>(__float_as_int(v)));        // quad_perm [1,0,3,2]
  v += __int_as_float(dpp_i<0x4e>(__float_as_int(v)));        // quad_perm [2,3,0,1]
  v += __int_as_float(dpp_i<0x141>(__float_as_int(v)));       // row_half_mirror
  v += __int_as_float(dpp_i<0x140>(__float_as_int(v)));       // row_mirror
  v += __int_as_float(dpp_i<0x142, 0xa>(__float_as_int(v)));  // row_bcast:15
  v += __int_as_float(dpp_i<0x143, 0xc>(__float_as_int(v)));  // row_bcast:31
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// Descriptor of a no-allocation call's job, but for its first tile; all zero for
// a job that is rejected.
__device__ inline VecBatchDesc vec_plan_job(const VecPlanArgs& a, const set_vec_job& v) {
  VecBatchDesc d{};
  const bool ok = v.n >= 1 && v.n <= a.max_n && v.x_off <= a.pool_len && v.n <= a.pool_len - v.x_off &&
                  v.y_off <= a.pool_len && v.n <= a.pool_len - v.y_off;
  if (ok) {
    d.x_off = v.x_off;
    d.y_off = v.y_off;
    d.a = v.a;
    vec_set_tiles(d, (uint32_t)v.n, a.item_elems[63 - __builtin_clzll(v.n)], kBlock, a.split != 0);
  }
  return d;
}
// Sum of one vector job's tile partials by one wave: a work item's tiles in
// order, lane l the items l, l + 64, ..., then the lanes' sums.  Items whose
// tiles are whole hold the same sum already, so the order depends only on n
// and the item and block sizes.
__device__ inline float vec_job_total(const float* partials, uint32_t count, uint32_t per_item) {
  float s = 0.f;
  for (uint32_t k = (threadIdx.x & 63u) * per_item; k < count; k += 64 * per_item) {
    float v[kVecUnitsPerItem];
#pragma unroll
    for (int u = 0; u < kVecUnitsPerItem; ++u) v[u] = u < (int)per_item && k + u < count ? partials[k + u] : 0.f;
    float item = v[0];
#pragma unroll
    for (int u = 1; u < kVecUnitsPerItem; ++u)
      if (u < (int)per_item && k + u < count) item += v[u];
    s += item;
  }
  return wave_total_f32(s);
}
#endif

// BLOCK threads per block: 128, 256, 512 or 1024 (the template's block).
template <int BLOCK>
__global__ void k_vec_batch_tiles(VecBatchArgs a);
__global__ void k_vec_batch_final(VecBatchFinalArgs a);
__global__ void k_scan_reduce_i32(ScanReduceArgs a);
__global__ void k_scan_spine_i64(ScanSpineArgs a);
template <int PREFIX>
__global__ void k_scan_down_i32_i64(ScanDownArgs a);

}  // namespace setrt
