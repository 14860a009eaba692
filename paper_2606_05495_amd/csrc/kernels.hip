// Stage kernels for CDNA4 (gfx950), wave64.  No MFMA: nothing here is a dense
// contraction.  Image stages stage their tile plus halo in LDS; reductions use
// wave shuffles and LDS in a fixed order, so every result depends only on the
// job's input and size (bit-identical whatever stream, slot or neighbour ran
// beside it); the histogram uses LDS atomics on per-wave private bins.
//
// Cross-block results are combined by a separate single-block kernel that runs
// after the producing kernel has finished (the kernel boundary is the
// synchronisation: no per-block device-scope fences, which on this multi-XCD
// part write back the issuing XCD's L2 and cost tens of microseconds when a
// thousand blocks issue them).  The one-kernel images and the last kernel of vector
// batches leave it to the block that arrives last, by agent-scope stores and loads
// without a fence.  What
// combines the per-block partials does so in a fixed order, checks the slot's
// canaries and publishes the output header.
#include <type_traits>

#include "kernels.hpp"

namespace setrt {

// ------------------------------------------------------------------ helpers
__device__ inline void write_slot_hdr(DevSlotHdr* hdr, const JobScalars& js) {
  hdr->job_id = js.job_id;
  hdr->seq = js.seq;
  hdr->user_tag = js.user_tag;
  hdr->worker = js.worker;
  hdr->slot = js.slot;
  hdr->n = js.n;
}

// The output header in two halves, so that a kernel can ask for the slot's
// words before its own work and write them behind it.  The canary tests are
// combined without short-circuit: every load goes out at once.  One thread.
struct OutWords {
  DevSlotHdr h;
  bool canaries;
};
__device__ inline OutWords load_out(const SlotConst& sc) {
  OutWords w;
  w.h = *sc.hdr;
  w.canaries = (w.h.canary_head == sc.canary_head) & (*sc.tail == sc.canary_tail);
  return w;
}
__device__ inline void store_out(const SlotConst& sc, const OutWords& w, bool extra_ok) {
  set_out_header* o = sc.outh;
  o->job_id = w.h.job_id;
  o->seq = w.h.seq;
  o->worker = w.h.worker;
  o->slot = w.h.slot;
  o->magic = extra_ok ? SET_OUT_MAGIC : 0xBAD0BAD0u;
  o->canary_ok = w.canaries ? 1u : 0u;
  o->user_tag = w.h.user_tag;
  o->reserved[0] = 0;
  o->reserved[1] = 0;
  o->reserved[2] = 0;
}
__device__ inline void publish_out(const SlotConst& sc, bool extra_ok) { store_out(sc, load_out(sc), extra_ok); }

// End of a kernel, by the one block that wrote the job's output to host memory
// itself: where the template completes by words, the word is stored once every wave's
// stores have been acknowledged.  All threads of the block.
__device__ inline void complete_out(const SlotConst& sc, uint64_t seq) {
  if (!sc.word) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(sc.word, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Blocks' arrivals at the end of a kernel whose last block to arrive finishes the
// job; the others leave their partial results and are done.  A word counts up to
// kArriveGroup blocks and, in a launch of more, one at the root the groups' last
// blocks: one word takes about 70 additions a microsecond, so every group's is in
// lines of its own.  A word rests at all ones, which a poisoned slot holds too,
// and the last to arrive puts it back.
//
// Partials are stored and read by relaxed agent-scope operations (put_partial,
// get_partial), which act where the XCDs' caches meet; every wave waits for the
// acknowledgement of its stores before the block arrives.  A release fence
// would write the XCD's whole L2 back instead.
template <typename T>
__device__ inline void put_partial(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline T get_partial(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline bool arrive(uint32_t* word, uint32_t count) {
  const uint32_t before = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const bool last = before + 2u == count;  // the first to arrive finds all ones
  if (last) __hip_atomic_store(word, ~0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return last;
}
// All threads of block b of nblocks, behind their put_partials.
__device__ inline bool arrives_last(uint32_t* words, uint32_t b, uint32_t nblocks) {
  __shared__ uint32_t s_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t g = b / kArriveGroup, first = g * kArriveGroup;
    const uint32_t in_group = nblocks - first < kArriveGroup ? nblocks - first : kArriveGroup;
    bool last = arrive(words + (size_t)g * (kArriveBytes / 4), in_group);
    if (last && nblocks > kArriveGroup)
      last = arrive(words + kArriveBytes / 8, (nblocks + kArriveGroup - 1) / kArriveGroup);
    s_last = last ? 1u : 0u;
  }
  __syncthreads();
  return s_last != 0;
}
// The output header of the job whose scalars a kernel carries itself (the slot's
// copy of them was written by another block of it).
__device__ inline OutWords load_out(const SlotConst& sc, const JobScalars& js) {
  OutWords w;
  w.h.job_id = js.job_id;
  w.h.seq = js.seq;
  w.h.user_tag = js.user_tag;
  w.h.worker = js.worker;
  w.h.slot = js.slot;
  w.canaries = (sc.hdr->canary_head == sc.canary_head) & (*sc.tail == sc.canary_tail);
  return w;
}

__device__ inline float wave_sum_f32(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ inline uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Block sums in a fixed order: lane 0 of each wave, then waves 0..3 pairwise.
// Every thread returns the same value.
__device__ inline float block_sum_f32(float v, float* s4) {
  v = wave_sum_f32(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) s4[wave] = v;
  __syncthreads();
  return (s4[0] + s4[1]) + (s4[2] + s4[3]);
}
__device__ inline uint32_t block_sum_u32(uint32_t v, uint32_t* s4) {
  v = wave_sum_u32(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) s4[wave] = v;
  __syncthreads();
  return (s4[0] + s4[1]) + (s4[2] + s4[3]);
}

// Partial sums of whole blocks are combined in float64 where a job is dispatched on its
// own (vec_final) and in one-kernel images: they are few, and their
// float32 sum rounded as much as all of the blocks' did.  Root mean square error
// against float64, relative: 3000 uneven vector jobs 1.3e-7 -> 9.9e-8, images of
// 333 x 250 4.1e-8 -> 2.5e-8.  The register-window images' finaliser (sobel_final) and
// batches' and no-allocation calls' jobs (vec_job_total) add in float32, as they always
// have; a batch and a call without allocation give the same bits.  The steps are wave_total_f32's.
template <int CTRL, int ROWS = 0xf>
__device__ inline double dpp_f64(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)dpp_i<CTRL, ROWS>((int)(uint32_t)u), hi = (uint32_t)dpp_i<CTRL, ROWS>((int)(u >> 32));
  return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
__device__ inline double wave_total_f64(double v) {
  v += dpp_f64<0xb1>(v);
  v += dpp_f64<0x4e>(v);
  v += dpp_f64<0x141>(v);
  v += dpp_f64<0x140>(v);
  v += dpp_f64<0x142, 0xa>(v);
  v += dpp_f64<0x143, 0xc>(v);
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(u >> 32), 63);
  return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Stage outputs (the blurred image, the mask, a heat step's grid, the scan's
// sums) are stored with the nontemporal hint.  On cold buffers this takes the
// Gaussian from 4.12 to 3.60 us at 1024x1024 and from 9.19 to 8.62 us at
// 2048x2048, Sobel from 6.36 to 6.01 us and the heat step from 10.69 to
// 10.15 us at 2048x2048; the next stage, which reads them, did not slow
// (thermal jobs of 16 steps ran at the same rate either way).
typedef float v4f_t __attribute__((ext_vector_type(4)));
// Four floats at any float's address: gfx950 moves 16 bytes at 4-byte alignment.
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef long long v2i64_t __attribute__((ext_vector_type(2)));
typedef unsigned v4u_t __attribute__((ext_vector_type(4)));
__device__ inline void store_nt(float* p, float x, float y, float z, float w) {
  __builtin_nontemporal_store(v4f_t{x, y, z, w}, reinterpret_cast<v4f_t*>(p));
}
__device__ inline void store_nt(int64_t* p, int64_t x, int64_t y) {
  __builtin_nontemporal_store(v2i64_t{x, y}, reinterpret_cast<v2i64_t*>(p));
}
__device__ inline void store_nt(uint32_t* p, uint32_t x, uint32_t y, uint32_t z, uint32_t w) {
  __builtin_nontemporal_store(v4u_t{x, y, z, w}, reinterpret_cast<v4u_t*>(p));
}
__device__ inline void store_nt(uint32_t* p, uint32_t x) { __builtin_nontemporal_store(x, p); }
// Global-memory (address space 1) views of an integer address.  A row base
// held in scalar registers as an integer, plus a lane's 32-bit byte offset,
// then loads and stores as global_load/store with a scalar base, where the
// compiler would otherwise form one 64-bit vector address per row.
typedef v4f_t __attribute__((address_space(1))) GlobalV4f;
typedef const float __attribute__((address_space(1))) GlobalF32;
__device__ inline v4f_t make_v4f(float x, float y, float z, float w) { return v4f_t{x, y, z, w}; }

// The hardware square root (v_sqrt_f32, within 1 ulp for normal inputs)
// instead of the correctly rounded library sequence, which costs about 15
// instructions per call; the Sobel magnitudes here are normal numbers and
// their parity bound is 1e-5 relative.
__device__ inline float sqrt_hw(float x) { return __builtin_amdgcn_sqrtf(x); }

// Fill an LDS tile of N elements (row-major, LW per row, stored with pitch
// P) from global memory: every thread issues all of its loads before its
// first LDS write, so one memory latency covers the whole tile.  get(r, c)
// returns the element for tile row r, column c.
template <typename T, int LW, int LH, int P, class Get>
__device__ inline void stage_tile(T (*tile)[P], Get get) {
  constexpr int N = LW * LH;
  constexpr int PER = (N + kBlock - 1) / kBlock;
  T vals[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = threadIdx.x + k * kBlock;
    const int r = i / LW, c = i - r * LW;
    vals[k] = (i < N) ? get(r, c) : T(0);
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = threadIdx.x + k * kBlock;
    const int r = i / LW, c = i - r * LW;
    if (i < N) tile[r][c] = vals[k];
  }
}

// ------------------------------------------------------------------ copy kernels (H2D pull / D2H push)
// Grid-stride over 16-byte words with four independent loads in flight per
// thread, then a byte tail.  Source and destination are 16-byte aligned (slot
// buffers are 256-aligned; host buffers are checked by the binder).  The two
// directions are separate kernels only so that a kernel trace tells them
// apart (input-copy idle time, batch boundaries).
__device__ __forceinline__ void copy_bytes(const CopyArgs& a) {
  const uint64_t nvec = a.bytes >> 4;
  const uint4* __restrict__ src = reinterpret_cast<const uint4*>(a.src);
  uint4* __restrict__ dst = reinterpret_cast<uint4*>(a.dst);
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  for (; i + 3 * stride < nvec; i += 4 * stride) {
    const uint4 v0 = src[i], v1 = src[i + stride], v2 = src[i + 2 * stride], v3 = src[i + 3 * stride];
    dst[i] = v0;
    dst[i + stride] = v1;
    dst[i + 2 * stride] = v2;
    dst[i + 3 * stride] = v3;
  }
  for (; i < nvec; i += stride) dst[i] = src[i];
  const uint64_t tail = nvec << 4;
  const uint64_t t = tail + (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (t < a.bytes) reinterpret_cast<uint8_t*>(a.dst)[t] = reinterpret_cast<const uint8_t*>(a.src)[t];
}
__global__ __launch_bounds__(kBlock) void k_copy_in(CopyArgs a) { copy_bytes(a); }
__global__ __launch_bounds__(kBlock) void k_ref_copy(RefCopyArgs a) {
  const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < a.nvec) static_cast<uint4*>(a.dst)[i] = static_cast<const uint4*>(a.src)[i];
}
__global__ __launch_bounds__(kBlock) void k_copy_out(CopyArgs a) { copy_bytes(a); }
__global__ __launch_bounds__(kBlock) void k_copy_out_publish(CopyOutArgs a) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.sc.outh = static_cast<set_out_header*>(a.c.dst);
    publish_out(a.sc, true);
  }
  copy_bytes(CopyArgs{static_cast<const char*>(a.c.src) + sizeof(set_out_header),
                      static_cast<char*>(a.c.dst) + sizeof(set_out_header), a.c.bytes - sizeof(set_out_header)});
}

// ------------------------------------------------------------------ completion word
// Runs after the job's device-to-host copy node; the kernel boundary orders
// the copy's host writes before this store.
__global__ __launch_bounds__(64) void k_done_flag(DoneFlagArgs a) {
  if (threadIdx.x == 0) __hip_atomic_store(a.word, a.hdr->seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ------------------------------------------------------------------ memory-safety stress
__global__ __launch_bounds__(kBlock) void k_poison(PoisonArgs a) {
  const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u);
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  const uint64_t zv = a.zero_word >> 2;  // the 16-byte word that holds the zero word, if any
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < a.nvec; i += stride) {
    uint4 v = ones;
    if (i == zv) {
      const unsigned c = (unsigned)(a.zero_word & 3);
      v.x = c == 0 ? 0u : v.x;
      v.y = c == 1 ? 0u : v.y;
      v.z = c == 2 ? 0u : v.z;
      v.w = c == 3 ? 0u : v.w;
    }
    reinterpret_cast<uint4*>(a.p)[i] = v;
  }
}

// One wave; s_sleep 8 is 512 clocks, so the loop ends within max_sleeps
// iterations even if the clock does not advance.
__global__ __launch_bounds__(64) void k_stress_delay(DelayArgs a) {
  if (threadIdx.x != 0) return;
  const uint64_t t0 = (uint64_t)wall_clock64();
  for (uint64_t k = 0; k < a.max_sleeps && (uint64_t)wall_clock64() - t0 < a.ticks; ++k)
    __builtin_amdgcn_s_sleep(8);
}

// ------------------------------------------------------------------ bracket kernels of library-call jobs
__global__ __launch_bounds__(kBlock) void k_job_begin(JobBeginArgs a) {
  if (blockIdx.x == 0 && threadIdx.x == 0) write_slot_hdr(a.hdr, a.js);
}
__global__ __launch_bounds__(kBlock) void k_job_end(JobEndArgs a) {
  if (blockIdx.x == 0 && threadIdx.x == 0) publish_out(a.sc, true);
}

// ------------------------------------------------------------------ box sum, floor(s / 9) and histogram in one
// For templates that return the histogram alone: the sums and quotients stay in
// registers.  A thread takes 4 pixels of a row of the block's tile, which is 64 x 64
// or, for narrow images, wider or taller (box_hist_shift).  Of each of its three input rows it loads the 8 bytes from one
// left of its pixels, at any alignment (before the first and past the last row
// of the image they reach into the slot around it, and are masked), and adds
// them column-wise two to a word.  Quotients go to LDS bins, four copies.  The
// grid is at most the partial rows the slot has, so a block may take several
// tiles.
// Small images are launch and memory latency, of the code too: a kernel this
// short runs once over its instructions, cold (16 pixels a thread, unrolled with
// a byte path for ragged ends, 4.4 KB of code: 3.3 us for 256^2 and 6.5 for 333
// x 250; now 2.8 and 3.3; as three kernels 2.5 + 2.1 + 2.2).
typedef uint32_t v2u_any __attribute__((ext_vector_type(2), aligned(1)));
__global__ __launch_bounds__(kBoxHistBlock) void k_box_hist_u8(BoxHistArgs a) {
  __shared__ uint32_t wh[4][256];
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && tid == 0) write_slot_hdr(a.hdr, a.js);
  (&wh[0][0])[tid] = 0u;
  __syncthreads();
  uint32_t* bins = wh[(tid >> 6) & 3];
  const int lw = a.shift + 2, lh = __builtin_ctz(kBoxHistBlock) - a.shift;  // log2 of the tile's sides
  const int tiles_x = (a.w + (1 << lw) - 1) >> lw, tiles_y = (a.h + (1 << lh) - 1) >> lh;
  for (int t = blockIdx.x; t < tiles_x * tiles_y; t += gridDim.x) {
    const int by = t / tiles_x, bx = t - by * tiles_x;
    const int x = (bx << lw) + 4 * (tid & ((1 << a.shift) - 1)), y = (by << lh) + (tid >> a.shift);
    if (x >= a.w || y >= a.h) continue;
    uint32_t even0 = 0, odd0 = 0, even1 = 0, odd1 = 0;  // columns x-1, x+1 | x, x+2 | x+3 | x+4
#pragma unroll
    for (int k = -1; k <= 1; ++k) {
      const int yr = y + k;
      const v2u_any v = *reinterpret_cast<const v2u_any*>(a.in + (ptrdiff_t)clampi(yr, 0, a.h - 1) * a.w + x - 1);
      const uint32_t keep = yr >= 0 && yr < a.h ? 0x00FF00FFu : 0u;
      even0 += v.x & keep;
      odd0 += (v.x >> 8) & keep;
      even1 += v.y & keep;
      odd1 += (v.y >> 8) & keep;
    }
    uint32_t c[6] = {even0 & 0xFFFFu, odd0 & 0xFFFFu, even0 >> 16, odd0 >> 16, even1 & 0xFFFFu, odd1 & 0xFFFFu};
    if (x == 0) c[0] = 0;
#pragma unroll
    for (int i = 2; i < 6; ++i)
      if (x + i - 1 >= a.w) c[i] = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (x + i < a.w) atomicAdd(&bins[(c[i] + c[i + 1] + c[i + 2]) / 9u], 1u);
  }
  __syncthreads();
  if (tid < 256) a.partials[(size_t)blockIdx.x * 256 + tid] = wh[0][tid] + wh[1][tid] + wh[2][tid] + wh[3][tid];
}

// ------------------------------------------------------------------ 3x3 box sum (zero padded), uint8 -> uint16
// Output tile kBoxTW x kBoxTH, input tile + 1-pixel halo staged in LDS.
__global__ __launch_bounds__(kBlock) void k_box3_u8_u16(BoxArgs a) {
  constexpr int LW = kBoxTW + 2, LH = kBoxTH + 2;
  __shared__ uint8_t tile[LH][LW + 2];
  const int x0 = blockIdx.x * kBoxTW, y0 = blockIdx.y * kBoxTH;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) write_slot_hdr(a.hdr, a.js);
  stage_tile<uint8_t, LW, LH, LW + 2>(tile, [&](int r, int c) {
    const int gy = y0 + r - 1, gx = x0 + c - 1;
    return (gy >= 0 && gy < a.h && gx >= 0 && gx < a.w) ? a.in[(size_t)gy * a.w + gx] : (uint8_t)0;
  });
  __syncthreads();
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int y = y0 + ty;
  if (y >= a.h) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int lx = tx * 4 + k, x = x0 + lx;
    if (x < a.w) {
      unsigned s = 0;
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) s += tile[ty + dy][lx + dx];
      a.S[(size_t)y * a.w + x] = (uint16_t)s;
    }
  }
}

// ------------------------------------------------------------------ floor(s / 9), uint16 -> uint8
__global__ __launch_bounds__(kBlock) void k_div9_u16_u8(Div9Args a) {
  const int64_t i0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kDivPerThread;
  if (i0 + kDivPerThread <= a.npix) {
    const uint4 v = *reinterpret_cast<const uint4*>(a.S + i0);  // 8 x uint16, 16-byte aligned
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[2] = {0u, 0u};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t lo = (w[k] & 0xFFFFu) / 9u, hi = (w[k] >> 16) / 9u;
      o[k >> 1] |= (lo | (hi << 8)) << (16 * (k & 1));
    }
    *reinterpret_cast<uint2*>(a.Q + i0) = make_uint2(o[0], o[1]);
  } else {
    for (int64_t i = i0; i < a.npix; ++i) a.Q[i] = (uint8_t)(a.S[i] / 9u);
  }
}

// ------------------------------------------------------------------ 256-bin histogram of uint8
// Per-wave private LDS bins (4 x 256) take the LDS atomics; the block's sum of
// them goes to partials[block].
__global__ __launch_bounds__(kBlock) void k_hist256_u8(HistArgs a) {
  __shared__ uint32_t wh[4][256];
  const int tid = threadIdx.x, wave = tid >> 6;
  for (int i = tid; i < 4 * 256; i += kBlock) (&wh[0][0])[i] = 0u;
  __syncthreads();
  const int64_t base = ((int64_t)blockIdx.x * kBlock + tid) * kHistPerThread;
  if (base + kHistPerThread <= a.npix) {
    const uint4 v = *reinterpret_cast<const uint4*>(a.Q + base);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int b = 0; b < 4; ++b) atomicAdd(&wh[wave][(w[k] >> (8 * b)) & 255u], 1u);
  } else {
    for (int64_t i = base; i < a.npix; ++i) atomicAdd(&wh[wave][a.Q[i]], 1u);
  }
  __syncthreads();
  a.partials[(size_t)blockIdx.x * 256 + tid] = wh[0][tid] + wh[1][tid] + wh[2][tid] + wh[3][tid];
}

// One block: bin tid = sum of the blocks' partial counts (integer, exact in
// any order).  Four quarters of the block take every fourth row, 16 loads of
// each going out at a time with no branch between them (past the last row the
// index is clamped and the value dropped): one memory latency covers 64 rows.
// Like the other combining kernels it has two names: k_copy_out_* where it
// writes the job's output to host memory itself (it is then the job's output
// copy, and its completion where the template completes by words, which saves
// a launch or two of about 2 us each), k_*_final where a copy follows.
__device__ __forceinline__ void hist256_final(const HistFinalArgs& a) {
  __shared__ uint32_t part[4][256];
  const int tid = threadIdx.x & 255, quarter = threadIdx.x >> 8;
  const unsigned nb = a.nblocks;
  OutWords w{};
  if (threadIdx.x == 0) w = load_out(a.sc);
  uint32_t s = 0;
  for (unsigned b0 = quarter; b0 < nb; b0 += 64) {  // rows b0, b0 + 4, ..., b0 + 60
    uint32_t v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const unsigned b = b0 + 4 * k < nb ? b0 + 4 * k : nb - 1;
      v[k] = a.partials[(size_t)b * 256 + tid];
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) s += b0 + 4 * k < nb ? v[k] : 0u;
  }
  part[quarter][tid] = s;
  __syncthreads();
  if (threadIdx.x < 256) a.H[tid] = part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid];
  if (threadIdx.x == 0) store_out(a.sc, w, true);
  complete_out(a.sc, w.h.seq);
}
__global__ __launch_bounds__(kHistFinalBlock) void k_hist256_final(HistFinalArgs a) { hist256_final(a); }
__global__ __launch_bounds__(kHistFinalBlock) void k_copy_out_hist256(HistFinalArgs a) { hist256_final(a); }

// ------------------------------------------------------------------ separable 5-tap Gaussian, replicated borders
// Input tile (kGaussTH+4) x (kGaussTW+4) in LDS, horizontal pass into a
// second LDS tile (kGaussTH+4) x kGaussTW, vertical pass to global.
__global__ __launch_bounds__(kBlock) void k_gauss5_f32(GaussArgs a) {
  constexpr int IW = kGaussTW + 4, IH = kGaussTH + 4;
  __shared__ float tin[IH][IW + 1];
  __shared__ float tmid[IH][kGaussTW + 1];
  const int x0 = blockIdx.x * kGaussTW, y0 = blockIdx.y * kGaussTH;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) write_slot_hdr(a.hdr, a.js);
  const int wm = a.w - 1, hm = a.h - 1;
  stage_tile<float, IW, IH, IW + 1>(tin, [&](int r, int c) {
    return a.in[(size_t)clampi(y0 + r - 2, 0, hm) * a.w + clampi(x0 + c - 2, 0, wm)];
  });
  __syncthreads();
  const float g0 = a.g0, g1 = a.g1, g2 = a.g2;
  for (int i = threadIdx.x; i < IH * kGaussTW; i += kBlock) {
    const int r = i / kGaussTW, c = i - r * kGaussTW;
    float acc = g0 * tin[r][c];
    acc = fmaf(g1, tin[r][c + 1], acc);
    acc = fmaf(g2, tin[r][c + 2], acc);
    acc = fmaf(g1, tin[r][c + 3], acc);
    acc = fmaf(g0, tin[r][c + 4], acc);
    tmid[r][c] = acc;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kGaussTH * kGaussTW; i += kBlock) {
    const int r = i / kGaussTW, c = i - r * kGaussTW;
    const int y = y0 + r, x = x0 + c;
    if (y < a.h && x < a.w) {
      float acc = g0 * tmid[r][c];
      acc = fmaf(g1, tmid[r + 1][c], acc);
      acc = fmaf(g2, tmid[r + 2][c], acc);
      acc = fmaf(g1, tmid[r + 3][c], acc);
      acc = fmaf(g0, tmid[r + 4][c], acc);
      a.out[(size_t)y * a.w + x] = acc;
    }
  }
}

// ------------------------------------------------------------------ Sobel magnitude + threshold + count/sum
// gx = (right column) - (left column) with weights 1,2,1; gy = (row below) -
// (row above); mag = sqrt(gx^2 + gy^2); mask = mag > thr.  Each block writes
// its count and its magnitude sum (fixed-order block reduction).
__global__ __launch_bounds__(kBlock) void k_sobel_thresh_f32(SobelArgs a) {
  constexpr int IW = kSobelTW + 2, IH = kSobelTH + 2;
  __shared__ float t[IH][IW + 1];
  __shared__ float s4f[4];
  __shared__ uint32_t s4u[4];
  const int x0 = blockIdx.x * kSobelTW, y0 = blockIdx.y * kSobelTH;
  const int wm = a.w - 1, hm = a.h - 1;
  stage_tile<float, IW, IH, IW + 1>(t, [&](int r, int c) {
    return a.blur[(size_t)clampi(y0 + r - 1, 0, hm) * a.w + clampi(x0 + c - 1, 0, wm)];
  });
  __syncthreads();
  float sum = 0.f;
  uint32_t cnt = 0;
  for (int i = threadIdx.x; i < kSobelTH * kSobelTW; i += kBlock) {
    const int r = i / kSobelTW, c = i - r * kSobelTW;
    const int y = y0 + r, x = x0 + c;
    if (y < a.h && x < a.w) {
      const float p00 = t[r][c], p01 = t[r][c + 1], p02 = t[r][c + 2];
      const float p10 = t[r + 1][c], p12 = t[r + 1][c + 2];
      const float p20 = t[r + 2][c], p21 = t[r + 2][c + 1], p22 = t[r + 2][c + 2];
      const float gx = (p02 + 2.f * p12 + p22) - (p00 + 2.f * p10 + p20);
      const float gy = (p20 + 2.f * p21 + p22) - (p00 + 2.f * p01 + p02);
      const float mag = sqrt_hw(gx * gx + gy * gy);
      const uint32_t on = mag > a.thr ? 1u : 0u;
      a.mask[(size_t)y * a.w + x] = (uint8_t)on;
      cnt += on;
      sum += mag;
    }
  }
  const unsigned b = blockIdx.y * gridDim.x + blockIdx.x;
  const float bs = block_sum_f32(sum, s4f);
  const uint32_t bc = block_sum_u32(cnt, s4u);
  if (threadIdx.x == 0) {
    a.psum[b] = bs;
    a.pcount[b] = bc;
  }
}

// ------------------------------------------------------------------ Gaussian + Sobel + threshold + count/sum in one
// For small images that return the count and the sum alone: the blurred image
// lives in LDS, one tile and a ring around it, and the mask is only counted.
// Replicated borders mean the blurred image's own border values beyond it, so
// a ring cell outside the image is the blur at the clamped place.  The
// arithmetic is that of the kernels it replaces, operation for operation:
// COLUMNS_FIRST for the register-window kernels (widths that are multiples of
// 4: vertical pass first, gy from column differences), rows first for the
// LDS-tile kernels.  A block's partials are those of its tile.
// Small images are launch and memory latency, which one kernel pays once: a
// 333 x 250 image 4.8 + 4.6 us as two kernels, four such jobs one after another
// 117 -> 103 us.  The tiles' partials are combined by the block that arrives last,
// which takes as long as a one-block kernel behind this one but is a launch less,
// where launches by one dispatcher thread set the pace: 64 jobs of 64 x 64 805-916
// -> 608-648 us, 16 of 333 x 250 266 -> 225, one after another and from 512 x 400
// up no difference.  Box/histogram and vector jobs have several threads that
// launch and mostly one job in flight to a worker: there it went neither way for
// the first, and 256 of the second, whose last block waits behind all the reads of
// the others, took 910 us and not 790.
template <bool COLUMNS_FIRST>
__global__ __launch_bounds__(kGsBlock) void k_gauss_sobel_f32(GaussSobelArgs a) {
  constexpr int BW = kSobelTW + 2, BH = kSobelTH + 2;  // blurred tile with its ring
  constexpr int IW = BW + 4, IH = BH + 4;              // input tile
  constexpr int MW = COLUMNS_FIRST ? IW : BW, MH = COLUMNS_FIRST ? BH : IH;  // first pass's output
  __shared__ float tin[IH][IW + 1];
  __shared__ float tmid[MH][MW + 1];
  float(*blur)[IW + 1] = tin;  // the second pass's output takes the input's place
  __shared__ float s_sum[kGsBlock / 64];
  __shared__ uint32_t s_count[kGsBlock / 64];
  const int x0 = blockIdx.x * kSobelTW, y0 = blockIdx.y * kSobelTH;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) write_slot_hdr(a.hdr, a.js);
  const int wm = a.w - 1, hm = a.h - 1, tid = threadIdx.x;
  constexpr int PER = (IW * IH + kGsBlock - 1) / kGsBlock;
  float v[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = tid + k * kGsBlock, r = i / IW, c = i - r * IW;
    v[k] = i < IW * IH ? a.in[(size_t)clampi(y0 + r - 3, 0, hm) * a.w + clampi(x0 + c - 3, 0, wm)] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = tid + k * kGsBlock, r = i / IW, c = i - r * IW;
    if (i < IW * IH) tin[r][c] = v[k];
  }
  __syncthreads();
  const float g0 = a.g0, g1 = a.g1, g2 = a.g2;
  auto taps = [&](const float* p, int step) {
    float acc = g0 * p[0];
    acc = fmaf(g1, p[step], acc);
    acc = fmaf(g2, p[2 * step], acc);
    acc = fmaf(g1, p[3 * step], acc);
    return fmaf(g0, p[4 * step], acc);
  };
  // rows and columns of the blurred tile are places of the image, clamped
  for (int i = tid; i < MW * MH; i += kGsBlock) {
    const int r = i / MW, c = i - r * MW;
    if constexpr (COLUMNS_FIRST)
      tmid[r][c] = taps(&tin[clampi(y0 + r - 1, 0, hm) - y0 + 1][c], IW + 1);
    else
      tmid[r][c] = taps(&tin[r][clampi(x0 + c - 1, 0, wm) - x0 + 1], 1);
  }
  __syncthreads();
  for (int i = tid; i < BW * BH; i += kGsBlock) {
    const int r = i / BW, c = i - r * BW;
    if constexpr (COLUMNS_FIRST)
      blur[r][c] = taps(&tmid[r][clampi(x0 + c - 1, 0, wm) - x0 + 1], 1);
    else
      blur[r][c] = taps(&tmid[clampi(y0 + r - 1, 0, hm) - y0 + 1][c], MW + 1);
  }
  __syncthreads();
  float sum = 0.f;
  uint32_t cnt = 0;
#pragma unroll
  for (int k = 0; k < kSobelTW * kSobelTH / kGsBlock; ++k) {
    const int i = tid + k * kGsBlock, r = i / kSobelTW, c = i - r * kSobelTW;
    if (y0 + r < a.h && x0 + c < a.w) {
      const float p00 = blur[r][c], p01 = blur[r][c + 1], p02 = blur[r][c + 2];
      const float p10 = blur[r + 1][c], p12 = blur[r + 1][c + 2];
      const float p20 = blur[r + 2][c], p21 = blur[r + 2][c + 1], p22 = blur[r + 2][c + 2];
      const float gx = (p02 + 2.f * p12 + p22) - (p00 + 2.f * p10 + p20);
      const float gy = COLUMNS_FIRST ? ((p20 - p00) + 2.f * (p21 - p01)) + (p22 - p02)
                                     : (p20 + 2.f * p21 + p22) - (p00 + 2.f * p01 + p02);
      const float mag = sqrt_hw(gx * gx + gy * gy);
      cnt += mag > a.thr ? 1u : 0u;
      sum += mag;
    }
  }
  const float ws = wave_total_f32(sum);
  const uint32_t wc = wave_total_u32(cnt);
  if ((tid & 63) == 0) {
    s_sum[tid >> 6] = ws;
    s_count[tid >> 6] = wc;
  }
  __syncthreads();
  const unsigned b = blockIdx.y * gridDim.x + blockIdx.x, nparts = gridDim.x * gridDim.y;
  if (tid == 0) {
    float s = 0.f;
    uint32_t n = 0;
#pragma unroll
    for (int k = 0; k < kGsBlock / 64; ++k) {
      s += s_sum[k];
      n += s_count[k];
    }
    put_partial(&a.psum[b], s);
    put_partial(&a.pcount[b], n);
  }
  if (!arrives_last(a.arrivals, b, nparts)) return;
  // The tiles' partials: thread t takes tiles t, t + kGsBlock, ..., four loads
  // of each going out together.
  __shared__ double s_total[kGsBlock / 64];
  OutWords w{};
  if (tid == 0) w = load_out(a.sc, a.js);
  double total = 0.0;
  cnt = 0;
  for (unsigned k = tid; k < nparts; k += 4 * kGsBlock) {
    float f[4];
    uint32_t u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned q = k + i * kGsBlock < nparts ? k + i * kGsBlock : nparts - 1;
      f[i] = get_partial(&a.psum[q]);
      u[i] = get_partial(&a.pcount[q]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (k + i * kGsBlock < nparts) {
        total += f[i];
        cnt += u[i];
      }
  }
  total = wave_total_f64(total);
  cnt = wave_total_u32(cnt);
  if ((tid & 63) == 0) {
    s_total[tid >> 6] = total;
    s_count[tid >> 6] = cnt;
  }
  __syncthreads();
  if (tid == 0) {
    total = 0.0;
    cnt = 0;
#pragma unroll
    for (int k = 0; k < kGsBlock / 64; ++k) {
      total += s_total[k];
      cnt += s_count[k];
    }
    *a.out_count = cnt;
    *a.out_sum = (float)total;
    store_out(a.sc, w, true);
  }
  complete_out(a.sc, w.h.seq);
}
template __global__ void k_gauss_sobel_f32<true>(GaussSobelArgs a);
template __global__ void k_gauss_sobel_f32<false>(GaussSobelArgs a);

// ------------------------------------------------------------------ register-window image kernels
// Path for float images whose width is a multiple of 4.  A lane owns 4
// adjacent columns (one 16-byte load or store per row), a wave 256 columns,
// and slides down R output rows with the window of input rows in
// registers: every input row of the wave is loaded before the first result
// is formed, so each wave has all its loads in flight at once.  Neighbouring
// columns come from the adjacent lanes by whole-wave lane shifts; lanes 0 and
// 63 take the columns beyond the wave from extra (clamped) loads.  A block is
// 4 waves stacked vertically.
//
// Blocks are dealt to the 8 XCDs round-robin in launch order.  xcd_tile
// renumbers them so each XCD owns a contiguous run of tiles in row-major
// order: vertically adjacent tiles, which read each other's halo rows, then
// share one L2.
__device__ inline void xcd_tile(unsigned& bx, unsigned& by) {
  const unsigned gx = gridDim.x, n = gx * gridDim.y;
  const unsigned L = blockIdx.y * gx + blockIdx.x;
  const unsigned q = n >> 3, rem = n & 7u, x = L & 7u, k = L >> 3;
  const unsigned t = x * q + (x < rem ? x : rem) + k;  // XCD x owns tiles [x*q + min(x, rem), ...)
  by = t / gx;
  bx = t - by * gx;
}

// Whole-wave shifts by one lane (DPP wave_shr:1 / wave_shl:1, a VALU move
// instead of an LDS permute).  from_left gives lane i the value of lane i-1,
// from_right the value of lane i+1.  With bound_ctrl off, the lane whose
// source lies outside the wave (lane 0 for from_left, lane 63 for
// from_right) keeps the old value, which is its own `edge`: the tile's halo
// column arrives without a per-lane select.
__device__ inline float from_left(float v, float edge) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ inline float from_right(float v, float edge) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x130, 0xf, 0xf, false));
}

// The neighbouring lane's value within a row of 16 lanes that wraps around (DPP
// row_ror:1 / row_ror:15): every lane has a source, so the move becomes part of
// the addition that uses it.
__device__ inline float row_from_left(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, true));
}
__device__ inline float row_from_right(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x12f, 0xf, 0xf, true));
}

// Register-window geometry of one lane.  The wave index goes through
// readfirstlane, so the wave's rows (and every row address, clamp and bounds
// test derived from them) live in scalar registers; a load or store is then a
// scalar row base plus the lane's 32-bit byte offset.  FULL: the width is a
// multiple of 256, so every lane's 4 columns lie inside the image.  Otherwise
// lanes past the right edge load the last 4 columns and keep only the border
// column (replicated), and store nothing.
template <bool FULL>
struct WinLane {
  int lane, y0;       // y0: first output row of the wave (wave-uniform)
  unsigned x;         // first of the lane's 4 columns
  unsigned xl;        // column the lane loads from
  bool past;          // lane lies beyond the right edge (never when FULL)
  __device__ WinLane(int w, unsigned bx, unsigned by, int rows) {
    lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    y0 = ((int)by * 4 + wave) * rows;
    x = bx * kWinCols + 4u * lane;
    past = FULL ? false : x >= (unsigned)w;
    xl = past ? (unsigned)w - 4u : x;
  }
  __device__ float4 load4(const float* row) const {
    const float4 t = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(row) + xl * 4u);
    return past ? make_float4(t.w, t.w, t.w, t.w) : t;
  }
};
__device__ inline float load1(const float* row, unsigned col) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + col * 4u);
}

// Separable 5-tap Gaussian on the register window, vertical pass first: each
// lane filters its own 4 columns down the R + 4 loaded rows (and lanes 0 and
// 63 the two columns beyond the wave's edge), then the horizontal pass takes
// the neighbouring columns' vertical results by lane shift.  Vertical first
// costs (R + 4)/R fewer lane shifts and FMAs than horizontal first, since the
// horizontal pass then runs on R rows instead of R + 4.
template <int R, bool FULL>
__global__ __launch_bounds__(kBlock) void k_gauss5_win_f32(GaussArgs a) {
  unsigned bx, by;
  xcd_tile(bx, by);
  if (bx == 0 && by == 0 && threadIdx.x == 0) write_slot_hdr(a.hdr, a.js);
  const int w = a.w, h = a.h, wm = w - 1, hm = h - 1;
  const WinLane<FULL> L(w, bx, by, R);
  const int xw = (int)bx * kWinCols;
  // lane 0 needs columns xw-2, xw-1; lane 63 needs xw+256, xw+257
  const unsigned hx0 = clampi(L.lane == 0 ? xw - 2 : xw + kWinCols, 0, wm);
  const unsigned hx1 = clampi(L.lane == 0 ? xw - 1 : xw + kWinCols + 1, 0, wm);
  float4 v[R + 4];
  float e0[R + 4], e1[R + 4];
#pragma unroll
  for (int r = 0; r < R + 4; ++r) {
    const float* row = a.in + (size_t)clampi(L.y0 + r - 2, 0, hm) * w;
    v[r] = L.load4(row);
    e0[r] = load1(row, hx0);
    e1[r] = load1(row, hx1);
  }
  const float g0 = a.g0, g1 = a.g1, g2 = a.g2;
  auto vert = [&](float t0, float t1, float t2, float t3, float t4) {
    float acc = g0 * t0;
    acc = fmaf(g1, t1, acc);
    acc = fmaf(g2, t2, acc);
    acc = fmaf(g1, t3, acc);
    return fmaf(g0, t4, acc);
  };
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const float c0 = vert(v[r].x, v[r + 1].x, v[r + 2].x, v[r + 3].x, v[r + 4].x);
    const float c1 = vert(v[r].y, v[r + 1].y, v[r + 2].y, v[r + 3].y, v[r + 4].y);
    const float c2 = vert(v[r].z, v[r + 1].z, v[r + 2].z, v[r + 3].z, v[r + 4].z);
    const float c3 = vert(v[r].w, v[r + 1].w, v[r + 2].w, v[r + 3].w, v[r + 4].w);
    const float f0 = vert(e0[r], e0[r + 1], e0[r + 2], e0[r + 3], e0[r + 4]);
    const float f1 = vert(e1[r], e1[r + 1], e1[r + 2], e1[r + 3], e1[r + 4]);
    const float c[8] = {from_left(c2, f0), from_left(c3, f1), c0, c1, c2, c3, from_right(c0, f0), from_right(c1, f1)};
    float o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = vert(c[j], c[j + 1], c[j + 2], c[j + 3], c[j + 4]);
    const int y = L.y0 + r;
    if (y < h && !L.past)
      store_nt(reinterpret_cast<float*>(reinterpret_cast<char*>(a.out + (size_t)y * w) + L.x * 4u), o[0], o[1], o[2],
               o[3]);
  }
}
// Row bands, for widths that are a multiple of kBandCols: a block of
// kBandCols / 256 waves lies side by side across R whole rows (8, or 4 above
// 4096^2 pixels), each wave 256 columns as in the window kernel.  A wave's halo columns are
// its neighbours' outermost columns, whose vertical-pass results the
// neighbours already hold: each wave's lane 0 publishes its first two columns
// and lane 63 its last two in LDS, and after one barrier lanes 0 and 63 read
// the neighbouring waves' pairs.  Only the block's outer edges, where they lie
// inside the image, load their two halo columns (the first wave on the left,
// the last on the right); at the image border the clamped columns are the
// border column itself, whose vertical result the border lane already holds.
// Against the window kernel at 4 rows, which loads both halo pairs in every
// wave, a wave issues R + 4 vector loads instead of 3 (R + 4) and skips two
// columns' vertical passes, and at 8 rows it re-reads 1.5x its rows from L2
// instead of 2x; the barrier makes a wave wait for its block's slowest load,
// which costs more than that saves on images of a million pixels or fewer,
// where each SIMD holds one wave.  The arithmetic is the window kernel's,
// operation for operation.
template <int R>
__global__ __launch_bounds__(kBandCols / 4) void k_gauss5_band_f32(GaussArgs a) {
  constexpr int nw = kBandCols / kWinCols;
  unsigned bx, band;
  xcd_tile(bx, band);  // grid (column blocks, bands)
  if (bx == 0 && band == 0 && threadIdx.x == 0) write_slot_hdr(a.hdr, a.js);
  // lo[k + 1][r]: wave k's two first columns; hi[k + 1][r]: its two last.
  // hi[0] holds the pair left of the block, lo[nw + 1] the pair right of it.
  __shared__ float2 lo[nw + 2][R], hi[nw + 2][R];
  const int w = a.w, h = a.h, hm = h - 1;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int y0 = (int)band * R;
  const unsigned xb = bx * (unsigned)kBandCols;  // first column of the block
  const unsigned x = xb + (unsigned)wave * kWinCols + 4u * (unsigned)lane;
  const uint32_t pitch = (uint32_t)w * 4u;  // row bytes
  const bool left_out = wave == 0 && bx > 0;                    // halo left of the block inside the image
  const bool right_out = wave == nw - 1 && bx + 1 < gridDim.x;  // halo right of the block inside the image
  auto row_base = [&](const float* img, int r) {
    uint64_t row = reinterpret_cast<uint64_t>(img) + (uint64_t)(uint32_t)clampi(y0 + r - 2, 0, hm) * pitch;
    asm("" : "+s"(row));  // keeps the row base scalar: scalar base + 32-bit lane offset per load
    return row;
  };
  float e0[R + 4], e1[R + 4];
  if (left_out || right_out) {  // wave-uniform (same address in every lane), issued before the window rows
    const unsigned hc = (left_out ? xb - 2u : xb + (unsigned)kBandCols) * 4u;
#pragma unroll
    for (int r = 0; r < R + 4; ++r) {
      const uint64_t row = row_base(a.in, r);
      e0[r] = *reinterpret_cast<const GlobalF32*>(row + hc);
      e1[r] = *reinterpret_cast<const GlobalF32*>(row + hc + 4u);
    }
  }
  float4 v[R + 4];
#pragma unroll
  for (int r = 0; r < R + 4; ++r) {
    const v4f_t t = *reinterpret_cast<const GlobalV4f*>(row_base(a.in, r) + x * 4u);
    v[r] = make_float4(t.x, t.y, t.z, t.w);
  }
  const float g0 = a.g0, g1 = a.g1, g2 = a.g2;
  auto vert = [&](float t0, float t1, float t2, float t3, float t4) {
    float acc = g0 * t0;
    acc = fmaf(g1, t1, acc);
    acc = fmaf(g2, t2, acc);
    acc = fmaf(g1, t3, acc);
    return fmaf(g0, t4, acc);
  };
  float4 c[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    c[r] = make_float4(vert(v[r].x, v[r + 1].x, v[r + 2].x, v[r + 3].x, v[r + 4].x),
                       vert(v[r].y, v[r + 1].y, v[r + 2].y, v[r + 3].y, v[r + 4].y),
                       vert(v[r].z, v[r + 1].z, v[r + 2].z, v[r + 3].z, v[r + 4].z),
                       vert(v[r].w, v[r + 1].w, v[r + 2].w, v[r + 3].w, v[r + 4].w));
  if (left_out || right_out) {
    // the outer pair, vertical pass, published by the lane that borders it
    float2* dst = left_out ? &hi[0][0] : &lo[nw + 1][0];
    if (lane == (left_out ? 0 : 63))
#pragma unroll
      for (int r = 0; r < R; ++r)
        dst[r] = make_float2(vert(e0[r], e0[r + 1], e0[r + 2], e0[r + 3], e0[r + 4]),
                             vert(e1[r], e1[r + 1], e1[r + 2], e1[r + 3], e1[r + 4]));
  }
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < R; ++r) lo[wave + 1][r] = make_float2(c[r].x, c[r].y);
    if (wave == 0 && bx == 0)  // image border: the clamped columns repeat column 0
#pragma unroll
      for (int r = 0; r < R; ++r) hi[0][r] = make_float2(c[r].x, c[r].x);
  } else if (lane == 63) {
#pragma unroll
    for (int r = 0; r < R; ++r) hi[wave + 1][r] = make_float2(c[r].z, c[r].w);
    if (wave == nw - 1 && bx + 1 == gridDim.x)  // image border: column w - 1 repeated
#pragma unroll
      for (int r = 0; r < R; ++r) lo[nw + 1][r] = make_float2(c[r].w, c[r].w);
  }
  __syncthreads();
  // lane 0 takes the left neighbour's last pair, every other lane the right
  // neighbour's first pair (only lane 63 uses it)
  const float2* halo = lane == 0 ? &hi[wave][0] : &lo[wave + 2][0];
  float2 f[R];
#pragma unroll
  for (int r = 0; r < R; ++r) f[r] = halo[r];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const float cc[8] = {from_left(c[r].z, f[r].x), from_left(c[r].w, f[r].y), c[r].x, c[r].y,
                         c[r].z, c[r].w, from_right(c[r].x, f[r].x), from_right(c[r].y, f[r].y)};
    float o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = vert(cc[j], cc[j + 1], cc[j + 2], cc[j + 3], cc[j + 4]);
    const int y = y0 + r;
    if (y < h) {
      uint64_t orow = reinterpret_cast<uint64_t>(a.out) + (uint64_t)(uint32_t)y * pitch;
      asm("" : "+s"(orow));
      __builtin_nontemporal_store(make_v4f(o[0], o[1], o[2], o[3]), reinterpret_cast<GlobalV4f*>(orow + x * 4u));
    }
  }
}

template __global__ void k_gauss5_band_f32<4>(GaussArgs a);
template __global__ void k_gauss5_band_f32<8>(GaussArgs a);
template __global__ void k_gauss5_win_f32<2, true>(GaussArgs a);
template __global__ void k_gauss5_win_f32<4, true>(GaussArgs a);
template __global__ void k_gauss5_win_f32<2, false>(GaussArgs a);
template __global__ void k_gauss5_win_f32<4, false>(GaussArgs a);

// Sobel with the same window, vertical pass first.  The two 3x3 kernels
// factor into a vertical and a horizontal 3-tap pass: gx = horizontal
// difference of the vertical smoothing, gy = horizontal smoothing of the
// vertical difference.  Each lane forms both vertical terms for its 4 columns
// (lanes 0 and 63 also for the column beyond the wave's edge), then takes the
// neighbouring columns' terms by DPP lane shift.  Mask bytes of a lane go out
// as one 4-byte store, and their popcount is the lane's count for the row;
// each wave writes its own (count, sum) partial, so there is no block-wide
// barrier, and the final kernel combines the partials in a fixed order.
template <int R, bool FULL>
__global__ __launch_bounds__(kBlock) void k_sobel_thresh_win_f32(SobelArgs a) {
  unsigned bx, by;
  xcd_tile(bx, by);
  const int w = a.w, h = a.h, wm = w - 1, hm = h - 1;
  const WinLane<FULL> L(w, bx, by, R);
  const int xw = (int)bx * kWinCols;
  const unsigned hx = clampi(L.lane == 0 ? xw - 1 : xw + kWinCols, 0, wm);
  float4 v[R + 2];
  float e[R + 2];
#pragma unroll
  for (int r = 0; r < R + 2; ++r) {
    const float* row = a.blur + (size_t)clampi(L.y0 + r - 1, 0, hm) * w;
    v[r] = L.load4(row);
    e[r] = load1(row, hx);
  }
  const float thr = a.thr;
  float sum = 0.f;
  uint32_t cnt = 0;
  // GUARD: test each row against the image (the last row of blocks, and
  // lanes past a ragged right edge).  Full-width waves whose rows all lie
  // inside take the unguarded copy: their results are used unconditionally,
  // so the compiler keeps every load above this point (one memory round trip)
  // instead of sinking part of a row's load into the row's branch.  Both
  // copies accumulate in the same order.
  auto rows = [&](auto guard) {
    constexpr bool GUARD = decltype(guard)::value;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int y = L.y0 + r;
      float vs[4], vd[4];  // vertical smoothing (above + 2*centre + below) and difference (below - above)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float t0 = (&v[r].x)[j], t1 = (&v[r + 1].x)[j], t2 = (&v[r + 2].x)[j];
        vs[j] = (t0 + 2.f * t1) + t2;
        vd[j] = t2 - t0;
      }
      const float es = (e[r] + 2.f * e[r + 1]) + e[r + 2], ed = e[r + 2] - e[r];
      const float cs[6] = {from_left(vs[3], es), vs[0], vs[1], vs[2], vs[3], from_right(vs[0], es)};
      const float cd[6] = {from_left(vd[3], ed), vd[0], vd[1], vd[2], vd[3], from_right(vd[0], ed)};
      uint32_t packed = 0;
      float rsum;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float gx = cs[j + 2] - cs[j];
        const float gy = (cd[j] + 2.f * cd[j + 1]) + cd[j + 2];
        const float mag = sqrt_hw(gx * gx + gy * gy);
        packed |= (mag > thr ? 1u : 0u) << (8 * j);
        rsum = (j == 0) ? mag : rsum + mag;
      }
      if (!GUARD || (y < h && !L.past)) {
        uint8_t* mrow = a.mask + (size_t)y * w;  // wave-uniform row base
        store_nt(reinterpret_cast<uint32_t*>(mrow + L.x), packed);
        cnt += __builtin_popcount(packed);
        sum += rsum;
      }
    }
  };
  if (FULL && L.y0 + R <= h)
    rows(std::false_type{});
  else
    rows(std::true_type{});
  const float ws = wave_total_f32(sum);
  const uint32_t wc = wave_total_u32(cnt);
  if (L.lane == 0) {
    const unsigned part = (by * gridDim.x + bx) * 4 + (threadIdx.x >> 6);
    a.psum[part] = ws;
    a.pcount[part] = wc;
  }
}
template __global__ void k_sobel_thresh_win_f32<2, true>(SobelArgs a);
template __global__ void k_sobel_thresh_win_f32<4, true>(SobelArgs a);
template __global__ void k_sobel_thresh_win_f32<2, false>(SobelArgs a);
template __global__ void k_sobel_thresh_win_f32<4, false>(SobelArgs a);

// ------------------------------------------------------------------ thermal grid step
// T' = T + CP*P + CX*(N + S - 2T) + CX*(W + E - 2T) + CZ*(T_AMB - T), a
// neighbour outside the grid being the cell itself.  CZ = CX/64, so it is taken as
//   T' = T + [CX*((W + E - (4 + 1/64)*T) + (N + S)) + Q],  Q = CP*P + CZ*T_AMB,
// six instructions where the formula as it stands is nine, and Q once for all of
// a launch's steps.  4 + 1/64 is exact and every coefficient is CX's or CP's, so none
// of them heats or cools a grid by its rounding (a coefficient of 4 CX + CZ for T would:
// 1.7e-6 K a step, 80 times the formula's error on grids around zero).  The bracket is
// rounded at its own size and T once.  Largest error against float64 (96^2), the formula in
// float32 / so: grids of 320 to 340 K 1.3e-4 / 5.9e-5 over 8 steps and 2.4e-4 / 8.3e-5
// over 32; around zero (0 to 1) 9.2e-7 / 5.1e-7 and 5.3e-6 / 2.0e-6; 273 to 1000 K
// 5.1e-4 / 1.4e-4 over 32.  Finite while 4 |T| + 2 of the largest neighbour is.
namespace hotspot {
constexpr float CX = 0.1f, CP = 0.5f;
constexpr float OWN = 4.f + 1.f / 64.f;
constexpr float AMBIENT = (float)((double)CX / 64.0 * 300.0);
__device__ inline float source(float p) { return fmaf(CP, p, AMBIENT); }
__device__ inline float step(float t, float q, float n, float s, float w, float e) {
  return t + fmaf(CX, fmaf(-OWN, t, w + e) + (n + s), q);
}
}  // namespace hotspot

// One thread of a launch: the job's first writes its scalars into the slot, one
// that writes the output to host memory publishes its header there.
__device__ inline void hotspot_headers(const HotspotArgs& a) {
  if (a.first) write_slot_hdr(a.sc.hdr, a.js);
  if (a.publish) store_out(a.sc, load_out(a.sc, a.js), true);
}

// Register window as for the image stages: a lane owns 4 columns, a wave 256
// columns x kHotWinRows rows with its rows of T (plus one above and below)
// and of P loaded before the first result.
template <bool FULL>
__global__ __launch_bounds__(kBlock) void k_hotspot_win_f32(HotspotArgs a) {
  constexpr int R = kHotWinRows;
  unsigned bx, by;
  xcd_tile(bx, by);
  if (bx == 0 && by == 0 && threadIdx.x == 0) hotspot_headers(a);
  const int w = a.w, h = a.h, wm = w - 1, hm = h - 1;
  const WinLane<FULL> L(w, bx, by, R);
  const int xw = (int)bx * kWinCols;
  const unsigned hx = clampi(L.lane == 0 ? xw - 1 : xw + kWinCols, 0, wm);
  float4 v[R + 2], pv[R];
  float e[R + 2];
#pragma unroll
  for (int r = 0; r < R + 2; ++r) {
    const float* row = a.tin + (size_t)clampi(L.y0 + r - 1, 0, hm) * w;
    v[r] = L.load4(row);
    e[r] = load1(row, hx);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) pv[r] = L.load4(a.p + (size_t)clampi(L.y0 + r, 0, hm) * w);
  // Full-width waves whose rows all lie inside store unguarded, which keeps
  // every load (P's rows included) above this point: one memory round trip.
  auto rows = [&](auto guard) {
    constexpr bool GUARD = decltype(guard)::value;
#pragma unroll
    for (int r = 1; r <= R; ++r) {
      const int y = L.y0 + r - 1;
      const float c[6] = {from_left(v[r].w, e[r]), v[r].x, v[r].y, v[r].z, v[r].w, from_right(v[r].x, e[r])};
      const float n4[4] = {v[r - 1].x, v[r - 1].y, v[r - 1].z, v[r - 1].w};
      const float s4[4] = {v[r + 1].x, v[r + 1].y, v[r + 1].z, v[r + 1].w};
      const float p4[4] = {pv[r - 1].x, pv[r - 1].y, pv[r - 1].z, pv[r - 1].w};
      float o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = hotspot::step(c[j + 1], hotspot::source(p4[j]), n4[j], s4[j], c[j], c[j + 2]);
      if (!GUARD || (y < h && !L.past))
        store_nt(reinterpret_cast<float*>(reinterpret_cast<char*>(a.tout + (size_t)y * w) + L.x * 4u), o[0], o[1],
                 o[2], o[3]);
    }
  };
  if (FULL && L.y0 + R <= h)
    rows(std::false_type{});
  else
    rows(std::true_type{});
}
// Thermal step on row bands, for widths that are a multiple of kBandCols
// and grids of 2^22 to 2^24 cells: 8 waves side by side across R rows (8 up
// to 2^22 cells, 16 above), as the Gaussian's bands.  The halo is
// one raw column each side: lane 0 publishes its first column, lane 63 its
// last, for each of the R rows; after one barrier lanes 0 and 63 read the
// neighbouring waves' columns.  A block's outer columns inside the grid are
// loaded by its first and last wave; at the grid border the neighbour is the
// cell itself.  The per-cell arithmetic is the window kernel's.
template <int R>
__global__ __launch_bounds__(kBandCols / 4) void k_hotspot_band_f32(HotspotArgs a) {
  constexpr int nw = kBandCols / kWinCols;
  unsigned bx, band;
  xcd_tile(bx, band);  // grid (column blocks, bands)
  if (bx == 0 && band == 0 && threadIdx.x == 0) hotspot_headers(a);
  __shared__ float lo[nw + 2][R], hi[nw + 2][R];
  const int w = a.w, h = a.h, hm = h - 1;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int y0 = (int)band * R;
  const unsigned xb = bx * (unsigned)kBandCols;
  const unsigned x = xb + (unsigned)wave * kWinCols + 4u * (unsigned)lane;
  const uint32_t pitch = (uint32_t)w * 4u;
  const bool left_out = wave == 0 && bx > 0;
  const bool right_out = wave == nw - 1 && bx + 1 < gridDim.x;
  auto row_base = [&](const float* g, int r) {  // row y0 + r, clamped
    uint64_t row = reinterpret_cast<uint64_t>(g) + (uint64_t)(uint32_t)clampi(y0 + r, 0, hm) * pitch;
    asm("" : "+s"(row));
    return row;
  };
  float e[R];
  if (left_out || right_out) {
    const unsigned hc = (left_out ? xb - 1u : xb + (unsigned)kBandCols) * 4u;
#pragma unroll
    for (int r = 0; r < R; ++r) e[r] = *reinterpret_cast<const GlobalF32*>(row_base(a.tin, r) + hc);
  }
  float4 v[R + 2], pv[R];
#pragma unroll
  for (int r = 0; r < R + 2; ++r) {
    const v4f_t t = *reinterpret_cast<const GlobalV4f*>(row_base(a.tin, r - 1) + x * 4u);
    v[r] = make_float4(t.x, t.y, t.z, t.w);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const v4f_t t = *reinterpret_cast<const GlobalV4f*>(row_base(a.p, r) + x * 4u);
    pv[r] = make_float4(t.x, t.y, t.z, t.w);
  }
  if (left_out || right_out) {
    float* dst = left_out ? &hi[0][0] : &lo[nw + 1][0];
    if (lane == (left_out ? 0 : 63))
#pragma unroll
      for (int r = 0; r < R; ++r) dst[r] = e[r];
  }
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < R; ++r) lo[wave + 1][r] = v[r + 1].x;
    if (wave == 0 && bx == 0)
#pragma unroll
      for (int r = 0; r < R; ++r) hi[0][r] = v[r + 1].x;
  } else if (lane == 63) {
#pragma unroll
    for (int r = 0; r < R; ++r) hi[wave + 1][r] = v[r + 1].w;
    if (wave == nw - 1 && bx + 1 == gridDim.x)
#pragma unroll
      for (int r = 0; r < R; ++r) lo[nw + 1][r] = v[r + 1].w;
  }
  __syncthreads();
  const float* halo = lane == 0 ? &hi[wave][0] : &lo[wave + 2][0];
  float f[R];
#pragma unroll
  for (int r = 0; r < R; ++r) f[r] = halo[r];
#pragma unroll
  for (int r = 1; r <= R; ++r) {
    const int y = y0 + r - 1;
    const float c[6] = {from_left(v[r].w, f[r - 1]), v[r].x, v[r].y, v[r].z, v[r].w, from_right(v[r].x, f[r - 1])};
    const float n4[4] = {v[r - 1].x, v[r - 1].y, v[r - 1].z, v[r - 1].w};
    const float s4[4] = {v[r + 1].x, v[r + 1].y, v[r + 1].z, v[r + 1].w};
    const float p4[4] = {pv[r - 1].x, pv[r - 1].y, pv[r - 1].z, pv[r - 1].w};
    float o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = hotspot::step(c[j + 1], hotspot::source(p4[j]), n4[j], s4[j], c[j], c[j + 2]);
    if (y < h) {
      uint64_t orow = reinterpret_cast<uint64_t>(a.tout) + (uint64_t)(uint32_t)y * pitch;
      asm("" : "+s"(orow));
      __builtin_nontemporal_store(make_v4f(o[0], o[1], o[2], o[3]), reinterpret_cast<GlobalV4f*>(orow + x * 4u));
    }
  }
}
template __global__ void k_hotspot_band_f32<8>(HotspotArgs a);
template __global__ void k_hotspot_band_f32<16>(HotspotArgs a);
template __global__ void k_hotspot_win_f32<true>(HotspotArgs a);
template __global__ void k_hotspot_win_f32<false>(HotspotArgs a);

// Several steps in one launch.  A block holds a tile of 64 x 64 cells in
// registers (16 lanes of 4 columns by 16 groups of 4 rows: a group is a DPP
// row, so the left and right neighbours are lane shifts) and passes the groups'
// outer rows through LDS, one barrier a step.  What lies S = 4 HALO cells
// inside the tile's edge is right after up to S steps and is stored; tiles
// overlap by 2 S.  Cells beyond the grid are loaded as its mirror image: no heat
// crosses the border, so the image takes the same steps as the cells it
// mirrors, bit for bit (w + e and n + s commute), and the steps know no border.
// Nor do they know the tile's: its outer lanes take each other's values.
// The cells' arithmetic is the one-step kernels'.
// On a small grid a step is launch and memory latency, and 16 steps in one
// launch take about the time of three of one step; on a large one a launch is
// bound by the vector ALU (6 instructions a cell and step, 1.8 cells computed
// for each stored at S = 8; counted, 954 instructions a wave of 8 steps, issued for
// 11.5 of 17.0 us at 2048^2 and 34 of 46.7 at 4096^2, operands cached, 19.6 and 55.9
// us from memory) where one step was bound by memory.  64 jobs of
// 256^2 and 16 steps, a step / 16 to a launch: 1558 / 799 us; one of 2000 x 1500 and
// 32, a step / 8 to a launch: 942 / 765.
// The inner rows of a group are stepped between the LDS reads and their use:
// 8 steps of 4096^2 71.8 -> 62.3 us, 16 of 256^2 10.4 -> 10.1 us.  With 6
// instructions instead of 9 a cell, and the lane shifts within the additions
// (shifts that kept the edge lanes' own values cost two moves each), 50.6 and 8.4
// us, and 8 steps of 2000 x 1500 18.6 -> 14.8.
__device__ inline int mirror_index(int i, int n) {  // i any distance outside [0, n)
  if ((unsigned)i < (unsigned)n) return i;
  i = i < 0 ? -1 - i : i;
  if (i >= 2 * n) i %= 2 * n;  // tiles wider than the grid only
  return i < n ? i : 2 * n - 1 - i;
}
template <int HALO>
__global__ __launch_bounds__(kBlock) void k_hotspot_steps_f32(HotspotArgs a) {
  constexpr int R = 4, G = kBlock / 16, S = 4 * HALO, U = kHotTile - 2 * S;
  static_assert(G * R == kHotTile && 16 * 4 == kHotTile, "square tile");
  unsigned bx, by;
  xcd_tile(bx, by);
  if (bx == 0 && by == 0 && threadIdx.x == 0) hotspot_headers(a);
  __shared__ v4f_t s_top[2][G][16], s_bottom[2][G][16];
  const int lane = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int x = (int)bx * U - S + 4 * lane, y = (int)by * U - S + R * grp;
  size_t row[R];
#pragma unroll
  for (int r = 0; r < R; ++r) row[r] = (size_t)mirror_index(y + r, a.h) * a.w;
  v4f_t v[R], p[R];
  if (x >= 0 && x + 4 <= a.w) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      v[r] = *reinterpret_cast<const v4f_any*>(a.tin + row[r] + x);
      p[r] = *reinterpret_cast<const v4f_any*>(a.p + row[r] + x);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = mirror_index(x + j, a.w);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        v[r][j] = a.tin[row[r] + c];
        p[r][j] = a.p[row[r] + c];
      }
    }
  }
  v4f_t q[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < 4; ++j) q[r][j] = hotspot::source(p[r][j]);
  const int above = grp > 0 ? grp - 1 : 0, below = grp < G - 1 ? grp + 1 : G - 1;
  auto step_row = [&](v4f_t n, v4f_t t, v4f_t s, v4f_t qw) {
    const float c[6] = {row_from_left(t.w), t.x, t.y, t.z, t.w, row_from_right(t.x)};
    v4f_t o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = hotspot::step(c[j + 1], qw[j], n[j], s[j], c[j], c[j + 2]);
    return o;
  };
  s_top[0][grp][lane] = v[0];
  s_bottom[0][grp][lane] = v[R - 1];
  for (int k = 0;; ++k) {
    const int b = k & 1;
    __syncthreads();
    const v4f_t up = s_bottom[b][above][lane], down = s_top[b][below][lane];
    // the inner rows need no other group: they hide the LDS reads
    const v4f_t in1 = step_row(v[0], v[1], v[2], q[1]), in2 = step_row(v[1], v[2], v[3], q[2]);
    v[0] = step_row(up, v[0], v[1], q[0]);
    v[3] = step_row(v[2], v[3], down, q[3]);
    v[1] = in1;
    v[2] = in2;
    if (k + 1 == a.steps) break;
    s_top[b ^ 1][grp][lane] = v[0];
    s_bottom[b ^ 1][grp][lane] = v[R - 1];
  }
  if (lane < HALO || lane >= 16 - HALO || grp < HALO || grp >= G - HALO) return;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (y + r >= a.h) break;
    float* o = a.tout + (size_t)(y + r) * a.w + x;
    if (x + 4 <= a.w) {
      *reinterpret_cast<v4f_any*>(o) = v[r];
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (x + j < a.w) o[j] = v[r][j];
    }
  }
}
template __global__ void k_hotspot_steps_f32<1>(HotspotArgs a);
template __global__ void k_hotspot_steps_f32<2>(HotspotArgs a);
template __global__ void k_hotspot_steps_f32<3>(HotspotArgs a);
template __global__ void k_hotspot_steps_f32<4>(HotspotArgs a);

// Widths that are not a multiple of 4: one cell per thread.
__global__ __launch_bounds__(kBlock) void k_hotspot_f32(HotspotArgs a) {
  if (blockIdx.x == 0 && threadIdx.x == 0) hotspot_headers(a);
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= (int64_t)a.h * a.w) return;
  const int y = (int)(i / a.w), x = (int)(i - (int64_t)y * a.w);
  const int wm = a.w - 1, hm = a.h - 1;
  const float* T = a.tin;
  const float t = T[i];
  const float n = T[(size_t)clampi(y - 1, 0, hm) * a.w + x], s = T[(size_t)clampi(y + 1, 0, hm) * a.w + x];
  const float wv = T[(size_t)y * a.w + clampi(x - 1, 0, wm)], ev = T[(size_t)y * a.w + clampi(x + 1, 0, wm)];
  a.tout[i] = hotspot::step(t, hotspot::source(a.p[i]), n, s, wv, ev);
}

// One block: fixed-order combination of the partial counts and sums (one per
// wave on the window path, one per block on the LDS-tile path).
__device__ __forceinline__ void sobel_final(const SobelFinalArgs& a) {
  __shared__ float s4f[4];
  __shared__ uint32_t s4u[4];
  OutWords w{};
  if (threadIdx.x == 0) w = load_out(a.sc);
  // Thread t takes 16-byte groups t, t + 256, t + 512, ... (four partials
  // each), four groups per step with independent loads in flight, then the
  // last nparts % 4 partials.  The order depends only on nparts.  Both arrays
  // start 256-byte aligned.
  const float4* ps4 = reinterpret_cast<const float4*>(a.psum);
  const uint4* pc4 = reinterpret_cast<const uint4*>(a.pcount);
  const unsigned n4 = a.nparts >> 2;
  float s = 0.f;
  uint32_t c = 0;
  unsigned k = threadIdx.x;
  for (; k + 3 * kBlock < n4; k += 4 * kBlock) {
    float4 f[4];
    uint4 u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[i] = ps4[k + i * kBlock];
      u[i] = pc4[k + i * kBlock];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s += (f[i].x + f[i].y) + (f[i].z + f[i].w);
      c += (u[i].x + u[i].y) + (u[i].z + u[i].w);
    }
  }
  for (; k < n4; k += kBlock) {
    const float4 f = ps4[k];
    const uint4 u = pc4[k];
    s += (f.x + f.y) + (f.z + f.w);
    c += (u.x + u.y) + (u.z + u.w);
  }
  const unsigned t = 4 * n4 + threadIdx.x;
  if (t < a.nparts) {
    s += a.psum[t];
    c += a.pcount[t];
  }
  s = block_sum_f32(s, s4f);
  c = block_sum_u32(c, s4u);
  if (threadIdx.x == 0) {
    *a.out_count = c;
    *a.out_sum = s;
    store_out(a.sc, w, true);
  }
  complete_out(a.sc, w.h.seq);
}
__global__ __launch_bounds__(kBlock) void k_sobel_final(SobelFinalArgs a) { sobel_final(a); }
__global__ __launch_bounds__(kBlock) void k_copy_out_sobel(SobelFinalArgs a) { sobel_final(a); }

// ------------------------------------------------------------------ vector job: S = sum tanh(a*x + y)
// tanh in 33 instruction slots (a transcendental counts as four) where the
// library function takes about 45: two divergent branches, and most waves run
// both, which bounded every vector kernel on long jobs.  Here both forms are
// evaluated and one is selected:
//  |z| < 0.8: odd polynomial z + z*s*P(s), s = z^2.  P is the degree-5 minimax
//    fit of (tanh(z)/z - 1)/s, weighted to the relative error of the whole
//    (Lawson iteration over 4000 Chebyshev points; largest error 3.7e-9).
//  otherwise 1 - 2/(e + 1) with e = exp(2|z|) = 2^(2 log2(e) |z|) from the
//    hardware exponential and reciprocal (1 ulp each).  The rounding error of
//    the exponent and of its constant, lo, makes e short by e ln2 lo, which goes
//    in where a Newton step takes out the reciprocal's error.
//    |z| is capped at 10, where the result is 1 in float32 and e is finite.
// A NaN fails the comparison and leaves through the polynomial.
// Largest error in ulp over every float, library / this: 0.25 to 0.5 0.68 / 0.64,
// to 0.8 1.41 / 0.90, to 1 1.14 / 1.04, to 1.5 0.995 / 0.969, to 2 0.66 / 0.65, to
// 2.5 0.57 / 0.56, to 3 0.522 / 0.519, beyond the same.  Three instructions fewer,
// with lo added to e and the reciprocal as it comes, it was 1.32, 1.07 and 0.72 from
// 0.8 to 2, above the library's.
__device__ inline float tanh_f32(float z) {
  const float s = z * z;
  float p = fmaf(s, 0.00158475642f, -0.0074095577f);
  p = fmaf(s, p, 0.0213029906f);
  p = fmaf(s, p, -0.0538523309f);
  p = fmaf(s, p, 0.133322209f);
  p = fmaf(s, p, -0.333332986f);
  const float small = fmaf(z * s, p, z);
  const float w = fminf(fabsf(z), 10.f);
  const float x = w * 2.88539004f;  // 2 log2(e), rounded
  const float lo = fmaf(w, 3.851926e-08f, fmaf(w, 2.88539004f, -x));
  const float e = __builtin_amdgcn_exp2f(x), d = e + 1.f;
  float q = __builtin_amdgcn_rcpf(d);
  q = fmaf(q, fmaf(-e * (0.693147182f * lo), q, fmaf(-d, q, 1.f)), q);
  const float big = copysignf(fmaf(-2.f, q, 1.f), z);
  return fabsf(z) >= 0.8f ? big : small;
}

// Four elements of sum tanh(a*x + y).
__device__ inline float vec_quad(float av, v4f_any xv, v4f_any yv) {
  return (tanh_f32(fmaf(av, xv.x, yv.x)) + tanh_f32(fmaf(av, xv.y, yv.y))) +
         (tanh_f32(fmaf(av, xv.z, yv.z)) + tanh_f32(fmaf(av, xv.w, yv.w)));
}

// Thread's share of sum tanh(a*x + y) over len elements, by a block of BLOCK
// threads: thread j takes the 4-element groups j, j + BLOCK, ... in order, and
// thread 0 the last len % 4 elements.  The order depends on len and BLOCK only.
// U groups (2 U 16-byte loads a thread) are in flight at once; with one, a block
// moved 32 bytes a thread per memory round trip, and calls of a few long jobs
// were bound by latency.  U = 4 keeps the kernel within 64 registers, so that
// eight waves fit a SIMD.
// x, y and len are the same in every thread.
template <int BLOCK>
__device__ __forceinline__ float vec_range_sum(const float* x, const float* y, float av, uint64_t len) {
  constexpr int U = 4;
  constexpr uint64_t kRow = 16ull * BLOCK;  // bytes of one row of groups
  const uint64_t ng = len >> 2;
  const uint32_t off = 16u * threadIdx.x;
  uint64_t px = reinterpret_cast<uint64_t>(x), py = reinterpret_cast<uint64_t>(y);
  auto load = [&](uint64_t base) {
    uint32_t o = off;
    asm("" : "+s"(base), "+v"(o));  // scalar row base + 32-bit lane offset
    return *reinterpret_cast<const v4f_any __attribute__((address_space(1)))*>(base + o);
  };
  float acc = 0.f;
  auto quad = [&](v4f_any xv, v4f_any yv) { return vec_quad(av, xv, yv); };
  uint64_t g = 0;
  for (; g + U * BLOCK <= ng; g += U * BLOCK) {
    v4f_any xv[U], yv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      xv[u] = load(px + kRow * u);
      yv[u] = load(py + kRow * u);
    }
    __builtin_amdgcn_sched_barrier(0);  // every load goes out before the first result is formed
#pragma unroll
    for (int u = 0; u < U; ++u) acc += quad(xv[u], yv[u]);
    px += kRow * U;
    py += kRow * U;
  }
  // Less than U rows of groups are left, the last perhaps part of a row: all
  // loads first (a thread past the end loads nothing), then the sums.
  const uint32_t left = (uint32_t)(ng - g);
  v4f_any xv[U], yv[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u * BLOCK + threadIdx.x < left) {
      xv[u] = load(px + kRow * u);
      yv[u] = load(py + kRow * u);
    }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u * BLOCK + threadIdx.x < left) acc += quad(xv[u], yv[u]);
  if ((len & 3u) && threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < (int)(len & 3u)) acc += tanh_f32(fmaf(av, x[4 * ng + k], y[4 * ng + k]));
  }
  return acc;
}

// Block b reduces elements [b*C, min((b+1)*C, n)), C = vec_chunk(n, grid).
__global__ __launch_bounds__(kBlock) void k_saxpy_tanh_sum_f32(VecArgs a) {
  __shared__ float s4f[4];
  const JobScalars js = a.js;
  if (blockIdx.x == 0 && threadIdx.x == 0) write_slot_hdr(a.hdr, js);
  const uint64_t n = js.n;
  const uint64_t C = vec_chunk(n, gridDim.x);
  const uint64_t beg = (uint64_t)blockIdx.x * C;
  const uint64_t end = beg + C < n ? beg + C : n;
  float acc = 0.f;
  if (beg < end) acc = vec_range_sum<kBlock>(a.x + js.x_off + beg, a.y + js.y_off + beg, js.a, end - beg);
  const float bs = block_sum_f32(acc, s4f);
  if (threadIdx.x == 0) a.partials[blockIdx.x] = bs;
}

// One block: the job's partials (vec_blocks(n) of them) in a fixed order.
// The job's block count comes from n in the slot header.  Every thread loads
// its kVecGridCap / kBlock possible partials beside that load (the scratch
// holds kVecGridCap of them) and adds those below the count, in the order of
// the one-partial-per-step loop: one memory round trip instead of two.
__device__ __forceinline__ void vec_final(const VecFinalArgs& a) {
  __shared__ double s_total[kBlock / 64];
  OutWords w{};
  if (threadIdx.x == 0) w = load_out(a.sc);
  static_assert(kVecGridCap % kBlock == 0, "whole partials per thread");
  constexpr int PER = kVecGridCap / kBlock;
  float v[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) v[i] = a.partials[threadIdx.x + i * kBlock];
  const unsigned G = vec_blocks(a.sc.hdr->n);
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (threadIdx.x + i * kBlock < G) s += v[i];
  s = wave_total_f64(s);
  if ((threadIdx.x & 63) == 0) s_total[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    *a.out_sum = (float)((s_total[0] + s_total[1]) + (s_total[2] + s_total[3]));
    store_out(a.sc, w, true);
  }
  complete_out(a.sc, w.h.seq);
}
__global__ __launch_bounds__(kBlock) void k_vec_final(VecFinalArgs a) { vec_final(a); }
__global__ __launch_bounds__(kBlock) void k_copy_out_vec(VecFinalArgs a) { vec_final(a); }

// ------------------------------------------------------------------ vector batch: persistent (job, tile) kernel
// Pairwise sum of W values in a fixed tree ((s0+s1)+(s2+s3)) + ...
template <int W>
__device__ inline float tree_sum_f32(const float* s) {
  if constexpr (W == 1) {
    return s[0];
  } else {
    return tree_sum_f32<W / 2>(s) + tree_sum_f32<W / 2>(s + W / 2);
  }
}

// The job that owns tile t: the last descriptor whose first tile is <= t.  One
// wave; every round its 64 lanes test 64 evenly spaced descriptors, so a table
// of 4096 jobs takes two memory round trips where a binary search took twelve.
__device__ inline uint32_t vec_find_job(const VecBatchDesc* D, uint32_t count, uint32_t t) {
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t lo = 0, n = count;  // the job is in [lo, lo + n), and D[lo] starts at or before t
  while (n > 1) {
    const uint32_t step = (n + 63) / 64;
    const uint32_t at = lane * step;
    const bool le = at < n && D[lo + at].tile_start <= t;
    const uint32_t k = (uint32_t)__builtin_popcountll(__ballot(le)) - 1;  // lane 0 always tests true
    lo += k * step;
    n = n - k * step < step ? n - k * step : step;
  }
  return lo;
}

// A block's tiles: `first`, then what next(t) names after tile t, up to T (both
// the same in every thread; only thread 0's next counts).  next is asked before
// a tile's loads, so that a claim is answered behind them.  Wave 0 finds the
// next tile's job and leaves its descriptor in LDS; one barrier ends a tile (the
// LDS words are double, so the next tile's writes cannot meet this one's
// reads).  A tile's partial depends on its job and BLOCK only, so which block
// takes it changes no result.  A table that the library did not plan may hold
// items past their job's end, which sum to nothing.
template <int BLOCK, class Next>
__device__ __forceinline__ void vec_tiles(const VecBatchDesc* D, uint32_t count, uint32_t T, uint32_t first, bool planned,
                                          const float* px, const float* py, float* partials, Next next) {
  constexpr int W = BLOCK / 64;
  __shared__ float s_sum[2][kVecUnitsPerItem][W];
  __shared__ uint32_t s_tile[2];
  __shared__ VecBatchDesc s_desc[2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  constexpr int kDescWords = sizeof(VecBatchDesc) / 4;
  auto publish = [&](uint32_t t, int slot) {  // wave 0: tile t and its job's descriptor
    if (t < T) {
      const uint32_t j = vec_find_job(D, count, t);
      if (lane < kDescWords)
        reinterpret_cast<uint32_t*>(&s_desc[slot])[lane] = reinterpret_cast<const uint32_t*>(D + j)[lane];
    }
    if (lane == 0) s_tile[slot] = t;
  };
  int cur = 0;
  if (wave == 0) publish(first, 0);
  __syncthreads();
  while (true) {
    const uint32_t t = __builtin_amdgcn_readfirstlane(s_tile[cur]);
    if (t >= T) break;
    const uint32_t after = next(t);
    const VecBatchDesc& d = s_desc[cur];
    auto scalar = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    auto scalar64 = [&](uint64_t v) { return (uint64_t)scalar((uint32_t)(v >> 32)) << 32 | scalar((uint32_t)v); };
    const uint32_t te = scalar(d.tile_elems), n = scalar(d.n);
    const uint32_t ue = planned ? scalar(d.unit_elems) : vec_unit_elems(te, BLOCK);
    const uint64_t beg = (uint64_t)(t - scalar(d.tile_start)) * te;
    const uint64_t len = beg + te < n ? te : beg < n ? n - beg : 0;
    const float av = __int_as_float((int)scalar((uint32_t)__float_as_int(d.a)));
    const float* x = px + scalar64(d.x_off) + beg;
    const float* y = py + scalar64(d.y_off) + beg;
    int units = 0;
    for (uint64_t u = 0; u < len; u += ue, ++units) {
      const float ws = wave_total_f32(vec_range_sum<BLOCK>(x + u, y + u, av, len - u < ue ? len - u : ue));
      if (lane == 0) s_sum[cur][units][wave] = ws;
    }
    if (wave == 0) publish(scalar(after), cur ^ 1);
    __syncthreads();
    if (threadIdx.x == 0) {
      float s = units > 0 ? tree_sum_f32<W>(s_sum[cur][0]) : 0.f;
      for (int u = 1; u < units; ++u) s += tree_sum_f32<W>(s_sum[cur][u]);
      partials[t] = s;
    }
    cur ^= 1;
  }
}

// A batch's tiles are claimed in runs of H->claim.  Block b starts with run b;
// further runs come from the batch's counter.
// Bound by memory from about 100 MB a call: 7.1 TB/s over jobs of 2^20 and more
// at every block size (256 threads: 6.7 before, with one pair of loads in
// flight and the atomic and a binary search ahead of each unit).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK, 8) void k_vec_batch_tiles(VecBatchArgs a) {
  if (blockIdx.x == 0 && threadIdx.x == 0) write_slot_hdr(a.hdr, a.js);
  const VecBatchHdr* H = reinterpret_cast<const VecBatchHdr*>(a.tab);
  const VecBatchDesc* D = reinterpret_cast<const VecBatchDesc*>(a.tab + sizeof(VecBatchHdr));
  const bool planned = H->planned == kVecPlanned;
  const uint32_t T = H->total_tiles, run = planned ? H->claim : 1u;
  const uint64_t first = (uint64_t)blockIdx.x * run, dealt = (uint64_t)gridDim.x * run;
  if (first >= T) return;
  uint32_t left = run;  // tiles of the run still to do, the current one included
  vec_tiles<BLOCK>(D, H->count, T, (uint32_t)first, planned, a.x, a.y, a.partials, [&](uint32_t t) {
    if (--left != 0) return t + 1;
    left = run;
    uint32_t after = T;
    if (T > dealt && threadIdx.x == 0) {
      const uint64_t u =
          dealt + (uint64_t)run * __hip_atomic_fetch_add(a.work, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      after = u < T ? (uint32_t)u : T;
    }
    return after;
  });
}
template __global__ void k_vec_batch_tiles<128>(VecBatchArgs);
template __global__ void k_vec_batch_tiles<256>(VecBatchArgs);
template __global__ void k_vec_batch_tiles<512>(VecBatchArgs);
template __global__ void k_vec_batch_tiles<1024>(VecBatchArgs);

// The tile kernel of a no-allocation call of at most kBlock jobs: every block
// plans the call for itself, a job a thread, in LDS, and block 0 leaves the
// table for the totals.  Tiles are dealt in turn, without a counter.  Without
// the planning kernel and the claims a small call takes 12-14 us instead of 17,
// and 64 uneven jobs (310 MB) 56 us instead of 70 (181 before the loads of
// vec_range_sum went out together).
__global__ __launch_bounds__(kBlock, 8) void k_vec_few_tiles(VecFewArgs a) {
  __shared__ VecBatchDesc s_table[kBlock];
  __shared__ uint32_t s_wave[kBlock / 64];
  const uint32_t j = threadIdx.x, lane = j & 63u, wave = j >> 6;
  VecBatchDesc d{};
  if (j < a.plan.count) d = vec_plan_job(a.plan, a.plan.jobs[j]);
  const uint32_t upto = wave_inclusive_u32(d.ntiles);  // within the wave, then over the waves
  if (lane == 63) s_wave[wave] = upto;
  __syncthreads();
  uint32_t before = 0, T = 0;
#pragma unroll
  for (uint32_t k = 0; k < kBlock / 64; ++k) {
    if (k < wave) before += s_wave[k];
    T += s_wave[k];
  }
  d.tile_start = before + upto - d.ntiles;
  s_table[j] = d;
  if (blockIdx.x == 0) {
    VecBatchHdr* H = reinterpret_cast<VecBatchHdr*>(a.plan.tab);
    if (j < a.plan.count) reinterpret_cast<VecBatchDesc*>(a.plan.tab + sizeof(VecBatchHdr))[j] = d;
    if (j == 0) {
      H->count = a.plan.count;
      H->total_tiles = T;
    }
  }
  __syncthreads();
  if (blockIdx.x >= T) return;
  vec_tiles<kBlock>(s_table, a.plan.count, T, blockIdx.x, true, a.x, a.y, a.partials,
                    [&](uint32_t t) { return gridDim.x < T - t ? t + gridDim.x : T; });
}

// Sum of one item of len elements by one wave, to the bit what the tile kernel's
// block of 256 threads makes of it: lane l stands for its threads l, l + 64, l +
// 128 and l + 192, whose loads go out together.
__device__ __forceinline__ float vec_item_wave(const float* x, const float* y, float av, uint32_t len) {
  static_assert(kBlock == 256, "four lanes' worth of threads");
  const uint32_t lane = threadIdx.x & 63u, ng = len >> 2;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  for (uint32_t g0 = lane; g0 - lane < ng; g0 += kBlock) {
    v4f_any xv[4], yv[4];
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (g0 + 64 * w < ng) {
        xv[w] = reinterpret_cast<const v4f_any*>(x)[g0 + 64 * w];
        yv[w] = reinterpret_cast<const v4f_any*>(y)[g0 + 64 * w];
      }
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (g0 + 64 * w < ng) s[w] += vec_quad(av, xv[w], yv[w]);
  }
  if ((len & 3u) && lane == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < (int)(len & 3u)) s[0] += tanh_f32(fmaf(av, x[4 * ng + k], y[4 * ng + k]));
  }
#pragma unroll
  for (int w = 0; w < 4; ++w) s[w] = wave_total_f32(s[w]);
  return tree_sum_f32<4>(s);
}

// A no-allocation call of short jobs in one launch: a block a job, a wave an item.
// Nothing to plan, to find or to add up behind another kernel: the block reads its
// own job, and wave 0 adds the items' sums in vec_job_total's order.
__global__ __launch_bounds__(1024, 8) void k_vec_short_jobs(VecShortArgs a) {
  __shared__ float s_item[kVecShortItems];
  const VecBatchDesc d = vec_plan_job(a.plan, a.plan.jobs[blockIdx.x]);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (uint32_t k = wave; k < d.ntiles; k += blockDim.x >> 6) {
    const uint32_t beg = k * d.tile_elems;
    const float s = vec_item_wave(a.x + d.x_off + beg, a.y + d.y_off + beg, d.a,
                                  d.n - beg < d.tile_elems ? d.n - beg : d.tile_elems);
    if ((threadIdx.x & 63) == 0) s_item[k] = s;
  }
  __syncthreads();
  if (wave == 0) {
    const float s = wave_total_f32(threadIdx.x < d.ntiles ? 0.f + s_item[threadIdx.x] : 0.f);
    if (threadIdx.x == 0) a.results[blockIdx.x] = d.n == 0 ? __builtin_nanf("") : s;
  }
}

// Job j = wave: its tiles' partials in a fixed order.  Block 0 also rewinds the
// work counter for the slot's next batch and publishes the header; or, where the
// output is small and goes to host memory, the block that arrives last does, with
// every job's result, which saves a batch its copy and its completion kernel:
// calls of 2 jobs 76 -> 68 us, 4 (as many batches) 117 -> 99, 64 196 -> 188, 1024
// 833 -> 816.
__global__ __launch_bounds__(kBlock) void k_vec_batch_final(VecBatchFinalArgs a) {
  const VecBatchHdr* H = reinterpret_cast<const VecBatchHdr*>(a.tab);
  VecBatchDesc* D = reinterpret_cast<VecBatchDesc*>(a.tab + sizeof(VecBatchHdr));
  const uint32_t j = blockIdx.x * kVecFinalJobs + (threadIdx.x >> 6);
  OutWords w{};
  if (threadIdx.x == 0) w = load_out(a.sc);
  if (j < H->count) {
    const float s = vec_job_total(a.partials + D[j].tile_start, D[j].ntiles,
                                  H->planned == kVecPlanned ? D[j].per_item : 1u);
    if ((threadIdx.x & 63) == 0) {
      if (a.arrivals)
        put_partial(&D[j].sum, s);
      else
        a.results[j] = s;
    }
  }
  if (a.arrivals ? !arrives_last(a.arrivals, blockIdx.x, gridDim.x) : blockIdx.x != 0) return;
  if (a.arrivals)
    for (uint32_t k = threadIdx.x; k < a.n; k += kBlock) a.results[k] = get_partial(&D[k].sum);
  if (threadIdx.x == 0) {
    *a.work = 0u;
    store_out(a.sc, w, true);
  }
  complete_out(a.sc, w.h.seq);
}

// ------------------------------------------------------------------ inclusive scan int32 -> int64
// Reduce-then-scan: tile sums, an exclusive scan of the tile sums in one
// block, then each tile scans itself from its offset.  Up to 2^21 elements a
// tile's block adds up the sums before its own instead, and up to 2^17 the input
// before its own, in one kernel: short scans are launches and latency.  Integer
// addition is exact, so any order gives the same sums; no block waits on another.

// Loads the kScanItems values thread tid owns in tile t (zeros past n).
__device__ inline void scan_load(const int32_t* in, uint64_t n, unsigned t, int tid, int64_t v[kScanItems]) {
  const uint64_t base = (uint64_t)t * kScanTile + (uint64_t)tid * kScanItems;
  if (base + kScanItems <= n) {
    const int4 p0 = *reinterpret_cast<const int4*>(in + base);
    const int4 p1 = *reinterpret_cast<const int4*>(in + base + 4);
    v[0] = p0.x; v[1] = p0.y; v[2] = p0.z; v[3] = p0.w;
    v[4] = p1.x; v[5] = p1.y; v[6] = p1.z; v[7] = p1.w;
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) v[k] = (base + k < n) ? (int64_t)in[base + k] : 0;
  }
}

// One DPP move of a 64-bit value (both halves): lanes whose source lies
// outside their row, or whose row or bank the masks leave out, read 0.
template <int CTRL, int ROWS, int BANKS>
__device__ inline int64_t dpp_i64(int64_t v) {
  const uint64_t u = (uint64_t)v;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, BANKS, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, BANKS, false);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Inclusive scan of one int64 per lane over the wave, in registers: adding
// the input shifted right by 1, 2 and 3 lanes gives each lane the sum of its
// 4-lane window; row_shr:4 into banks 1-3 and row_shr:8 into banks 2-3 extend
// that to the lane's prefix of its 16-lane row; row_bcast:15 into rows 1 and
// 3 and row_bcast:31 into rows 2 and 3 add the totals of the rows below.
__device__ inline int64_t wave_inclusive_i64(int64_t x) {
  int64_t v = x;
  v += dpp_i64<0x111, 0xf, 0xf>(x);  // row_shr:1
  v += dpp_i64<0x112, 0xf, 0xf>(x);  // row_shr:2
  v += dpp_i64<0x113, 0xf, 0xf>(x);  // row_shr:3
  v += dpp_i64<0x114, 0xf, 0xe>(v);  // row_shr:4
  v += dpp_i64<0x118, 0xf, 0xc>(v);  // row_shr:8
  v += dpp_i64<0x142, 0xa, 0xf>(v);  // row_bcast:15
  v += dpp_i64<0x143, 0xc, 0xf>(v);  // row_bcast:31
  return v;
}

// Exclusive block scan of one int64 per thread; returns the thread's exclusive
// prefix and the block total.
__device__ inline int64_t block_exclusive_i64(int64_t x, int64_t* s_wave, int64_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t inc = wave_inclusive_i64(x);
  __syncthreads();
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  int64_t wave_excl = 0;
  for (int i = 0; i < wave; ++i) wave_excl += s_wave[i];
  *total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
  return wave_excl + inc - x;
}

__global__ __launch_bounds__(kBlock) void k_scan_reduce_i32(ScanReduceArgs a) {
  __shared__ int64_t s_wave[4];
  const JobScalars js = a.js;
  const unsigned t = blockIdx.x;
  if (t == 0 && threadIdx.x == 0) write_slot_hdr(a.hdr, js);
  if ((uint64_t)t * kScanTile >= js.n) return;
  int64_t v[kScanItems];
  scan_load(a.in, js.n, t, threadIdx.x, v);
  int64_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) s += v[k];
  int64_t total;
  block_exclusive_i64(s, s_wave, &total);
  if (threadIdx.x == 0) a.tile_sum[t] = total;
}

// A thread's 8 tile sums are four 16-byte loads with no branch around them:
// past the last tile it re-reads the last 8-sum group (inside the scratch,
// which is padded to 256 bytes) and drops what lies beyond.
__global__ __launch_bounds__(kBlock) void k_scan_spine_i64(ScanSpineArgs a) {
  __shared__ int64_t s_wave[4];
  const unsigned T = scan_tiles(a.n);
  const unsigned last = (T - 1) & ~(unsigned)(kScanItems - 1);
  int64_t carry = 0;
  for (unsigned base = 0; base < T; base += kScanTile) {
    int64_t v[kScanItems];
    const unsigned i0 = base + threadIdx.x * kScanItems;
    const longlong2* g = reinterpret_cast<const longlong2*>(a.tile_sum + (i0 < last ? i0 : last));
#pragma unroll
    for (int q = 0; q < kScanItems / 2; ++q) {
      const longlong2 t = g[q];
      v[2 * q] = t.x;
      v[2 * q + 1] = t.y;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) v[k] = (i0 + k < T) ? v[k] : 0;
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) s += v[k];
    int64_t total;
    const int64_t ex = block_exclusive_i64(s, s_wave, &total);
    int64_t run = carry + ex;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (i0 + k < T) a.tile_excl[i0 + k] = run;
      run += v[k];
    }
    carry += total;
  }
  if (threadIdx.x == 0) publish_out(a.sc, true);
}

// Results are computed in the blocked order the loads use (8 consecutive
// elements per thread), then pass through LDS so that each store instruction
// of a wave writes one contiguous 1 KiB run: a thread's own 64-byte run would
// make every store instruction touch 32 lines a quarter each.
template <int PREFIX>
__global__ __launch_bounds__(kBlock) void k_scan_down_i32_i64(ScanDownArgs a) {
  constexpr int kPitch = kScanItems + 2;  // LDS row of a thread (padding spreads the banks, keeps 16-byte alignment)
  __shared__ int64_t s_wave[4];
  __shared__ int64_t s_before[4];
  __shared__ __align__(16) int64_t s_out[kBlock * kPitch];
  const uint64_t n = a.js.n;
  const unsigned t = blockIdx.x;
  if (PREFIX != SCAN_FROM_SPINE && t == 0 && threadIdx.x == 0) {
    if (PREFIX == SCAN_FROM_INPUT) {
      write_slot_hdr(a.sc.hdr, a.js);
      store_out(a.sc, load_out(a.sc, a.js), true);
    } else {
      publish_out(a.sc, true);
    }
  }
  if ((uint64_t)t * kScanTile >= n) return;
  // The thread's 8 values as two 16-byte loads with no branch around them,
  // then the tile's prefix, held at this point by the empty asm statement
  // (the compiler would otherwise load it after the block scan, or after
  // waiting for the data behind a branch: a second memory round trip).  So
  // one memory latency covers both.  A thread past the end reads the last
  // 8-value group instead and zeroes what lies beyond n: the slot's input
  // region is padded to 256 bytes, so a 32-byte group that starts below n
  // lies inside it.
  const uint64_t base = (uint64_t)t * kScanTile + (uint64_t)threadIdx.x * kScanItems;
  const uint64_t last = (n - 1) & ~(uint64_t)(kScanItems - 1);
  const uint64_t ld = base < last ? base : last;
  const int4 q0 = *reinterpret_cast<const int4*>(a.in + ld);
  const int4 q1 = *reinterpret_cast<const int4*>(a.in + ld + 4);
  int64_t tile_off = 0, before = 0;  // the block's, or a thread's share of it
  if constexpr (PREFIX == SCAN_FROM_SPINE) {
    tile_off = a.tiles[t];
    asm volatile("" ::"s"(tile_off) : "memory");
  } else if constexpr (PREFIX == SCAN_FROM_SUMS) {
    int64_t w[kScanSumTiles / kBlock];
#pragma unroll
    for (unsigned k = 0; k < kScanSumTiles / kBlock; ++k) {
      const unsigned i = threadIdx.x + k * kBlock;
      w[k] = a.tiles[i < t ? i : 0];
    }
#pragma unroll
    for (unsigned k = 0; k < kScanSumTiles / kBlock; ++k) before += threadIdx.x + k * kBlock < t ? w[k] : 0;
  } else {
    // two 16-byte words of each tile to a thread, 16 words going out together
    const unsigned words = t * (kScanTile / 4 / kBlock);
    for (unsigned k0 = 0; k0 < words; k0 += 16) {
      int4 w[16];
#pragma unroll
      for (unsigned k = 0; k < 16; ++k)
        w[k] = reinterpret_cast<const int4*>(a.in)[k0 + k < words ? threadIdx.x + (k0 + k) * kBlock : threadIdx.x & 1];
#pragma unroll
      for (unsigned k = 0; k < 16; ++k)
        before += k0 + k < words ? ((int64_t)w[k].x + w[k].y) + ((int64_t)w[k].z + w[k].w) : 0;
    }
  }
  int64_t v[kScanItems] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) v[k] = (base + k < n) ? v[k] : 0;
#pragma unroll
  for (int k = 1; k < kScanItems; ++k) v[k] += v[k - 1];
  if constexpr (PREFIX != SCAN_FROM_SPINE) {
    before = wave_inclusive_i64(before);
    if ((threadIdx.x & 63) == 63) s_before[threadIdx.x >> 6] = before;
  }
  int64_t total;
  int64_t off0 = block_exclusive_i64(v[kScanItems - 1], s_wave, &total);  // its barriers are s_before's too
  if constexpr (PREFIX != SCAN_FROM_SPINE) tile_off = (s_before[0] + s_before[1]) + (s_before[2] + s_before[3]);
  off0 += tile_off;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) s_out[threadIdx.x * kPitch + k] = off0 + v[k];
  __syncthreads();
  const uint64_t tile0 = (uint64_t)t * kScanTile;
  auto at = [&](int e) { return s_out[(e / kScanItems) * kPitch + (e % kScanItems)]; };
  if (!a.low32) {
    int64_t* o = reinterpret_cast<int64_t*>(a.out) + tile0;
    if (tile0 + kScanTile <= n) {
#pragma unroll
      for (int k = 0; k < kScanItems / 2; ++k) {
        const int e = 2 * (k * kBlock + (int)threadIdx.x);  // element pairs in striped order
        store_nt(o + e, at(e), at(e + 1));
      }
    } else {
      for (int e = threadIdx.x; e < kScanTile; e += kBlock)
        if (tile0 + e < n) o[e] = at(e);
    }
  } else {
    uint32_t* o = reinterpret_cast<uint32_t*>(a.out) + tile0;
    if (tile0 + kScanTile <= n) {
#pragma unroll
      for (int k = 0; k < kScanItems / 4; ++k) {
        const int e = 4 * (k * kBlock + (int)threadIdx.x);  // element quads in striped order
        store_nt(o + e, (uint32_t)at(e), (uint32_t)at(e + 1), (uint32_t)at(e + 2), (uint32_t)at(e + 3));
      }
    } else {
      for (int e = threadIdx.x; e < kScanTile; e += kBlock)
        if (tile0 + e < n) o[e] = (uint32_t)at(e);
    }
  }
}
template __global__ void k_scan_down_i32_i64<SCAN_FROM_INPUT>(ScanDownArgs a);
template __global__ void k_scan_down_i32_i64<SCAN_FROM_SUMS>(ScanDownArgs a);
template __global__ void k_scan_down_i32_i64<SCAN_FROM_SPINE>(ScanDownArgs a);

}  // namespace setrt
