// Tile geometry and grid sizes of the stage kernels.  Plain C++ so host-only
// code (slot layout, scheduler, fake backend) shares it without HIP headers.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define SETRT_HD __host__ __device__
#else
#define SETRT_HD
#endif

namespace setrt {

constexpr int kBlock = 256;
constexpr int kBoxTW = 64, kBoxTH = 16;       // 3x3 box: output tile
constexpr int kDivPerThread = 8;              // floor(s/9): pixels per thread
constexpr int kHistPerThread = 16;            // histogram: pixels per thread
constexpr int kGaussTW = 64, kGaussTH = 16;   // separable Gaussian: output tile
constexpr int kSobelTW = 64, kSobelTH = 16;   // Sobel: output tile
constexpr int kVecChunk = 2048;               // vector job: elements per block (multiple of 4*kBlock)
constexpr int kVecGridCap = 2048;             // vector job: most blocks per job
// Words that count a launch's blocks as they arrive: one to a group of blocks,
// in kArriveBytes of its own; the root is in the first group's.
constexpr unsigned kArriveGroup = 128;
constexpr unsigned kArriveBytes = 256;
SETRT_HD inline uint64_t arrival_bytes(uint64_t blocks) {
  return (blocks + kArriveGroup - 1) / kArriveGroup * kArriveBytes;
}
constexpr int kScanItems = 8;                 // scan: items per thread
constexpr int kScanTile = kBlock * kScanItems;
constexpr int kCopyBlocks = 32;               // host<->device copy kernels: small grid, PCIe-bound
// Device-to-host copies of 1 MiB and more take 64 blocks: with a host-to-device
// pull running beside them, 32 + 64 blocks moved 67 GB/s in both directions
// together against 57 GB/s for 32 + 32.
inline unsigned d2h_copy_blocks(uint64_t bytes) { return bytes >= (1ull << 20) ? 64u : (unsigned)kCopyBlocks; }
constexpr int kVecBatchGrid = 1024;           // persistent vector-batch kernel: default grid

// Default work-item size for vector jobs of size bucket b = floor(log2 n):
// about eight items per job, a multiple of 1024 elements, within [1024, 65536].
inline uint32_t vec_default_tile(int b) {
  uint64_t t = (b >= 3) ? (1ull << (b - 3)) : 1ull;
  t = (t + 1023) / 1024 * 1024;
  if (t < 1024) t = 1024;
  if (t > 65536) t = 65536;
  return (uint32_t)t;
}

// A work item's elements are summed in up to four equal units, whose sums are
// added in order.  Where the batch's units fit the partials of its template (a
// batch that is long has no need of it), a block takes a unit instead of an
// item, with the same result: so a few long jobs still give every compute unit
// work (one job of 2^22 elements has 64 items of the default size), and the
// last blocks to finish hold less.  A unit keeps at least 64 elements a thread,
// four rounds of vec_range_sum's loads: after a unit of one round a block's
// waves are in step, loading and then computing together (1024 threads, jobs of
// 2^20 and more: 6.7 TB/s with 16384-element units against 6.9 with whole items
// of 65536).  Items are multiples of 1024, so units are multiples of 256; one that is
// not (a table submitted by hand, a serving call's tuning) stays whole, since it has
// no four equal parts.
SETRT_HD inline uint32_t vec_unit_elems(uint32_t item_elems, int block) {
  if (item_elems % 1024u) return item_elems;
  const uint32_t least = 64u * (uint32_t)block;
  return item_elems / 4u >= least ? item_elems / 4u : item_elems / 2u >= least ? item_elems / 2u : item_elems;
}
// Units a block claims at a time.  A claim is an atomic on one word of the whole
// device, which takes them at about 70 a microsecond: units of 1024 elements,
// claimed one by one, cannot run faster than 0.6 TB/s.  So short units are
// claimed in runs of about 16384 elements (what a longer unit holds by itself),
// and of at most a block's even share: then nothing is left to claim.  1024
// jobs of 4096 to 8192 elements: 91 us one by one, 30 us in runs.
SETRT_HD inline uint32_t vec_claim(uint64_t elems, uint32_t units, uint32_t grid) {
  if (units == 0 || grid == 0) return 1;
  // in float32 and 32 bits: the planning kernel's one thread took 2 us over the
  // divisions of 64 bits, and no result depends on the claim
  const uint32_t c = (uint32_t)(16384.f * (float)units / ((float)elems + (float)units));
  const uint32_t share = (units - 1) / grid + 1;
  return c < 1 ? 1 : c < share ? c : share;
}
constexpr int kVecUnitsPerItem = 4;  // most units of one work item
// A no-allocation call whose jobs have at most this many work items, of at most
// kVecShortItem elements each, takes a block to a job and a wave to an item.  In
// us, planned / so: 1 to 256 jobs of up to 8192 12.5-14 / 10-11, 1000 22.9 / 12.6,
// 2000 34.7 / 19.3, 2000 of up to 32767 61.6 / 42.6.  A wave takes a longer item in
// rounds of one memory latency each, and the largest job sets the time: items of
// 4096 took 300 jobs of up to 65535 21.2 / 22.8 (1000 46.5 / 41.1), of 8192 64 of up
// to 131071 14.1 / 24.6.
constexpr uint32_t kVecShortItems = 16;
constexpr uint32_t kVecShortItem = 2048;
constexpr int kVecFinalJobs = 4;     // jobs per block of the batch's last kernel: one wave each
// Up to this many jobs to a batch, the last block of that kernel writes the results
// to host memory, four to a thread; longer ones are left to the copy kernel's 32
// blocks.
constexpr uint32_t kVecFinishJobs = 1024;

struct Grid3 {
  unsigned x, y, z;
};

inline Grid3 box_grid(int h, int w) {
  return {(unsigned)((w + kBoxTW - 1) / kBoxTW), (unsigned)((h + kBoxTH - 1) / kBoxTH), 1u};
}
inline unsigned div9_blocks(int64_t npix) {
  return (unsigned)((npix + (int64_t)kBlock * kDivPerThread - 1) / ((int64_t)kBlock * kDivPerThread));
}
inline unsigned hist_blocks(int64_t npix) {
  return (unsigned)((npix + (int64_t)kBlock * kHistPerThread - 1) / ((int64_t)kBlock * kHistPerThread));
}
// Box sums, quotients and histogram in one kernel (templates without
// intermediate images): tiles of 4096 pixels, at most a block for each compute unit
// (one block combines the partial rows: of 2048^2 pixels 1024 rows took it 34
// us, 256 take it 4.6) and for each partial row of the slot's scratch, which
// hist_blocks sizes (ragged grids have more tiles).  A tile is 64 x 64, four
// pixels to a thread, unless half of it would lie beside a narrow image: it is then
// halved in width and doubled in height, or the other way round.  One job, us, at
// 64 x 64 / so: 1 x 262144 72 / 28, 262144 x 1 59 / 26, 65536 x 4 33 / 26 (the three
// kernels that return the images 44, 34, 32).
constexpr int kBoxHistBlock = 1024;
constexpr int kHistFinalBlock = 1024;
// log2 of the threads across a tile: 4 << s columns, kBoxHistBlock >> s rows.
inline int box_hist_shift(int h, int w) {
  int s = 4;
  while (s > 0 && w <= 2 << s) --s;
  while (s < 10 && 2 * (int64_t)h <= kBoxHistBlock >> s) ++s;
  return s;
}
inline unsigned box_hist_blocks(int h, int w) {
  const int s = box_hist_shift(h, w), tw = 4 << s, th = kBoxHistBlock >> s;
  const uint64_t t = (((uint64_t)w + tw - 1) / tw) * (((uint64_t)h + th - 1) / th);
  const unsigned hb = hist_blocks((int64_t)h * w);
  const uint64_t b = t < hb ? t : hb;
  return (unsigned)(b < 256 ? b : 256);
}
// Float images whose width is a multiple of 4 take the register-window
// kernels: a lane owns 4 adjacent columns (16-byte loads and stores), a wave
// 256 columns x R rows, a block 4 waves stacked vertically.  The Gaussian
// takes R = 2 below 1024^2 pixels and Sobel up to 1024^2, both R = 4 above
// (more blocks in flight pay on the smaller images, fewer re-read halo rows on
// the larger).  Other widths take the LDS-tile kernels.  The Gaussian of
// widths that are multiples of kBandCols takes the row-band kernel instead.
constexpr int kWinCols = 256;                 // columns per wave (and per block)
// Gaussian row bands for widths that are a multiple of kBandCols: blocks of
// 8 waves side by side (2048 columns) across R rows, R = 8 up to 4096^2
// pixels and 4 above.  Measured on cold buffers (window kernel / band R = 4 /
// band R = 8): 8.6 / 8.1 / 7.2 us at 2048^2, 29.2 / 28.3 / 28.0 us at 4096^2,
// 99.7 / 92.4 / 94.3 us at 8192^2.  At 1024^2 (blocks of 4 waves across the
// width) a 4-row band was the slower, 3.7 against 3.6 us, and 16-wave blocks
// across 4096 columns took 31 us.
constexpr int kBandCols = 2048;
inline bool gauss_band_path(int w) { return w > 0 && (w % kBandCols) == 0; }
inline int gauss_band_rows(int h, int w) { return (int64_t)h * w <= (int64_t)4096 * 4096 ? 8 : 4; }
inline bool image_window_path(int w) { return w > 0 && (w % 4) == 0; }
// Every tile of the window path full width: no lane lies past the right edge.
inline bool window_full_width(int w) { return w > 0 && (w % kWinCols) == 0; }
inline int gauss_win_rows(int h, int w) { return (int64_t)h * w < (int64_t)1024 * 1024 ? 2 : 4; }
inline int sobel_win_rows(int h, int w) { return (int64_t)h * w <= (int64_t)1024 * 1024 ? 2 : 4; }
inline Grid3 window_grid(int h, int w, int rows_per_wave) {
  const int rows = 4 * rows_per_wave;
  return {(unsigned)((w + kWinCols - 1) / kWinCols), (unsigned)((h + rows - 1) / rows), 1u};
}
inline Grid3 gauss_grid(int h, int w) {
  if (gauss_band_path(w)) {
    const int r = gauss_band_rows(h, w);
    return {(unsigned)(w / kBandCols), (unsigned)((h + r - 1) / r), 1u};
  }
  if (image_window_path(w)) return window_grid(h, w, gauss_win_rows(h, w));
  return {(unsigned)((w + kGaussTW - 1) / kGaussTW), (unsigned)((h + kGaussTH - 1) / kGaussTH), 1u};
}
inline Grid3 sobel_grid(int h, int w) {
  if (image_window_path(w)) return window_grid(h, w, sobel_win_rows(h, w));
  return {(unsigned)((w + kSobelTW - 1) / kSobelTW), (unsigned)((h + kSobelTH - 1) / kSobelTH), 1u};
}
// Sobel's partial (count, sum) pairs: one per wave on the window path, one per
// block on the LDS-tile path.
inline uint64_t sobel_partials(int h, int w) {
  const Grid3 g = sobel_grid(h, w);
  return (uint64_t)g.x * g.y * (image_window_path(w) ? 4u : 1u);
}
// Gaussian and Sobel in one kernel (templates without intermediate images), 64
// x 16 tiles of 512 threads: below 1024^2 pixels, and at any size for widths
// that are not a multiple of 4, whose pair of kernels stages tiles in LDS as
// well, twice.  Four jobs in the synchronous model, us, as a pair / in one:
// 128^2 93 / 80, 333 x 250 117 / 103, 512^2 161 / 155, 1023 x 700 306 / 293,
// 1501 x 1400 722 / 703; one of 4097^2 1264 / 1260, of 16383 x 16381, near the largest
// allowed, 19834 / 19830; on the register windows 1024^2 390 / 384 and 2048^2
// 1300 / 1309, so the line is drawn where the pair's second pass over memory
// stops costing more than the one kernel's passes through LDS.
constexpr int kGsBlock = 512;
inline bool gauss_sobel_in_one(int h, int w) { return !image_window_path(w) || (int64_t)h * w < (int64_t)1024 * 1024; }
inline Grid3 gauss_sobel_grid(int h, int w) {
  return {(unsigned)((w + kSobelTW - 1) / kSobelTW), (unsigned)((h + kSobelTH - 1) / kSobelTH), 1u};
}
// Thermal-grid step: the register window (4 columns x kHotWinRows rows per
// lane) for widths that are multiples of 4, one pixel per thread otherwise.
constexpr int kHotWinRows = 2;
// Row bands (the Gaussian's layout) for widths that are a multiple of
// kBandCols and grids of 2^22 to 2^24 cells: 8 rows per band up to 2^22
// cells, 16 above; 0 = not the band path.  Measured cold per step (window /
// 8-row / 16-row band): 10.3 / 9.0 / 10.4 us at 2048^2, 10.3 / 9.4 us at
// 4096x1024, 38.9 / 39.6 / 37.4 us at 4096^2; at 2048x1024 the 8-row band
// was the slower (6.9 against 6.1 us).
inline int hotspot_band_rows(int h, int w) {
  const int64_t n = (int64_t)h * w;
  if (w <= 0 || (w % kBandCols) != 0 || n < ((int64_t)1 << 22) || n > ((int64_t)1 << 24)) return 0;
  return n <= ((int64_t)1 << 22) ? 8 : 16;
}
inline Grid3 hotspot_grid(int h, int w) {
  if (const int r = hotspot_band_rows(h, w)) return {(unsigned)(w / kBandCols), (unsigned)((h + r - 1) / r), 1u};
  if (image_window_path(w)) return window_grid(h, w, kHotWinRows);
  const uint64_t n = (uint64_t)h * w;
  return {(unsigned)((n + kBlock - 1) / kBlock), 1u, 1u};
}
// Steps of a job that one launch takes (k_hotspot_steps_f32): up to 16 on grids
// of 512^2 cells or fewer, 8 above; K steps are dealt evenly over the launches,
// and a launch of one step takes the one-step kernels.  The tile's halo is the
// steps rounded up to 4 cells.  On a small grid a launch is latency and more
// steps cost little; on a large one the halo's cells are computed for nothing
// (3 of 4 at 16 steps).  One job, us from submit to drained, at 1 (the one-step
// kernels) / 4 / 8 / 16 steps a launch: 256^2, K = 16: 98 / 74 / 64 / 62;
// 512^2, K = 16: 145 / 132 / 122 / 120; 700^2, K = 16: 216 / 177 / 169 / 169; 1024^2,
// K = 16: 339 / 324 / 307 / 311; 2000 x 1500, K = 32: 942 / 785 / 765 / 784; 4096^2,
// K = 16: 4214 / 3824 / 3766 / 3838; 64 jobs of 256^2 1558 / 961 / 850 / 799.
// The one-step kernels serve jobs of one step: cold, us, one of them / the steps kernel
// with one step: 64^2 2.9 / 4.6, 333 x 250 7.7 / 9.2, 1024^2 3.8 / 6.8, 2048^2 8.8 /
// 13.7, 8192^2 135 / 160 (of eleven sizes only odd 4099^2 the other way, 52 / 45).
constexpr int kHotTile = 64;
// Up to this many cells a job's last launch writes the grid to host memory itself.
// Jobs, us, with an output copy / so: 64 of 32^2 402-465 / 354-396, one 47-51 / 40,
// 64 of 128^2 658 / 601, of 256^2 891 / 871, 32 of 333^2 746 / 731; from 512^2 up
// the link sets the time either way, and its stores hold the launch's blocks.
constexpr int64_t kHotHostCells = 1 << 17;
inline int hotspot_steps_max(int h, int w) { return (int64_t)h * w <= (int64_t)512 * 512 ? 16 : 8; }
inline int hotspot_launches(int h, int w, int K) {
  const int m = hotspot_steps_max(h, w);
  return (K + m - 1) / m;
}
inline int hotspot_steps(int h, int w, int K, int launch) {
  const int n = hotspot_launches(h, w, K);
  return K / n + (launch < K % n ? 1 : 0);
}
inline int hotspot_halo(int steps) { return (steps + 3) / 4; }
inline Grid3 hotspot_steps_grid(int h, int w, int halo) {
  const int u = kHotTile - 8 * halo;
  return {(unsigned)((w + u - 1) / u), (unsigned)((h + u - 1) / u), 1u};
}
// Vector job: blocks for length n.  Deterministic in n, so the reduction
// order of a job depends only on its length.
SETRT_HD inline unsigned vec_blocks(uint64_t n) {
  uint64_t b = (n + kVecChunk - 1) / kVecChunk;
  if (b < 1) b = 1;
  if (b > (uint64_t)kVecGridCap) b = kVecGridCap;
  return (unsigned)b;
}
// Elements per block for length n over g blocks (a multiple of 4*kBlock).
SETRT_HD inline uint64_t vec_chunk(uint64_t n, unsigned g) {
  uint64_t c = (n + g - 1) / g;
  const uint64_t q = 4ull * kBlock;
  return (c + q - 1) / q * q;
}
SETRT_HD inline unsigned scan_tiles(uint64_t n) { return (unsigned)((n + kScanTile - 1) / kScanTile); }
// Where a downsweep block has the sum of the tiles before its own from, by the
// template's largest length: it adds up to kScanRawTiles - 1 tiles of the input
// itself (one kernel a job, which also writes the output to host memory), up to
// kScanSumTiles - 1 tile sums (two kernels), or reads the spine's prefix (three).
// 32 jobs, us, three kernels and a copy / two / one: 1000 elements 258 / 227 / 202,
// 16000 341 / 330 / 282, 65000 - / 546 / 488, 100000 842 / 813 / 717, 130000 - / 958 /
// 860; from there the input is read too often (200000 by one kernel: one job 98 /
// 104), and output written by the downsweep is held up in its many blocks (2^21,
// one job 540 / 595, where two kernels and a copy take what three took).  Where the
// output goes by a memcpy node or a copy kernel all the same (to_host false), one
// kernel saves less and its reading shows earlier: 24 jobs, us, three / one, 16384
// elements 881 / 810, 32768 940 / 916, 50000 1017 / 1040, 131072 1432 / 1600.
constexpr unsigned kScanRawTiles = 64, kScanRawTilesCopied = 16, kScanSumTiles = 1024;
enum { SCAN_FROM_INPUT, SCAN_FROM_SUMS, SCAN_FROM_SPINE };
inline int scan_prefix(uint64_t max_n, bool to_host) {
  const unsigned t = scan_tiles(max_n);
  return t <= (to_host ? kScanRawTiles : kScanRawTilesCopied) ? SCAN_FROM_INPUT : t <= kScanSumTiles ? SCAN_FROM_SUMS : SCAN_FROM_SPINE;
}

// Byte layout of one buffer slot of a template (offsets from the slot base,
// all 256-byte aligned).  In debug templates the intermediate images live
// inside the output block so the D2H copy returns them.
struct SlotLayout {
  uint64_t hdr;        // DevSlotHdr
  uint64_t in;         // H2D destination
  uint64_t in_cap;
  uint64_t out;        // output block: set_out_header + payload (+ debug images)
  uint64_t out_cap;
  uint64_t b1, b2;     // intermediates (box: S, Q in debug templates; gauss: blur, mask, or arrival words)
  uint64_t scratch;    // partials, counters, tile states
  uint64_t scratch_bytes;
  uint64_t tail;       // tail canary
  uint64_t total;
};

}  // namespace setrt
