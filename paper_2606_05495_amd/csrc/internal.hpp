// Internal declarations shared by the scheduler core, the HIP backend and the
// CPU fake backend.  Nothing here is part of the C ABI.
#pragma once

#include <atomic>
#include <chrono>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <string>

#include "set.h"
#include "tiles.hpp"

namespace setrt {

inline uint64_t now_ns() {
  return (uint64_t)std::chrono::duration_cast<std::chrono::nanoseconds>(
             std::chrono::steady_clock::now().time_since_epoch())
      .count();
}

// Message that set_last_error(NULL) returns on the calling thread (calls
// that have no context: a failed set_ctx_create, the no-allocation call).
void set_thread_error(const std::string& msg);

// Threads per block of the vector-batch work-item kernel of template t.
inline int vec_batch_block(const set_job_template& t) { return t.block > 0 ? t.block : kBlock; }

constexpr int kMaxWorkers = 256;     // b: workers (streams) of a context
constexpr int kMaxThreads = 64;      // dispatcher threads, input-copy streams
constexpr int kStatWorkers = 64;     // workers whose launches set_stats lists
constexpr int kMaxSlots = 64;
constexpr int kMaxTemplates = 16;
constexpr int kMaxStages = 40;
constexpr int kMaxHotspotSteps = 32;  // thermal-grid template: steps per job (one kernel each)

// Per-job scalar arguments.  Passed by value to the first kernel of a chain
// (a kernel-node placeholder, Section 4.1) and written by it into the slot's
// device header, where later stages read it.
struct JobScalars {
  uint64_t job_id;
  uint64_t seq;
  uint64_t user_tag;
  uint64_t n;
  uint64_t x_off;
  uint64_t y_off;
  uint32_t worker;
  uint32_t slot;
  float a;
  uint32_t flags;
};
static_assert(sizeof(JobScalars) == 64, "JobScalars layout");

// Device-side slot header (first bytes of every slot).  The first stage of a
// job writes job_id/seq/worker/slot/user_tag; the last stage copies them into
// the output header after checking the head and tail canaries.
struct DevSlotHdr {
  uint64_t canary_head;
  uint64_t job_id;
  uint64_t seq;
  uint64_t user_tag;
  uint32_t worker;
  uint32_t slot;
  uint64_t n;  // job length (vector / scan pipelines), read by later stages
  uint32_t pad[4];
};
static_assert(sizeof(DevSlotHdr) == 64, "DevSlotHdr layout");
static_assert(sizeof(set_out_header) == 64, "set_out_header layout");
static_assert(sizeof(set_config) == 104, "set_config layout");
static_assert(sizeof(set_job_template) == 96, "set_job_template layout");

// Descriptor table of a vector batch (host-written, copied to the slot by
// the batch's H2D): a 64-byte header, then one 48-byte descriptor per job.
// Each job carries its own work-item size, so one batch may mix size buckets
// while every job's result still depends only on (n, its item size).  A tile is
// what a block takes: a work item, or one of its units (vec_unit_elems).
// `claim`, `unit_elems` and `per_item` are read only where `planned` says that the
// library built the table: in one submitted by hand they are padding, every tile is a
// whole work item and is claimed by itself.
constexpr uint64_t kVecPlanned = 0x73656C6974636576ull;
struct VecBatchHdr {
  uint32_t count;        // jobs in the batch
  uint32_t total_tiles;  // tiles in the batch
  uint32_t claim;        // tiles a block claims at a time (vec_claim)
  uint32_t pad0;
  uint64_t planned;      // kVecPlanned
  uint32_t pad[10];
};
struct VecBatchDesc {
  uint64_t x_off, y_off;
  uint32_t n;
  float a;
  uint32_t tile_start;   // first tile of this job (non-decreasing)
  uint32_t ntiles;       // ceil(n / tile_elems)
  uint32_t tile_elems;   // elements per tile, multiple of 256
  uint32_t unit_elems;   // elements per unit: tile_elems, or an equal part of it
  uint32_t per_item;     // tiles per work item
  float sum;             // the job's result, on its way to the block that collects them
};
// Tile geometry of a job of n elements with work items of item_elems, for
// blocks of `block` threads; split: tiles are units.
SETRT_HD inline void vec_set_tiles(VecBatchDesc& d, uint32_t n, uint32_t item_elems, int block, bool split) {
  d.n = n;
  d.unit_elems = vec_unit_elems(item_elems, block);
  d.tile_elems = split ? d.unit_elems : item_elems;
  d.per_item = item_elems / d.tile_elems;
  d.ntiles = n ? (n - 1) / d.tile_elems + 1 : 0;
  d.sum = 0.f;
}
inline uint64_t vec_units(uint64_t n, uint32_t item_elems, int block) {
  const uint32_t u = vec_unit_elems(item_elems, block);
  return (n + u - 1) / u;
}
static_assert(sizeof(VecBatchHdr) == 64, "VecBatchHdr layout");
static_assert(sizeof(VecBatchDesc) == 48, "VecBatchDesc layout");

inline uint64_t canary_value(int tmpl, int w, int s, int which) {
  return 0x5E7CA9A200000000ull ^ ((uint64_t)which << 60) ^ ((uint64_t)tmpl << 24) ^ ((uint64_t)w << 12) ^
         (uint64_t)s;
}

// A submitted job (M5 of the method: id, prepared parameters, is_stolen).
struct JobRec {
  uint64_t id;
  int tmpl;
  set_job_args args;
  int worker;     // worker whose slot the job is bound to
  int slot;       // bound slot
  int stolen;     // retargeted by a thief (Algorithm 2)
  uint64_t seq;   // binding sequence number of that slot
  uint64_t footprint;
  uint64_t t_submit, t_launch, t_done;
  int status;
  int64_t serve_ref;  // serving: request index (>= 0), vector batch -(2 + ring entry), or -1
  JobRec* next;   // free list / intrusive links
};

// Sizes one template needs, computed on the host.
struct TemplateSizes {
  uint64_t slot_bytes;
  int num_stages;
  uint64_t stage_bytes[kMaxStages];
  char stage_names[kMaxStages][32];
};

// Image templates that take the Gaussian and Sobel in one kernel, whose last block
// publishes the output.
inline bool one_kernel_image(const set_job_template& t) {
  return t.pipeline == SET_PIPE_GAUSS_SOBEL_F32 && !(t.flags & SET_TF_DEBUG) &&
         gauss_sobel_in_one((int)t.height, (int)t.width);
}
// Partial counts and sums of an image job: one to a tile of the one kernel, or of the
// Sobel kernel's blocks or waves.
inline uint64_t image_partials(const set_job_template& t) {
  if (!one_kernel_image(t)) return sobel_partials((int)t.height, (int)t.width);
  const Grid3 g = gauss_sobel_grid((int)t.height, (int)t.width);
  return (uint64_t)g.x * g.y;
}
// Where a scan template's blocks have the sums before their tiles from.
inline int scan_prefix(const set_job_template& t) {
  return scan_prefix(t.max_n, t.copy_mode != SET_COPY_NODES && !(t.flags & SET_TF_DEBUG));
}
// Templates whose last stage writes the job's output to host memory itself: small
// outputs without intermediate images, of copy modes whose output copy is a kernel.
// The block that has all of it does (and stores the completion word), or, for
// one-kernel scans and thermal grids, every block its part.
inline bool writes_out(const set_job_template& t) {
  return t.copy_mode != SET_COPY_NODES && !(t.flags & SET_TF_DEBUG) &&
         (t.pipeline == SET_PIPE_BOX_HIST_U8 || t.pipeline == SET_PIPE_GAUSS_SOBEL_F32 ||
          t.pipeline == SET_PIPE_SAXPY_TANH_SUM_F32 ||
          (t.pipeline == SET_PIPE_SCAN_I32_I64 && scan_prefix(t) == SCAN_FROM_INPUT) ||
          (t.pipeline == SET_PIPE_HOTSPOT_F32 && (int64_t)t.width * t.height <= kHotHostCells) ||
          (t.pipeline == SET_PIPE_SAXPY_BATCH_F32 && t.batch_max <= kVecFinishJobs));
}
// Templates whose output copy kernel publishes the header: no stage of theirs
// runs in one block behind the others.
inline bool publishes_in_copy(const set_job_template& t) {
  return t.copy_mode != SET_COPY_NODES && t.pipeline == SET_PIPE_HOTSPOT_F32 && !writes_out(t);
}
// Static per-job sizes of a template (in/out bytes for a job with length n).
uint64_t pipeline_in_bytes(const set_job_template& t, uint64_t n);
uint64_t pipeline_out_bytes(const set_job_template& t, uint64_t n);
int pipeline_validate(const set_job_template& t, std::string* why);
int pipeline_validate_job(const set_job_template& t, const set_job_args& a, std::string* why);
// Implemented by the HIP pipeline code (needs kernel tile constants); the fake
// backend uses the same sizes so footprints agree.
int pipeline_sizes(const set_job_template& t, TemplateSizes* out);
SlotLayout slot_layout(const set_job_template& t);

// Completion hook the scheduler core hands to a backend launch.
using DoneFn = void (*)(void* ctx, JobRec* job, int status);

// Execution backend: owns device resources of every template.
class Backend {
 public:
  virtual ~Backend() {}
  // Create per-worker resources (streams are borrowed or created here).
  virtual int init(const set_config& cfg, std::string* err) = 0;
  // Allocate/lay out slots and build per-slot graphs (SET/GRAPH) or the batch graph (BATCH_SYNC).
  virtual int define_template(int id, const set_job_template& t, std::string* err) = 0;
  // UpdateGraphParams(J, i): bind job to slot (worker, slot) of its template.
  virtual int bind(JobRec* job, std::string* err) = 0;
  // GraphLaunch + AddCallback: launch the bound slot's executable on the
  // worker's stream and arrange for done(ctx, job, status) after it finishes.
  virtual int launch(JobRec* job, DoneFn done, void* ctx, std::string* err) = 0;
  // Queue model: launch the bound slot's executable and record its completion
  // event without any callback; is_done() queries that event.
  virtual int launch_polled(JobRec* job, std::string* err) = 0;
  virtual int is_done(JobRec* job, bool* done, std::string* err) = 0;
  // Baselines, run on the caller's thread.
  virtual int run_sync(JobRec* job, int stream_index, std::string* err) = 0;
  virtual int run_graph(JobRec* job, int stream_index, std::string* err) = 0;
  virtual int run_batch(JobRec** jobs, int count, std::string* err) = 0;
  virtual int time_stage(int tmpl, int stage, int worker, int reps, double* avg_us, std::string* err) = 0;
  // A plain device copy of `bytes` (half read, half written), cold; see set_time_device_copy.
  virtual int time_device_copy(uint64_t bytes, int reps, double* avg_us, std::string* err) = 0;
  virtual uint64_t host_ns_sync() const { return 0; }
  // Pinned host staging owned by the library (descriptor tables, results).
  virtual void* alloc_host(uint64_t bytes) = 0;
  virtual void free_host(void* p) = 0;
  virtual void shutdown() = 0;
};

Backend* make_hip_backend();
Backend* make_fake_backend();

}  // namespace setrt
