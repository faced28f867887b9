// libfp8lm: FP8 gradient quantisation and FP8 Adam step of FP8-LM (arXiv 2310.18313, Sec. 2.1, 2.2,
// Appendix A) for MI355X / gfx950.  See include/fp8lm.h for the boundary.  This file holds the host side
// (context, validation, launches); the kernels live in the headers it includes:
//   walk.hpp      tables, reductions, the chunk walk every kernel shares, access helpers, tuning knobs
//   quantize.hpp  amax + scale, FP8 cast + auto-scaling, delayed scaling, Eq. 4-6 (re-quantise, sum)
//   adam.hpp      master-weight initialisation and the two passes of the FP8 Adam step
//   stats.hpp     quantisation-error statistics, metadata initialisation, streaming copy
//   formats.hpp   FP8 / FP16 / bf16 conversions and the power-of-two scale rule
//
// Shape of every hot kernel
//   * The tensor list is cut into chunks of `chunk_elems` elements that never straddle a tensor, a chunk into units
//     of one, two or four tiles (the update one, the cast of 16-bit sources two, amax and re-quantisation four; see the
//     end of walk.hpp).  A 256-thread workgroup takes one unit and ends, so that the chip
//     sweeps through the buffers in order; a 5 K-element bias and a 250 M-element matrix are served by the same launch.
//   * A thread handles 16 elements of a 4096-element tile, with 128-bit (64-bit on 8-bit
//     streams of the update and cast kernels) accesses that are contiguous over the whole workgroup.
//   * Per-tensor statistics (amax, counters) stay in registers while a workgroup is inside one tensor,
//     then go wavefront -> LDS -> one record per unit.  A second, tiny launch (one workgroup per tensor, more
//     for a large one) combines the records and runs the scalar epilogue (scale update,
//     auto-scaling state, metadata); a single-pass form with a per-tensor ticket is selectable.
//   * These kernels are HBM-bandwidth bound (2..12 bytes per element against ~10-60 ALU operations); no
//     matrix cores are involved.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <numeric>
#include <queue>
#include <string>
#include <vector>

#include "fp8lm.h"
#include "formats.hpp"

#include "walk.hpp"
#include "quantize.hpp"
#include "adam.hpp"
#include "stats.hpp"


// ====================================================================================================
// Fixed device array for fp8lm_adam_step_fp8_static (callers that cannot allocate)
// ====================================================================================================
namespace fp8lm {

// Everything a context keeps in hipMalloc'd memory, at fixed maximum sizes.
constexpr int kStaticChunkElems = 16384;
constexpr int kStaticRecords = 4 << 20;                   // bytes of records
constexpr int kStaticChunks = kStaticRecords / 64;        // chunks of a launch; longer lists have larger chunks
constexpr int kStaticEpilogue = FP8LM_STATIC_MAX_TENSORS + kStaticChunks / kEpilogueChunks;
struct StaticArena {
  TensorDesc desc[FP8LM_STATIC_MAX_TENSORS];              // 128 KiB
  Scratch scratch[FP8LM_STATIC_MAX_TENSORS];              // 512 KiB
  unsigned char records[kStaticRecords];                  // 4 MiB
  unsigned long long totals[(size_t)kStaticEpilogue * kTotalWords];   // 528 KiB
  EpilogueDesc epi[kStaticEpilogue];                      // 198 KiB
  ChunkDesc chunks[kStaticChunks];                        // 1 MiB
};

// A batch of tensor descriptors travels as kernel arguments: no copy from host memory is enqueued.
constexpr int kDescBatch = 96;                            // 3 KiB of arguments per launch
struct DescBatch {
  TensorDesc d[kDescBatch];
  int32_t first, count;
};
__global__ void static_desc_kernel(DescBatch b, TensorDesc* desc) {
  const int i = threadIdx.x;
  if (i < b.count) desc[b.first + i] = b.d[i];
}
}  // namespace fp8lm

// The array itself.  In host code this name is only a handle for hipGetSymbolAddress: the device address is
// looked up once per GPU (static_arena_of) and that pointer is what kernels and launches are given.
static __device__ __align__(256) unsigned char scratch[sizeof(fp8lm::StaticArena)];

// ====================================================================================================
// Host side: context, validation, launches
// ====================================================================================================
using namespace fp8lm;

static thread_local std::string g_hip_error;

constexpr int32_t kLibraryChooses = 1 << 30;      // default of single_pass_min_chunks

struct fp8lm_ctx {
  int device = 0;
  int n_tensors = 0;
  int num_cus = 0;
  std::vector<fp8lm_tensor> tensors;
  std::vector<uint32_t> tensor_flags;   // FP8LM_TENSOR_* per tensor
  int32_t chunk_elems = 16384;
  int32_t blocks_per_cu = kMaxBlocksPerCu;
  int32_t single_pass_min_chunks = kLibraryChooses;
  int32_t n_chunks = 0;
  TensorDesc* d_desc = nullptr;
  ChunkDesc* d_chunks = nullptr;
  Scratch* d_scratch = nullptr;
  unsigned char* d_records = nullptr;   // one record per unit
  size_t record_bytes = 0;
  unsigned long long* d_totals = nullptr;
  EpilogueDesc* d_epi = nullptr;
  int32_t n_epi = 0;
  Partial* d_partials = nullptr;    // [num_cus * kMaxBlocksPerCu + n_tensors], error statistics
  // speculation: number of the last call and, on the device, of the last one that marked a tensor; running totals (calls,
  // tensors done again, elements done again) for the gradient and for the first moment
  uint32_t spec_call = 0;
  uint32_t* d_marked_call = nullptr;
  uint32_t* d_redo = nullptr;           // [n_tensors, whole quads] marks
  int spec_kind = 0;                    // what the call speculates about: 0 gradient scales, 1 first-moment scales
  unsigned long long* d_spec_totals = nullptr;
  // what the last fused cast measured for (checked by the Adam step that wants to use it)
  struct Fused { bool valid; const uint8_t* grad; const uint8_t* m; const fp8lm_meta* m_meta; float b1; int fmt; };
  Fused fused{false, nullptr, nullptr, nullptr, 0.0f, 0};
  // timing
  bool timing = false;
  struct Stamp { int kernel; hipEvent_t a, b; };
  std::vector<Stamp> stamps;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> free_events;
};

#define HIP_TRY(expr)                                                      \
  do {                                                                     \
    hipError_t e_ = (expr);                                                \
    if (e_ != hipSuccess) {                                                \
      g_hip_error = std::string(#expr) + ": " + hipGetErrorString(e_);     \
      return FP8LM_ERR_HIP;                                                \
    }                                                                      \
  } while (0)

namespace {

struct DeviceGuard {
  int prev = -1;
  bool ok = true;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) { ok = false; return; }
    if (prev != dev && hipSetDevice(dev) != hipSuccess) ok = false;
    if (prev == dev) prev = -1;
  }
  ~DeviceGuard() { if (prev >= 0) (void)hipSetDevice(prev); }
};

void free_tables(fp8lm_ctx* c) {
  for (void* p : {(void*)c->d_desc, (void*)c->d_chunks, (void*)c->d_epi, (void*)c->d_records, (void*)c->d_totals})
    if (p) (void)hipFree(p);
}

// Elements per chunk of a context (or a call without one) that has not been given a tuning: 16384, which keeps the chunk
// table small, unless the tensors are so small that most of the units such chunks are cut into would be empty.
template <class NumelOf> int32_t default_chunk(int n, NumelOf numel_of) {
  long long chunks = 0, tiles = 0;
  for (int t = 0; t < n; ++t) {
    chunks += (numel_of(t) + 4 * kTile - 1) / (4 * kTile);
    tiles += (numel_of(t) + kTile - 1) / kTile;
  }
  return 4 * chunks > tiles + tiles / 4 ? kTile : 4 * kTile;
}

// Builds the tensor and chunk tables for chunks of chunk_elems elements and installs them.  On failure the
// context keeps the tables (and the chunk size) it had.
fp8lm_status build_tables(fp8lm_ctx* c, int32_t chunk_elems) {
  std::vector<TensorDesc> desc(c->n_tensors);
  long long total_chunks = 0;
  int32_t n_epi = 0;
  for (int t = 0; t < c->n_tensors; ++t) {
    const long long n = c->tensors[t].numel;
    const long long nc = (n + chunk_elems - 1) / chunk_elems;
    if (total_chunks + nc > 0x7FFFFFF0LL) return FP8LM_ERR_TOO_LARGE;
    desc[t] = TensorDesc{c->tensors[t].offset, n, (int32_t)total_chunks, (int32_t)nc, c->tensor_flags[t], n_epi};
    if (nc > 0) n_epi += epilogue_groups((int32_t)nc);
    total_chunks += nc;
  }
  // records: 32 bytes for each 4096 elements (units are not smaller than that), and a chunk can always be one unit
  const size_t record_bytes = std::max<size_t>(1, (size_t)total_chunks) * std::max(64, chunk_elems / kTile * 32);
  // everything in one list, so that a failure gives back what had been allocated
  struct Piece { void** at; size_t bytes; const void* from; };
  TensorDesc* d_desc = nullptr;
  ChunkDesc* d_chunks = nullptr;
  EpilogueDesc* d_epi = nullptr;
  unsigned char* d_records = nullptr;
  unsigned long long* d_totals = nullptr;
  const Piece pieces[] = {
      {(void**)&d_desc, desc.size() * sizeof(TensorDesc), desc.data()},
      {(void**)&d_chunks, (size_t)total_chunks * sizeof(ChunkDesc), nullptr},
      {(void**)&d_epi, (size_t)n_epi * sizeof(EpilogueDesc), nullptr},
      {(void**)&d_records, record_bytes, nullptr},
      {(void**)&d_totals, (size_t)n_epi * kTotalWords * sizeof(unsigned long long), nullptr},
  };
  hipError_t e = hipSuccess;
  for (const Piece& q : pieces) {
    if (e == hipSuccess) e = hipMalloc(q.at, std::max<size_t>(16, q.bytes));
    if (e == hipSuccess && q.from && q.bytes) e = hipMemcpy(*q.at, q.from, q.bytes, hipMemcpyHostToDevice);
  }
  if (e == hipSuccess && total_chunks > 0) {     // the per-chunk tables are written on the device
    hipLaunchKernelGGL(chunk_tables_kernel, dim3(std::min(c->n_tensors, 1024)), dim3(kThreads), 0, nullptr, d_desc, d_chunks,
                       d_epi, c->d_scratch, chunk_elems, c->n_tensors);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipDeviceSynchronize();
  }
  if (e != hipSuccess) {
    g_hip_error = std::string("chunk tables: ") + hipGetErrorString(e);
    for (const Piece& q : pieces)
      if (*q.at) (void)hipFree(*q.at);
    return FP8LM_ERR_HIP;
  }
  free_tables(c);
  c->d_desc = d_desc;
  c->d_chunks = d_chunks;
  c->d_epi = d_epi;
  c->d_records = d_records;
  c->d_totals = d_totals;
  c->record_bytes = record_bytes;
  c->n_epi = n_epi;
  c->chunk_elems = chunk_elems;
  c->n_chunks = (int32_t)total_chunks;
  return FP8LM_OK;
}

// Workgroups of a persistent launch: blocks_per_cu per compute unit, but never more than there are chunks.
int grid_of(const fp8lm_ctx* c) {
  const long long full = (long long)c->num_cus * c->blocks_per_cu;
  return (int)std::max<long long>(1, std::min<long long>(full, c->n_chunks));
}

// Tables of a launch whose workgroups take up to `un` tiles at once and leave records of `record` bytes, and its grid.
// By default a workgroup per unit.  A unit is `un` tiles where that gives every compute unit four workgroups, otherwise
// fewer (a small launch needs workgroups more than it needs loads in flight), and more where the record memory would not
// do.  A persistent grid where the caller asked for a limit (fp8lm_set_tuning), where there would be more workgroups than
// a launch can have, and for `ranges`.
constexpr long long kMaxGrid = 1ll << 23;          // x 256 threads stays below 2^32
Tables tables_of(const fp8lm_ctx* c, int un, int record, int* grid, bool ranges = false) {
  Tables tb{};
  tb.desc = c->d_desc;
  tb.chunks = c->d_chunks;
  tb.scratch = c->d_scratch;
  tb.records = c->d_records;
  tb.totals = c->d_totals;
  tb.epi = c->d_epi;
  tb.n_tensors = c->n_tensors;
  tb.call = c->spec_call;
  tb.marked_call = c->d_marked_call;
  tb.redo = c->d_redo;
  tb.spec_totals = c->d_spec_totals ? c->d_spec_totals + 3 * c->spec_kind : nullptr;
  tb.n_epi = c->n_epi;
  tb.n_chunks = c->n_chunks;
  tb.unit_elems = c->chunk_elems;
  auto units = [&] { return (long long)c->n_chunks << tb.unit_shift; };
  if (c->blocks_per_cu >= kMaxBlocksPerCu && !ranges) {
    while (tb.unit_elems % (2 * kTile) == 0 && (tb.unit_elems > un * kTile || units() < 4ll * c->num_cus) &&
           (size_t)(2 * units() * record) <= c->record_bytes) {
      tb.unit_elems /= 2;
      ++tb.unit_shift;
    }
    tb.one_unit = units() <= kMaxGrid;
  }
  *grid = tb.one_unit ? (int)units() : grid_of(c);
  // In the deferred form a second launch finishes the tensors; see walk.hpp for the two forms' costs.  Unless told otherwise
  // tickets are for launches of at most 64 units, where they win whatever the list: a step of one tensor of 64 units takes
  // 25.4 us with and 30.5 without them, one of 50 small tensors 25.1 and 30.5.  Above, it depends on the list (one tensor of 256
  // units 27.1 and 30.6; 120 small tensors 30.9 and 30.5, 200 39.5 and 30.7), and at 512 units one tensor loses too (36.9 and 32.5).
  // A caller's threshold is compared with the chunks per workgroup of this launch.
  constexpr int kTicketUnits = 64;
  tb.deferred = c->single_pass_min_chunks == kLibraryChooses
                    ? units() > kTicketUnits
                    : c->single_pass_min_chunks > 0 && c->n_chunks / *grid < c->single_pass_min_chunks;
  // Tickets that a caller wants at any size: of a persistent grid of at most a workgroup per chunk, which has a ticket for each
  // workgroup and tensor and not one for each unit.  amax and cast of two tensors, us, units / persistent: 256 units in all
  // 16.3 / 16.5, 512 20.6 / 16.4, 1024 33.6 / 16.8, 8192 241 / 165; of a GPT-7B layer 3050 / 570.
  if (!tb.deferred && tb.one_unit && units() > 256) {
    tb.unit_elems = c->chunk_elems;
    tb.unit_shift = tb.one_unit = 0;
    *grid = grid_of(c);
  }
  return tb;
}
// The tables and the grid of the second round of a speculation (walk_marked), from the tables of the first: the marks are
// counts of its units.
Tables marked_tables_of(const fp8lm_ctx* c, const Tables& first, int* grid) {
  Tables tb = first;
  const long long units = (long long)c->n_chunks << tb.unit_shift;
  // Mostly nothing is marked, and then a launch to finish with is 1.7 us for nothing, so tickets go up to more units than in
  // the first round.  quantize_fp8 with nothing / everything marked, tickets against launch, us: 160 units 16.1 / 24.2
  // against 17.7 / 23.1; 256 units 16.2 / 25.9 against 17.9 / 23.5; 400 units 16.5 / 28.6 against 18.1 / 24.3.
  if (c->single_pass_min_chunks == kLibraryChooses) tb.deferred = units > 256;
  // Four workgroups per compute unit: with nothing marked they only cost their start, and more are no faster with much marked
  // (two of eight tensors of 2^21 34.9 us with four, 38.8 with eight; of 2^27 699 and 707; all eight of 2^25 304 and 312;
  // a step of a GPT-175B layer with two thirds marked 5455 and 5449).
  *grid = (int)std::min<long long>((long long)std::min(4, c->blocks_per_cu) * c->num_cus, units);
  return tb;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct Timed {
  fp8lm_ctx* c;
  hipStream_t s;
  int kernel;
  hipEvent_t a = nullptr, b = nullptr;
  Timed(fp8lm_ctx* c_, hipStream_t s_, int k) : c(c_), s(s_), kernel(k) {
    if (!c->timing || c->free_events.empty()) return;
    a = c->free_events.back().first;
    b = c->free_events.back().second;
    c->free_events.pop_back();
    (void)hipEventRecord(a, s);
  }
  ~Timed() {
    if (!a) return;
    (void)hipEventRecord(b, s);
    c->stamps.push_back({kernel, a, b});
  }
};

fp8lm_status after_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    g_hip_error = std::string("kernel launch: ") + hipGetErrorString(e);
    return FP8LM_ERR_HIP;
  }
  return FP8LM_OK;
}

// Launches a kernel that walks the units and, in the deferred form, the launch that finishes its tensors.
template <class Stats> struct RecordOf;
template <int NV, int NC> struct RecordOf<BlockStats<NV, NC>> { static constexpr int bytes = kRecordBytes<NC>; };
template <class Op, bool MARKED = false, class Params, class Kernel>
void launch_walk_on(fp8lm_ctx* c, hipStream_t s, Kernel kernel, const Params& p, const Tables& tb, int grid) {
  const dim3 b(kThreads);
  hipLaunchKernelGGL(kernel, dim3(grid), b, 0, s, tb, p);
  if (tb.deferred) hipLaunchKernelGGL((epilogue_kernel<Op, Params, MARKED>), dim3(std::min<int>(c->n_epi, 8 * c->num_cus)), b, 0, s, tb, p);
}
// ... on the usual tables, which it returns.
template <class Op, class Params, class Kernel>
Tables launch_walk(fp8lm_ctx* c, hipStream_t s, Kernel kernel, const Params& p, int un = 1, bool ranges = false) {
  int grid = 0;
  const Tables tb = tables_of(c, un, RecordOf<typename Op::Stats>::bytes, &grid, ranges);
  launch_walk_on<Op>(c, s, kernel, p, tb, grid);
  return tb;
}
// The amax pass reads one stream and writes nothing, so the order of the walk brings it little, and from 1 GiB on what a
// workgroup does once per unit costs more: a persistent grid then.  us, a workgroup per unit / persistent: fp32 2^27 elements 84 /
// 87, 2^30 645 / 622, 2^32 2565 / 2472; bf16 2^27 45 / 46, 2^30 326 / 321, 2^32 1281 / 1259.
template <int MODE, int SRC> void launch_amax(fp8lm_ctx* c, hipStream_t s, const AmaxParams& p) {
  const long long bytes = (long long)c->n_chunks * c->chunk_elems * (long long)sizeof(typename SrcTraits<SRC>::elem_t);
  launch_walk<AmaxOp<MODE, SRC>>(c, s, amax_kernel<MODE, SRC>, p, kUnAmax<SRC>, bytes >= 1ll << 30);
}

// Selects the adam_update_kernel instantiation.
template <int GFMT, int WCOPY>
Tables launch_update(fp8lm_ctx* c, hipStream_t s, const AdamParams& p, bool fast, bool stats) {
#define FP8LM_UPDATE(F, S) launch_walk<AdamUpdateOp<GFMT, WCOPY, F, S>>(c, s, adam_update_kernel<GFMT, WCOPY, F, S>, p, kUnUpdate)
  if (fast) return stats ? FP8LM_UPDATE(true, true) : FP8LM_UPDATE(true, false);
  return stats ? FP8LM_UPDATE(false, true) : FP8LM_UPDATE(false, false);
#undef FP8LM_UPDATE
}

// Selects the adam_update_var_kernel instantiation (every master / second-moment format pair except the default).
template <int GFMT>
void launch_update_variant_g(fp8lm_ctx* c, hipStream_t s, const AdamParams& p, int master, int vfmt) {
#define FP8LM_VAR(M, V) launch_walk<AdamUpdateVarOp<GFMT, M, V>>(c, s, adam_update_var_kernel<GFMT, M, V>, p)
  if (vfmt == kStF16) {
    if (master == kStBF16) FP8LM_VAR(kStBF16, kStF16);
    else if (master == kStE4M3) FP8LM_VAR(kStE4M3, kStF16);
    else FP8LM_VAR(kStF32, kStF16);
  } else {
    if (master == kStF16) FP8LM_VAR(kStF16, kStE4M3);
    else if (master == kStBF16) FP8LM_VAR(kStBF16, kStE4M3);
    else if (master == kStE4M3) FP8LM_VAR(kStE4M3, kStE4M3);
    else FP8LM_VAR(kStF32, kStE4M3);
  }
#undef FP8LM_VAR
}
void launch_update_variant(fp8lm_ctx* c, hipStream_t s, const AdamParams& p, bool e5, int master, int vfmt) {
  if (e5) launch_update_variant_g<kE5M2>(c, s, p, master, vfmt);
  else launch_update_variant_g<kE4M3>(c, s, p, master, vfmt);
}

bool src_ok(fp8lm_src t) { return t == FP8LM_SRC_BF16 || t == FP8LM_SRC_F16 || t == FP8LM_SRC_F32; }
AutoscaleRule rule_of(const fp8lm_autoscale_cfg* cfg) {
  return AutoscaleRule{cfg->sat_num, cfg->sat_den, cfg->ramp_steps, cfg->mu_rule, cfg->mu_min_exp};
}
bool cfg_ok(const fp8lm_autoscale_cfg* cfg) {
  if (cfg && cfg->mu_rule != FP8LM_MU_SET_HALF &&
      !(cfg->mu_rule == FP8LM_MU_HALVE && cfg->mu_min_exp >= -64 && cfg->mu_min_exp <= -1))
    return false;
  // sat_num, sat_den <= 2^24: the overflow test multiplies them with element counts in 64 bits
  return cfg && cfg->sat_num >= 0 && cfg->sat_num <= (1 << 24) && cfg->sat_den > 0 && cfg->sat_den <= (1 << 24) &&
         cfg->ramp_steps >= 2 && cfg->hist_window >= 1 &&
         cfg->hist_window <= FP8LM_HIST && cfg->margin >= -64 && cfg->margin <= 64;
}

}  // namespace

extern "C" {

const char* fp8lm_status_string(fp8lm_status s) {
  switch (s) {
    case FP8LM_OK: return "ok";
    case FP8LM_ERR_INVALID_ARGUMENT: return "invalid argument";
    case FP8LM_ERR_MISALIGNED: return "misaligned offset or buffer";
    case FP8LM_ERR_OVERLAP: return "tensors overlap";
    case FP8LM_ERR_HIP: return "HIP runtime error";
    case FP8LM_ERR_TOO_LARGE: return "too many chunks or tensors";
  }
  return "unknown status";
}

const char* fp8lm_last_hip_error(void) { return g_hip_error.c_str(); }
uint32_t fp8lm_sizeof_meta(void) { return (uint32_t)sizeof(fp8lm_meta); }

fp8lm_status fp8lm_create(fp8lm_ctx** out, const fp8lm_tensor* tensors, int32_t n, int device) {
  if (!out || n < 0 || (n > 0 && !tensors)) return FP8LM_ERR_INVALID_ARGUMENT;
  *out = nullptr;
  for (int t = 0; t < n; ++t) {
    if (tensors[t].numel < 0 || tensors[t].offset < 0) return FP8LM_ERR_INVALID_ARGUMENT;
    if (tensors[t].offset % 16 != 0) return FP8LM_ERR_MISALIGNED;
  }
  {
    std::vector<std::pair<long long, long long>> spans;
    for (int t = 0; t < n; ++t)
      if (tensors[t].numel > 0) spans.emplace_back(tensors[t].offset, tensors[t].offset + tensors[t].numel);
    std::sort(spans.begin(), spans.end());
    for (size_t i = 1; i < spans.size(); ++i)
      if (spans[i].first < spans[i - 1].second) return FP8LM_ERR_OVERLAP;
  }
  int count = 0;
  HIP_TRY(hipGetDeviceCount(&count));
  if (device < 0 || device >= count) return FP8LM_ERR_INVALID_ARGUMENT;
  DeviceGuard guard(device);
  if (!guard.ok) { g_hip_error = "hipSetDevice failed"; return FP8LM_ERR_HIP; }
  hipDeviceProp_t prop;
  HIP_TRY(hipGetDeviceProperties(&prop, device));
  fp8lm_ctx* c = new fp8lm_ctx();
  c->device = device;
  c->n_tensors = n;
  c->num_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
  c->tensors.assign(tensors, tensors + n);
  c->tensor_flags.assign((size_t)n, 0u);
  const size_t bytes = std::max<size_t>(1, (size_t)n) * sizeof(Scratch);
  hipError_t e = hipMalloc((void**)&c->d_scratch, bytes);
  if (e == hipSuccess) e = hipMemset(c->d_scratch, 0, bytes);
  if (e != hipSuccess) g_hip_error = hipGetErrorString(e);
  c->chunk_elems = default_chunk(n, [&](int t) { return tensors[t].numel; });
  fp8lm_status st = e == hipSuccess ? build_tables(c, c->chunk_elems) : FP8LM_ERR_HIP;
  if (st == FP8LM_OK) {
    const size_t records = (size_t)c->num_cus * kMaxBlocksPerCu + (size_t)n + 1;
    if (e == hipSuccess) e = hipMalloc((void**)&c->d_partials, records * sizeof(Partial));
    if (e == hipSuccess) e = hipMemset(c->d_partials, 0, records * sizeof(Partial));
    if (e == hipSuccess) e = hipMalloc((void**)&c->d_marked_call, sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemset(c->d_marked_call, 0, sizeof(uint32_t));
    const size_t marks = ((size_t)n + 3) / 4 * 16 + 16;
    if (e == hipSuccess) e = hipMalloc((void**)&c->d_redo, marks);
    if (e == hipSuccess) e = hipMemset(c->d_redo, 0, marks);
    if (e == hipSuccess) e = hipMalloc((void**)&c->d_spec_totals, 6 * sizeof(unsigned long long));     // gradient, first moment
    if (e == hipSuccess) e = hipMemset(c->d_spec_totals, 0, 6 * sizeof(unsigned long long));
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) { g_hip_error = hipGetErrorString(e); st = FP8LM_ERR_HIP; }
  }
  if (st != FP8LM_OK) { fp8lm_destroy(c); return st; }
  *out = c;
  return FP8LM_OK;
}

fp8lm_status fp8lm_destroy(fp8lm_ctx* c) {
  if (!c) return FP8LM_OK;
  DeviceGuard guard(c->device);
  free_tables(c);
  if (c->d_scratch) (void)hipFree(c->d_scratch);
  if (c->d_partials) (void)hipFree(c->d_partials);
  if (c->d_marked_call) (void)hipFree(c->d_marked_call);
  if (c->d_redo) (void)hipFree(c->d_redo);
  if (c->d_spec_totals) (void)hipFree(c->d_spec_totals);
  for (auto& s : c->stamps) { (void)hipEventDestroy(s.a); (void)hipEventDestroy(s.b); }
  for (auto& e : c->free_events) { (void)hipEventDestroy(e.first); (void)hipEventDestroy(e.second); }
  delete c;
  return FP8LM_OK;
}

fp8lm_status fp8lm_set_tuning(fp8lm_ctx* c, int32_t chunk_elems, int32_t blocks_per_cu, int32_t single_pass_min_chunks) {
  if (!c || chunk_elems < kTile || chunk_elems > (1 << 20) || chunk_elems % kTile != 0 || blocks_per_cu < 1 ||
      blocks_per_cu > kMaxBlocksPerCu || single_pass_min_chunks < 0 || single_pass_min_chunks > (1 << 30))
    return FP8LM_ERR_INVALID_ARGUMENT;
  DeviceGuard guard(c->device);
  HIP_TRY(hipDeviceSynchronize());   // no launch may still be reading the tables that are about to go
  const fp8lm_status st = build_tables(c, chunk_elems);
  if (st != FP8LM_OK) return st;
  c->blocks_per_cu = blocks_per_cu;
  c->single_pass_min_chunks = single_pass_min_chunks;
  return FP8LM_OK;
}

fp8lm_status fp8lm_set_tensor_flags(fp8lm_ctx* c, const uint32_t* flags, int32_t n) {
  if (!c || n != c->n_tensors || (n > 0 && !flags)) return FP8LM_ERR_INVALID_ARGUMENT;
  for (int t = 0; t < n; ++t)
    if (flags[t] & ~(uint32_t)FP8LM_TENSOR_NO_WEIGHT_DECAY) return FP8LM_ERR_INVALID_ARGUMENT;
  DeviceGuard guard(c->device);
  HIP_TRY(hipDeviceSynchronize());   // no launch may still be reading the tables that are about to go
  const std::vector<uint32_t> before = c->tensor_flags;
  c->tensor_flags.assign(flags, flags + n);
  const fp8lm_status st = build_tables(c, c->chunk_elems);
  if (st != FP8LM_OK) c->tensor_flags = before;
  return st;
}

fp8lm_status fp8lm_meta_init(fp8lm_ctx* c, fp8lm_meta* meta, const fp8lm_autoscale_cfg* cfg, void* stream) {
  if (!c || !cfg_ok(cfg) || (c->n_tensors > 0 && !meta)) return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_tensors == 0) return FP8LM_OK;
  DeviceGuard guard(c->device);
  const int blocks = (c->n_tensors + 255) / 256;
  hipLaunchKernelGGL(meta_init_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, meta, c->n_tensors,
                     cfg->mu_rule == FP8LM_MU_HALVE ? 0 : cfg->ramp_steps / 2);
  return after_launch();
}

fp8lm_status fp8lm_amax_scale(fp8lm_ctx* c, const void* src, fp8lm_src src_type, fp8lm_fmt target, fp8lm_meta* meta,
                              const fp8lm_autoscale_cfg* cfg, void* stream) {
  if (!c || !cfg_ok(cfg) || !src_ok(src_type) || (target != FP8LM_E4M3 && target != FP8LM_E5M2))
    return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_chunks == 0) return FP8LM_OK;
  if (!src || !meta) return FP8LM_ERR_INVALID_ARGUMENT;
  if (!aligned16(src)) return FP8LM_ERR_MISALIGNED;
  DeviceGuard guard(c->device);
  AmaxParams p{src, meta, target == FP8LM_E4M3 ? kBitsE4M3Max : kBitsE5M2Max, cfg->hist_window, cfg->margin};
  hipStream_t s = (hipStream_t)stream;
  Timed tm(c, s, FP8LM_K_AMAX);
  if (src_type == FP8LM_SRC_F32) launch_amax<kAmaxForGradient, kSrcF32>(c, s, p);
  else if (src_type == FP8LM_SRC_F16) launch_amax<kAmaxForGradient, kSrcF16>(c, s, p);
  else launch_amax<kAmaxForGradient, kSrcBF16>(c, s, p);
  return after_launch();
}

// Common body of the three cast entry points.
enum CastMode { kCastPlain = 0, kCastDelayed = 1, kCastSpeculative = 2 };
static fp8lm_status cast_impl(fp8lm_ctx* c, const void* src, fp8lm_src src_type, uint8_t* dst, fp8lm_fmt fmt,
                              fp8lm_meta* meta, const fp8lm_autoscale_cfg* cfg, int mode, bool fuse,
                              const uint8_t* m, const fp8lm_meta* m_meta, float beta1, void* stream) {
  const bool delayed = mode != kCastPlain;        // the first pass of a speculation is a delayed-scaling cast
  if (!c || !cfg_ok(cfg) || !src_ok(src_type) || (fmt != FP8LM_E4M3 && fmt != FP8LM_E5M2))
    return FP8LM_ERR_INVALID_ARGUMENT;
  c->fused.valid = false;
  if (fuse && !(beta1 >= 0.0f && beta1 < 1.0f)) return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_chunks == 0) return FP8LM_OK;
  if (!src || !dst || !meta || (fuse && (!m || !m_meta))) return FP8LM_ERR_INVALID_ARGUMENT;
  if (!aligned16(src) || !aligned16(dst) || (fuse && !aligned16(m))) return FP8LM_ERR_MISALIGNED;
  DeviceGuard guard(c->device);
  hipStream_t s = (hipStream_t)stream;
  const uint32_t fmax_bits = fmt == FP8LM_E4M3 ? kBitsE4M3Max : kBitsE5M2Max;
  if (mode == kCastSpeculative) {
    ++c->spec_call;
    c->spec_kind = 0;
  }
  CastParams p{};
  p.speculative = mode == kCastSpeculative ? 1 : 0;
  p.fmax_bits = fmax_bits;
  p.margin = cfg->margin;
  p.src = src;
  p.dst = dst;
  p.meta = meta;
  p.rule = rule_of(cfg);
  p.hist_window = cfg->hist_window;
  p.m = m;
  p.m_meta = m_meta;
  p.b1 = beta1;
  p.omb1 = (float)(1.0 - (double)beta1);
  Tables tb;
  {
    Timed tm(c, s, FP8LM_K_CAST);
#define FP8LM_CAST_LAUNCH(F, S)                                                                           \
    do {                                                                                                    \
      if (delayed && fuse) tb = launch_walk<CastOp<F, true, true, S>>(c, s, cast_kernel<F, true, true, S>, p, kUnCast<S>);     \
      else if (delayed) tb = launch_walk<CastOp<F, true, false, S>>(c, s, cast_kernel<F, true, false, S>, p, kUnCast<S>);       \
      else if (fuse) tb = launch_walk<CastOp<F, false, true, S>>(c, s, cast_kernel<F, false, true, S>, p, kUnCast<S>);          \
      else tb = launch_walk<CastOp<F, false, false, S>>(c, s, cast_kernel<F, false, false, S>, p, kUnCast<S>);                   \
    } while (0)
#define FP8LM_CAST_SRC(S)                                                                                   \
    do {                                                                                                    \
      if (fmt == FP8LM_E4M3) FP8LM_CAST_LAUNCH(kE4M3, S);                                                   \
      else FP8LM_CAST_LAUNCH(kE5M2, S);                                                                     \
    } while (0)
    if (src_type == FP8LM_SRC_F32) FP8LM_CAST_SRC(kSrcF32);
    else if (src_type == FP8LM_SRC_F16) FP8LM_CAST_SRC(kSrcF16);
    else FP8LM_CAST_SRC(kSrcBF16);
#undef FP8LM_CAST_SRC
#undef FP8LM_CAST_LAUNCH
  }
  fp8lm_status st = after_launch();
  if (st == FP8LM_OK && mode == kCastSpeculative) {
    // the tensors whose scale turned out different, with the plain cast
    {
      int grid = 0;
      const Tables rt = marked_tables_of(c, tb, &grid);
      p.speculative = 0;
      Timed tm(c, s, FP8LM_K_CAST);
#define FP8LM_REDO_LAUNCH(F, S)                                                                            \
      do {                                                                                                  \
        if (fuse) launch_walk_on<CastOp<F, false, true, S>, true>(c, s, cast_marked_kernel<F, true, S>, p, rt, grid);    \
        else launch_walk_on<CastOp<F, false, false, S>, true>(c, s, cast_marked_kernel<F, false, S>, p, rt, grid);       \
      } while (0)
#define FP8LM_REDO_SRC(S)                                                                                  \
      do {                                                                                                  \
        if (fmt == FP8LM_E4M3) FP8LM_REDO_LAUNCH(kE4M3, S);                                                 \
        else FP8LM_REDO_LAUNCH(kE5M2, S);                                                                   \
      } while (0)
      if (src_type == FP8LM_SRC_F32) FP8LM_REDO_SRC(kSrcF32);
      else if (src_type == FP8LM_SRC_F16) FP8LM_REDO_SRC(kSrcF16);
      else FP8LM_REDO_SRC(kSrcBF16);
#undef FP8LM_REDO_SRC
#undef FP8LM_REDO_LAUNCH
      st = after_launch();
    }
  }
  if (st == FP8LM_OK && fuse) c->fused = {true, dst, m, m_meta, p.b1, fmt};
  return st;
}

fp8lm_status fp8lm_cast_fp8(fp8lm_ctx* c, const void* src, fp8lm_src src_type, uint8_t* dst, fp8lm_fmt fmt,
                            fp8lm_meta* meta, const fp8lm_autoscale_cfg* cfg, void* stream) {
  return cast_impl(c, src, src_type, dst, fmt, meta, cfg, kCastPlain, false, nullptr, nullptr, 0.0f, stream);
}

fp8lm_status fp8lm_cast_fp8_delayed(fp8lm_ctx* c, const void* src, fp8lm_src src_type, uint8_t* dst, fp8lm_fmt fmt,
                                    fp8lm_meta* meta, const fp8lm_autoscale_cfg* cfg, void* stream) {
  return cast_impl(c, src, src_type, dst, fmt, meta, cfg, kCastDelayed, false, nullptr, nullptr, 0.0f, stream);
}

fp8lm_status fp8lm_cast_fp8_for_adam(fp8lm_ctx* c, const void* src, fp8lm_src src_type, uint8_t* dst, fp8lm_fmt fmt,
                                     fp8lm_meta* meta, const fp8lm_autoscale_cfg* cfg, int32_t delayed,
                                     const uint8_t* m, const fp8lm_meta* m_meta, float beta1, void* stream) {
  return cast_impl(c, src, src_type, dst, fmt, meta, cfg, delayed != 0 ? kCastDelayed : kCastPlain, true, m, m_meta, beta1,
                   stream);
}

fp8lm_status fp8lm_quantize_fp8(fp8lm_ctx* c, const void* src, fp8lm_src src_type, uint8_t* dst, fp8lm_fmt fmt,
                                fp8lm_meta* meta, const fp8lm_autoscale_cfg* cfg, void* stream) {
  return cast_impl(c, src, src_type, dst, fmt, meta, cfg, kCastSpeculative, false, nullptr, nullptr, 0.0f, stream);
}

fp8lm_status fp8lm_quantize_fp8_for_adam(fp8lm_ctx* c, const void* src, fp8lm_src src_type, uint8_t* dst, fp8lm_fmt fmt,
                                         fp8lm_meta* meta, const fp8lm_autoscale_cfg* cfg, const uint8_t* m,
                                         const fp8lm_meta* m_meta, float beta1, void* stream) {
  return cast_impl(c, src, src_type, dst, fmt, meta, cfg, kCastSpeculative, true, m, m_meta, beta1, stream);
}

fp8lm_status fp8lm_get_speculation_stats(fp8lm_ctx* c, uint64_t* calls, uint64_t* tensors_redone, uint64_t* elems_redone,
                                         void* stream) {
  if (!c || !calls || !tensors_redone || !elems_redone) return FP8LM_ERR_INVALID_ARGUMENT;
  DeviceGuard guard(c->device);
  unsigned long long h[3] = {0, 0, 0};
  HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
  HIP_TRY(hipMemcpy(h, c->d_spec_totals, sizeof(h), hipMemcpyDeviceToHost));
  *calls = h[0]; *tensors_redone = h[1]; *elems_redone = h[2];
  return FP8LM_OK;
}

fp8lm_status fp8lm_shared_scale(fp8lm_ctx* c, const fp8lm_meta* const* metas, int32_t n_ranks, float* shared,
                                void* stream) {
  if (!c || !metas || n_ranks < 1 || n_ranks > kMaxRanks) return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_tensors == 0) return FP8LM_OK;
  if (!shared) return FP8LM_ERR_INVALID_ARGUMENT;
  RankMetas rm{};
  rm.n_ranks = n_ranks;
  for (int r = 0; r < n_ranks; ++r) {
    if (!metas[r]) return FP8LM_ERR_INVALID_ARGUMENT;
    rm.m[r] = metas[r];
  }
  DeviceGuard guard(c->device);
  Timed tm(c, (hipStream_t)stream, FP8LM_K_SCALARS);
  hipLaunchKernelGGL(shared_scale_kernel, dim3((c->n_tensors + 255) / 256), dim3(256), 0, (hipStream_t)stream, rm,
                     c->n_tensors, shared);
  return after_launch();
}

fp8lm_status fp8lm_requantize_fp8(fp8lm_ctx* c, const uint8_t* src, fp8lm_fmt fmt, const fp8lm_meta* src_meta,
                                  const float* shared, uint8_t* dst, fp8lm_meta* dst_meta, void* stream) {
  if (!c || (fmt != FP8LM_E4M3 && fmt != FP8LM_E5M2)) return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_chunks == 0) return FP8LM_OK;
  if (!src || !src_meta || !shared || !dst || !dst_meta || src_meta == dst_meta) return FP8LM_ERR_INVALID_ARGUMENT;
  if (!aligned16(src) || !aligned16(dst)) return FP8LM_ERR_MISALIGNED;
  DeviceGuard guard(c->device);
  RequantParams p{src, src_meta, shared, dst, dst_meta};
  Timed tm(c, (hipStream_t)stream, FP8LM_K_REQUANT);
  if (fmt == FP8LM_E4M3)
    launch_walk<RequantOp<kE4M3>>(c, (hipStream_t)stream, requantize_kernel<kE4M3>, p, kUnRequant);
  else
    launch_walk<RequantOp<kE5M2>>(c, (hipStream_t)stream, requantize_kernel<kE5M2>, p, kUnRequant);
  return after_launch();
}

fp8lm_status fp8lm_sum_fp8(fp8lm_ctx* c, const uint8_t* const* payloads, int32_t n_ranks, fp8lm_fmt fmt,
                           const float* shared, uint8_t* dst, fp8lm_meta* dst_meta, const fp8lm_autoscale_cfg* cfg,
                           void* stream) {
  if (!c || !cfg_ok(cfg) || !payloads || n_ranks < 1 || n_ranks > kMaxRanks || (fmt != FP8LM_E4M3 && fmt != FP8LM_E5M2))
    return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_chunks == 0) return FP8LM_OK;
  if (!shared || !dst || !dst_meta) return FP8LM_ERR_INVALID_ARGUMENT;
  SumParams p{};
  p.in.n_ranks = n_ranks;
  for (int r = 0; r < n_ranks; ++r) {
    if (!payloads[r]) return FP8LM_ERR_INVALID_ARGUMENT;
    if (!aligned16(payloads[r])) return FP8LM_ERR_MISALIGNED;
    p.in.p[r] = payloads[r];
  }
  if (!aligned16(dst)) return FP8LM_ERR_MISALIGNED;
  p.shared = shared; p.dst = dst; p.dst_meta = dst_meta;
  p.rule = rule_of(cfg);
  DeviceGuard guard(c->device);
  Timed tm(c, (hipStream_t)stream, FP8LM_K_SUM);
  hipStream_t s = (hipStream_t)stream;
#define FP8LM_SUM_N(N)                                                                          \
  case N:                                                                                       \
    if (fmt == FP8LM_E4M3) launch_walk<SumOp<kE4M3, N>>(c, s, sum_fp8_kernel<kE4M3, N>, p, sum_tiles(N));   \
    else launch_walk<SumOp<kE5M2, N>>(c, s, sum_fp8_kernel<kE5M2, N>, p, sum_tiles(N));                    \
    break
  static_assert(kUnrolledRanks == 8, "one case per unrolled rank count");
  switch (n_ranks) {
    FP8LM_SUM_N(1); FP8LM_SUM_N(2); FP8LM_SUM_N(3); FP8LM_SUM_N(4);
    FP8LM_SUM_N(5); FP8LM_SUM_N(6); FP8LM_SUM_N(7); FP8LM_SUM_N(8);
    default:          // any larger number of ranks: the kernel that loops over them
      if (fmt == FP8LM_E4M3) launch_walk<SumOp<kE4M3, 0>>(c, s, sum_fp8_kernel<kE4M3, 0>, p);
      else launch_walk<SumOp<kE5M2, 0>>(c, s, sum_fp8_kernel<kE5M2, 0>, p);
      break;
  }
#undef FP8LM_SUM_N
  return after_launch();
}

fp8lm_status fp8lm_autoscale_broadcast(fp8lm_ctx* c, const fp8lm_meta* from, fp8lm_meta* const* metas, int32_t n_ranks,
                                       void* stream) {
  if (!c || !metas || n_ranks < 1 || n_ranks > kMaxRanks) return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_tensors == 0) return FP8LM_OK;
  if (!from) return FP8LM_ERR_INVALID_ARGUMENT;
  RankMetasOut rm{};
  rm.n_ranks = n_ranks;
  for (int r = 0; r < n_ranks; ++r) {
    if (!metas[r] || metas[r] == from) return FP8LM_ERR_INVALID_ARGUMENT;
    rm.m[r] = metas[r];
  }
  DeviceGuard guard(c->device);
  Timed tm(c, (hipStream_t)stream, FP8LM_K_SCALARS);
  hipLaunchKernelGGL(autoscale_broadcast_kernel, dim3((c->n_tensors + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                     from, rm, c->n_tensors);
  return after_launch();
}

fp8lm_status fp8lm_set_mu(fp8lm_ctx* c, fp8lm_meta* meta, int32_t mu_exp, void* stream) {
  if (!c || mu_exp < -64 || mu_exp > 1) return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_tensors == 0) return FP8LM_OK;
  if (!meta) return FP8LM_ERR_INVALID_ARGUMENT;
  DeviceGuard guard(c->device);
  Timed tm(c, (hipStream_t)stream, FP8LM_K_SCALARS);
  hipLaunchKernelGGL(set_mu_kernel, dim3((c->n_tensors + 255) / 256), dim3(256), 0, (hipStream_t)stream, meta,
                     c->n_tensors, mu_exp);
  return after_launch();
}

fp8lm_status fp8lm_init_master_as(fp8lm_ctx* c, const void* w_bf16, void* w_out, fp8lm_meta* w_meta,
                                  fp8lm_state_fmt master_fmt, void* stream) {
  if (!c || (int)master_fmt < 0 || (int)master_fmt > 3) return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_chunks == 0) return FP8LM_OK;
  if (!w_bf16 || !w_out || !w_meta) return FP8LM_ERR_INVALID_ARGUMENT;
  if (!aligned16(w_bf16) || !aligned16(w_out)) return FP8LM_ERR_MISALIGNED;
  DeviceGuard guard(c->device);
  hipStream_t s = (hipStream_t)stream;
  Timed tm(c, s, FP8LM_K_INIT_MASTER);
  const uint32_t fmax_bits = master_fmt == FP8LM_STATE_F16 ? kBitsF16Max : (master_fmt == FP8LM_STATE_E4M3 ? kBitsE4M3Max : 0u);
  AmaxParams pa{static_cast<const uint16_t*>(w_bf16), w_meta, fmax_bits, 1, 0};
  launch_amax<kAmaxForMaster, kSrcBF16>(c, s, pa);
  fp8lm_status st = after_launch();
  if (st != FP8LM_OK) return st;
  InitParams pi{static_cast<const uint16_t*>(w_bf16), w_out, w_meta};
  switch (master_fmt) {
    case FP8LM_STATE_F16: launch_walk<InitCastOp<kStF16>>(c, s, init_master_cast_kernel<kStF16>, pi); break;
    case FP8LM_STATE_BF16: launch_walk<InitCastOp<kStBF16>>(c, s, init_master_cast_kernel<kStBF16>, pi); break;
    case FP8LM_STATE_E4M3: launch_walk<InitCastOp<kStE4M3>>(c, s, init_master_cast_kernel<kStE4M3>, pi); break;
    default: launch_walk<InitCastOp<kStF32>>(c, s, init_master_cast_kernel<kStF32>, pi); break;
  }
  return after_launch();
}

fp8lm_status fp8lm_init_master(fp8lm_ctx* c, const void* w_bf16, uint16_t* w_f16, fp8lm_meta* w_meta, void* stream) {
  return fp8lm_init_master_as(c, w_bf16, w_f16, w_meta, FP8LM_STATE_F16, stream);
}

// Validation of everything but the context (shared by the two Adam entry points).
static fp8lm_status adam_args_ok(const uint8_t* grad, fp8lm_fmt grad_fmt, const fp8lm_meta* grad_meta, uint8_t* m,
                                 fp8lm_meta* m_meta, void* v, fp8lm_meta* v_meta, void* w, fp8lm_meta* w_meta, void* wcopy,
                                 fp8lm_meta* wcopy_meta, const fp8lm_adam_hparams* hp, bool have_chunks) {
  if (!hp || (grad_fmt != FP8LM_E4M3 && grad_fmt != FP8LM_E5M2)) return FP8LM_ERR_INVALID_ARGUMENT;
  if (hp->wcopy != FP8LM_WCOPY_E4M3 && hp->wcopy != FP8LM_WCOPY_BF16) return FP8LM_ERR_INVALID_ARGUMENT;
  if (hp->m_scale_mode < 0 || hp->m_scale_mode > 2) return FP8LM_ERR_INVALID_ARGUMENT;
  if (hp->master_fmt < 0 || hp->master_fmt > 3 || (hp->v_fmt != FP8LM_STATE_F16 && hp->v_fmt != FP8LM_STATE_E4M3))
    return FP8LM_ERR_INVALID_ARGUMENT;
  const bool variant = hp->master_fmt != FP8LM_STATE_F16 || hp->v_fmt != FP8LM_STATE_F16;
  if (variant && (hp->wcopy != FP8LM_WCOPY_E4M3 || hp->stats)) return FP8LM_ERR_INVALID_ARGUMENT;
  if (!(hp->lr >= 0.0f && hp->lr <= 1024.0f) || !(hp->beta1 >= 0.0f && hp->beta1 < 1.0f) ||
      !(hp->beta2 >= 0.0f && hp->beta2 < 1.0f) || !(hp->eps >= 0x1p-36f && hp->eps < INFINITY) ||
      !(hp->weight_decay >= 0.0f && hp->weight_decay <= 1024.0f) || hp->step < 1)
    return FP8LM_ERR_INVALID_ARGUMENT;
  if (!have_chunks) return FP8LM_OK;
  if (!grad || !grad_meta || !m || !m_meta || !v || !v_meta || !w || !w_meta || !wcopy || !wcopy_meta)
    return FP8LM_ERR_INVALID_ARGUMENT;
  if (!aligned16(grad) || !aligned16(m) || !aligned16(v) || !aligned16(w) || !aligned16(wcopy)) return FP8LM_ERR_MISALIGNED;
  // the one pair of buffers that may be the same: an E4M3 weight copy written over the gradient it was computed from
  if (static_cast<const void*>(grad) == wcopy && hp->wcopy != FP8LM_WCOPY_E4M3) return FP8LM_ERR_INVALID_ARGUMENT;
  return FP8LM_OK;
}

static fp8lm_status adam_launch(fp8lm_ctx* c, const uint8_t* grad, fp8lm_fmt grad_fmt, const fp8lm_meta* grad_meta,
                                uint8_t* m, fp8lm_meta* m_meta, void* v, fp8lm_meta* v_meta, void* w, fp8lm_meta* w_meta,
                                void* wcopy, fp8lm_meta* wcopy_meta, const fp8lm_adam_hparams* hp, hipStream_t s,
                                const uint8_t* m_in = nullptr);

fp8lm_status fp8lm_adam_step_fp8(fp8lm_ctx* c, const uint8_t* grad, fp8lm_fmt grad_fmt, const fp8lm_meta* grad_meta,
                                 uint8_t* m, fp8lm_meta* m_meta, void* v, fp8lm_meta* v_meta, void* w,
                                 fp8lm_meta* w_meta, void* wcopy, fp8lm_meta* wcopy_meta, const fp8lm_adam_hparams* hp,
                                 void* stream) {
  if (!c) return FP8LM_ERR_INVALID_ARGUMENT;
  const fp8lm_status ok = adam_args_ok(grad, grad_fmt, grad_meta, m, m_meta, v, v_meta, w, w_meta, wcopy, wcopy_meta, hp,
                                       c->n_chunks > 0);
  if (ok != FP8LM_OK) return ok;
  if (c->n_chunks == 0) return FP8LM_OK;
  DeviceGuard guard(c->device);
  return adam_launch(c, grad, grad_fmt, grad_meta, m, m_meta, v, v_meta, w, w_meta, wcopy, wcopy_meta, hp,
                     (hipStream_t)stream);
}

// The launches of one Adam step on the tables `c` points to (a context's own, or the fixed device array).
// m_in: null for the in-place step; otherwise the buffer the first moment is read from, and its scale is speculated.
static fp8lm_status adam_launch(fp8lm_ctx* c, const uint8_t* grad, fp8lm_fmt grad_fmt, const fp8lm_meta* grad_meta,
                                uint8_t* m, fp8lm_meta* m_meta, void* v, fp8lm_meta* v_meta, void* w, fp8lm_meta* w_meta,
                                void* wcopy, fp8lm_meta* wcopy_meta, const fp8lm_adam_hparams* hp, hipStream_t s,
                                const uint8_t* m_in) {
  const bool variant = hp->master_fmt != FP8LM_STATE_F16 || hp->v_fmt != FP8LM_STATE_F16;
  const bool spec_m = m_in != nullptr;

  AdamParams p{};
  p.grad = grad; p.grad_meta = grad_meta; p.m = m; p.m_meta = m_meta; p.v = v; p.v_meta = v_meta;
  p.w = w; p.w_meta = w_meta; p.wcopy = wcopy; p.wcopy_meta = wcopy_meta;
  // scalars derived once on the host, in double, then rounded to fp32
  p.b1 = hp->beta1;
  p.b2 = hp->beta2;
  p.omb1 = (float)(1.0 - (double)p.b1);
  p.omb2 = (float)(1.0 - (double)p.b2);
  p.rbc1 = (float)(1.0 / (1.0 - std::pow((double)p.b1, (double)hp->step)));
  p.rbc2 = (float)(1.0 / (1.0 - std::pow((double)p.b2, (double)hp->step)));
  p.lr = hp->lr;
  p.eps = hp->eps;
  p.decay = (float)(1.0 - (double)hp->lr * (double)hp->weight_decay);
  p.v_scaled = (hp->v_scaled || hp->v_fmt == FP8LM_STATE_E4M3) ? 1 : 0;
  p.v_fmax_bits = hp->v_fmt == FP8LM_STATE_E4M3 ? kBitsE4M3Max : kBitsF16Max;
  p.w_fmax_bits = hp->master_fmt == FP8LM_STATE_F16 ? kBitsF16Max : (hp->master_fmt == FP8LM_STATE_E4M3 ? kBitsE4M3Max : 0u);
  p.m_in = spec_m ? m_in : m;
  p.speculative_m = spec_m ? 1 : 0;

  const bool stats = hp->stats != 0, fast = hp->exact == 0;
  if (spec_m) {
    ++c->spec_call;
    c->spec_kind = 1;
  }
  int grid = 0;
  const Tables tb = tables_of(c, 1, 16, &grid);      // for the per-tensor kernels, which only need the tables
  const bool e5 = grad_fmt == FP8LM_E5M2, q8 = hp->wcopy == FP8LM_WCOPY_E4M3;
  if (spec_m) {
    Timed tm(c, s, FP8LM_K_SCALARS);
    const dim3 gs((c->n_tensors + 255) / 256), bs(256);
    if (q8) hipLaunchKernelGGL((adam_speculate_scales_kernel<FP8LM_WCOPY_E4M3>), gs, bs, 0, s, tb, p, c->n_tensors);
    else hipLaunchKernelGGL((adam_speculate_scales_kernel<FP8LM_WCOPY_BF16>), gs, bs, 0, s, tb, p, c->n_tensors);
  } else if (hp->m_scale_mode == FP8LM_MSCALE_FROM_CAST) {
    const fp8lm_ctx::Fused f = c->fused;
    c->fused.valid = false;
    if (!f.valid || f.grad != grad || f.m != m || f.m_meta != m_meta || f.b1 != p.b1 || f.fmt != (int)grad_fmt)
      return FP8LM_ERR_INVALID_ARGUMENT;
    Timed tm(c, s, FP8LM_K_SCALARS);
    const dim3 gs((c->n_tensors + 255) / 256), bs(256);
    if (q8) hipLaunchKernelGGL((adam_scales_from_cast_kernel<FP8LM_WCOPY_E4M3>), gs, bs, 0, s, tb, p, c->n_tensors);
    else hipLaunchKernelGGL((adam_scales_from_cast_kernel<FP8LM_WCOPY_BF16>), gs, bs, 0, s, tb, p, c->n_tensors);
  } else if (hp->m_scale_mode == FP8LM_MSCALE_PREDICTED) {
    Timed tm(c, s, FP8LM_K_SCALARS);
    const dim3 gs((c->n_tensors + 255) / 256), bs(256);
    if (q8) hipLaunchKernelGGL((adam_predict_scales_kernel<FP8LM_WCOPY_E4M3>), gs, bs, 0, s, tb, p, c->n_tensors);
    else hipLaunchKernelGGL((adam_predict_scales_kernel<FP8LM_WCOPY_BF16>), gs, bs, 0, s, tb, p, c->n_tensors);
  } else {
    Timed tm(c, s, FP8LM_K_ADAM_AMAX);
    if (e5 && q8) launch_walk<AdamAmaxOp<kE5M2, FP8LM_WCOPY_E4M3>>(c, s, adam_amax_kernel<kE5M2, FP8LM_WCOPY_E4M3>, p, kUnRead);
    else if (e5) launch_walk<AdamAmaxOp<kE5M2, FP8LM_WCOPY_BF16>>(c, s, adam_amax_kernel<kE5M2, FP8LM_WCOPY_BF16>, p, kUnRead);
    else if (q8) launch_walk<AdamAmaxOp<kE4M3, FP8LM_WCOPY_E4M3>>(c, s, adam_amax_kernel<kE4M3, FP8LM_WCOPY_E4M3>, p, kUnRead);
    else launch_walk<AdamAmaxOp<kE4M3, FP8LM_WCOPY_BF16>>(c, s, adam_amax_kernel<kE4M3, FP8LM_WCOPY_BF16>, p, kUnRead);
  }
  fp8lm_status st = after_launch();
  if (st != FP8LM_OK) return st;
  Tables first{};
  if (variant) {
    Timed tm(c, s, FP8LM_K_ADAM_UPDATE);
    launch_update_variant(c, s, p, e5, hp->master_fmt, hp->v_fmt);
  } else {
    Timed tm(c, s, FP8LM_K_ADAM_UPDATE);
    if (e5 && q8) first = launch_update<kE5M2, FP8LM_WCOPY_E4M3>(c, s, p, fast, stats);
    else if (e5) first = launch_update<kE5M2, FP8LM_WCOPY_BF16>(c, s, p, fast, stats);
    else if (q8) first = launch_update<kE4M3, FP8LM_WCOPY_E4M3>(c, s, p, fast, stats);
    else first = launch_update<kE4M3, FP8LM_WCOPY_BF16>(c, s, p, fast, stats);
  }
  st = after_launch();
  if (st != FP8LM_OK || !spec_m) return st;
  // tensors whose first-moment scale turned out different: the moment once more
  {
    int grid = 0;
    const Tables rt = marked_tables_of(c, first, &grid);
    const dim3 g(grid), b(kThreads);
    Timed tm(c, s, FP8LM_K_ADAM_AMAX);
    if (e5) hipLaunchKernelGGL((adam_moment_redo_kernel<kE5M2>), g, b, 0, s, rt, p);
    else hipLaunchKernelGGL((adam_moment_redo_kernel<kE4M3>), g, b, 0, s, rt, p);
  }
  return after_launch();
}

fp8lm_status fp8lm_adam_step_fp8_m2(fp8lm_ctx* c, const uint8_t* grad, fp8lm_fmt grad_fmt, const fp8lm_meta* grad_meta,
                                    const uint8_t* m_in, uint8_t* m_out, fp8lm_meta* m_meta, void* v, fp8lm_meta* v_meta,
                                    void* w, fp8lm_meta* w_meta, void* wcopy, fp8lm_meta* wcopy_meta,
                                    const fp8lm_adam_hparams* hp, void* stream) {
  if (!c) return FP8LM_ERR_INVALID_ARGUMENT;
  const fp8lm_status ok = adam_args_ok(grad, grad_fmt, grad_meta, m_out, m_meta, v, v_meta, w, w_meta, wcopy, wcopy_meta, hp,
                                       c->n_chunks > 0);
  if (ok != FP8LM_OK) return ok;
  // the exact-amax scale only, default storage formats, no element counters (they would have to be recounted)
  if (hp->m_scale_mode != FP8LM_MSCALE_EXACT_PASS || hp->master_fmt != FP8LM_STATE_F16 || hp->v_fmt != FP8LM_STATE_F16 || hp->stats)
    return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_chunks == 0) return FP8LM_OK;
  if (!m_in || m_in == m_out) return FP8LM_ERR_INVALID_ARGUMENT;
  if (!aligned16(m_in)) return FP8LM_ERR_MISALIGNED;
  if (static_cast<const void*>(grad) == wcopy) return FP8LM_ERR_OVERLAP;     // the repair reads the gradient again
  {
    // the two buffers must not share an element of any tensor
    long long extent = 0;
    for (const fp8lm_tensor& T : c->tensors) extent = std::max<long long>(extent, T.numel > 0 ? T.offset + T.numel : 0);
    const uintptr_t a = reinterpret_cast<uintptr_t>(m_in), b = reinterpret_cast<uintptr_t>(m_out);
    if (a < b + (uintptr_t)extent && b < a + (uintptr_t)extent) return FP8LM_ERR_OVERLAP;
  }
  DeviceGuard guard(c->device);
  c->fused.valid = false;
  return adam_launch(c, grad, grad_fmt, grad_meta, m_out, m_meta, v, v_meta, w, w_meta, wcopy, wcopy_meta, hp,
                     (hipStream_t)stream, m_in);
}

fp8lm_status fp8lm_get_moment_speculation_stats(fp8lm_ctx* c, uint64_t* calls, uint64_t* tensors_redone,
                                                uint64_t* elems_redone, void* stream) {
  if (!c || !calls || !tensors_redone || !elems_redone) return FP8LM_ERR_INVALID_ARGUMENT;
  DeviceGuard guard(c->device);
  unsigned long long h[3] = {0, 0, 0};
  HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
  HIP_TRY(hipMemcpy(h, c->d_spec_totals + 3, sizeof(h), hipMemcpyDeviceToHost));
  *calls = h[0]; *tensors_redone = h[1]; *elems_redone = h[2];
  return FP8LM_OK;
}

// ---- the Adam step without a context: tables, scales and reduction records in the fixed device array ----------
namespace {

constexpr int kMaxDevices = 64;
struct StaticDevice {
  StaticArena* arena = nullptr;      // device address of `scratch` on this GPU
  int num_cus = 0;
};
std::mutex g_static_mutex;
StaticDevice g_static_dev[kMaxDevices];

// Device address of the fixed array on `device` (which must be current) and that GPU's size; looked up on the
// first call per GPU.  Each GPU holds its own copy of the array at its own address.
fp8lm_status static_arena_of(int device, StaticDevice* out) {
  std::lock_guard<std::mutex> lock(g_static_mutex);
  StaticDevice& d = g_static_dev[device];
  if (!d.arena) {
    void* ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) { g_hip_error = "hipGetSymbolAddress returned a null address"; return FP8LM_ERR_HIP; }
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device));
    d.num_cus = cus > 0 ? cus : 256;
    d.arena = static_cast<StaticArena*>(ptr);
  }
  *out = d;
  return FP8LM_OK;
}

}  // namespace

fp8lm_status fp8lm_adam_step_fp8_static(int device, const fp8lm_tensor* tensors, int32_t n, const uint32_t* tensor_flags,
                                        const uint8_t* grad, fp8lm_fmt grad_fmt, const fp8lm_meta* grad_meta, uint8_t* m,
                                        fp8lm_meta* m_meta, void* v, fp8lm_meta* v_meta, void* w, fp8lm_meta* w_meta,
                                        void* wcopy, fp8lm_meta* wcopy_meta, const fp8lm_adam_hparams* hp, void* stream) {
  if (n < 0 || (n > 0 && !tensors) || device < 0 || device >= kMaxDevices) return FP8LM_ERR_INVALID_ARGUMENT;
  if (n > FP8LM_STATIC_MAX_TENSORS) return FP8LM_ERR_TOO_LARGE;
  // the tensor list: same rules as fp8lm_create; everything below lives on this thread's stack
  long long total_chunks = 0;
  {
    std::pair<long long, long long> spans[FP8LM_STATIC_MAX_TENSORS];
    int n_spans = 0;
    for (int t = 0; t < n; ++t) {
      if (tensors[t].numel < 0 || tensors[t].offset < 0) return FP8LM_ERR_INVALID_ARGUMENT;
      if (tensors[t].offset % 16 != 0) return FP8LM_ERR_MISALIGNED;
      if (tensor_flags && (tensor_flags[t] & ~(uint32_t)FP8LM_TENSOR_NO_WEIGHT_DECAY)) return FP8LM_ERR_INVALID_ARGUMENT;
      if (tensors[t].numel > 0) spans[n_spans++] = {tensors[t].offset, tensors[t].offset + tensors[t].numel};
      total_chunks += (tensors[t].numel + kStaticChunkElems - 1) / kStaticChunkElems;
      if (total_chunks > FP8LM_STATIC_MAX_CHUNKS) return FP8LM_ERR_TOO_LARGE;
    }
    std::sort(spans, spans + n_spans);
    for (int i = 1; i < n_spans; ++i)
      if (spans[i].first < spans[i - 1].second) return FP8LM_ERR_OVERLAP;
  }
  const fp8lm_status ok = adam_args_ok(grad, grad_fmt, grad_meta, m, m_meta, v, v_meta, w, w_meta, wcopy, wcopy_meta, hp,
                                       total_chunks > 0);
  if (ok != FP8LM_OK) return ok;
  if (hp->m_scale_mode == FP8LM_MSCALE_FROM_CAST) return FP8LM_ERR_INVALID_ARGUMENT;   // needs the fused cast's context
  int count = 0;
  HIP_TRY(hipGetDeviceCount(&count));
  if (device >= count) return FP8LM_ERR_INVALID_ARGUMENT;
  if (total_chunks == 0) return FP8LM_OK;
  DeviceGuard guard(device);
  if (!guard.ok) { g_hip_error = "hipSetDevice failed"; return FP8LM_ERR_HIP; }
  StaticDevice dev;
  const fp8lm_status got = static_arena_of(device, &dev);
  if (got != FP8LM_OK) return got;
  StaticArena* A = dev.arena;
  hipStream_t s = (hipStream_t)stream;

  // 1. the tensor table, a batch of descriptors per launch, then the chunk table
  DescBatch batch;
  int32_t first_chunk = 0, first_epi = 0;
  // the usual chunks or, where the units of a launch would be too many for the records, larger ones
  int32_t chunk_elems = default_chunk(n, [&](int t) { return tensors[t].numel; });
  auto chunks_of = [&](int64_t numel) { return (numel + chunk_elems - 1) / chunk_elems; };
  for (;; chunk_elems *= 2) {
    total_chunks = 0;
    for (int t = 0; t < n; ++t) total_chunks += chunks_of(tensors[t].numel);
    if (total_chunks <= kStaticChunks) break;
  }
  for (int t0 = 0; t0 < n; t0 += kDescBatch) {
    batch.first = t0;
    batch.count = std::min(kDescBatch, n - t0);
    for (int i = 0; i < batch.count; ++i) {
      const fp8lm_tensor& T = tensors[t0 + i];
      const int32_t nc = (int32_t)chunks_of(T.numel);
      batch.d[i] = TensorDesc{T.offset, T.numel, first_chunk, nc, tensor_flags ? tensor_flags[t0 + i] : 0u, first_epi};
      first_chunk += nc;
      if (nc > 0) first_epi += epilogue_groups(nc);
    }
    for (int i = batch.count; i < kDescBatch; ++i) batch.d[i] = TensorDesc{0, 0, 0, 0, 0u, 0};
    hipLaunchKernelGGL(static_desc_kernel, dim3(1), dim3(kDescBatch), 0, s, batch, A->desc);
  }
  hipLaunchKernelGGL(chunk_tables_kernel, dim3(std::min(n, 1024)), dim3(kThreads), 0, s, A->desc, A->chunks, A->epi, A->scratch,
                     chunk_elems, n);
  fp8lm_status st = after_launch();
  if (st != FP8LM_OK) return st;

  // 2. the two passes, on a context-shaped view of the array (no vectors in it are ever filled: nothing allocates)
  fp8lm_ctx view;
  view.device = device;
  view.n_tensors = n;
  view.num_cus = dev.num_cus;
  view.chunk_elems = chunk_elems;
  view.n_chunks = (int32_t)total_chunks;
  view.d_desc = A->desc;
  view.d_chunks = A->chunks;
  view.d_scratch = A->scratch;
  view.d_records = A->records;
  view.record_bytes = sizeof(A->records);
  view.d_totals = A->totals;
  view.d_epi = A->epi;
  view.n_epi = first_epi;
  return adam_launch(&view, grad, grad_fmt, grad_meta, m, m_meta, v, v_meta, w, w_meta, wcopy, wcopy_meta, hp, s);
}

fp8lm_status fp8lm_quant_error_stats(fp8lm_ctx* c, const void* ref, fp8lm_src ref_type, const uint8_t* q, fp8lm_fmt fmt,
                                     const fp8lm_meta* q_meta, fp8lm_quant_stats* out, void* stream) {
  if (!c || !src_ok(ref_type) || (fmt != FP8LM_E4M3 && fmt != FP8LM_E5M2)) return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_tensors == 0) return FP8LM_OK;
  if (!out || (c->n_chunks > 0 && (!ref || !q || !q_meta))) return FP8LM_ERR_INVALID_ARGUMENT;
  if (c->n_chunks > 0 && (!aligned16(ref) || !aligned16(q))) return FP8LM_ERR_MISALIGNED;
  DeviceGuard guard(c->device);
  hipStream_t s = (hipStream_t)stream;
  if (c->n_chunks == 0) {                        // only empty tensors
    Timed tm(c, s, FP8LM_K_SCALARS);
    hipLaunchKernelGGL(quant_stats_zero_kernel, dim3((c->n_tensors + 255) / 256), dim3(256), 0, s, out, c->n_tensors);
    return after_launch();
  }
  StatsParams p{ref, q, q_meta, out, c->d_partials};
  int unused = 0;
  const Tables tb = tables_of(c, 1, 16, &unused);    // for its chunk table; the grid is persistent (see stats.hpp)
  const int grid = grid_of(c);
  const dim3 ge(std::min<int>(c->n_tensors, 8 * c->num_cus));
  Timed tm(c, s, FP8LM_K_STATS);
#define FP8LM_STATS_LAUNCH(F, S)                                                                             \
  do {                                                                                                       \
    hipLaunchKernelGGL((quant_stats_kernel<F, S>), dim3(grid), dim3(kThreads), 0, s, tb, p);                 \
    hipLaunchKernelGGL((quant_stats_epilogue_kernel<F, S>), ge, dim3(kThreads), 0, s, tb, p, grid, c->n_tensors); \
  } while (0)
#define FP8LM_STATS_SRC(S)                                                                                   \
  do {                                                                                                       \
    if (fmt == FP8LM_E4M3) FP8LM_STATS_LAUNCH(kE4M3, S);                                                     \
    else FP8LM_STATS_LAUNCH(kE5M2, S);                                                                       \
  } while (0)
  if (ref_type == FP8LM_SRC_F32) FP8LM_STATS_SRC(kSrcF32);
  else if (ref_type == FP8LM_SRC_F16) FP8LM_STATS_SRC(kSrcF16);
  else FP8LM_STATS_SRC(kSrcBF16);
#undef FP8LM_STATS_SRC
#undef FP8LM_STATS_LAUNCH
  return after_launch();
}

// Host only.  Whole-tensor greedy distribution of Sec. 2.3, Alg. 1, with a heap over the GPUs.
fp8lm_status fp8lm_greedy_partition(const int64_t* sizes, int32_t n, int32_t n_gpus, int32_t* owner, int64_t* usage) {
  if (n < 0 || n_gpus < 1 || (n > 0 && (!sizes || !owner)) || !usage) return FP8LM_ERR_INVALID_ARGUMENT;
  for (int32_t i = 0; i < n; ++i)
    if (sizes[i] < 0) return FP8LM_ERR_INVALID_ARGUMENT;
  std::vector<int32_t> order(n);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return sizes[a] > sizes[b]; });
  typedef std::pair<int64_t, int32_t> Load;   // (memory in use, gpu): the smallest pair is the next receiver
  std::priority_queue<Load, std::vector<Load>, std::greater<Load>> heap;
  for (int32_t j = 0; j < n_gpus; ++j) heap.emplace(0, j);
  for (int32_t i : order) {
    Load top = heap.top();
    heap.pop();
    owner[i] = top.second;
    top.first += sizes[i];
    heap.push(top);
  }
  for (int32_t j = 0; j < n_gpus; ++j) usage[j] = 0;
  for (int32_t i = 0; i < n; ++i) usage[owner[i]] += sizes[i];
  return FP8LM_OK;
}

fp8lm_status fp8lm_copy_bytes(fp8lm_ctx* c, const void* src, void* dst, int64_t bytes, void* stream) {
  if (!c || !src || !dst || bytes < 0 || bytes % 16 != 0) return FP8LM_ERR_INVALID_ARGUMENT;
  if (!aligned16(src) || !aligned16(dst)) return FP8LM_ERR_MISALIGNED;
  if (bytes == 0) return FP8LM_OK;
  DeviceGuard guard(c->device);
  const long long n16 = bytes / 16;
  const long long want = (long long)c->num_cus * c->blocks_per_cu;
  const int grid = (int)std::max<long long>(1, std::min<long long>(want, (n16 + kThreads - 1) / kThreads));
  Timed tm(c, (hipStream_t)stream, FP8LM_K_COPY);
  hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(kThreads), 0, (hipStream_t)stream, static_cast<const uint4*>(src),
                     static_cast<uint4*>(dst), n16);
  return after_launch();
}

fp8lm_status fp8lm_memory_skeleton(fp8lm_ctx* c, int32_t shape, void* const* bufs, int64_t n_elems, void* stream) {
  static const int n_bufs[] = {1, 2, 1, 1, 2, 5, 5, 5, 5};
  if (!c || shape < 0 || shape > FP8LM_SKEL_UPDATE_RANGES || !bufs || n_elems < 0 || n_elems % kTile != 0)
    return FP8LM_ERR_INVALID_ARGUMENT;
  for (int i = 0; i < n_bufs[shape]; ++i) {
    if (!bufs[i]) return FP8LM_ERR_INVALID_ARGUMENT;
    if (!aligned16(bufs[i])) return FP8LM_ERR_MISALIGNED;
  }
  if (n_elems == 0) return FP8LM_OK;
  DeviceGuard guard(c->device);
  SkeletonParams p{};
  p.n_tiles = n_elems / kTile;
  p.sink = reinterpret_cast<uint32_t*>(c->d_partials);
  const dim3 b(kThreads);
  p.ranges = shape == FP8LM_SKEL_UPDATE_RANGES || c->blocks_per_cu < kMaxBlocksPerCu ? 1 : 0;
  auto grid = [&](int un) {
    const long long all = (p.n_tiles + un - 1) / un;
    return dim3((unsigned)std::min(p.ranges ? (long long)c->num_cus * c->blocks_per_cu : kMaxGrid, all));
  };
  hipStream_t s = (hipStream_t)stream;
  Timed tm(c, s, FP8LM_K_SKELETON);
  switch (shape) {
    case FP8LM_SKEL_READ16:
      p.s2[0] = static_cast<const uint16_t*>(bufs[0]);
      hipLaunchKernelGGL((skeleton_kernel<0, 1, 0, 0, kUnRead>), grid(kUnRead), b, 0, s, p);
      break;
    case FP8LM_SKEL_READ8X2:
      p.s1[0] = static_cast<const uint8_t*>(bufs[0]); p.s1[1] = static_cast<const uint8_t*>(bufs[1]);
      hipLaunchKernelGGL((skeleton_kernel<2, 0, 0, 0, kUnRead>), grid(kUnRead), b, 0, s, p);
      break;
    case FP8LM_SKEL_WRITE16:
      p.d2[0] = static_cast<uint16_t*>(bufs[0]);
      hipLaunchKernelGGL((skeleton_kernel<0, 0, 0, 1, 1>), grid(1), b, 0, s, p);
      break;
    case FP8LM_SKEL_WRITE8:
      p.d1[0] = static_cast<uint8_t*>(bufs[0]);
      hipLaunchKernelGGL((skeleton_kernel<0, 0, 1, 0, 1>), grid(1), b, 0, s, p);
      break;
    case FP8LM_SKEL_CAST:
      p.s2[0] = static_cast<const uint16_t*>(bufs[0]); p.d1[0] = static_cast<uint8_t*>(bufs[1]);
      hipLaunchKernelGGL((skeleton_kernel<0, 1, 1, 0, kUnCast<kSrcBF16>>), grid(kUnCast<kSrcBF16>), b, 0, s, p);
      break;
    default:   // the update shapes: reads g, m, v, w; writes m, v, w in place and the weight copy; or one half of that
      p.s1[0] = static_cast<const uint8_t*>(bufs[0]); p.s1[1] = static_cast<const uint8_t*>(bufs[1]);
      p.s2[0] = static_cast<const uint16_t*>(bufs[2]); p.s2[1] = static_cast<const uint16_t*>(bufs[3]);
      p.d1[0] = static_cast<uint8_t*>(bufs[1]); p.d1[1] = static_cast<uint8_t*>(bufs[4]);
      p.d2[0] = static_cast<uint16_t*>(bufs[2]); p.d2[1] = static_cast<uint16_t*>(bufs[3]);
      if (shape == FP8LM_SKEL_UPDATE || shape == FP8LM_SKEL_UPDATE_RANGES) hipLaunchKernelGGL((skeleton_kernel<2, 2, 2, 2, kUnUpdate>), grid(kUnUpdate), b, 0, s, p);
      else if (shape == FP8LM_SKEL_UPDATE_READS) hipLaunchKernelGGL((skeleton_kernel<2, 2, 0, 0, kUnUpdate>), grid(kUnUpdate), b, 0, s, p);
      else hipLaunchKernelGGL((skeleton_kernel<0, 0, 2, 2, kUnUpdate>), grid(kUnUpdate), b, 0, s, p);
      break;
  }
  return after_launch();
}

// ---- device memory piece by piece (HIP virtual memory management); see fp8lm.h ---------------------------------
namespace {
hipMemAllocationProp vmm_prop(int device) {
  hipMemAllocationProp prop = {};
  prop.type = hipMemAllocationTypePinned;
  prop.location.type = hipMemLocationTypeDevice;
  prop.location.id = device;
  return prop;
}
fp8lm_status vmm_granularity_of(int device, size_t* g) {
  const hipMemAllocationProp prop = vmm_prop(device);
  HIP_TRY(hipMemGetAllocationGranularity(g, &prop, hipMemAllocationGranularityRecommended));
  if (*g == 0) *g = 4096;
  return FP8LM_OK;
}
}  // namespace

fp8lm_status fp8lm_vmm_granularity(int device, uint64_t* bytes) {
  if (!bytes || device < 0) return FP8LM_ERR_INVALID_ARGUMENT;
  int ok = 0;
  HIP_TRY(hipDeviceGetAttribute(&ok, hipDeviceAttributeVirtualMemoryManagementSupported, device));
  if (!ok) { g_hip_error = "virtual memory management is not supported on this device"; return FP8LM_ERR_HIP; }
  size_t g = 0;
  const fp8lm_status st = vmm_granularity_of(device, &g);
  if (st == FP8LM_OK) *bytes = g;
  return st;
}

fp8lm_status fp8lm_vmm_reserve(uint64_t bytes, void** va) {
  if (!va || bytes == 0) return FP8LM_ERR_INVALID_ARGUMENT;
  *va = nullptr;
  HIP_TRY(hipMemAddressReserve(va, bytes, 0, nullptr, 0));
  return FP8LM_OK;
}

fp8lm_status fp8lm_vmm_free(void* va, uint64_t bytes) {
  if (!va || bytes == 0) return FP8LM_ERR_INVALID_ARGUMENT;
  HIP_TRY(hipMemAddressFree(va, bytes));
  return FP8LM_OK;
}

fp8lm_status fp8lm_vmm_create(int device, uint64_t bytes, uint64_t* piece) {
  if (!piece || bytes == 0 || device < 0) return FP8LM_ERR_INVALID_ARGUMENT;
  size_t g = 0;
  const fp8lm_status st = vmm_granularity_of(device, &g);
  if (st != FP8LM_OK) return st;
  if (bytes % g != 0) return FP8LM_ERR_INVALID_ARGUMENT;
  const hipMemAllocationProp prop = vmm_prop(device);
  hipMemGenericAllocationHandle_t h{};
  HIP_TRY(hipMemCreate(&h, bytes, &prop, 0));
  static_assert(sizeof(h) <= sizeof(uint64_t), "the handle travels as 64 bits");
  *piece = 0;
  std::memcpy(piece, &h, sizeof(h));
  return FP8LM_OK;
}

fp8lm_status fp8lm_vmm_destroy(uint64_t piece) {
  if (piece == 0) return FP8LM_ERR_INVALID_ARGUMENT;
  hipMemGenericAllocationHandle_t h{};
  std::memcpy(&h, &piece, sizeof(h));
  HIP_TRY(hipMemRelease(h));
  return FP8LM_OK;
}

fp8lm_status fp8lm_vmm_map(void* va, uint64_t bytes, uint64_t piece, int device) {
  if (!va || bytes == 0 || piece == 0 || device < 0) return FP8LM_ERR_INVALID_ARGUMENT;
  hipMemGenericAllocationHandle_t h{};
  std::memcpy(&h, &piece, sizeof(h));
  HIP_TRY(hipMemMap(va, bytes, 0, h, 0));
  hipMemAccessDesc acc = {};
  acc.location.type = hipMemLocationTypeDevice;
  acc.location.id = device;
  acc.flags = hipMemAccessFlagsProtReadWrite;
  const hipError_t e = hipMemSetAccess(va, bytes, &acc, 1);
  if (e != hipSuccess) {
    g_hip_error = std::string("hipMemSetAccess: ") + hipGetErrorString(e);
    (void)hipMemUnmap(va, bytes);
    return FP8LM_ERR_HIP;
  }
  return FP8LM_OK;
}

fp8lm_status fp8lm_vmm_unmap(void* va, uint64_t bytes) {
  if (!va || bytes == 0) return FP8LM_ERR_INVALID_ARGUMENT;
  HIP_TRY(hipDeviceSynchronize());     // no kernel may still be using the mapping
  HIP_TRY(hipMemUnmap(va, bytes));
  return FP8LM_OK;
}

fp8lm_status fp8lm_set_timing(fp8lm_ctx* c, int32_t enable) {
  if (!c) return FP8LM_ERR_INVALID_ARGUMENT;
  DeviceGuard guard(c->device);
  if (enable && c->free_events.empty() && c->stamps.empty()) {
    c->stamps.reserve(4096);           // launches are stamped without touching the host allocator
    c->free_events.reserve(4096);
    for (int i = 0; i < 4096; ++i) {
      hipEvent_t a = nullptr, b = nullptr;
      HIP_TRY(hipEventCreate(&a));
      if (hipError_t e = hipEventCreate(&b); e != hipSuccess) {
        (void)hipEventDestroy(a);
        g_hip_error = std::string("hipEventCreate: ") + hipGetErrorString(e);
        return FP8LM_ERR_HIP;
      }
      c->free_events.emplace_back(a, b);
    }
  }
  c->timing = enable != 0;
  return FP8LM_OK;
}

fp8lm_status fp8lm_get_timing(fp8lm_ctx* c, int32_t* launches, double* total_ms) {
  if (!c || !launches || !total_ms) return FP8LM_ERR_INVALID_ARGUMENT;
  DeviceGuard guard(c->device);
  for (int k = 0; k < FP8LM_K_COUNT; ++k) { launches[k] = 0; total_ms[k] = 0.0; }
  for (auto& s : c->stamps) {
    HIP_TRY(hipEventSynchronize(s.b));
    float ms = 0.0f;
    HIP_TRY(hipEventElapsedTime(&ms, s.a, s.b));
    launches[s.kernel] += 1;
    total_ms[s.kernel] += ms;
    c->free_events.emplace_back(s.a, s.b);
  }
  c->stamps.clear();
  return FP8LM_OK;
}

}  // extern "C"
