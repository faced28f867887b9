// Shared by every kernel of libfp8lm: tensor and chunk tables, wavefront / workgroup / grid-wide
// reductions, the chunk walk, 128-bit and 64-bit access helpers and the build-time tuning knobs.
#ifndef FP8LM_WALK_HPP
#define FP8LM_WALK_HPP

#include "fp8lm.h"
#include "formats.hpp"

namespace fp8lm {

constexpr int kThreads = 256;
constexpr int kGroup = 16;                 // elements per thread per iteration
constexpr int kTile = kThreads * kGroup;   // elements per workgroup per iteration
constexpr int kWaves = kThreads / 64;
constexpr int kMaxBlocksPerCu = 16;        // upper limit of the launch tuning; this value, the default, means "no limit"

struct TensorDesc {
  int64_t offset;
  int64_t numel;
  int32_t first_chunk;
  int32_t n_chunks;
  uint32_t flags;       // FP8LM_TENSOR_* attributes of the tensor
  int32_t epi0;         // the first of the workgroups that combine its records (epilogue_kernel)
};
struct alignas(16) ChunkDesc {
  int64_t base;         // its first element in the flat buffers
  int32_t len;
  int32_t tensor;
};
// A workgroup of the launch that combines records: its tensor, and which of the tensor's workgroups it is.
struct alignas(16) EpilogueDesc {
  TensorDesc d;
  int32_t tensor, k;
  int32_t pad[2];
};
// How many workgroups combine a tensor's records.
constexpr int kEpilogueChunks = 512, kMaxEpilogue = 64;
__host__ __device__ inline int epilogue_groups(int32_t n_chunks) {
  const int k = (n_chunks + kEpilogueChunks - 1) / kEpilogueChunks;
  return k < 1 ? 1 : (k > kMaxEpilogue ? kMaxEpilogue : k);
}

// Per-tensor scratch.  The ticket is zero between launches; the `pend` block carries the scales chosen
// by the first Adam pass to the second, and what else that needs to know of a tensor.
struct alignas(128) Scratch {
  uint32_t ticket;                // units finished, or epilogue workgroups
  uint32_t pad;
  float old_scale, old_inv;       // the scale the first moment's meta held before its speculation
  struct Pending {
    float sm, ism, sv, isv, sw, isw, sq, isq;
    uint32_t fm, fv, fw, fq;      // flags gathered while choosing the scales
    uint32_t careful;
    uint32_t amax_m_bits;   // written by a fused cast: bit pattern of max |m'|
    uint32_t tame;          // the update may take the short arithmetic, with these coefficients (tame_range)
    float c[8];
    float inv_sg, inv_sm, inv_sv, inv_sw, decay;      // inverse scales of the inputs; 1 - lr * weight_decay, or 1 if exempt
  } pend;
};

// What one workgroup found in its part of one tensor, for statistics whose order of summation has to be fixed (float64
// sums).  One record per (workgroup, tensor) pair.
struct alignas(64) Partial {
  double fs[2];
  unsigned long long ct[4];
};

struct Tables {
  const TensorDesc* desc;
  const ChunkDesc* chunks;
  Scratch* scratch;
  unsigned char* records;         // one record per unit (see leave_record)
  unsigned long long* totals;     // [epilogue workgroups][kTotalWords] what those of a large tensor hand to the last of them
  const EpilogueDesc* epi;        // [n_epi]
  int32_t n_epi;
  int32_t n_chunks;
  int32_t unit_elems;             // a chunk is cut into 2^unit_shift units of unit_elems elements, the work of a workgroup
  int32_t unit_shift;
  int32_t one_unit;               // 1: the grid has one workgroup per unit; 0: a workgroup walks a contiguous range of units
  int32_t deferred;               // 1: workgroups only leave their records; an epilogue launch finishes the tensors
  int32_t n_tensors;
  // speculation: the number of this call, where the last call that marked a tensor leaves its number, the marks (a tensor's
  // units, which have to be done again, or 0; padded with zeros to whole quads), running totals (calls, tensors done
  // again, elements done again)
  uint32_t call;
  uint32_t* marked_call;
  uint32_t* redo;
  unsigned long long* spec_totals;
};

// A load from an address all lanes share, through the scalar cache and whatever stores come before it: the compiler takes
// what it reads as constant.  So only for what the launch does not write, or writes only once every workgroup that could
// read it has done so: a tensor's metadata before its units, never in its scalar epilogue (finalize).
template <class T> __device__ __forceinline__ T uniform_load(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "words");
  struct Words { uint32_t w[sizeof(T) / 4]; } v;
  const auto* q = reinterpret_cast<const __attribute__((address_space(4))) uint32_t*>(reinterpret_cast<uintptr_t>(p));
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 4; ++i) v.w[i] = q[i];
  return __builtin_bit_cast(T, v);
}

// Writes the chunk and epilogue tables from the tensor table and returns the tickets to zero; workgroup t (and t + grid,
// ...) does tensor t's part.
__global__ void chunk_tables_kernel(const TensorDesc* desc, ChunkDesc* chunks, EpilogueDesc* epi, Scratch* scratch, int chunk_elems, int n) {
  for (int t = blockIdx.x; t < n; t += gridDim.x) {
    const TensorDesc d = desc[t];
    for (int i = threadIdx.x; i < d.n_chunks; i += blockDim.x) {
      const long long e0 = (long long)i * chunk_elems, rest = d.numel - e0;
      chunks[d.first_chunk + i] = ChunkDesc{d.offset + e0, (int32_t)(rest < chunk_elems ? rest : chunk_elems), t};
    }
    if (d.n_chunks > 0)
      for (int i = threadIdx.x; i < epilogue_groups(d.n_chunks); i += blockDim.x) epi[d.epi0 + i] = EpilogueDesc{d, t, i, {0, 0}};
    if (threadIdx.x == 0) scratch[t].ticket = 0;
  }
}

// ---- reductions ----------------------------------------------------------------------------------
// Over a wavefront by data-parallel-primitive moves (rows of 16 lanes, then the two row broadcasts): the moves are part
// of the vector instruction, no LDS traffic.  The total is valid in lane 63.
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
template <class F> __device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t v, F f) {   // f(x, 0) == x
  v = f(v, dpp_or_zero<0x111, 0xF>(v));   // row_shr:1
  v = f(v, dpp_or_zero<0x112, 0xF>(v));   // row_shr:2
  v = f(v, dpp_or_zero<0x114, 0xF>(v));   // row_shr:4
  v = f(v, dpp_or_zero<0x118, 0xF>(v));   // row_shr:8: lane 15 of every row holds the row's total
  v = f(v, dpp_or_zero<0x142, 0xA>(v));   // row_bcast:15 into rows 1 and 3
  v = f(v, dpp_or_zero<0x143, 0xC>(v));   // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  return wave_reduce_u32(v, [](uint32_t a, uint32_t b) { return max(a, b); });
}
__device__ __forceinline__ uint32_t wave_or_u32(uint32_t v) {
  return wave_reduce_u32(v, [](uint32_t a, uint32_t b) { return a | b; });
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
  return wave_reduce_u32(v, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t last_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {   // valid in every lane
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// NV maxima, NC counters and one OR-mask of a tensor: per lane while a workgroup works on it (CT = uint32_t; a unit
// has at most 2^20 elements), and as the tensor's totals.
template <int NV, int NC, class CT = unsigned long long>
struct BlockStats {
  static constexpr int kNV = NV, kNC = NC;
  uint32_t mx[NV > 0 ? NV : 1];
  CT ct[NC > 0 ? NC : 1];
  uint32_t orv;
};
constexpr int kTotalWords = 16;       // 4 words of maxima and mask, up to 8 counters

// Cross-workgroup reduction of a tensor's statistics.
//
// A workgroup combines what its lanes found in one unit (wavefront, then LDS) and leaves it as a record of 16 bytes
// (maxima and OR-mask), 32 (and two counters) or 64 (and eight).  The units of a tensor are consecutive, so are their
// records.  How the tensors are finished has two forms with the same results:
//
//  * deferred: a second, tiny launch combines the records and runs the tensors' scalar epilogues: one workgroup per
//    tensor, or one per 512 chunks of a large one, of which the last to arrive adds up what the others left.
//  * single pass: every workgroup bumps a per-tensor ticket when it leaves the tensor, the one that completes it reads the
//    records of the tensor.  A ticket costs 15 to 50 ns that do not overlap with those of other workgroups, most of it the
//    agent-scope release in front of it, which makes the record visible outside the workgroup's L2 and writes back what
//    else is in there (cast of a GPT-7B layer, 4096 persistent workgroups: 200 us more than the deferred form).
//
// Measured and not used: adding to per-tensor slots with fire-and-forget atomics instead of leaving records.  At device
// scope they are served outside the L2s at about 15 ns each whichever line they go to: the update pass of 1.8e9
// elements (442 000 workgroups) took 29 ms instead of 4.
template <int NC> constexpr int kRecordBytes = NC == 0 ? 16 : (NC <= 4 ? 32 : 64);

// Combines s over the workgroup; the results end up in the first lanes of the first wavefront: lane 0 holds the maxima and the
// mask, lane 1 counters 0..3, lane 2 counters 4..7 (that is, lane i holds the i-th 16 bytes of the record).
template <int NV, int NC>
__device__ __forceinline__ uint4 block_combine(const BlockStats<NV, NC, uint32_t>& s) {
  constexpr int kWords = NC == 0 ? 4 : (NC <= 4 ? 8 : 12);
  __shared__ uint4 l_v[kWaves][kWords / 4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t v[kWords];
#pragma unroll
  for (int i = 0; i < 3; ++i) v[i] = i < NV ? wave_max_u32(s.mx[i < NV ? i : 0]) : 0u;
  v[3] = wave_or_u32(s.orv);
#pragma unroll
  for (int i = 4; i < kWords; ++i) v[i] = i - 4 < NC ? wave_sum_u32(s.ct[i - 4 < NC ? i - 4 : 0]) : 0u;
  __syncthreads();   // the previous use of the LDS array is over
  if (lane == 63) {
#pragma unroll
    for (int i = 0; i < kWords / 4; ++i) l_v[wave][i] = make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
  }
  __syncthreads();
  uint4 r = make_uint4(0, 0, 0, 0);
  if (threadIdx.x < kWords / 4) {
    r = l_v[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      const uint4 o = l_v[w][threadIdx.x];
      if (threadIdx.x == 0) r = make_uint4(max(r.x, o.x), max(r.y, o.y), max(r.z, o.z), r.w | o.w);
      else r = make_uint4(r.x + o.x, r.y + o.y, r.z + o.z, r.w + o.w);
    }
  }
  return r;
}

// Adds up records [u0, u1) with the whole workgroup; the totals are valid in thread 0.
template <int NV, int NC>
__device__ __forceinline__ void gather_records(const Tables& tb, long long u0, long long u1, BlockStats<NV, NC>& s) {
  constexpr int kQuads = kRecordBytes<NC> / 16;
  BlockStats<NV, NC> a;
#pragma unroll
  for (int i = 0; i < NV; ++i) a.mx[i] = 0;
#pragma unroll
  for (int i = 0; i < NC; ++i) a.ct[i] = 0;
  a.orv = 0;
#pragma unroll 4
  for (long long u = u0 + threadIdx.x; u < u1; u += kThreads) {
    const uint4* rec = reinterpret_cast<const uint4*>(tb.records + u * kRecordBytes<NC>);
    const uint4 h = rec[0];
    const uint32_t m[3] = {h.x, h.y, h.z};
#pragma unroll
    for (int i = 0; i < NV; ++i) a.mx[i] = max(a.mx[i], m[i]);
    a.orv |= h.w;
    if constexpr (NC > 0) {
      uint32_t c[8];
#pragma unroll
      for (int q = 1; q < (kQuads < 3 ? kQuads : 3); ++q) {
        const uint4 k = rec[q];
        c[4 * q - 4] = k.x; c[4 * q - 3] = k.y; c[4 * q - 2] = k.z; c[4 * q - 1] = k.w;
      }
#pragma unroll
      for (int i = 0; i < NC; ++i) a.ct[i] += c[i];
    }
  }
  __shared__ uint32_t l_m[kWaves][4];
  __shared__ unsigned long long l_c[kWaves][NC > 0 ? NC : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < NV; ++i) a.mx[i] = wave_max_u32(a.mx[i]);
  a.orv = wave_or_u32(a.orv);
#pragma unroll
  for (int i = 0; i < NC; ++i) a.ct[i] = wave_sum_u64(a.ct[i]);
  __syncthreads();
  if (lane == 63) {
#pragma unroll
    for (int i = 0; i < NV; ++i) l_m[wave][i] = a.mx[i];
    l_m[wave][3] = a.orv;
#pragma unroll
    for (int i = 0; i < NC; ++i) l_c[wave][i] = a.ct[i];
  }
  __syncthreads();
  s = a;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) s.mx[i] = max(max(l_m[0][i], l_m[1][i]), max(l_m[2][i], l_m[3][i]));
    s.orv = l_m[0][3] | l_m[1][3] | l_m[2][3] | l_m[3][3];
#pragma unroll
    for (int i = 0; i < NC; ++i) s.ct[i] = l_c[0][i] + l_c[1][i] + l_c[2][i] + l_c[3][i];
  }
  static_assert(kWaves == 4, "four partial results");
}

// Adds `add` to a tensor's ticket; true in the workgroup that makes it `want`, which then sees everything the others wrote
// before they came here.  Called by all threads after the first wavefront wrote what the others are to see.
__device__ __forceinline__ bool ticket_last(const Tables& tb, int t, uint32_t add, uint32_t want) {
  __shared__ int l_last;
  if (threadIdx.x < 64) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");        // the stores of all lanes of this wavefront
    if (threadIdx.x == 0) {
      uint32_t* ticket = &tb.scratch[t].ticket;
      // (relaxed: the fences on both sides order it, and a release of its own would write the L2 back a second time)
      const bool last = __hip_atomic_fetch_add(ticket, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add == want;
      if (last) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
      }
      l_last = last;
    }
  }
  __syncthreads();
  const bool last = l_last != 0;
  __syncthreads();                 // l_last may be rewritten by the next call
  if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return last;
}

__device__ __forceinline__ uint32_t units_of(const Tables& tb, const TensorDesc& d) {
  return (uint32_t)((d.numel + tb.unit_elems - 1) / tb.unit_elems);
}

// Called by all threads at the end of unit u: its record.
template <int NV, int NC>
__device__ __forceinline__ void collect(const Tables& tb, long long u, const BlockStats<NV, NC, uint32_t>& s) {
  const uint4 r = block_combine(s);
  constexpr int kStored = NC == 0 ? 1 : (NC <= 4 ? 2 : 3);
  if (threadIdx.x < kStored) reinterpret_cast<uint4*>(tb.records + u * kRecordBytes<NC>)[threadIdx.x] = r;
}
// The single-pass form, called by all threads when the workgroup has collected the last of `done` units of tensor t in a
// row: one ticket for all of them.  The workgroup that completes the tensor runs its scalar epilogue.
template <class Op>
__device__ __forceinline__ void finish_by_ticket(const Tables& tb, Op& op, int t, uint32_t done) {
  const TensorDesc d = tb.desc[t];
  const uint32_t n = units_of(tb, d);
  if (!ticket_last(tb, t, done, n)) return;
  const long long u0 = (long long)d.first_chunk << tb.unit_shift;
  typename Op::Stats total;
  gather_records(tb, u0, u0 + n, total);
  if (threadIdx.x == 0) op.finalize(t, d, total);
}

// The second launch of the deferred form.  MARKED: of the second round of a speculation (walk_marked), for the tensors it did.
template <class Op, class Params, bool MARKED = false>
__global__ __launch_bounds__(kThreads) void epilogue_kernel(Tables tb, Params p) {
  if (MARKED && uniform_load(tb.marked_call) != tb.call) return;
  Op op(p, tb);
  for (int i = blockIdx.x; i < tb.n_epi; i += gridDim.x) {
    const EpilogueDesc e = tb.epi[i];
    const TensorDesc& d = e.d;
    const int t = e.tensor, K = epilogue_groups(d.n_chunks);
    if (MARKED && uniform_load(tb.redo + t) == 0) continue;
    const long long n = units_of(tb, d), u0 = (long long)d.first_chunk << tb.unit_shift;
    typename Op::Stats s;
    gather_records(tb, u0 + n * e.k / K, u0 + n * (e.k + 1) / K, s);
    if (K > 1) {
      constexpr int NV = Op::Stats::kNV, NC = Op::Stats::kNC;
      if (threadIdx.x == 0) {
        unsigned long long* w = tb.totals + (long long)i * kTotalWords;
        for (int j = 0; j < NV; ++j) w[j] = s.mx[j];
        w[3] = s.orv;
        for (int j = 0; j < NC; ++j) w[4 + j] = s.ct[j];
      }
      if (!ticket_last(tb, t, 1u, (uint32_t)K)) continue;
      if (threadIdx.x < 64) {                    // a lane per workgroup
        static_assert(kMaxEpilogue <= 64, "one wavefront");
        const bool have = threadIdx.x < K;
        const unsigned long long* w = tb.totals + (long long)(d.epi0 + (have ? threadIdx.x : 0)) * kTotalWords;
#pragma unroll
        for (int j = 0; j < NV; ++j) s.mx[j] = last_lane(wave_max_u32(have ? (uint32_t)w[j] : 0u));
        s.orv = last_lane(wave_or_u32(have ? (uint32_t)w[3] : 0u));
#pragma unroll
        for (int j = 0; j < NC; ++j) s.ct[j] = wave_sum_u64(have ? w[4 + j] : 0ull);
      }
    }
    if (threadIdx.x == 0) op.finalize(t, d, s);
  }
}

// ---- the walk shared by all kernels -------------------------------------------------------
// Op must provide: begin(t); fast() (uniform: may the vector path be used for this tensor); Regs<UN>, the registers
// of UN complete 4096-element tiles, with load(r, pos) (issues the loads of the tiles starting at element `pos` of the
// flat buffers; does not depend on the tensor) and tiles(r, pos) (the rest, the whole workgroup together; the op chooses
// which 16 elements of a tile a thread takes); full_group(pos): the 16 consecutive elements starting at `pos`, handled by
// the calling thread alone with vector accesses (any subset of the threads may call it); group(pos, valid) with
// 1 <= valid <= 16 for everything else, element by element; flush(unit) (called by all threads at the end of a
// unit: it fills a BlockStats and hands it to `collect`); and for the tensor's scalar epilogue
// finalize(t, desc, stats), run by one thread once the totals of all workgroups are known.
//
// Order of the walk.  By default a workgroup takes one unit (UN tiles) and ends: the dispatcher starts workgroups in order, so
// at any time the chip works on a few hundred neighbouring tiles of every buffer, a window that sweeps through memory and
// finds the DRAM rows it needs open.  A persistent grid in which every workgroup walked a range of its own (or a
// round-robin share: the workgroups drift apart) touched a few thousand places at once and lost more the more it wrote:
// XOR-only traffic of 1.8e9 elements in one HBM region, TB/s, persistent / one tile per workgroup: update shape 5.13 / 5.5
// (5.9 with two or three workgroups per compute unit), cast shape 5.37 / 6.45, one-to-one copy 5.23 / 6.54, reads alone
// 6.95 / 6.95.  Two tiles per workgroup cost 5 % of the cast shape, four consecutive ones 2 to 8 % of the update shape.
// Unit u.  Returns its tensor and adds 1 to `done`, unless the unit is empty.
template <int UN, class Op>
__device__ __forceinline__ int walk_unit(const Tables& tb, Op& op, long long u, uint32_t& done) {
  const ChunkDesc c = uniform_load(tb.chunks + (u >> tb.unit_shift));
  const int e0 = ((int)u & ((1 << tb.unit_shift) - 1)) * tb.unit_elems;
  const int len = min(c.len - e0, tb.unit_elems);
  const int t = c.tensor;
  if (len <= 0) return t;                      // the last chunk of a tensor can have fewer units
  const long long base = c.base + e0;
  const int ntiles = len / kTile;
  // the loads of the first tiles go out before anything about the tensor but its address is known
  typename Op::template Regs<UN> r;
  if (ntiles >= UN) op.load(r, base);
  op.begin(t);
  int tile = 0;
  if (op.fast()) {
    while (tile + UN <= ntiles) {
      op.tiles(r, base + (long long)tile * kTile);
      tile += UN;
      if (tile + UN <= ntiles) op.load(r, base + (long long)tile * kTile);
    }
    if constexpr (UN > 1) {
      for (; tile < ntiles; ++tile) {
        typename Op::template Regs<1> q;
        op.load(q, base + (long long)tile * kTile);
        op.tiles(q, base + (long long)tile * kTile);
      }
    }
  }
  // what is left (less than a tile; a whole small tensor): complete 16-element groups still take 128-bit accesses
  const int whole = len & ~(kGroup - 1);
  for (int i = tile * kTile + threadIdx.x * kGroup; i < whole; i += kTile) {
    if (op.fast()) op.full_group(base + i);
    else op.group(base + i, kGroup);
  }
  // the last, incomplete group of a tensor goes element by element, a thread each: one thread alone with up to 15 in-place
  // elements waits for every load in turn (the update of 600 ragged tensors: 38 us, 14 us this way)
  const int last = whole + kThreads - 1 - (int)threadIdx.x;
  if (last < len) op.group(base + last, 1);
  op.flush(u);
  ++done;
  return t;
}

template <int UN, class Op>
__device__ __forceinline__ void walk_units(const Tables& tb, Op& op) {
  long long u = blockIdx.x, end = u + 1;
  if (!tb.one_unit) {
    const long long U = (long long)tb.n_chunks << tb.unit_shift, b = blockIdx.x, G = gridDim.x;
    u = b * U / G;
    end = (b + 1) * U / G;
  }
  uint32_t done = 0;
  for (; u < end; ++u) {
    const int t = walk_unit<UN>(tb, op, u, done);
    if (tb.deferred || done == 0) continue;
    if (u + 1 < end && uniform_load(tb.chunks + ((u + 1) >> tb.unit_shift)).tensor == t) continue;
    finish_by_ticket(tb, op, t, done);
    done = 0;
  }
}

// ---- the second round of a speculation ------------------------------------------------------------------
// The scalar epilogue of a speculative pass marks the tensors whose speculation failed (mark_redo); this walk does their
// units once more.  Mostly nothing is marked: then a workgroup reads
// one word and ends.  Otherwise every workgroup adds up the marked units of all tensors and takes a contiguous share
// of them, so that one marked tensor keeps the whole chip busy as well as many do.  (Two small kernels that built a list
// before it cost 10 us per call whether or not there was anything to do.)  The marks lie side by side, a thread adds up those
// of a segment of neighbouring tensors, and only the segments of the workgroup's share are looked at one by one; the running
// totals are kept by the first workgroup.  (One word per 128 bytes, 256 tensors at a time, and two device-scope atomics per
// marked tensor for the totals: 459 us for 20 000 tensors of which a third is marked, 198 us this way.)  The tensors
// are finished by tickets or by a launch of their own, as after any other pass.
__device__ __forceinline__ void mark_redo(const Tables& tb, int t, const TensorDesc& d, bool redo) {
  tb.redo[t] = redo ? units_of(tb, d) : 0u;
  if (redo) __hip_atomic_store(tb.marked_call, tb.call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);    // the next kernel reads it
}
struct alignas(16) Quad4 { uint32_t n[4]; };
template <int UN, class Op>
__device__ __forceinline__ void walk_marked(const Tables& tb, Op& op) {
  if (blockIdx.x == 0 && threadIdx.x == 0) tb.spec_totals[0] += 1;
  if (uniform_load(tb.marked_call) != tb.call) return;
  __shared__ uint32_t l_sum[kWaves], l_count[kWaves];
  __shared__ struct { uint32_t at; int32_t t; } l_share[kThreads];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // a thread per segment of `per` tensors: its marked units
  const int per = 4 * ((tb.n_tensors + 4 * kThreads - 1) / (4 * kThreads)), t0 = per * (int)threadIdx.x;
  const int n4 = (tb.n_tensors + 3) & ~3;
  uint32_t n = 0;                                // (all units of a launch fit 32 bits)
  for (int t = t0; t < min(t0 + per, n4); t += 4) {
    const Quad4 q = *reinterpret_cast<const Quad4*>(tb.redo + t);
    n += (q.n[0] + q.n[1]) + (q.n[2] + q.n[3]);
  }
  if (blockIdx.x == 0) {
    unsigned long long tensors = 0, elems = 0;
    for (int t = t0; t < min(t0 + per, tb.n_tensors); ++t) {
      if (tb.redo[t] == 0) continue;
      tensors += 1;
      elems += (unsigned long long)tb.desc[t].numel;
    }
    tensors = wave_sum_u64(tensors);
    elems = wave_sum_u64(elems);
    if (lane == 0) {
      (void)__hip_atomic_fetch_add(&tb.spec_totals[1], tensors, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      (void)__hip_atomic_fetch_add(&tb.spec_totals[2], elems, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  // where the segments' units lie among all
  uint32_t upto = n;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t x = (uint32_t)__shfl_up((int)upto, o, 64);
    if (lane >= o) upto += x;
  }
  if (lane == 63) l_sum[wave] = upto;
  __syncthreads();
  uint32_t at = upto - n;
  long long total = 0;
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) at += l_sum[w];
    total += l_sum[w];
  }
  // the segments that this workgroup's share reaches into, in order
  const long long lo = total * blockIdx.x / gridDim.x, hi = total * (blockIdx.x + 1) / gridDim.x;
  const bool share = n && lo < hi && (long long)at < hi && (long long)at + n > lo;
  const unsigned long long ballot = __ballot(share);
  if (lane == 0) l_count[wave] = (uint32_t)__popcll(ballot);
  __syncthreads();
  int count = 0, place = __popcll(ballot & ((1ull << lane) - 1));
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) place += (int)l_count[w];
    count += (int)l_count[w];
  }
  if (share) {
    l_share[place].at = at;
    l_share[place].t = t0;
  }
  __syncthreads();
  for (int i = 0; i < count; ++i) {
    const int s0 = __builtin_amdgcn_readfirstlane(l_share[i].t);
    long long first = (uint32_t)__builtin_amdgcn_readfirstlane((int)l_share[i].at);
    for (int s = s0; s < min(s0 + per, n4) && first < hi; s += 4) {
      const Quad4 q = uniform_load(reinterpret_cast<const Quad4*>(tb.redo + s));
      const long long quad = (long long)q.n[0] + q.n[1] + q.n[2] + q.n[3];
      if (first + quad <= lo) {
        first += quad;
        continue;
      }
#pragma unroll 1
      for (int t = s; t < s + 4; ++t) {
        const long long units = uniform_load(tb.redo + t);
        const long long k0 = max(lo - first, 0ll), k1 = min(hi - first, units);
        first += units;
        if (k0 >= k1) continue;
        const long long u0 = (long long)uniform_load(&tb.desc[t].first_chunk) << tb.unit_shift;
        uint32_t done = 0;
        for (long long k = k0; k < k1; ++k) walk_unit<UN>(tb, op, u0 + k, done);
        if constexpr (Op::kFinishes) {
          if (!tb.deferred) finish_by_ticket(tb, op, t, done);
        }
      }
    }
  }
}

// Build-time tuning knobs (defaults are the measured best on MI355X).
#ifndef FP8LM_NT_MASK
#define FP8LM_NT_MASK 15  // bit0 non-temporal loads of read-only streams, bit1 non-temporal stores of write-only
                          // streams, bit2 / bit3 the same for the in-place (read-modify-write) streams.  All four
                          // measured best with the split access layout (bits 2+3 together: -1 % on the update
                          // kernel; bit 3 alone: +0.7 %)
#endif
// Tiles a workgroup takes at once (all their loads are issued before the first is used).  One tile keeps the window of
// walk_units smallest, but then a workgroup's fixed costs (the chain table -> data, two barriers, the record) come once per 4096
// elements: cast of GPT-125M with bf16 gradients, 1 / 2 / 4 tiles: 69 / 62 / 71 us (4: 207 registers, two wavefronts
// per SIMD; kUnCast); re-quantisation 55 / 48 / 47 us; cast of fp32 gradients (201e6 elements) 228 / 240 us for 1 / 2.  The update pass
// does 40 to 70 instructions per element in the meantime and has no registers for a second tile.
constexpr int kUnRead = 4;
constexpr int kUnRequant = 4;
constexpr int kUnUpdate = 1;
__host__ __device__ constexpr int sum_tiles(int ranks) { return ranks == 0 ? 1 : ranks <= 2 ? 4 : ranks <= 4 ? 2 : 1; }
constexpr bool kNtLoadRO = (FP8LM_NT_MASK & 1) != 0, kNtStoreWO = (FP8LM_NT_MASK & 2) != 0;
constexpr bool kNtLoadRW = (FP8LM_NT_MASK & 4) != 0, kNtStoreRW = (FP8LM_NT_MASK & 8) != 0;

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
template <bool NT = false> __device__ __forceinline__ uint4 ld16(const void* p) {
  if constexpr (NT) {
    const u32x4_t r = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(r.x, r.y, r.z, r.w);
  } else {
    return *reinterpret_cast<const uint4*>(p);
  }
}
template <bool NT = false> __device__ __forceinline__ void st16(void* p, uint4 v) {
  if constexpr (NT) {
    const u32x4_t r = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(r, reinterpret_cast<u32x4_t*>(p));
  } else {
    *reinterpret_cast<uint4*>(p) = v;
  }
}

template <bool NT = false> __device__ __forceinline__ uint32_t ld4(const void* p) {
  if constexpr (NT) return __builtin_nontemporal_load(static_cast<const uint32_t*>(p));
  else return *static_cast<const uint32_t*>(p);
}
template <bool NT = false> __device__ __forceinline__ void st4(void* p, uint32_t v) {
  if constexpr (NT) __builtin_nontemporal_store(v, static_cast<uint32_t*>(p));
  else *static_cast<uint32_t*>(p) = v;
}

typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
template <bool NT = false> __device__ __forceinline__ uint2 ld8(const void* p) {
  if constexpr (NT) {
    const u32x2_t r = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(p));
    return make_uint2(r.x, r.y);
  } else {
    return *reinterpret_cast<const uint2*>(p);
  }
}
template <bool NT = false> __device__ __forceinline__ void st8(void* p, uint2 v) {
  if constexpr (NT) {
    const u32x2_t r = {v.x, v.y};
    __builtin_nontemporal_store(r, reinterpret_cast<u32x2_t*>(p));
  } else {
    *reinterpret_cast<uint2*>(p) = v;
  }
}

}  // namespace fp8lm

#endif
