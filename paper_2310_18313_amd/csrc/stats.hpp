// Quantisation-error statistics of an FP8 gradient (Sec. 3.3, communication ablation) and the small
// utility kernels (metadata initialisation, streaming copy).
#ifndef FP8LM_STATS_HPP
#define FP8LM_STATS_HPP

#include <type_traits>

#include "walk.hpp"

namespace fp8lm {

// ================================================================================================
// Quantisation error of an FP8 gradient against a high-precision reference (Sec. 3.3, the figure
// of the communication ablation: SNR, underflow rate, overflow rate)
// ================================================================================================
struct StatsParams {
  const void* ref;
  const uint8_t* q;
  const fp8lm_meta* meta;
  fp8lm_quant_stats* out;
  Partial* partials;       // [grid + n_tensors]
};

template <int FMT, int SRC>
struct QuantStatsOp {
  using elem_t = typename SrcTraits<SRC>::elem_t;
  static constexpr int kPer = 16 / (int)sizeof(elem_t);
  static constexpr int kLoads = kGroup / kPer;
  static constexpr int kW = kSrcWords<SRC>;
  const StatsParams& p;
  const Tables& tb;
  double rs, signal, noise;
  uint32_t n_nonzero, n_under, n_over, n_nonfinite;
  __device__ QuantStatsOp(const StatsParams& p_, const Tables& tb_) : p(p_), tb(tb_) {}
  __device__ __forceinline__ void begin(int t) {
    rs = 1.0 / (double)p.meta[t].scale;
    signal = noise = 0.0;
    n_nonzero = n_under = n_over = n_nonfinite = 0;
  }
  __device__ __forceinline__ void add_error(float r, float pv) {
    const double rd = (double)r;
    const double e = __builtin_fma(-(double)pv, rs, rd);
    signal = __builtin_fma(rd, rd, signal);
    noise = __builtin_fma(e, e, noise);
  }
  __device__ __forceinline__ void one(uint32_t rbits, uint32_t code) {
    const float r = SrcTraits<SRC>::dec(rbits);
    const float pv = fp8_to_f32<FMT>(code);
    if (!(fabsf(r) <= 3.4028234664e38f) || !(fabsf(pv) <= 3.4028234664e38f)) {
      ++n_nonfinite;
      return;
    }
    add_error(r, pv);
    const uint32_t mag = code & 0x7Fu;
    n_nonzero += (r != 0.0f);
    n_under += (r != 0.0f) && mag == 0u;
    n_over += mag == Fp8Traits<FMT>::kTop;
  }
  // 16 elements, kRuns runs of consecutive ones: a whole tile's groups take 16 bytes of the reference at a time, contiguous over the
  // workgroup.  What bounds this is the vector unit: two conversions and three float64 fused multiply-adds per element
  // are what it cannot do without, so everything else is asked of the group as a whole first, by integer maxima and
  // minima of the reference's bits and tests of four codes at a time: mostly nothing is zero, on the top code or not finite.
  // Only a group with something that is not finite goes element by element.  1.3e8 elements, fp32 reference, E4M3: 136 us,
  // 140 where every wavefront meets zeros (element by element: 25 instructions, 215 us; 340 where a group with a zero was left to
  // a loop that picks its elements out of registers).
  static constexpr int kRuns = kLoads, kRun = kGroup / kRuns;
  struct Regs { uint4 r[kLoads]; uint32_t q[4]; };
  template <bool kSplit> __device__ __forceinline__ void load(Regs& g, long long pos0) const {
    constexpr int kStep = kSplit ? kTile / kRuns : kRun;
    const long long pos = pos0 + threadIdx.x * (kSplit ? kRun : kGroup);
    const elem_t* rp = static_cast<const elem_t*>(p.ref) + pos;
#pragma unroll
    for (int k = 0; k < kLoads; ++k) g.r[k] = ld16<kNtLoadRO>(rp + k * kStep);
#pragma unroll
    for (int k = 0; k < kRuns; ++k) {
      if constexpr (kRun == 8) {
        const uint2 c = ld8<kNtLoadRO>(p.q + pos + k * kStep);
        g.q[2 * k] = c.x;
        g.q[2 * k + 1] = c.y;
      } else {
        g.q[k] = ld4<kNtLoadRO>(p.q + pos + k * kStep);
      }
    }
  }
  // bit 7 of byte i: element 4 k + i of the reference is not zero
  static __device__ __forceinline__ uint32_t nonzero_refs(const uint32_t (&w)[kW], int k) {
    if constexpr (kSrc16<SRC>) {
      const uint32_t lo = (w[2 * k] & 0x7FFF7FFFu) + 0x7FFF7FFFu, hi = (w[2 * k + 1] & 0x7FFF7FFFu) + 0x7FFF7FFFu;
      return __builtin_amdgcn_perm(hi, lo, 0x07050301u) & 0x80808080u;
    } else {
      auto m = [&](int i) { return (w[4 * k + i] & 0x7FFFFFFFu) + 0x7FFFFFFFu; };
      return (__builtin_amdgcn_perm(m(1), m(0), 0x0C0C0703u) | __builtin_amdgcn_perm(m(3), m(2), 0x07030C0Cu)) & 0x80808080u;
    }
  }
  __device__ __forceinline__ void accumulate(const Regs& g) {
    uint32_t w[kW];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      w[4 * k] = g.r[k].x; w[4 * k + 1] = g.r[k].y; w[4 * k + 2] = g.r[k].z; w[4 * k + 3] = g.r[k].w;
    }
    uint32_t gmax = 0, gmin = 0xFFFFFFFFu, all_nz = 0x80808080u, top = 0;
#pragma unroll
    for (int j = 0; j < kW; ++j) {
      src_fold<SRC>(gmax, w[j]);
      src_fold_min<SRC>(gmin, w[j]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t mag = g.q[k] & 0x7F7F7F7Fu;
      all_nz &= mag + 0x7F7F7F7Fu;                                         // bit 7 of a byte: its magnitude is not zero
      top |= mag + (0x80808080u - Fp8Traits<FMT>::kTopX4);                 // ... it is the top code or beyond it
    }
    if (src_final<SRC>(gmax) >= SrcTraits<SRC>::kNonfinite || src_final_min<SRC>(gmin) == 0 || all_nz != 0x80808080u || (top & 0x80808080u)) {
      uint32_t beyond = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) beyond |= (g.q[k] & 0x7F7F7F7Fu) + (0x7F7F7F7Fu - Fp8Traits<FMT>::kTopX4);
      if (src_final<SRC>(gmax) >= SrcTraits<SRC>::kNonfinite || (beyond & 0x80808080u)) {
#pragma unroll 1
        for (int j = 0; j < 16; ++j) {
          uint32_t bits = 0, code = 0;                                     // (no dynamic index into registers)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            if (i != j) continue;
            bits = kSrc16<SRC> ? (w[(i >> 1) % kW] >> ((i & 1) * 16)) & 0xFFFFu : w[i % kW];
            code = (g.q[i >> 2] >> ((i & 3) * 8)) & 0xFFu;
          }
          one(bits, code);
        }
        return;
      }
      // zeros or top codes among them (a gradient with unused rows, one that underflows): counted four at a time
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t mag = g.q[k] & 0x7F7F7F7Fu, nz_code = mag + 0x7F7F7F7Fu, nz = nonzero_refs(w, k);
        n_nonzero += __popc(nz);
        n_under += __popc(nz & ~nz_code);
        n_over += 4 - nonzero_bytes7(mag ^ Fp8Traits<FMT>::kTopX4);
      }
    } else {
      n_nonzero += kGroup;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float2_t lo = fp8x2_to_f32<FMT, false>(g.q[k]), hi = fp8x2_to_f32<FMT, true>(g.q[k]);
      const float pv[4] = {lo.x, lo.y, hi.x, hi.y};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = 4 * k + i;
        add_error(SrcTraits<SRC>::dec(kSrc16<SRC> ? (w[(j >> 1) % kW] >> ((j & 1) * 16)) & 0xFFFFu : w[j % kW]), pv[i]);
      }
    }
  }
  template <bool kSplit> __device__ __forceinline__ void group16(long long pos0) {
    Regs g;
    load<kSplit>(g, pos0);
    accumulate(g);
  }
  __device__ __forceinline__ void group(long long pos, int valid) {
    const elem_t* rp = static_cast<const elem_t*>(p.ref) + pos;
    for (int j = 0; j < valid; ++j) one(rp[j], p.q[pos + j]);
  }
  // The workgroup's totals as one record (every step in a fixed order).
  __device__ __forceinline__ void flush(Partial* rec) { combine(Partial{{signal, noise}, {n_nonzero, n_under, n_over, n_nonfinite}}, rec); }
  static __device__ __forceinline__ void combine(Partial s, Partial* rec) {
    __shared__ Partial l_p[kWaves];
#pragma unroll
    for (int i = 0; i < 2; ++i) s.fs[i] = wave_sum_f64(s.fs[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) s.ct[i] = wave_sum_u64(s.ct[i]);
    __syncthreads();             // the previous use of the LDS array is over
    if ((threadIdx.x & 63) == 0) l_p[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < kWaves; ++w) add(s, l_p[w]);
      *rec = s;
    }
  }
  static __device__ __forceinline__ void add(Partial& s, const Partial& o) {
    s.fs[0] += o.fs[0];
    s.fs[1] += o.fs[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) s.ct[i] += o.ct[i];
  }
};

// float64 sums are only reproducible if they are added in a fixed order, so these statistics do not go through slots: a
// persistent grid, workgroup b walking the chunks [b*C/G, (b+1)*C/G), one record per (workgroup, tensor) pair.  The
// workgroups that touch tensor t are consecutive and a workgroup touches consecutive tensors, so record b + t is unique
// and the records of a tensor are contiguous.  (The kernel only reads: the order of the walk costs nothing here.)
// Seven wavefronts per SIMD: with an fp32 reference the allocator would take 75 registers, three too many for that, for the
// paths that are seldom taken (72 do without spilling).
template <int FMT, int SRC>
__global__ __launch_bounds__(kThreads, 7) void quant_stats_kernel(Tables tb, StatsParams p) {
  QuantStatsOp<FMT, SRC> op(p, tb);
  const long long C = tb.n_chunks, b = blockIdx.x, G = gridDim.x;
  int cur = -1;
  for (long long c = b * C / G; c < (b + 1) * C / G; ++c) {
    const ChunkDesc k = uniform_load(tb.chunks + c);
    if (k.tensor != cur) {
      if (cur >= 0) op.flush(p.partials + (b + cur));
      cur = k.tensor;
      op.begin(cur);
    }
    int tile = 0;
    for (; tile + kTile <= k.len; tile += kTile) op.template group16<true>(k.base + tile);
    const int whole = k.len & ~(kGroup - 1), i = tile + threadIdx.x * kGroup;
    if (i < whole) op.template group16<false>(k.base + tile);
    const int last = whole + kThreads - 1 - (int)threadIdx.x;              // the incomplete group, a thread per element
    if (last < k.len) op.group(k.base + last, 1);
  }
  if (cur >= 0) op.flush(p.partials + (b + cur));
}

// One workgroup per tensor adds up its records: lane by lane, then over the workgroup, in a fixed order.
template <int FMT, int SRC>
__global__ __launch_bounds__(kThreads) void quant_stats_epilogue_kernel(Tables tb, StatsParams p, int main_grid, int n_tensors) {
  typedef QuantStatsOp<FMT, SRC> Op;
  __shared__ Partial l_total;
  for (int t = blockIdx.x; t < n_tensors; t += gridDim.x) {
    const TensorDesc d = tb.desc[t];
    if (d.n_chunks == 0) {                       // an empty tensor
      if (threadIdx.x == 0) p.out[t] = fp8lm_quant_stats{0.0, 0.0, 0, 0, 0, 0};
      continue;
    }
    // owner(c) = the b with b*C/G <= c < (b+1)*C/G
    const long long C = tb.n_chunks, c0 = d.first_chunk, c1 = c0 + d.n_chunks - 1;
    const long long b_lo = ((c0 + 1) * main_grid - 1) / C, b_hi = ((c1 + 1) * main_grid - 1) / C;
    Partial s{};
    for (long long b = b_lo + threadIdx.x; b <= b_hi; b += kThreads) Op::add(s, p.partials[b + t]);
    Op::combine(s, &l_total);
    if (threadIdx.x == 0)
      p.out[t] = fp8lm_quant_stats{l_total.fs[0], l_total.fs[1], l_total.ct[0], l_total.ct[1], l_total.ct[2], l_total.ct[3]};
  }
}

__global__ void quant_stats_zero_kernel(fp8lm_quant_stats* out, int n) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) out[t] = fp8lm_quant_stats{0.0, 0.0, 0, 0, 0, 0};
}

__global__ void meta_init_kernel(fp8lm_meta* meta, int n, int clean0) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  fp8lm_meta M;
  M.scale = 1.0f; M.inv_scale = 1.0f; M.amax = 0.0f; M.amax_deq = 0.0f;
  for (int h = 0; h < FP8LM_HIST; ++h) M.amax_hist[h] = 0.0f;
  M.hist_pos = 0; M.mu_exp = 0; M.clean_steps = clean0; M.flags = 0; M.n_sat = 0; M.n_underflow = 0;
  meta[t] = M;
}

// Plain streaming copy: every workgroup owns one contiguous range, four 128-bit loads in flight per
// thread, non-temporal on both sides.
__global__ __launch_bounds__(kThreads) void copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, long long n16) {
  const long long b0 = n16 * blockIdx.x / gridDim.x, b1 = n16 * (blockIdx.x + 1) / gridDim.x;
  long long i = b0 + threadIdx.x;
  for (; i + 3 * kThreads < b1; i += 4 * kThreads) {
    const uint4 a = ld16<true>(src + i), b = ld16<true>(src + i + kThreads), c = ld16<true>(src + i + 2 * kThreads),
                d = ld16<true>(src + i + 3 * kThreads);
    st16<true>(dst + i, a);
    st16<true>(dst + i + kThreads, b);
    st16<true>(dst + i + 2 * kThreads, c);
    st16<true>(dst + i + 3 * kThreads, d);
  }
  for (; i < b1; i += kThreads) st16<true>(dst + i, ld16<true>(src + i));
}

// Memory-only skeletons of the hot kernels: the same grid, walk, access widths, access layout and
// cache policies as the kernels they stand for, with the arithmetic replaced by XORs.  What they reach is the
// bandwidth ceiling of that access pattern on this machine; the real kernels are measured against it.
//   NS1 / NS2 : number of 8-bit / 16-bit streams read;  ND1 / ND2 : number of 8-bit / 16-bit streams written.
// A thread takes elements [8L, 8L+8) of both halves of a 4096-element tile (L = thread index), like the update and
// cast kernels: 64-bit accesses on 8-bit streams, 128-bit accesses on 16-bit streams, contiguous over the workgroup.
struct SkeletonParams {
  const uint8_t* s1[2];
  const uint16_t* s2[2];
  uint8_t* d1[2];
  uint16_t* d2[2];
  long long n_tiles;
  int32_t ranges;        // 0: a workgroup takes UN tiles and ends, as the kernels do; 1: a persistent grid, every workgroup walking a
                         // range of its own, as they do under a limit on workgroups; shows where a buffer lies in HBM more clearly
  uint32_t* sink;        // a word that pure reads could write, so that they cannot be optimised away
};
template <int NS1, int NS2, int ND1, int ND2, int UN>
__global__ __launch_bounds__(kThreads) void skeleton_kernel(SkeletonParams p) {
  const long long t0 = p.ranges ? p.n_tiles * blockIdx.x / gridDim.x : (long long)blockIdx.x * UN;
  const long long t1 = p.ranges ? p.n_tiles * (blockIdx.x + 1) / gridDim.x : p.n_tiles;
  const long long stride = p.ranges ? UN : (long long)gridDim.x * UN;      // one round unless the grid is at its limit
  uint32_t acc = 0;
  auto body = [&](long long tile, auto un_tag) {
    constexpr int U = decltype(un_tag)::value;
    uint2 a1[U][NS1 > 0 ? NS1 : 1][2];
    uint4 a2[U][NS2 > 0 ? NS2 : 1][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long a = (tile + u) * kTile + threadIdx.x * 8, b = a + kTile / 2;
#pragma unroll
      for (int i = 0; i < NS1; ++i) { a1[u][i][0] = ld8<true>(p.s1[i] + a); a1[u][i][1] = ld8<true>(p.s1[i] + b); }
#pragma unroll
      for (int i = 0; i < NS2; ++i) { a2[u][i][0] = ld16<true>(p.s2[i] + a); a2[u][i][1] = ld16<true>(p.s2[i] + b); }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long a = (tile + u) * kTile + threadIdx.x * 8, b = a + kTile / 2;
      uint32_t x = acc, y = ~acc;
#pragma unroll
      for (int i = 0; i < NS1; ++i) { x ^= a1[u][i][0].x ^ a1[u][i][1].y; y ^= a1[u][i][0].y ^ a1[u][i][1].x; }
#pragma unroll
      for (int i = 0; i < NS2; ++i) {
        x ^= a2[u][i][0].x ^ a2[u][i][0].z ^ a2[u][i][1].y ^ a2[u][i][1].w;
        y ^= a2[u][i][0].y ^ a2[u][i][0].w ^ a2[u][i][1].x ^ a2[u][i][1].z;
      }
      acc = x + y;
#pragma unroll
      for (int i = 0; i < ND1; ++i) { st8<true>(p.d1[i] + a, make_uint2(x, y)); st8<true>(p.d1[i] + b, make_uint2(y, x)); }
#pragma unroll
      for (int i = 0; i < ND2; ++i) { st16<true>(p.d2[i] + a, make_uint4(x, y, y, x)); st16<true>(p.d2[i] + b, make_uint4(y, x, x, y)); }
    }
  };
  long long tile = t0;
  for (; tile + UN <= t1; tile += stride) body(tile, std::integral_constant<int, UN>{});
  for (int u = 0; u < UN && tile < t1; ++u, ++tile) body(tile, std::integral_constant<int, 1>{});
  if constexpr (ND1 + ND2 == 0) {
    if (acc == 0x9E3779B9u) *p.sink = acc;
  }
}

}  // namespace fp8lm

#endif
