// Gradient quantisation (Sec. 2.1, Appendix A): amax + scale update, scaled saturating FP8 cast with the
// auto-scaling state, delayed scaling, and the shared-scale re-quantisation and FP8 sum of Eq. 4-6.
#ifndef FP8LM_QUANTIZE_HPP
#define FP8LM_QUANTIZE_HPP

#include "walk.hpp"

namespace fp8lm {

// ================================================================================================
// Kernel 1: per-tensor amax of a bf16 buffer, then the scale update (Appendix A.2; Sec. 2.1 Eq. 3)
// ================================================================================================
// |x| of a bf16 is monotone in (bits & 0x7FFF), so the maximum is taken on packed 16-bit integers:
// exact, order independent, and inf/NaN show up as a result >= 0x7F80.
enum : int { kAmaxForGradient = 0, kAmaxForMaster = 1 };

// The high-precision source of a cast: bf16, IEEE half or fp32 (Sec. 2.1 casts "high-precision"
// gradients).  |x| is monotone in the magnitude bits of all three, so the amax is an integer maximum;
// for the 16-bit types two maxima are kept packed in one register.
enum : int { kSrcBF16 = 0, kSrcF16 = 1, kSrcF32 = 2 };
template <int SRC> struct SrcTraits;
template <> struct SrcTraits<kSrcBF16> {
  using elem_t = uint16_t;
  static constexpr uint32_t kNonfinite = 0x7F80u;
  static __device__ __forceinline__ float dec(uint32_t bits) { return u2f(bits << 16); }
};
template <> struct SrcTraits<kSrcF16> {
  using elem_t = uint16_t;
  static constexpr uint32_t kNonfinite = 0x7C00u;
  static __device__ __forceinline__ float dec(uint32_t bits) { return f16_to_f32(bits); }
};
template <> struct SrcTraits<kSrcF32> {
  using elem_t = uint32_t;
  static constexpr uint32_t kNonfinite = 0x7F800000u;
  static __device__ __forceinline__ float dec(uint32_t bits) { return u2f(bits); }
};
// Tiles a workgroup of the amax pass takes at once: 32 KiB of either width (four tiles of fp32 take 146 registers: 131 us for
// 201e6 elements, 125 this way).
template <int SRC> constexpr int kUnAmax = SRC == kSrcF32 ? kUnRead / 2 : kUnRead;
template <int SRC> constexpr int kUnCast = SRC == kSrcF32 ? 1 : 2;      // tiles a workgroup of the cast takes at once (walk.hpp)
template <int SRC> constexpr bool kSrc16 = sizeof(typename SrcTraits<SRC>::elem_t) == 2;
template <int SRC> constexpr int kSrcWords = kSrc16<SRC> ? 8 : 16;     // 32-bit words of a 16-element group
// folds one 32-bit word of the source (two 16-bit elements or one fp32) into a running maximum
template <int SRC> __device__ __forceinline__ void src_fold(uint32_t& acc, uint32_t word) {
  if constexpr (kSrc16<SRC>)
    acc = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, acc),
                                                                 __builtin_bit_cast(ushort2_t, word & 0x7FFF7FFFu)));
  else
    acc = max(acc, word & 0x7FFFFFFFu);
}
// ... and into a running minimum
template <int SRC> __device__ __forceinline__ void src_fold_min(uint32_t& acc, uint32_t word) {
  if constexpr (kSrc16<SRC>)
    acc = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(ushort2_t, acc),
                                                                 __builtin_bit_cast(ushort2_t, word & 0x7FFF7FFFu)));
  else
    acc = min(acc, word & 0x7FFFFFFFu);
}
template <int SRC> __device__ __forceinline__ uint32_t src_final_min(uint32_t acc) {
  if constexpr (kSrc16<SRC>) return min(acc & 0xFFFFu, acc >> 16);
  else return acc;
}
// the same (maximum) for a single element given by its bit pattern
template <int SRC> __device__ __forceinline__ void src_fold1(uint32_t& acc, uint32_t bits) {
  if constexpr (kSrc16<SRC>) acc = (acc & 0xFFFF0000u) | max(acc & 0xFFFFu, bits & 0x7FFFu);
  else acc = max(acc, bits & 0x7FFFFFFFu);
}
template <int SRC> __device__ __forceinline__ uint32_t src_final(uint32_t acc) {
  if constexpr (kSrc16<SRC>) return max(acc & 0xFFFFu, acc >> 16);
  else return acc;
}

struct AmaxParams {
  const void* src;
  fp8lm_meta* meta;
  uint32_t fmax_bits;     // gradient mode: largest finite value of the target format
  int32_t hist_window;
  int32_t margin;
};

// Exponent of a gradient tensor's scale from the amax history as it stands (the rule of scale_from_history), or kKeepScale
// if the history is all zero, without writing anything.  UNIFORM: for a whole workgroup that is about to cast with it; integer
// arithmetic on values all lanes share, so it runs on the scalar unit (bit patterns of values that are not negative are ordered
// like they are; of a negative one the pattern is negative too).  The scalar epilogue, which goes on to write the history, reads it with ordinary loads.
constexpr int kKeepScale = 1000;
template <bool UNIFORM> __device__ __forceinline__ int predicted_exponent(const fp8lm_meta* M, uint32_t fmax_bits, int hist_window, int margin) {
  auto load = [](const auto* q) { if constexpr (UNIFORM) return uniform_load(q); else return *q; };
  const int H = hist_window < 1 ? 1 : (hist_window > FP8LM_HIST ? FP8LM_HIST : hist_window);
  int bits = 0;
  for (int h = 0; h < H; ++h) {
    const int b = (int)f2u(load(&M->amax_hist[h]));
    bits = b <= 0x7F800000 ? max(bits, b) : bits;          // a NaN (of a caller's making) is smaller than nothing there
  }
  if (bits == 0) return kKeepScale;
  const int k = pow2_exp(fmax_bits, u2f((uint32_t)bits)) + load(&M->mu_exp) - margin;
  return k < -126 ? -126 : (k > 126 ? 126 : k);
}
// Sets the scale from the amax history as it stands: the largest of the last H entries, times 2^(mu_exp - margin).
// Returns the flags (amax zero / clamped) and leaves the scale alone when the history is all zero.
__device__ __forceinline__ uint32_t scale_from_history(fp8lm_meta& M, uint32_t fmax_bits, int hist_window, int margin) {
  const int H = hist_window < 1 ? 1 : (hist_window > FP8LM_HIST ? FP8LM_HIST : hist_window);
  float Aeff = 0.0f;
  for (int h = 0; h < H; ++h) Aeff = M.amax_hist[h] > Aeff ? M.amax_hist[h] : Aeff;
  if (Aeff == 0.0f) return FP8LM_FLAG_AMAX_ZERO;
  uint32_t flags = 0;
  const int k = pow2_exp(fmax_bits, Aeff) + M.mu_exp - margin;
  const int e = k < -126 ? -126 : (k > 126 ? 126 : k);
  if (e != k) flags |= FP8LM_FLAG_SCALE_CLAMPED;
  M.scale = pow2f(e);
  M.inv_scale = pow2f(-e);
  return flags;
}
__device__ __forceinline__ void push_history(fp8lm_meta& M, float A, int hist_window) {
  const int H = hist_window < 1 ? 1 : (hist_window > FP8LM_HIST ? FP8LM_HIST : hist_window);
  const int slot = M.hist_pos % H;
  M.amax_hist[slot] = A;
  M.hist_pos = (slot + 1) % H;
}

template <int MODE, int SRC>
struct AmaxOp {
  using elem_t = typename SrcTraits<SRC>::elem_t;
  static constexpr int kPer = 16 / (int)sizeof(elem_t);   // elements per 128-bit load
  static constexpr int kLoads = kGroup / kPer;            // loads per thread and tile
  const AmaxParams& p;
  const Tables& tb;
  uint32_t acc;   // running maximum of the magnitude bits (two packed maxima for 16-bit sources)
  __device__ AmaxOp(const AmaxParams& p_, const Tables& tb_) : p(p_), tb(tb_), acc(0) {}
  __device__ __forceinline__ void begin(int) { acc = 0; }
  __device__ __forceinline__ bool fast() const { return true; }
  template <int UN> struct Regs { uint4 r[UN][kLoads]; };
  // a pure reduction: each load instruction of a wavefront covers 1 KiB contiguous
  template <int UN> __device__ __forceinline__ void load(Regs<UN>& g, long long pos) {
    const elem_t* q = static_cast<const elem_t*>(p.src) + pos + threadIdx.x * kPer;
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int k = 0; k < kLoads; ++k) g.r[u][k] = ld16<kNtLoadRO>(q + u * kTile + k * (kThreads * kPer));
  }
  template <int UN> __device__ __forceinline__ void tiles(const Regs<UN>& g, long long) {
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int k = 0; k < kLoads; ++k) {
        src_fold<SRC>(acc, g.r[u][k].x);
        src_fold<SRC>(acc, g.r[u][k].y);
        src_fold<SRC>(acc, g.r[u][k].z);
        src_fold<SRC>(acc, g.r[u][k].w);
      }
  }
  // 16 consecutive elements at `pos`, by this thread alone
  __device__ __forceinline__ void full_group(long long pos) {
    const elem_t* q = static_cast<const elem_t*>(p.src) + pos;
    uint4 r[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) r[k] = ld16<kNtLoadRO>(q + k * kPer);
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      src_fold<SRC>(acc, r[k].x);
      src_fold<SRC>(acc, r[k].y);
      src_fold<SRC>(acc, r[k].z);
      src_fold<SRC>(acc, r[k].w);
    }
  }
  __device__ __forceinline__ void group(long long pos, int valid) {
    const elem_t* q = static_cast<const elem_t*>(p.src) + pos;
    for (int j = 0; j < valid; ++j) src_fold1<SRC>(acc, q[j]);
  }
  using Stats = BlockStats<1, 0>;
  __device__ __forceinline__ void flush(long long u) {
    BlockStats<1, 0, uint32_t> s;
    s.mx[0] = src_final<SRC>(acc);
    s.orv = 0;
    collect(tb, u, s);
  }
  // scalar epilogue, one thread per tensor
  __device__ void finalize(int t, const TensorDesc&, const Stats& s) {
    const uint32_t abits = s.mx[0];
    fp8lm_meta& M = p.meta[t];
    if constexpr (MODE == kAmaxForMaster) {
      // an initialisation has no earlier scale to keep: zero tensors, non-finite ones and unscaled formats get 1
      M.scale = 1.0f;
      M.inv_scale = 1.0f;
    }
    if (abits >= SrcTraits<SRC>::kNonfinite) {
      M.amax = __builtin_inff();
      M.flags = FP8LM_FLAG_NONFINITE;
      return;
    }
    const float A = SrcTraits<SRC>::dec(abits);
    M.amax = A;
    uint32_t flags = 0;
    if constexpr (MODE == kAmaxForGradient) {
      push_history(M, A, p.hist_window);
      M.flags = scale_from_history(M, p.fmax_bits, p.hist_window, p.margin);
    } else {
      // master weights: one binade of headroom; flags and the rest are completed by the cast pass
      if (A == 0.0f) {
        flags |= FP8LM_FLAG_AMAX_ZERO;
      } else if (p.fmax_bits != 0u) {      // 0: BF16 / FP32 master weights carry no scale
        const int k = pow2_exp(p.fmax_bits, A) - 1;
        const int e = k < -126 ? -126 : (k > 126 ? 126 : k);
        if (e != k) flags |= FP8LM_FLAG_SCALE_CLAMPED;
        M.scale = pow2f(e);
        M.inv_scale = pow2f(-e);
      }
      M.flags = flags;
    }
  }
};

template <int MODE, int SRC>
__global__ __launch_bounds__(kThreads) void amax_kernel(Tables tb, AmaxParams p) {
  AmaxOp<MODE, SRC> op(p, tb);
  walk_units<kUnAmax<SRC>>(tb, op);
}

// ================================================================================================
// Kernel 2: scaled saturating FP8 cast + auto-scaling state (Sec. 2.1; Appendix A.1)
// ================================================================================================
// The auto-scaling state machine of Sec. 2.1 (text after Eq. 3), shared by the cast and the sum.
// mu_rule 0: an overflow sets mu to 1/2; mu then follows the count of clean steps (1/2, 1, 2 as it passes
// 0, ramp_steps/2, ramp_steps).  mu_rule 1, the other reading of the same sentence: every overflowing step
// halves mu down to 2^mu_min_exp, every ramp_steps/2 clean steps in a row double it up to 2.
struct AutoscaleRule {
  int32_t sat_num, sat_den, ramp_steps, mu_rule, mu_min_exp;
};
__device__ __forceinline__ void autoscale_update(fp8lm_meta& M, unsigned long long n_sat, long long numel,
                                                 const AutoscaleRule& a) {
  const int R = a.ramp_steps < 2 ? 2 : a.ramp_steps;
  const bool overflow = (long long)n_sat * (long long)a.sat_den > numel * (long long)a.sat_num;
  if (a.mu_rule == 1) {
    if (overflow) {
      M.mu_exp = M.mu_exp - 1 < a.mu_min_exp ? a.mu_min_exp : M.mu_exp - 1;
      M.clean_steps = 0;
    } else if (M.clean_steps + 1 >= R / 2) {
      M.mu_exp = M.mu_exp + 1 > 1 ? 1 : M.mu_exp + 1;
      M.clean_steps = 0;
    } else {
      M.clean_steps = M.clean_steps + 1;
    }
    return;
  }
  const int clean = overflow ? 0 : (M.clean_steps + 1 > R ? R : M.clean_steps + 1);
  M.clean_steps = clean;
  const int ramp = (2 * clean) / R;
  M.mu_exp = -1 + (ramp > 2 ? 2 : ramp);
}

// max |m'| of one element's new first moment is taken on m' = fma(beta1, m / s_m, (1-beta1) * (g / s_g)).  Scales are
// powers of two, so they can go into the coefficients without changing a rounding, unless something gets subnormal or
// overflows on the way: false then (or if a scale is no power of two, as that of an FP8 sum can be).
__device__ __forceinline__ bool fold_moment_scales(float b1, float omb1, float isg, float ism, float& cg, float& cm) {
  const uint32_t g = f2u(isg), m = f2u(ism);
  cg = omb1 * isg;
  cm = b1 * ism;
  return ((g | m) & 0x807FFFFFu) == 0 && (g >> 23) - 47u <= 160u && (m >> 23) - 47u <= 160u &&     // 2^-80 .. 2^80
         (b1 == 0.0f || b1 >= 0x1p-20f);
}
// the largest bit pattern of four |m'|, inf and NaN above all others
template <int FMT> __device__ __forceinline__ uint32_t folded_moment_max(uint32_t gw, uint32_t mw, float cg, float cm) {
  const float2_t g01 = fp8x2_to_f32<FMT, false>(gw), g23 = fp8x2_to_f32<FMT, true>(gw);
  const float2_t m01 = fp8x2_to_f32<kE4M3, false>(mw), m23 = fp8x2_to_f32<kE4M3, true>(mw);
  auto bits = [&](float dg, float dm) { return f2u(__builtin_fmaf(cm, dm, cg * dg)) & 0x7FFFFFFFu; };
  return max(max(bits(g01.x, m01.x), bits(g01.y, m01.y)), max(bits(g23.x, m23.x), bits(g23.y, m23.y)));
}

struct CastParams {
  const void* src;
  uint8_t* dst;
  fp8lm_meta* meta;
  AutoscaleRule rule;
  int32_t hist_window;   // delayed scaling and speculation
  int32_t speculative;   // DELAYED pass of the speculative just-in-time quantisation (see CastOp::speculation_verdict)
  uint32_t fmax_bits;    // speculation: largest finite value of the target format
  int32_t margin;
  // fused first pass of the Adam step (FUSE): the first moment as it stands and beta1
  const uint8_t* m;
  const fp8lm_meta* m_meta;
  float b1, omb1;
};

// number of non-zero bytes among the four 7-bit fields of x (each byte of x must be <= 0x7F)
__device__ __forceinline__ uint32_t nonzero_bytes7(uint32_t x) { return __popc((x + 0x7F7F7F7Fu) & 0x80808080u); }

// DELAYED: the scale was fixed from the amax history before the launch (Appendix A.2, delayed
// scaling); this pass also measures the amax of the source for the history, and since no amax pass
// has looked for inf/NaN it checks every 16-element group itself.
// FUSE: on one GPU the Adam step follows the cast directly, so this pass also measures what the Adam
// step's first pass would: max |fma(beta1, m, (1-beta1) * g)| with g the value just stored in FP8.
template <int FMT, bool DELAYED, bool FUSE, int SRC>
struct CastOp {
  using elem_t = typename SrcTraits<SRC>::elem_t;
  static constexpr int kPer = 16 / (int)sizeof(elem_t);   // elements per 128-bit load
  static constexpr int kLoads = kGroup / kPer;            // loads per 16-element group
  static constexpr int kW = kSrcWords<SRC>;
  const CastParams& p;
  const Tables& tb;
  float scale;
  bool careful;
  bool measure;           // a speculation with nothing to go by: only the amax is wanted
  float inv_sg, inv_sm;   // FUSE
  float cm, cg;           // FUSE: beta1 / s_m and (1 - beta1) / s_g, if folding the scales changes no rounding
  bool fold;
  uint32_t macc;          // FUSE: running max of the |m'| bit patterns
  uint32_t amax16;        // DELAYED: running maximum of the source's magnitude bits (packed pair for 16-bit types)
  float vmax;             // max |clamped scaled value|
  // counted elements: tails and the groups that have a code on the top or at zero at all
  uint32_t n_elems;
  uint32_t nz_top;        // codes whose magnitude differs from the top code
  uint32_t nz_code;       // codes with non-zero magnitude
  uint32_t z_in;          // inputs that are +-0
  __device__ CastOp(const CastParams& p_, const Tables& tb_) : p(p_), tb(tb_) {}
  __device__ __forceinline__ void reset() { vmax = 0.0f; n_elems = nz_top = nz_code = z_in = 0; amax16 = 0; macc = 0; }
  __device__ __forceinline__ void begin(int t) {
    scale = uniform_load(&p.meta[t].scale);
    int e = kKeepScale;
    if constexpr (DELAYED) {
      e = predicted_exponent<true>(p.meta + t, p.fmax_bits, p.hist_window, p.margin);
      if (e != kKeepScale) scale = pow2f(e);
    }
    measure = DELAYED && p.speculative && e == kKeepScale;
    careful = !DELAYED && (uniform_load(&p.meta[t].flags) & FP8LM_FLAG_NONFINITE) != 0;
    if constexpr (FUSE) {
      inv_sg = e != kKeepScale ? pow2f(-e) : uniform_load(&p.meta[t].inv_scale);
      inv_sm = uniform_load(&p.m_meta[t].inv_scale);
      fold = fold_moment_scales(p.b1, p.omb1, inv_sg, inv_sm, cg, cm);
    }
    reset();
  }
  // FUSE: the new first moment of one element, from the decoded FP8 gradient and moment codes
  __device__ __forceinline__ void moment(float dg, float dm) {
    const float g = dg * inv_sg, m0 = dm * inv_sm;
    const float m1 = __builtin_fmaf(p.b1, m0, p.omb1 * g);
    macc = max(macc, f2u(m1) & 0x7FFFFFFFu);
  }
  __device__ __forceinline__ void moment_word(uint32_t gw, uint32_t mw) {
    if (fold) {
      macc = max(macc, folded_moment_max<FMT>(gw, mw, cg, cm));
      return;
    }
    const float2_t g01 = fp8x2_to_f32<FMT, false>(gw), g23 = fp8x2_to_f32<FMT, true>(gw);
    const float2_t m01 = fp8x2_to_f32<kE4M3, false>(mw), m23 = fp8x2_to_f32<kE4M3, true>(mw);
    moment(g01.x, m01.x);
    moment(g01.y, m01.y);
    moment(g23.x, m23.x);
    moment(g23.y, m23.y);
  }
  // four consecutive elements of a group (quad q = 0..3) widened to fp32
  __device__ __forceinline__ float4 widen(const uint32_t (&w)[kW], int q) const {
    if constexpr (SRC == kSrcBF16) {
      return make_float4(bf16lo_to_f32(w[2 * q]), bf16hi_to_f32(w[2 * q]), bf16lo_to_f32(w[2 * q + 1]), bf16hi_to_f32(w[2 * q + 1]));
    } else if constexpr (SRC == kSrcF16) {
      const float2_t lo = f16x2_to_f32(w[2 * q]), hi = f16x2_to_f32(w[2 * q + 1]);
      return make_float4(lo.x, lo.y, hi.x, hi.y);
    } else {
      return make_float4(u2f(w[4 * q]), u2f(w[4 * q + 1]), u2f(w[4 * q + 2]), u2f(w[4 * q + 3]));
    }
  }
  template <bool CLAMP> __device__ __forceinline__ uint32_t quad(const uint32_t (&w)[kW], int q) {
    const float4 f = widen(w, q);
    float y0 = f.x * scale, y1 = f.y * scale, y2 = f.z * scale, y3 = f.w * scale;
    if constexpr (CLAMP) {
      y0 = clamp_fp8<FMT>(y0); y1 = clamp_fp8<FMT>(y1); y2 = clamp_fp8<FMT>(y2); y3 = clamp_fp8<FMT>(y3);
    }
    return f32x2_to_fp8<FMT, true>(y2, y3, f32x2_to_fp8<FMT, false>(y0, y1, 0u));
  }
  // the counters of one group's codes
  __device__ __forceinline__ void count(const uint32_t (&w)[kW], const uint4& o) {
    const uint32_t c[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t mag = c[q] & 0x7F7F7F7Fu;
      nz_code += nonzero_bytes7(mag);
      nz_top += nonzero_bytes7(mag ^ Fp8Traits<FMT>::kTopX4);
      const float4 f = widen(w, q);
      z_in += (f.x == 0.0f) + (f.y == 0.0f) + (f.z == 0.0f) + (f.w == 0.0f);
    }
    n_elems += kGroup;
  }
  __device__ __forceinline__ uint32_t one(uint32_t bits, uint32_t mcode) {
    const float f = SrcTraits<SRC>::dec(bits);
    const float y = f * scale;
    uint32_t c;
    if (y != y) {
      c = 0x7Fu;
    } else {
      const float yc = clamp_fp8<FMT>(y);
      vmax = fmaxf(vmax, fabsf(yc));
      c = f32x2_to_fp8<FMT, false>(yc, 0.0f, 0u) & 0xFFu;
    }
    z_in += (f == 0.0f);
    nz_code += (c & 0x7Fu) != 0;
    nz_top += (c & 0x7Fu) != Fp8Traits<FMT>::kTop;
    if constexpr (DELAYED) src_fold1<SRC>(amax16, bits);
    if constexpr (FUSE) moment(fp8_to_f32<FMT>(c), fp8_to_f32<kE4M3>(mcode));
    return c;
  }
  __device__ __forceinline__ bool fast() const { return !careful; }
  // kSplit: the thread's 16 elements are kRuns runs, [8L, 8L+8) of each half of the tile for 16-bit sources, [4L, 4L+4)
  // of each quarter for fp32: every 128-bit load is contiguous over the workgroup, the stores have 64 or 32 bits.
  // Otherwise 16 consecutive elements.  (fp32 sources with 16 consecutive elements per thread, 201e6 of them: 228 us.)
  static constexpr int kRuns = kLoads, kRun = kGroup / kRuns;
  template <int UN> struct Regs { uint4 r[UN][kLoads], mm[FUSE ? UN : 1]; };
  template <int UN> __device__ __forceinline__ void load(Regs<UN>& g, long long pos0) { load_as<true>(g, pos0); }
  template <int UN> __device__ __forceinline__ void tiles(const Regs<UN>& g, long long pos0) { tiles_as<true>(g, pos0); }
  template <bool kSplit, int UN> __device__ __forceinline__ void load_as(Regs<UN>& g, long long pos0) {
    constexpr int kStep = kTile / kRuns;
    const long long pos = pos0 + threadIdx.x * (kSplit ? kRun : kGroup);
    const elem_t* q = static_cast<const elem_t*>(p.src) + pos;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
#pragma unroll
      for (int k = 0; k < kLoads; ++k) g.r[u][k] = ld16<kNtLoadRO>(q + u * kTile + k * (kSplit ? kStep : kPer));
      if constexpr (FUSE) {
        const uint8_t* m = p.m + pos + u * kTile;
        if constexpr (kSplit && kRuns == 2) {
          const uint2 lo = ld8<kNtLoadRO>(m), hi = ld8<kNtLoadRO>(m + kStep);
          g.mm[u] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        } else if constexpr (kSplit) {
          g.mm[u] = make_uint4(ld4<kNtLoadRO>(m), ld4<kNtLoadRO>(m + kStep), ld4<kNtLoadRO>(m + 2 * kStep), ld4<kNtLoadRO>(m + 3 * kStep));
        } else {
          g.mm[u] = ld16<kNtLoadRO>(m);
        }
      }
    }
  }
  template <bool kSplit, int UN> __device__ __forceinline__ void tiles_as(const Regs<UN>& g, long long pos0) {
    constexpr int kStep = kTile / kRuns;
    const long long pos = pos0 + threadIdx.x * (kSplit ? kRun : kGroup);
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      uint32_t w[kW];
#pragma unroll
      for (int k = 0; k < kLoads; ++k) {
        w[4 * k] = g.r[u][k].x; w[4 * k + 1] = g.r[u][k].y; w[4 * k + 2] = g.r[u][k].z; w[4 * k + 3] = g.r[u][k].w;
      }
      // The largest and the smallest magnitude of the group, by integer maxima of the source's bits (packed pairs for 16-bit
      // types): scaling is monotone, so they tell whether any element saturates, lands on the top code or underflows.
      // Mostly none does, and the elements are only scaled and converted: 5.5 instructions each instead of 10, which is
      // what kept the pass off the memory's pace.
      uint32_t gmax = 0, gmin = 0xFFFFFFFFu;
#pragma unroll
      for (int j = 0; j < kW; ++j) {
        src_fold<SRC>(gmax, w[j]);
        src_fold_min<SRC>(gmin, w[j]);
      }
      const uint32_t top = src_final<SRC>(gmax);
      if constexpr (DELAYED) {
        src_fold1<SRC>(amax16, top);
        // Without a history (the first call) the speculation of a tensor cannot hold unless all of it is zero, so only zeros are
        // written: 5 bytes per element in both rounds, as amax pass and cast have, instead of 6 (125e6 elements: 160 us, 137 this way).
        if (measure && top != 0) continue;
        if (top >= SrcTraits<SRC>::kNonfinite) {
          // rare: this group holds inf/NaN; element by element, and again from memory: no registers for it
          if constexpr (kSplit) {
            for (int k = 0; k < kRuns; ++k) group(pos + u * kTile + k * kStep, kRun);
          } else {
            group(pos + u * kTile, kGroup);
          }
          continue;
        }
      }
      const float ymax = SrcTraits<SRC>::dec(top) * scale, ymin = SrcTraits<SRC>::dec(src_final_min<SRC>(gmin)) * scale;
      uint4 o;
      if (!(ymax <= Fp8Traits<FMT>::kMax)) {
        o = make_uint4(quad<true>(w, 0), quad<true>(w, 1), quad<true>(w, 2), quad<true>(w, 3));
      } else {
        // one quad after the other: interleaved, as the compiler would have them, they take registers that other
        // wavefronts make better use of
        o.x = quad<false>(w, 0);
        __builtin_amdgcn_sched_barrier(0);
        o.y = quad<false>(w, 1);
        __builtin_amdgcn_sched_barrier(0);
        o.z = quad<false>(w, 2);
        __builtin_amdgcn_sched_barrier(0);
        o.w = quad<false>(w, 3);
      }
      vmax = fmaxf(vmax, fminf(ymax, Fp8Traits<FMT>::kMax));
      if (ymax >= Fp8Traits<FMT>::kFirstTop || ymin <= Fp8Traits<FMT>::kLastZero) count(w, o);
      if constexpr (FUSE) {
        const uint4 mm = g.mm[u];
        moment_word(o.x, mm.x);
        moment_word(o.y, mm.y);
        moment_word(o.z, mm.z);
        moment_word(o.w, mm.w);
      }
      uint8_t* dst = p.dst + pos + u * kTile;
      if constexpr (kSplit && kRuns == 2) {
        st8<kNtStoreWO>(dst, make_uint2(o.x, o.y));
        st8<kNtStoreWO>(dst + kStep, make_uint2(o.z, o.w));
      } else if constexpr (kSplit) {
        st4<kNtStoreWO>(dst, o.x);
        st4<kNtStoreWO>(dst + kStep, o.y);
        st4<kNtStoreWO>(dst + 2 * kStep, o.z);
        st4<kNtStoreWO>(dst + 3 * kStep, o.w);
      } else {
        st16<kNtStoreWO>(dst, o);
      }
    }
  }
  // 16 consecutive elements at `pos`, by this thread alone (the layout without the split)
  __device__ __forceinline__ void full_group(long long pos) {
    Regs<1> g;
    load_as<false>(g, pos - (long long)threadIdx.x * kGroup);
    tiles_as<false>(g, pos - (long long)threadIdx.x * kGroup);
  }
  __device__ __forceinline__ void group(long long pos, int valid) {
    const elem_t* q = static_cast<const elem_t*>(p.src) + pos;
#pragma unroll 1
    for (int j = 0; j < valid; ++j) p.dst[pos + j] = (uint8_t)one(q[j], FUSE ? p.m[pos + j] : 0u);
    n_elems += valid;
  }
  static constexpr bool kFinishes = true;      // walk_marked
  using Stats = BlockStats<3, 2>;
  __device__ __forceinline__ void flush(long long u) {
    BlockStats<3, 2, uint32_t> s;
    s.mx[0] = f2u(vmax);
    s.mx[1] = src_final<SRC>(amax16);
    s.mx[2] = macc;
    s.ct[0] = n_elems - nz_top;                 // codes on the top magnitude
    s.ct[1] = (n_elems - nz_code) - z_in;       // zero codes that did not come from zero inputs
    s.orv = 0;
    collect(tb, u, s);
  }
  __device__ void finalize(int t, const TensorDesc& d, const Stats& s) {
    const float vm = u2f(s.mx[0]);
    const uint32_t abits = s.mx[1];
    if constexpr (FUSE) tb.scratch[t].pend.amax_m_bits = s.mx[2];
    const unsigned long long n_sat = s.ct[0], n_und = s.ct[1];
    if constexpr (DELAYED) {
      if (p.speculative) {
        const bool held = speculation_verdict(t, abits);
        mark_redo(tb, t, d, !held);
        if (held) finish(t, d, vm, n_sat, n_und);
        return;
      }
      fp8lm_meta& M = p.meta[t];
      M.flags = scale_from_history(M, p.fmax_bits, p.hist_window, p.margin);     // the scale the pass has used
      if (abits >= SrcTraits<SRC>::kNonfinite) {
        M.amax = __builtin_inff();
        M.flags |= FP8LM_FLAG_NONFINITE;
      } else {
        M.amax = SrcTraits<SRC>::dec(abits);
        push_history(M, M.amax, p.hist_window);
      }
    }
    finish(t, d, vm, n_sat, n_und);
  }
  // Speculative just-in-time quantisation (Appendix A.2): this pass has cast the tensor with the scale its amax
  // history predicted and measured the true amax on the way.  Now the metadata is brought to exactly what the amax
  // pass of the two-pass form would have left (scale from the true amax, history pushed, flags); if that scale is
  // the one the cast used, the codes already written are the just-in-time result and the caller finishes the cast's
  // bookkeeping; otherwise the tensor has to be cast again.  Returns true if the speculation held.
  __device__ bool speculation_verdict(int t, uint32_t abits) {
    fp8lm_meta& M = p.meta[t];
    const int e = predicted_exponent<false>(p.meta + t, p.fmax_bits, p.hist_window, p.margin);
    const float used = e != kKeepScale ? pow2f(e) : M.scale;
    bool held;
    if (abits >= SrcTraits<SRC>::kNonfinite) {
      M.amax = __builtin_inff();
      M.flags = FP8LM_FLAG_NONFINITE;       // the second cast takes the path that knows NaN
      held = false;
    } else {
      const float A = SrcTraits<SRC>::dec(abits);
      M.amax = A;
      push_history(M, A, p.hist_window);
      M.flags = scale_from_history(M, p.fmax_bits, p.hist_window, p.margin);
      held = M.scale == used && (e != kKeepScale || abits == 0);      // (without a history only zeros have been cast)
    }
    return held;
  }
  __device__ void finish(int t, const TensorDesc& d, float vm, unsigned long long n_sat, unsigned long long n_und) {
    fp8lm_meta& M = p.meta[t];
    M.n_sat = n_sat;
    M.n_underflow = n_und;
    M.amax_deq = fp8_to_f32<FMT>(encode1_fp8<FMT>(vm)) * M.inv_scale;
    M.flags = n_sat ? (M.flags | FP8LM_FLAG_SATURATED) : (M.flags & ~FP8LM_FLAG_SATURATED);
    autoscale_update(M, n_sat, d.numel, p.rule);
  }
};

template <int FMT, bool DELAYED, bool FUSE, int SRC>
__global__ __launch_bounds__(kThreads) void cast_kernel(Tables tb, CastParams p) {
  CastOp<FMT, DELAYED, FUSE, SRC> op(p, tb);
  walk_units<kUnCast<SRC>>(tb, op);
}

// The second round of a speculative quantisation: the marked tensors, with the scale that is now in their metadata.
template <int FMT, bool FUSE, int SRC>
__global__ __launch_bounds__(kThreads) void cast_marked_kernel(Tables tb, CastParams p) {
  CastOp<FMT, false, FUSE, SRC> op(p, tb);
  walk_marked<kUnCast<SRC>>(tb, op);
}

// ================================================================================================
// Shared-scale re-quantisation and the FP8 gradient sum (Sec. 2.1, Eq. 4-6)
// ================================================================================================
constexpr int kMaxRanks = 128;      // rank pointers travel as kernel arguments (1 KiB)
constexpr int kUnrolledRanks = 8;   // rank counts up to this have a kernel of their own
struct RankMetas { const fp8lm_meta* m[kMaxRanks]; int32_t n_ranks; };
struct RankPayloads { const uint8_t* p[kMaxRanks]; int32_t n_ranks; };

// Eq. 4: one thread per tensor takes the smallest scale among the ranks.
__global__ void shared_scale_kernel(RankMetas rm, int n, float* shared) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  float s = rm.m[0][t].scale;
  for (int r = 1; r < rm.n_ranks; ++r) s = rm.m[r][t].scale < s ? rm.m[r][t].scale : s;
  shared[t] = s;
}

// Sec. 2.1, text after Eq. 3: the factor mu chosen from the summed gradient's statistic is what every rank
// applies to its next gradient.  One thread per tensor copies the auto-scaling state into the ranks' metas.
struct RankMetasOut { fp8lm_meta* m[kMaxRanks]; int32_t n_ranks; };
__global__ void autoscale_broadcast_kernel(const fp8lm_meta* from, RankMetasOut rm, int n) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int32_t mu_exp = from[t].mu_exp, clean = from[t].clean_steps;
  for (int r = 0; r < rm.n_ranks; ++r) {
    rm.m[r][t].mu_exp = mu_exp;
    rm.m[r][t].clean_steps = clean;
  }
}
// Sec. 2.1, Eq. 1-2: a fixed factor mu = 2^mu_exp (pre-scaling 1/N, post-scaling 1) for every tensor.
__global__ void set_mu_kernel(fp8lm_meta* meta, int n, int32_t mu_exp) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) meta[t].mu_exp = mu_exp;
}

struct RequantParams {
  const uint8_t* src;
  const fp8lm_meta* src_meta;
  const float* shared;
  uint8_t* dst;
  fp8lm_meta* dst_meta;
};

// Eq. 5: dst = FP8(s_g * (src / s')).  Both scales are powers of two with s_g <= s': an exponent shift
// that can only lose bits at the bottom of the range.
template <int FMT>
struct RequantOp {
  const RequantParams& p;
  const Tables& tb;
  float inv_src, sg;
  bool careful;
  bool same;              // the shared scale is the source's: the codes stay as they are
  uint32_t cmax;          // ... and the largest magnitude among them (two packed maxima)
  float vmax;
  uint32_t n_elems, nz_top, nz_code, nz_in, nonfinite;
  __device__ RequantOp(const RequantParams& p_, const Tables& tb_) : p(p_), tb(tb_) {}
  __device__ __forceinline__ void begin(int t) {
    inv_src = uniform_load(&p.src_meta[t].inv_scale);
    sg = uniform_load(p.shared + t);
    // codes that stand for more than fp32 holds (amax of the last binade) come out as the top code, element by element
    careful = (uniform_load(&p.src_meta[t].flags) & FP8LM_FLAG_NONFINITE) != 0 ||
              !(inv_src * Fp8Traits<FMT>::kMax <= 3.4028234663852886e38f);
    same = ((f2u(inv_src) | f2u(sg)) & 0x807FFFFFu) == 0 && inv_src * sg == 1.0f;      // powers of two
    cmax = 0;
    vmax = 0.0f;
    n_elems = nz_top = nz_code = nz_in = nonfinite = 0;
  }
  __device__ __forceinline__ bool fast() const { return !careful; }
  // Four codes.  The counters only of groups where they can change: `count`.
  __device__ __forceinline__ uint32_t word(uint32_t w) {
    const float2_t a = fp8x2_to_f32<FMT, false>(w), b = fp8x2_to_f32<FMT, true>(w);
    const float y0 = (a.x * inv_src) * sg, y1 = (a.y * inv_src) * sg, y2 = (b.x * inv_src) * sg, y3 = (b.y * inv_src) * sg;
    vmax = fmaxf(fmaxf(vmax, fmaxf(fabsf(y0), fabsf(y1))), fmaxf(fabsf(y2), fabsf(y3)));
    return encode4_fp8<FMT>(y0, y1, y2, y3);
  }
  __device__ __forceinline__ void count(uint32_t w, uint32_t c) {
    const uint32_t mag = c & 0x7F7F7F7Fu;
    nz_in += nonzero_bytes7(w & 0x7F7F7F7Fu);
    nz_code += nonzero_bytes7(mag);
    nz_top += nonzero_bytes7(mag ^ Fp8Traits<FMT>::kTopX4);
  }
  // 16 codes.  Ranks whose amax lies in the same binade share their scale already: then there is nothing to convert (the
  // tensors with NaN codes, which would get their canonical form, take the careful path).  No code on the top and none
  // zero: nothing to count.  (Converting and counting everything, 8 instructions per code: 51 us for 125e6 codes.)
  __device__ __forceinline__ uint4 codes16(const uint4& in) {
    uint4 o = in;
    if (!same) o = make_uint4(word(in.x), word(in.y), word(in.z), word(in.w));
    const uint32_t w[4] = {in.x, in.y, in.z, in.w}, c[4] = {o.x, o.y, o.z, o.w};
    uint32_t all_nz = 0x80808080u, any = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t mag = c[k] & 0x7F7F7F7Fu;
      all_nz &= mag + 0x7F7F7F7Fu;                                         // bit 7 of a byte: its magnitude is not zero
      any |= mag + (0x80808080u - Fp8Traits<FMT>::kTopX4);                 // ... it is the top code
      if (same) {
        src_fold<kSrcBF16>(cmax, mag & 0x007F007Fu);
        src_fold<kSrcBF16>(cmax, (mag >> 8) & 0x007F007Fu);
      }
    }
    if (all_nz != 0x80808080u || (any & 0x80808080u)) {
#pragma unroll
      for (int k = 0; k < 4; ++k) count(w[k], c[k]);
      n_elems += kGroup;
    }
    return o;
  }
  template <int UN> struct Regs { uint4 a[UN]; };
  template <int UN> __device__ __forceinline__ void load(Regs<UN>& g, long long pos0) {
    const long long pos = pos0 + threadIdx.x * kGroup;
#pragma unroll
    for (int u = 0; u < UN; ++u) g.a[u] = ld16<kNtLoadRW>(p.src + pos + u * kTile);
  }
  template <int UN> __device__ __forceinline__ void tiles(const Regs<UN>& g, long long pos0) {
    const long long pos = pos0 + threadIdx.x * kGroup;
#pragma unroll
    for (int u = 0; u < UN; ++u)
      st16<kNtStoreRW>(p.dst + pos + u * kTile, codes16(g.a[u]));
  }
  // 16 consecutive elements at `pos`, by this thread alone: the tile body with the thread's own offset taken out
  __device__ __forceinline__ void full_group(long long pos) {
    Regs<1> g;
    load(g, pos - (long long)threadIdx.x * kGroup);
    tiles(g, pos - (long long)threadIdx.x * kGroup);
  }
  __device__ __forceinline__ void group(long long pos, int valid) {
    for (int j = 0; j < valid; ++j) {
      const uint32_t in = p.src[pos + j];
      const float y = (fp8_to_f32<FMT>(in) * inv_src) * sg;
      const uint32_t c = encode1_fp8_careful<FMT>(y);
      if (y == y) vmax = fmaxf(vmax, fabsf(clamp_fp8<FMT>(y)));
      nonfinite |= !(fabsf(y) <= 3.4028234663852886e38f);
      nz_in += (in & 0x7Fu) != 0;
      nz_code += (c & 0x7Fu) != 0;
      nz_top += (c & 0x7Fu) != Fp8Traits<FMT>::kTop;
      p.dst[pos + j] = (uint8_t)c;
    }
    n_elems += valid;
  }
  using Stats = BlockStats<1, 2>;
  __device__ __forceinline__ void flush(long long u) {
    BlockStats<1, 2, uint32_t> s;
    s.mx[0] = f2u(fmaxf(vmax, fp8_to_f32<FMT>(src_final<kSrcBF16>(cmax))));
    s.ct[0] = n_elems - nz_top;
    s.ct[1] = nz_in - nz_code;                 // non-zero codes in, zero codes out (a NaN code is non-zero on both sides)
    s.orv = nonfinite;
    collect(tb, u, s);
  }
  __device__ void finalize(int t, const TensorDesc&, const Stats& s) {
    const float vm = u2f(s.mx[0]);
    const unsigned long long n_sat = s.ct[0], n_und = s.ct[1];
    const uint32_t nf = s.orv;
    fp8lm_meta& M = p.dst_meta[t];
    const float src_amax = p.src_meta[t].amax, sg = p.shared[t];
    const float inv = 1.0f / sg;
    M.scale = sg;
    M.inv_scale = inv;
    M.amax = nf ? __builtin_inff() : src_amax;
    M.amax_deq = fp8_to_f32<FMT>(encode1_fp8<FMT>(vm)) * inv;
    M.n_sat = n_sat;
    M.n_underflow = n_und;
    M.flags = (nf ? FP8LM_FLAG_NONFINITE : 0u) | (n_sat ? FP8LM_FLAG_SATURATED : 0u);
  }
};

template <int FMT>
__global__ __launch_bounds__(kThreads) void requantize_kernel(Tables tb, RequantParams p) {
  RequantOp<FMT> op(p, tb);
  walk_units<kUnRequant>(tb, op);
}

struct SumParams {
  RankPayloads in;
  const float* shared;
  uint8_t* dst;
  fp8lm_meta* dst_meta;
  AutoscaleRule rule;
};

// Eq. 6 on one GPU: the payloads of all ranks (same shared scale) are added in rank order in fp32 and
// rounded once to FP8, saturating; the result carries the scale N * s_g.
template <int FMT, int NR>
struct SumOp {
  const SumParams& p;
  const Tables& tb;
  float vmax;
  uint32_t amax_bits, n_top, n_und;            // n_top / n_und: counted element by element (tails, NaN groups)
  uint32_t n_fast, nz_top, nz_code, z_acc;     // whole groups: counted on the packed codes, as in the cast
  __device__ SumOp(const SumParams& p_, const Tables& tb_) : p(p_), tb(tb_) {}
  __device__ __forceinline__ void begin(int) {
    vmax = 0.0f;
    amax_bits = n_top = n_und = n_fast = nz_top = nz_code = z_acc = 0;
  }
  __device__ __forceinline__ bool fast() const { return true; }
  __device__ __forceinline__ uint32_t finish_one(float acc) {
    const uint32_t c = encode1_fp8_careful<FMT>(acc);
    amax_bits = max(amax_bits, f2u(acc) & 0x7FFFFFFFu);
    if (acc == acc) vmax = fmaxf(vmax, fabsf(clamp_fp8<FMT>(acc)));
    n_top += (c & 0x7Fu) == Fp8Traits<FMT>::kTop;
    n_und += (acc != 0.0f) && ((c & 0x7Fu) == 0);
    return c;
  }
  // four sums without a NaN among them: clamp, convert in pairs, count on the packed codes
  __device__ __forceinline__ uint32_t finish_quad(const float* acc) {
    const float y0 = clamp_fp8<FMT>(acc[0]), y1 = clamp_fp8<FMT>(acc[1]);
    const float y2 = clamp_fp8<FMT>(acc[2]), y3 = clamp_fp8<FMT>(acc[3]);
    vmax = fmaxf(fmaxf(vmax, fmaxf(fabsf(y0), fabsf(y1))), fmaxf(fabsf(y2), fabsf(y3)));
    amax_bits = max(max(amax_bits, max(f2u(acc[0]) & 0x7FFFFFFFu, f2u(acc[1]) & 0x7FFFFFFFu)),
                    max(f2u(acc[2]) & 0x7FFFFFFFu, f2u(acc[3]) & 0x7FFFFFFFu));
    z_acc += (acc[0] == 0.0f) + (acc[1] == 0.0f) + (acc[2] == 0.0f) + (acc[3] == 0.0f);
    uint32_t c = f32x2_to_fp8<FMT, false>(y0, y1, 0u);
    c = f32x2_to_fp8<FMT, true>(y2, y3, c);
    const uint32_t mag = c & 0x7F7F7F7Fu;
    nz_code += nonzero_bytes7(mag);
    nz_top += nonzero_bytes7(mag ^ Fp8Traits<FMT>::kTopX4);
    return c;
  }
  // one rank's 16 payloads added to the running sums: rank order, one fp32 addition per rank
  __device__ __forceinline__ void add_rank(float* acc, const uint4& a) {
    const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float2_t lo = fp8x2_to_f32<FMT, false>(w[k]), hi = fp8x2_to_f32<FMT, true>(w[k]);
      acc[4 * k + 0] = acc[4 * k + 0] + lo.x;
      acc[4 * k + 1] = acc[4 * k + 1] + lo.y;
      acc[4 * k + 2] = acc[4 * k + 2] + hi.x;
      acc[4 * k + 3] = acc[4 * k + 3] + hi.y;
    }
  }
  // rounds 16 sums to FP8 and stores them
  __device__ __forceinline__ void finish_group(const float* acc, long long pos) {
    bool any_nan = false;
#pragma unroll
    for (int j = 0; j < kGroup; ++j) any_nan |= acc[j] != acc[j];
    uint32_t o[4] = {0, 0, 0, 0};
    if (!any_nan) {
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = finish_quad(acc + 4 * k);
      n_fast += kGroup;
    } else {
#pragma unroll
      for (int j = 0; j < kGroup; ++j) o[j >> 2] |= finish_one(acc[j]) << ((j & 3) * 8);
    }
    st16<kNtStoreWO>(p.dst + pos, make_uint4(o[0], o[1], o[2], o[3]));
  }
  // NR > 0: that many ranks, all loads of UN tiles issued up front.  NR == 0: any number of ranks
  // (p.in.n_ranks), loaded eight at a time.
  template <int UN> struct Regs { uint4 a[UN][NR > 0 ? NR : 1]; };
  template <int UN> __device__ __forceinline__ void load(Regs<UN>& g, long long pos0) {
    const long long pos = pos0 + threadIdx.x * kGroup;
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int r = 0; r < NR; ++r) g.a[u][r] = ld16<kNtLoadRO>(p.in.p[r] + pos + u * kTile);
  }
  template <int UN> __device__ __forceinline__ void tiles(const Regs<UN>& g, long long pos0) {
    const long long pos = pos0 + threadIdx.x * kGroup;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      float acc[kGroup];
#pragma unroll
      for (int j = 0; j < kGroup; ++j) acc[j] = 0.0f;
      if constexpr (NR == 0) {
        const int n = p.in.n_ranks;
        for (int r0 = 0; r0 < n; r0 += kUnrolledRanks) {
          uint4 a[kUnrolledRanks];
#pragma unroll
          for (int k = 0; k < kUnrolledRanks; ++k)
            if (r0 + k < n) a[k] = ld16<kNtLoadRO>(p.in.p[r0 + k] + pos + u * kTile);
#pragma unroll
          for (int k = 0; k < kUnrolledRanks; ++k)
            if (r0 + k < n) add_rank(acc, a[k]);
        }
      } else {
#pragma unroll
        for (int r = 0; r < NR; ++r) add_rank(acc, g.a[u][r]);
      }
      finish_group(acc, pos + u * kTile);
    }
  }
  // 16 consecutive elements at `pos`, by this thread alone: the tile body with the thread's own offset taken out
  __device__ __forceinline__ void full_group(long long pos) {
    Regs<1> g;
    load(g, pos - (long long)threadIdx.x * kGroup);
    tiles(g, pos - (long long)threadIdx.x * kGroup);
  }
  __device__ __forceinline__ void group(long long pos, int valid) {
    for (int j = 0; j < valid; ++j) {
      float acc = 0.0f;
      const int n = NR > 0 ? NR : p.in.n_ranks;
      for (int r = 0; r < n; ++r) acc = acc + fp8_to_f32<FMT>(p.in.p[r][pos + j]);
      p.dst[pos + j] = (uint8_t)finish_one(acc);
    }
  }
  using Stats = BlockStats<2, 2>;
  __device__ __forceinline__ void flush(long long u) {
    BlockStats<2, 2, uint32_t> s;
    s.mx[0] = f2u(vmax);
    s.mx[1] = amax_bits;
    s.ct[0] = n_top + (n_fast - nz_top);              // codes on the top magnitude
    s.ct[1] = n_und + ((n_fast - nz_code) - z_acc);   // zero codes that did not come from zero sums
    s.orv = 0;
    collect(tb, u, s);
  }
  __device__ void finalize(int t, const TensorDesc& d, const Stats& s) {
    const float vm = u2f(s.mx[0]);
    const uint32_t ab = s.mx[1];
    const unsigned long long n_sat = s.ct[0], n_under = s.ct[1];
    fp8lm_meta& M = p.dst_meta[t];
    const float sc_out = (float)p.in.n_ranks * p.shared[t];
    const bool nf = ab >= 0x7F800000u;
    M.scale = sc_out;
    M.inv_scale = 1.0f / sc_out;
    M.amax = nf ? __builtin_inff() : u2f(ab) * M.inv_scale;
    M.amax_deq = fp8_to_f32<FMT>(encode1_fp8<FMT>(vm)) * M.inv_scale;
    M.n_sat = n_sat;
    M.n_underflow = n_under;
    M.flags = (nf ? FP8LM_FLAG_NONFINITE : 0u) | (n_sat ? FP8LM_FLAG_SATURATED : 0u);
    autoscale_update(M, n_sat, d.numel, p.rule);
  }
};

template <int FMT, int NR>
__global__ __launch_bounds__(kThreads) void sum_fp8_kernel(Tables tb, SumParams p) {
  SumOp<FMT, NR> op(p, tb);
  walk_units<sum_tiles(NR)>(tb, op);   // about eight 128-bit loads in flight per thread
}

}  // namespace fp8lm

#endif
