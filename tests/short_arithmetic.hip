// What the short root and division of the update pass rest on (adam.hpp: short_root, short_quotient), tried out:
// quotients() on the host, over the quotients that lie closest to a rounding boundary; roots_and_reciprocals() on the GPU, over
// every significand; tame() says which tensors take them.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <thread>
#include <vector>

#include "fp8lm.h"
#include "adam.hpp"

namespace {
float as_float(uint32_t u) { float f; std::memcpy(&f, &u, 4); return f; }
uint32_t as_bits(float f) { uint32_t u; std::memcpy(&u, &f, 4); return u; }
uint64_t pow_mod(uint64_t b, uint64_t e, uint64_t m) {
  uint64_t r = 1 % m;
  for (b %= m; e; e >>= 1, b = (unsigned __int128)b * b % m)
    if (e & 1) r = (unsigned __int128)r * b % m;
  return r;
}

__global__ void estimates_kernel(uint32_t base, float* rcp, float* root, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float x = fp8lm::u2f(base + i);
  rcp[i] = __builtin_amdgcn_rcpf(x);
  root[i] = fp8lm::short_root(x, __builtin_amdgcn_rsqf(x));
}
}  // namespace

extern "C" {
// hp: b1, 1 - b1, 1 / (1 - b1^t), b2, 1 - b2, 1 / (1 - b2^t), eps; inverse: of the scales of gradient, moments and weight.
int tame(const float* hp, const float* inverse, float decay) {
  fp8lm::AdamParams p{};
  p.b1 = hp[0]; p.omb1 = hp[1]; p.rbc1 = hp[2]; p.b2 = hp[3]; p.omb2 = hp[4]; p.rbc2 = hp[5]; p.eps = hp[6];
  float c[8];
  return fp8lm::tame_range(p, inverse[0], inverse[1], inverse[2], inverse[3], decay, c);
}

// With significands A and D of 24 bits and k = 23 or 24 (so that the quotient of a = A / 2^23 and d = D / 2^23 has 24 bits), a / d is
// A 2^k / D in units of its last place: close to a boundary between two roundings if 2 ((A 2^k) mod D) is close to D.  For every
// `stride`-th D the A with a difference of at most 32 are solved for, and every quotient is taken with the reciprocal estimate
// off by -1, 0 and 1 ulp.  out: cases, wrong with the nearest estimate, wrong with another; wrong_d: the divisors of the latter
// (bit patterns, up to 64).  Returns -1 if a case is not what it was solved for.
int quotients(uint32_t first, uint32_t stride, int64_t* out, uint32_t* wrong_d) {
  const int threads = 8;
  std::atomic<long long> cases(0), wrong_nearest(0), wrong_off(0), failed(0);
  auto work = [&](int t) {
    long long mine = 0;
    for (uint64_t D = (1u << 23) + first + (uint64_t)stride * t; D < (1u << 24); D += (uint64_t)stride * threads) {
      const float d = as_float(0x3F800000u | ((uint32_t)D & 0x7FFFFFu));
      const uint32_t nearest = as_bits(1.0f / d);
      for (int k = 23; k <= 24; ++k) {
        const uint64_t lo = k == 24 ? (1u << 23) : D, hi = k == 24 ? D : (1u << 24);      // a < d or a >= d
        if (lo >= hi) continue;
        const int twos = std::min(__builtin_ctzll(D), k);
        const uint64_t m = D >> twos, inverse = m > 1 ? pow_mod((m + 1) / 2, k - twos, m) : 0;
        for (int diff = -32; diff <= 32; ++diff) {
          const int64_t twice = (int64_t)D + diff;
          if ((twice & 1) || twice < 0 || twice >= 2 * (int64_t)D) continue;
          const uint64_t rest = (uint64_t)twice / 2;                                      // (A 2^k) mod D
          if (rest & ((1ull << twos) - 1)) continue;
          const uint64_t a0 = m > 1 ? (rest >> twos) % m * inverse % m : 0;
          for (uint64_t A = a0 + (lo > a0 ? (lo - a0 + m - 1) / m * m : 0); A < hi; A += m) {
            if ((A << k) % D != rest) { ++failed; return; }
            const float a = as_float(0x3F800000u | ((uint32_t)A & 0x7FFFFFu));
            const uint32_t want = as_bits(a / d);
            ++mine;
            for (int off = -1; off <= 1; ++off) {
              if (as_bits(fp8lm::short_quotient(a, d, as_float(nearest + off))) == want) continue;
              if (off == 0) { ++wrong_nearest; continue; }
              const long long at = wrong_off++;
              if (at < 64) wrong_d[at] = as_bits(d);
            }
          }
        }
      }
    }
    cases += mine;
  };
  std::vector<std::thread> pool;
  for (int t = 0; t < threads; ++t) pool.emplace_back(work, t);
  for (auto& t : pool) t.join();
  out[0] = cases;
  out[1] = wrong_nearest;
  out[2] = wrong_off;
  return failed ? -1 : 0;
}

// Two binades from 2^(exponent - 127) on, all 2^24 values.  out: short roots that differ from the correctly rounded one; reciprocal
// estimates more than one ulp from the nearest; how far the estimate of the last value but 0 and but 2 of either binade is off.
int roots_and_reciprocals(uint32_t exponent, int64_t* out) {
  if (exponent < 2 || exponent > 250) return -1;
  const uint32_t n = 1u << 24, base = exponent << 23;
  float *d_rcp = nullptr, *d_root = nullptr;
  if (hipMalloc((void**)&d_rcp, (size_t)n * 4) != hipSuccess) return -2;
  if (hipMalloc((void**)&d_root, (size_t)n * 4) != hipSuccess) { (void)hipFree(d_rcp); return -2; }
  hipLaunchKernelGGL(estimates_kernel, dim3(n / 256), dim3(256), 0, nullptr, base, d_rcp, d_root, n);
  std::vector<float> rcp(n), root(n);
  bool ok = hipGetLastError() == hipSuccess;
  ok = ok && hipMemcpy(rcp.data(), d_rcp, (size_t)n * 4, hipMemcpyDeviceToHost) == hipSuccess;
  ok = ok && hipMemcpy(root.data(), d_root, (size_t)n * 4, hipMemcpyDeviceToHost) == hipSuccess;
  (void)hipFree(d_rcp);
  (void)hipFree(d_root);
  if (!ok) return -3;
  out[0] = out[1] = 0;
  for (uint32_t i = 0; i < n; ++i) {
    const float x = as_float(base + i);
    out[0] += as_bits(root[i]) != as_bits(std::sqrt(x));
    const int64_t off = (int64_t)as_bits(rcp[i]) - (int64_t)as_bits(1.0f / x);
    out[1] += off > 1 || off < -1;
  }
  int64_t* at = out + 2;
  for (uint32_t binade = 0; binade < 2; ++binade)
    for (uint32_t s : {0x7FFFFFu, 0x7FFFFDu}) {
      const uint32_t i = (binade << 23) | s;
      *at++ = (int64_t)as_bits(rcp[i]) - (int64_t)as_bits(1.0f / as_float(base + i));
    }
  return 0;
}
}  // extern "C"
