// How token selection divides the order keys of the scores into bins: between
// 64 sorted sample keys (the splitters), so that every interval holds about a
// 64th of the tokens whatever the scores look like.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace sva {

constexpr int kSamples = 64;
constexpr int kIntervals = kSamples + 1;
constexpr int kKeyBins = 4096;                            // at most

// The token whose key is sample i of n: one of the i-th 64th of the tokens, at a
// hashed place in it.  (The first of each 64th would be at 2 places of the frame
// for 32 frames, 4 for 16: a score that depends on the place then has splitters
// that say nothing about the others.)
__host__ __device__ __forceinline__ int sample_index(int i, int n) {
  const int64_t from = (int64_t)i * n >> 6, to = (int64_t)(i + 1) * n >> 6;
  const uint32_t hash = (uint32_t)(i + 1) * 2654435761u;  // 2^32 over the golden ratio
  return (int)(from + (int64_t)(((uint64_t)hash * (uint64_t)(to - from)) >> 32));
}

// Interval t of the splitters s[0..63], ascending: t = 0 the keys below s[0], else
// those from s[t - 1] up to the next splitter.  Its first key has a bin of its own (a
// score that many tokens share is a splitter).  The others are in per - 1 equal
// parts in the intervals from .. to, where the k-th largest key is expected, and
// in one part elsewhere.
struct KeyBins {
  const unsigned long long* s;
  int from, to, per;
};

// The number of samples below the k-th largest of n keys has mean 64 (1 - p), p =
// k / n, and standard deviation of at most 8 sqrt(p (1 - p)) where the hashed
// places have nothing to do with the scores; four of them on either side.
__host__ __device__ __forceinline__ KeyBins make_bins(const unsigned long long* s, int n, int k) {
  const float p = (float)k / (float)n;
  const float mid = 64.0f * (1.0f - p), margin = 32.0f * sqrtf(fmaxf(p * (1.0f - p), 0.0f)) + 1.0f;
  KeyBins b;
  b.s = s;
  b.from = (int)fmaxf(floorf(mid - margin), 0.0f);
  b.to = (int)fminf(ceilf(mid + margin), (float)kSamples);
  const int fine = b.to - b.from + 1;
  b.per = (kKeyBins - 2 * (kIntervals - fine)) / fine;
  return b;
}

struct KeyInterval {
  uint64_t lo, hi;                                        // inclusive
  int first;                                              // its first bin
  int shift;                                              // of the distance to lo + 1; -1: one part
};

__host__ __device__ __forceinline__ KeyInterval key_interval(const KeyBins& b, int t) {
  KeyInterval v;
  const int fine = t < b.from ? 0 : (t <= b.to ? t - b.from : b.to - b.from + 1);   // intervals before it in parts
  v.first = 2 * (t - fine) + fine * b.per;
  v.lo = t == 0 ? 0 : b.s[t - 1];
  v.hi = t == kSamples ? ~0ull : (b.s[t] == 0 ? 0 : b.s[t] - 1);
  if (t < b.from || t > b.to) {
    v.shift = -1;
    return v;
  }
  const uint64_t last = v.hi - v.lo > 1 ? v.hi - v.lo - 1 : 0;   // distance of the last key to lo + 1
  const int bits = last == 0 ? 0 : 64 - __builtin_clzll(last), want = 31 - __builtin_clz(b.per);
  v.shift = bits > want ? bits - want : 0;
  if (v.shift > 0 && (last >> (v.shift - 1)) <= (uint64_t)(b.per - 2)) --v.shift;
  if ((last >> v.shift) > (uint64_t)(b.per - 2)) ++v.shift;
  return v;
}

__host__ __device__ __forceinline__ int key_bin(const KeyBins& b, uint64_t key) {
  int t = 0;                                              // splitters <= key
#pragma unroll
  for (int step = kSamples / 2; step > 0; step >>= 1)
    if (b.s[t + step - 1] <= key) t += step;
  if (b.s[t] <= key) ++t;                                 // t <= 63 here
  const KeyInterval v = key_interval(b, t);
  const uint64_t d = key - v.lo;
  if (d == 0) return v.first;
  return v.first + 1 + (v.shift < 0 ? 0 : (int)((d - 1) >> v.shift));
}

// the keys of a bin: lo .. hi, inclusive
__host__ __device__ __forceinline__ void bin_range(const KeyBins& b, int bin, uint64_t& lo, uint64_t& hi) {
  const int fine = b.to - b.from + 1, in = bin - 2 * b.from;
  const int t = in < 0 ? bin / 2 : (in < fine * b.per ? b.from + in / b.per : b.to + 1 + (in - fine * b.per) / 2);
  const KeyInterval v = key_interval(b, t);
  const int part = bin - v.first;
  lo = hi = v.lo;
  if (part == 0) return;
  lo = v.lo + 1;
  hi = v.hi;
  if (v.shift < 0) return;
  lo += (uint64_t)(part - 1) << v.shift;
  const uint64_t rest = (1ull << v.shift) - 1;            // 2^64 is not crossed
  hi = v.hi - lo < rest ? v.hi : lo + rest;
}

}  // namespace sva
