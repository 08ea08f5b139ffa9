// feat_norm token pruning (Section 4.2.3 token pruning; Appendix A.2.2 keeps
// 50% of the video tokens by the feat_norm saliency score): token scores, the
// kept-token selection, and the gather / scatter around the pruned span.
//
//   score  s[b, n] = sum_c x[b, n, c]^2 in float64 (the products of bf16 values
//          are exact there); one wave per token, 16-byte loads.
//   select the k largest scores of each batch entry (ties to the lower token
//          index), listed in ascending order: two grid-wide passes over the
//          scores' order keys find the k-th largest key, then a write pass over
//          token segments emits kept_idx (ascending) and kept_pos (the position
//          of each kept token, -1 for the others).
//   gather x_kept[b, j] = x[b, kept_idx[b, j]]; scatter out[b, n] = y_kept[b,
//          kept_pos[b, n]] for kept tokens and base[b, n] for the others.  One
//          wave per row, 16-byte loads and stores.
#include <mutex>

#include "sva_internal.h"
#include "token_bins.h"

namespace sva {
namespace {

__device__ __forceinline__ float lo16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ uint64_t order_key(double s) {
  if (s == 0.0) s = 0.0;           // -0 and +0 compare equal: give them one key
  const uint64_t b = (uint64_t)__double_as_longlong(s);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// ---- selection of the k-th largest order key, grid-wide ----
//
// Two passes over the scores instead of one per digit, because what such a pass
// costs is not its reads (0.5 MB at 63,240 tokens) but its launch and the
// hand-off to the last workgroup, 11-12 us together:
//   bins     64 sampled keys, sorted, are the splitters of 4096 bins (token_bins.h);
//            every key is counted in its bin (an LDS histogram per workgroup,
//            flushed to the batch entry's); the last workgroup to finish (a ticket
//            counter, no waiting) picks the bin of the k-th largest key.
//   resolve  per token segment: the keys above that bin and in it, the latter
//            also listed (a few dozen of 63,240 tokens); the last workgroup
//            finds the threshold among them and turns the counts into output
//            offsets and tie quotas.
// A bin of one repeated key is its threshold as it stands.  One of more than kCand
// different keys, which takes very many tokens whose scores crowd inside one
// 64th of them, is left to a radix select over all keys by the last workgroup
// alone.  Then the write pass emits kept_idx and kept_pos in token order.
// Splitters, not equal bins over a bracket around the sampled k-th key: where
// that bracket missed, or reached from rows of zeros to the scores of the others,
// most keys fell into one bin.  63,240 tokens x 512, select in us, six digit passes
// and a counting pass / bracket / splitters: 70 / 49 / 52 with random scores, 61 /
// 224 / 50 with 30% zero rows, 66 / 193 / 46 for 32 frames of 30 x 52 with scores by
// place (scores included, 14 us).

constexpr int kDigitBits = 12;
constexpr int kBins = 1 << kDigitBits;
constexpr int kCand = kBins;                     // listed keys, in the histogram's place
constexpr int kRank = 512;                       // of which this many are ranked against each other
constexpr int kSegThreads = 512;
constexpr int kMaxSegs = 1024;
// tokens per segment (one workgroup each): fewer, larger segments cut the
// per-workgroup cost of the cross-workgroup hand-off (a release fence and a
// ticket atomic); 2048 measured fastest at 111600 tokens
constexpr int kSegTokens = 2048;

struct SelState {                // per batch entry, at the head of its workspace slice
  unsigned long long threshold;  // the k-th largest key
  unsigned long long lo, hi;     // its bin, inclusive
  unsigned long long kmin, kmax; // smallest and largest key in the bin
  unsigned int cand;             // keys in the bin
  unsigned int ticket;           // workgroups finished in the current pass
  int need_eq;                   // keys equal to the threshold that are kept
};

static_assert(sizeof(SelState) + sizeof(uint32_t) * kBins + 4 * sizeof(int) * kMaxSegs <=
                  kTokenSelectWsStride, "workspace slice per batch entry");

struct SelWs {
  SelState* st;
  uint32_t* hist;            // [kBins], then the token indices of the bin's keys
  int* gt;                   // [kMaxSegs] per segment: keys above the threshold
  int* eq;                   // [kMaxSegs] per segment: keys equal to it
  int* kept_before;          // [kMaxSegs] exclusive offsets into kept_idx
  int* eq_before;            // [kMaxSegs] equal keys in earlier segments
};

__device__ __forceinline__ SelWs sel_ws(unsigned char* ws, int b) {
  unsigned char* p = ws + (size_t)b * kTokenSelectWsStride;
  SelWs w;
  w.st = reinterpret_cast<SelState*>(p);
  w.hist = reinterpret_cast<uint32_t*>(p + sizeof(SelState));
  w.gt = reinterpret_cast<int*>(w.hist + kBins);
  w.eq = w.gt + kMaxSegs;
  w.kept_before = w.eq + kMaxSegs;
  w.eq_before = w.kept_before + kMaxSegs;
  return w;
}

// workgroup-wide exclusive prefix sum (and the total) of one value per thread;
// every thread calls it
__device__ int block_scan(int v, int* red, int& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(incl, off, 64);
    if (lane >= off) incl += o;
  }
  if (lane == 63) red[w] = incl;
  __syncthreads();
  int before = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kSegThreads / 64; ++i) {
    const int r = red[i];
    before += i < w ? r : 0;
    tot += r;
  }
  __syncthreads();
  total = tot;
  return before + incl - v;
}

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

// Sixteen bytes, non-temporal (NT) where the tensor is too large for the caches to
// keep anything of it for the next reader: such traffic then leaves in the 256 MB
// memory-side cache what a later kernel does read again.
template <bool NT>
__device__ __forceinline__ u32x4 load16(const uint16_t* p) {
  if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return *reinterpret_cast<const u32x4*>(p);
}
template <bool NT>
__device__ __forceinline__ void store16(uint16_t* p, u32x4 v) {
  if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
  else *reinterpret_cast<u32x4*>(p) = v;
}

// scores: one wave per token, four 16-byte loads in flight per lane; blocks below
// B also initialise the selection state
__global__ __launch_bounds__(256) void token_score_kernel(const uint16_t* __restrict__ x,
                                                          double* __restrict__ scores,
                                                          unsigned char* __restrict__ ws, int B,
                                                          int rows, int C) {
  if (blockIdx.x < (unsigned)B) {
    const SelWs w = sel_ws(ws, blockIdx.x);
    for (int i = threadIdx.x; i < kBins; i += 256) w.hist[i] = 0;
    if (threadIdx.x == 0) {
      w.st->kmin = ~0ull;
      w.st->kmax = 0;
      w.st->cand = 0;
      w.st->ticket = 0;
    }
  }
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const uint16_t* p = x + (size_t)row * C;
  double acc = 0.0;
  auto add = [&](u32x4 q) {
    const float v[8] = {lo16(q[0]), hi16(q[0]), lo16(q[1]), hi16(q[1]), lo16(q[2]), hi16(q[2]), lo16(q[3]), hi16(q[3])};
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fma((double)v[e], (double)v[e], acc);
  };
  int c = lane * 8;
  for (; c + 3 * 512 < C; c += 4 * 512) {
    u32x4 q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u] = load16<false>(p + c + u * 512);
#pragma unroll
    for (int u = 0; u < 4; ++u) add(q[u]);
  }
  for (; c < C; c += 512) add(load16<false>(p + c));
  acc = wave_sum(acc);
  if (lane == 0) scores[row] = acc;
}

// true in the one workgroup that finishes the pass last (all threads call it)
__device__ bool last_to_finish(unsigned int* ticket, int* flag) {
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) *flag = atomicAdd(ticket, 1u) == gridDim.x - 1;
  __syncthreads();
  const bool last = *flag;
  if (last) __threadfence();
  return last;
}

// the splitters: n keys' 64 samples in ascending order, by one wave
__device__ void sort_samples(const double* s, int n, unsigned long long* sorted) {
  const int lane = threadIdx.x & 63;
  const uint64_t key = order_key(s[sample_index(lane, n)]);
  int pos = 0;
#pragma unroll 8
  for (int j = 0; j < 64; ++j) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)key, j), hi = __builtin_amdgcn_readlane((uint32_t)(key >> 32), j);
    const uint64_t o = (uint64_t)hi << 32 | lo;
    pos += (o < key || (o == key && j < lane)) ? 1 : 0;
  }
  sorted[pos] = key;
}

// the bin (from the top) that holds the need-th largest of the counted keys: pick
// = {bin, keys above it, keys in it}, or bin -1.  Every thread passes its own
// kBins / kSegThreads counts, in bin order.
__device__ void pick_bin(const uint32_t (&mine)[kBins / kSegThreads], int need, int* red, int (&pick)[3]) {
  constexpr int BPT = kBins / kSegThreads;
  int sum = 0;
#pragma unroll
  for (int e = 0; e < BPT; ++e) sum += (int)mine[e];
  if (threadIdx.x == 0) pick[0] = -1;
  int total;
  const int excl = block_scan(sum, red, total);             // (two barriers)
  int above = total - excl - sum;                           // keys in higher bins
#pragma unroll
  for (int e = BPT - 1; e >= 0; --e) {
    const int c = (int)mine[e];
    if (above < need && need <= above + c) {
      pick[0] = threadIdx.x * BPT + e;
      pick[1] = above;
      pick[2] = c;
    }
    above += c;
  }
  __syncthreads();
}

// grid (segments, B)
__global__ __launch_bounds__(kSegThreads) void token_bins_kernel(const double* __restrict__ scores,
                                                                 unsigned char* __restrict__ ws,
                                                                 int N, int seg_len, int k) {
  __shared__ uint32_t h[kBins];
  __shared__ unsigned long long splitters[kSamples];
  __shared__ int red[kSegThreads / 64];
  __shared__ int flag;
  __shared__ int pick[3];
  static_assert(kKeyBins <= kBins, "bins");
  const int b = blockIdx.y;
  const SelWs w = sel_ws(ws, b);
  for (int i = threadIdx.x; i < kBins; i += kSegThreads) h[i] = 0;
  const double* s = scores + (size_t)b * N;
  if (threadIdx.x < 64) sort_samples(s, N, splitters);
  __syncthreads();
  const KeyBins bins = make_bins(splitters, N, k);
  const int n0 = blockIdx.x * seg_len, n1 = min(N, n0 + seg_len);
  for (int n = n0 + threadIdx.x; n < n1; n += kSegThreads) atomicAdd(&h[key_bin(bins, order_key(s[n]))], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < kBins; i += kSegThreads)
    if (h[i]) atomicAdd(&w.hist[i], h[i]);
  if (!last_to_finish(&w.st->ticket, &flag)) return;

  constexpr int BPT = kBins / kSegThreads;                  // bins per thread
  uint32_t mine[BPT];
#pragma unroll
  for (int e = 0; e < BPT; ++e)
    mine[e] = __hip_atomic_load(&w.hist[threadIdx.x * BPT + e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  pick_bin(mine, k, red, pick);
  if (threadIdx.x == 0) {
    uint64_t lo, hi;
    bin_range(bins, pick[0], lo, hi);                       // every key was counted: a bin holds the k-th
    w.st->lo = lo;
    w.st->hi = hi;
    w.st->ticket = 0;
  }
}

// The need-th largest of the keys in [lo, hi] among key_at(0 .. count-1), by one
// workgroup: digits of 12 bits from the highest in which lo and hi differ.
template <class KeyAt>
__device__ uint64_t radix_pick(int count, KeyAt key_at, uint64_t lo, uint64_t hi, int need, uint32_t* h, int* red,
                               int (&pick)[3]) {
  int top = lo == hi ? 0 : 64 - __builtin_clzll(lo ^ hi);   // bits below `top` are open
  uint64_t prefix = lo;
  while (top > 0) {
    const int width = min(kDigitBits, top), low = top - width;
    for (int i = threadIdx.x; i < kBins; i += kSegThreads) h[i] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < count; i += kSegThreads) {
      const uint64_t key = key_at(i);
      if (key >= lo && key <= hi && (top == 64 || (key >> top) == (prefix >> top)))
        atomicAdd(&h[(key >> low) & ((1ull << width) - 1)], 1u);
    }
    __syncthreads();
    constexpr int BPT = kBins / kSegThreads;
    uint32_t mine[BPT];
#pragma unroll
    for (int e = 0; e < BPT; ++e) mine[e] = h[threadIdx.x * BPT + e];
    pick_bin(mine, need, red, pick);
    prefix = (((prefix >> low) & ~((1ull << width) - 1)) | (uint64_t)pick[0]) << low;
    need -= pick[1];
    top = low;
    __syncthreads();                                        // pick and h are reused
  }
  return prefix;
}

// grid (segments, B)
__global__ __launch_bounds__(kSegThreads) void token_resolve_kernel(const double* __restrict__ scores,
                                                                    unsigned char* __restrict__ ws,
                                                                    int N, int seg_len, int k) {
  __shared__ uint32_t h[kBins];                             // also: the candidates' keys
  __shared__ int red[kSegThreads / 64];
  __shared__ int flag;
  __shared__ int pick[3];
  __shared__ unsigned long long thr, mm[2];
  __shared__ int seg_gt[kMaxSegs], seg_eq[kMaxSegs];
  const int b = blockIdx.y, lane = threadIdx.x & 63;
  const SelWs w = sel_ws(ws, b);
  const uint64_t lo = w.st->lo, hi = w.st->hi;
  int* list = reinterpret_cast<int*>(w.hist);
  const double* s = scores + (size_t)b * N;
  const int n0 = blockIdx.x * seg_len, n1 = min(N, n0 + seg_len);
  if (threadIdx.x == 0) {
    mm[0] = ~0ull;
    mm[1] = 0;
  }
  __syncthreads();
  int gt = 0, in = 0;
  uint64_t kmin = ~0ull, kmax = 0;
  for (int base = n0; base < n1; base += kSegThreads) {     // uniform trip count
    const int n = base + threadIdx.x;
    const uint64_t key = n < n1 ? order_key(s[n]) : 0;
    const bool here = n < n1 && key >= lo && key <= hi;
    gt += n < n1 && key > hi ? 1 : 0;
    const uint64_t m = __builtin_amdgcn_ballot_w64(here);
    if (m != 0) {                                           // one atomic per wave
      unsigned at = 0;
      if (lane == 0) at = atomicAdd(&w.st->cand, (unsigned)__builtin_popcountll(m));
      at = __builtin_amdgcn_readfirstlane(at) + (unsigned)__builtin_popcountll(m & ((1ull << lane) - 1));
      if (here) {
        ++in;
        kmin = min(kmin, key);
        kmax = max(kmax, key);
        if (at < kCand) list[at] = n;
      }
    }
  }
  int tg, ti;
  block_scan(gt, red, tg);
  block_scan(in, red, ti);
  if (in != 0) {
    atomicMin(&mm[0], (unsigned long long)kmin);
    atomicMax(&mm[1], (unsigned long long)kmax);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    w.gt[blockIdx.x] = tg;
    w.eq[blockIdx.x] = ti;
    if (ti != 0) {
      atomicMin(&w.st->kmin, mm[0]);
      atomicMax(&w.st->kmax, mm[1]);
    }
  }
  if (!last_to_finish(&w.st->ticket, &flag)) return;

  const int nseg = gridDim.x;
  constexpr int SPT = kMaxSegs / kSegThreads;               // segments per thread
  int g[SPT], e[SPT], sg = 0, se = 0;
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    const int sgi = threadIdx.x * SPT + i;
    g[i] = sgi < nseg ? __hip_atomic_load(&w.gt[sgi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    e[i] = sgi < nseg ? __hip_atomic_load(&w.eq[sgi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    seg_gt[sgi] = seg_eq[sgi] = 0;
    sg += g[i];
  }
  int all_gt;
  block_scan(sg, red, all_gt);
  const int count = (int)__hip_atomic_load(&w.st->cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t first = __hip_atomic_load(&w.st->kmin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t last = __hip_atomic_load(&w.st->kmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int need = k - all_gt;                              // 1 .. count
  auto cand_at = [&](int i) { return __hip_atomic_load(&list[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  uint64_t T;
  if (first == last) {                                      // one key, however often: counts as they stand
    T = first;
  } else if (count <= kCand) {
    if (count <= kRank) {
      uint64_t* keys = reinterpret_cast<uint64_t*>(h);
      uint64_t key = 0;
      if ((int)threadIdx.x < count) keys[threadIdx.x] = key = order_key(s[cand_at(threadIdx.x)]);
      __syncthreads();
      if ((int)threadIdx.x < count) {
        int n_gt = 0, n_ge = 0;
        for (int i = 0; i < count; ++i) {
          n_gt += keys[i] > key ? 1 : 0;
          n_ge += keys[i] >= key ? 1 : 0;
        }
        if (n_gt < need && need <= n_ge) thr = key;         // equal keys write the same value
      }
      __syncthreads();
      T = thr;
    } else {
      T = radix_pick(count, [&](int i) { return order_key(s[cand_at(i)]); }, first, last, need, h, red, pick);
    }
    for (int i = threadIdx.x; i < count; i += kSegThreads) {
      const int n = cand_at(i);
      const uint64_t key = order_key(s[n]);
      if (key > T) atomicAdd(&seg_gt[n / seg_len], 1);
      if (key == T) atomicAdd(&seg_eq[n / seg_len], 1);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      g[i] += seg_gt[threadIdx.x * SPT + i];
      e[i] = seg_eq[threadIdx.x * SPT + i];
    }
  } else {
    T = radix_pick(N, [&](int i) { return order_key(s[i]); }, first, last, need, h, red, pick);
    for (int sgi = threadIdx.x >> 6; sgi < nseg; sgi += kSegThreads / 64) {
      int n_gt = 0, n_eq = 0;
      const int end = min(N, (sgi + 1) * seg_len);
      for (int n = sgi * seg_len + lane; n < end; n += 64) {
        const uint64_t key = order_key(s[n]);
        n_gt += key > T ? 1 : 0;
        n_eq += key == T ? 1 : 0;
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        n_gt += __shfl_xor(n_gt, off, 64);
        n_eq += __shfl_xor(n_eq, off, 64);
      }
      if (lane == 0) {
        seg_gt[sgi] = n_gt;
        seg_eq[sgi] = n_eq;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      g[i] = seg_gt[threadIdx.x * SPT + i];
      e[i] = seg_eq[threadIdx.x * SPT + i];
    }
  }
  sg = 0;
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    sg += g[i];
    se += e[i];
  }
  int all_eq;
  block_scan(sg, red, all_gt);
  int eb = block_scan(se, red, all_eq);
  const int need_eq = k - all_gt;                           // equal keys kept, lowest index first
  int take[SPT], st = 0;
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    take[i] = max(0, min(e[i], need_eq - eb));
    eb += e[i];
    st += g[i] + take[i];
  }
  int unused;
  int kb = block_scan(st, red, unused);
  eb -= se;
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    const int sgi = threadIdx.x * SPT + i;
    if (sgi < nseg) {
      w.kept_before[sgi] = kb;
      w.eq_before[sgi] = eb;
    }
    kb += g[i] + take[i];
    eb += e[i];
  }
  if (threadIdx.x == 0) {
    w.st->threshold = T;
    w.st->need_eq = need_eq;
  }
}

// kept_idx (ascending) and kept_pos, segment by segment in token order.  grid (segments, B)
__global__ __launch_bounds__(kSegThreads) void token_write_kernel(const double* __restrict__ scores,
                                                                  const unsigned char* __restrict__ ws,
                                                                  int32_t* __restrict__ kept_idx,
                                                                  int32_t* __restrict__ kept_pos,
                                                                  int N, int seg_len, int k) {
  __shared__ int red[kSegThreads / 64];
  const int b = blockIdx.y;
  const SelWs w = sel_ws(const_cast<unsigned char*>(ws), b);
  const uint64_t T = w.st->threshold;
  const int need_eq = w.st->need_eq;
  int pos = w.kept_before[blockIdx.x], ties = w.eq_before[blockIdx.x];
  const double* s = scores + (size_t)b * N;
  const int n0 = blockIdx.x * seg_len, n1 = min(N, n0 + seg_len);
  for (int base = n0; base < n1; base += kSegThreads) {      // uniform trip count
    const int n = base + threadIdx.x;
    uint64_t key = 0;
    if (n < n1) key = order_key(s[n]);
    const bool in = n < n1;
    const int is_eq = (in && key == T) ? 1 : 0;
    int n_eq;
    const int eq_rank = ties + block_scan(is_eq, red, n_eq);
    const int kp = (in && (key > T || (is_eq && eq_rank < need_eq))) ? 1 : 0;
    int n_kp;
    const int p = pos + block_scan(kp, red, n_kp);
    if (in) {
      if (kp && p < k) kept_idx[(size_t)b * k + p] = n;
      kept_pos[(size_t)b * N + n] = (kp && p < k) ? p : -1;
    }
    ties += n_eq;
    pos += n_kp;
  }
}

// one row by one wave, four loads in flight per lane
template <bool NT>
__device__ __forceinline__ void copy_row(uint16_t* dst, const uint16_t* src, int C, int lane) {
  int c = lane * 8;
  for (; c + 3 * 512 < C; c += 4 * 512) {
    u32x4 q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u] = load16<NT>(src + c + u * 512);
#pragma unroll
    for (int u = 0; u < 4; ++u) store16<NT>(dst + c + u * 512, q[u]);
  }
  for (; c < C; c += 512) store16<NT>(dst + c, load16<NT>(src + c));
}

// x_kept[b, j] = x[b, kept_idx[b, j]]; one wave per kept row
template <bool NT>
__global__ __launch_bounds__(256) void token_gather_kernel(const uint16_t* __restrict__ x,
                                                           const int32_t* __restrict__ kept_idx,
                                                           uint16_t* __restrict__ x_kept, int B,
                                                           int N, int C, int k) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);   // b * k + j
  if (row >= B * k) return;
  const int b = row / k;
  const int n = kept_idx[row];
  uint16_t* dst = x_kept + (size_t)row * C;
  if (n < 0 || n >= N) {                     // not a token of this entry: zeros
    for (int c = lane * 8; c < C; c += 512) *reinterpret_cast<uint4*>(dst + c) = make_uint4(0, 0, 0, 0);
    return;
  }
  const uint16_t* src = x + ((size_t)b * N + n) * C;
  copy_row<NT>(dst, src, C, lane);
}

// out[b, n] = y_kept[b, kept_pos[b, n]] if kept, else base[b, n]; one wave per row
template <bool NT>
__global__ __launch_bounds__(256) void token_scatter_kernel(const uint16_t* __restrict__ y_kept,
                                                            const int32_t* __restrict__ kept_pos,
                                                            const uint16_t* __restrict__ base,
                                                            uint16_t* __restrict__ out, int B,
                                                            int N, int C, int k) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);   // b * N + n
  if (row >= B * N) return;
  const int b = row / N;
  const int pos = kept_pos[row];
  const uint16_t* src = (pos >= 0 && pos < k) ? y_kept + ((size_t)b * k + pos) * C : base + (size_t)row * C;
  uint16_t* dst = out + (size_t)row * C;
  copy_row<NT>(dst, src, C, lane);
}

// Gather and scatter of tensors past the caches stream (select, gather and scatter
// together, us, plain / streaming): 33 MB 52.1 / 53.0, 131 MB 127.8 / 111.6,
// 518 MB 423 / 354, 1.2 GB 960 / 840.  The scores' reads
// do not: gather and scatter find the end of x in the cache (518 MB 356 / 372, 1.03
// GB 704 / 721).
bool streams_past_caches(int B, int N, int C) { return (int64_t)B * N * C * 2 >= (64 << 20); }

}  // namespace

int token_select_segments(int N) {
  const int nseg = (N + kSegTokens - 1) / kSegTokens;
  return nseg < kMaxSegs ? nseg : kMaxSegs;
}

hipError_t launch_token_select(int B, int N, int C, int k, const uint16_t* x, double* scores,
                               int32_t* kept_idx, int32_t* kept_pos, void* workspace,
                               hipStream_t stream) {
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  const int rows = B * N;
  const int grid = max((rows + 3) / 4, B);
  hipLaunchKernelGGL(token_score_kernel, dim3(grid), dim3(256), 0, stream, x, scores, ws, B, rows, C);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nseg = token_select_segments(N);
  const int seg_len = (N + nseg - 1) / nseg;
  hipLaunchKernelGGL(token_bins_kernel, dim3(nseg, B), dim3(kSegThreads), 0, stream, scores, ws, N, seg_len, k);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(token_resolve_kernel, dim3(nseg, B), dim3(kSegThreads), 0, stream, scores, ws, N, seg_len, k);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(token_write_kernel, dim3(nseg, B), dim3(kSegThreads), 0, stream, scores, ws,
                     kept_idx, kept_pos, N, seg_len, k);
  return hipGetLastError();
}

// Workspace of the allocation-free token selection (sva_token_select_noalloc):
// kTokenSelectStaticBatch slices.  Each GPU the library runs on holds its own
// copy until the process ends; host code never passes the array's name to a
// kernel (in host code it is a stand-in, not a device address), only the
// per-device address hipGetSymbolAddress returns.
static __device__ __align__(256) unsigned char scratch[kTokenSelectStaticBatch * kTokenSelectWsStride];

hipError_t token_select_scratch(hipStream_t stream, void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = stream ? hipStreamGetDevice(stream, &dev) : hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    // once per device, with that device current
    int cur = 0;
    if ((e = hipGetDevice(&cur)) != hipSuccess) return e;
    if (cur != dev && (e = hipSetDevice(dev)) != hipSuccess) return e;
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    const hipError_t back = cur != dev ? hipSetDevice(cur) : hipSuccess;
    if (e != hipSuccess) return e;
    if (back != hipSuccess) return back;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t launch_token_gather(int B, int N, int C, int k, const uint16_t* x, const int32_t* kept_idx,
                               uint16_t* x_kept, hipStream_t stream) {
  const int rows = B * k;
  if (streams_past_caches(B, N, C))
    hipLaunchKernelGGL(token_gather_kernel<true>, dim3((rows + 3) / 4), dim3(256), 0, stream, x, kept_idx,
                     x_kept, B, N, C, k);
  else
    hipLaunchKernelGGL(token_gather_kernel<false>, dim3((rows + 3) / 4), dim3(256), 0, stream, x, kept_idx,
                     x_kept, B, N, C, k);
  return hipGetLastError();
}

hipError_t launch_token_scatter(int B, int N, int C, int k, const uint16_t* y_kept,
                                const int32_t* kept_pos, const uint16_t* base, uint16_t* out,
                                hipStream_t stream) {
  const int rows = B * N;
  if (streams_past_caches(B, N, C))
    hipLaunchKernelGGL(token_scatter_kernel<true>, dim3((rows + 3) / 4), dim3(256), 0, stream, y_kept,
                     kept_pos, base, out, B, N, C, k);
  else
    hipLaunchKernelGGL(token_scatter_kernel<false>, dim3((rows + 3) / 4), dim3(256), 0, stream, y_kept,
                     kept_pos, base, out, B, N, C, k);
  return hipGetLastError();
}

}  // namespace sva
