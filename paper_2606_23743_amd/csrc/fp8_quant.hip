// fp8 (e4m3) quantisation of Q, K, V for 8-bit attention (Section 4.2.4
// points to 8-bit attention with outlier smoothing, the SageAttention series).
//
// Scales are powers of two 2^e (the MX e8m0 scales the gfx950 matrix
// instructions apply themselves): for a group with largest magnitude a, e is
// the smallest exponent with a <= 448 * 2^e, so x * 2^-e is exact in float32
// and the hardware conversion (round to nearest even) gives the code.
//   stats  the float64 channel sums of K over all N tokens (mean rounded once
//          to bf16: the smoothing vector) and the channel maxima of |V| (V's
//          per-channel exponents): segment partials, then a fixed-order sum.
//   Q, K   one workgroup per (tensor, b, h, block): Q is first multiplied by
//          the softmax scale in base 2 (float32), so the code product is the
//          logit in base-2 units; K subtracts the smoothing vector in float32;
//          the block's largest magnitude sets its exponent; codes are written
//          [B, H, Np, DP] (Np = nB * S, rows past N zero).
//   V      one workgroup per (b, h, block): codes with the channel exponents,
//          transposed through LDS into 64-key tiles [B, H, Np/64, DP, 64], the
//          layout the attention kernel stages directly.
// DP is D rounded up to a multiple of 64 (the fp8 matrix instructions take 64
// channels per step): at D = 112 the codes of channels 112..127 are zero and
// their V exponent is 0.
#include "sva_internal.h"

namespace sva {
namespace {

constexpr int kThreads = 256;
constexpr int kFinalThreads = 1024;
constexpr int kStatRows = 256;               // tokens per statistics workgroup

__device__ __forceinline__ float lo16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// smallest e in [-127, 127] with amax <= 448 * 2^e; 0 for amax = 0.
// 448 = 0.875 * 2^9 and amax = f * 2^x with f in [0.5, 1).
__device__ __forceinline__ int scale_exp(float amax) {
  if (!(amax > 0.0f)) return 0;
  int x;
  const float f = frexpf(amax, &x);
  const int e = f <= 0.875f ? x - 9 : x - 8;
  return e < -127 ? -127 : (e > 127 ? 127 : e);
}

// four float32 values -> four e4m3 codes (round to nearest even), packed
__device__ __forceinline__ uint32_t pack4_e4m3(float a, float b, float c, float d) {
  int w = 0;
  w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, w, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
  return (uint32_t)w;
}

typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

// Where the tensors exceed the caches (NT, see streams_past_caches) the
// quantiser's loads and stores are non-temporal: they then push no K or V that
// the statistics left in the memory-side cache out of it.
template <bool NT>
__device__ __forceinline__ uint4 load16(const uint16_t* p) {
  if constexpr (NT) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
  }
  return *reinterpret_cast<const uint4*>(p);
}
template <bool NT>
__device__ __forceinline__ void store8(uint8_t* p, uint2 o) {
  const u32x2 v = {o.x, o.y};
  if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<u32x2*>(p));
  else *reinterpret_cast<u32x2*>(p) = v;
}

// a float64 value rounded once to bf16 (nearest, ties to even), as bf16 bits
__device__ __forceinline__ uint16_t round_bf16_bits(double x) {
  if (x == 0.0) return (uint16_t)(__double_as_longlong(x) >> 48);
  int e;
  (void)frexp(x, &e);
  const int sh = e - 8 > -133 ? e - 8 : -133;          // spacing of bf16 values near x
  const double r = ldexp(rint(ldexp(x, -sh)), sh);     // exact: a bf16 value
  return (uint16_t)(__float_as_uint((float)r) >> 16);
}

// Channel statistics in two steps, so that every CU takes part: segment
// workgroups of kStatRows tokens write float64 partial sums of K and float32
// partial maxima of |V| per channel, then one workgroup per (b, h) adds them in
// a fixed order (deterministic).  The partials are staged in the head's K-code
// region, which the quantiser overwrites right after (it is at least
// 12 * nseg * DP bytes: Np >= 64 tokens of DP bytes each).
//
// Bound by reading K and V once.  A wave adds its rows in registers and lanes
// and the four waves meet in 6 KB of LDS, so that five workgroups share a CU
// (one of 1024 threads with 96 KB of LDS filled a CU before).  256 rows: 180.4 us
// for the whole quantiser at 20 heads of 32,760 x 112, 512 rows 182.4, 1024
// rows 184.
template <int D>
__global__ __launch_bounds__(kThreads) void fp8_stats_partial_kernel(Fp8QuantArgs a) {
  constexpr int DP = (D + 63) / 64 * 64;
  constexpr int TPR = DP / 8;                 // lanes per token row
  constexpr int RPP = kThreads / TPR;         // rows per pass
  constexpr int NW = kThreads / 64;
  __shared__ double part_s[NW][DP];
  __shared__ float part_m[NW][DP];
  const int seg = blockIdx.x, bh = blockIdx.y;
  const int nseg = gridDim.x;
  const int N = a.N;
  const int r0 = threadIdx.x / TPR, c = threadIdx.x % TPR;
  const bool live = c < D / 8;                // D = 112: lanes 14, 15 hold no channel
  const uint16_t* K = a.k + (size_t)bh * N * D;
  const uint16_t* V = a.v + (size_t)bh * N * D;
  const int n0 = seg * kStatRows, n1 = min(N, n0 + kStatRows);
  double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  float m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  auto add = [&](const uint4& kw, const uint4& vw) {
    const float kx[8] = {lo16(kw.x), hi16(kw.x), lo16(kw.y), hi16(kw.y), lo16(kw.z), hi16(kw.z), lo16(kw.w), hi16(kw.w)};
    const float vx[8] = {lo16(vw.x), hi16(vw.x), lo16(vw.y), hi16(vw.y), lo16(vw.z), hi16(vw.z), lo16(vw.w), hi16(vw.w)};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      s[e] += (double)kx[e];
      m[e] = fmaxf(m[e], fabsf(vx[e]));
    }
  };
  if (live) {
    constexpr int U = 4;                      // row pairs in flight per lane
    int r = n0 + r0;
    for (; r + (U - 1) * RPP < n1; r += U * RPP) {
      uint4 kw[U], vw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        kw[u] = *reinterpret_cast<const uint4*>(K + (size_t)(r + u * RPP) * D + c * 8);
        vw[u] = *reinterpret_cast<const uint4*>(V + (size_t)(r + u * RPP) * D + c * 8);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) add(kw[u], vw[u]);
    }
    for (; r < n1; r += RPP)
      add(*reinterpret_cast<const uint4*>(K + (size_t)r * D + c * 8),
          *reinterpret_cast<const uint4*>(V + (size_t)r * D + c * 8));
  }
  // the wave's rows: lanes with the same c, in pairs at distance TPR, 2 TPR, ..
#pragma unroll
  for (int off = TPR; off < 64; off <<= 1)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      s[e] += __shfl_xor(s[e], off, 64);
      m[e] = fmaxf(m[e], __shfl_xor(m[e], off, 64));
    }
  if ((threadIdx.x & 63) < TPR) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      part_s[threadIdx.x >> 6][c * 8 + e] = s[e];
      part_m[threadIdx.x >> 6][c * 8 + e] = m[e];
    }
  }
  __syncthreads();
  if (threadIdx.x < DP) {
    const int d = threadIdx.x;
    double t = 0.0;
    float mx = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {           // fixed order: deterministic
      t += part_s[w][d];
      mx = fmaxf(mx, part_m[w][d]);
    }
    unsigned char* scratch = a.k8 + (size_t)bh * a.Np * DP;
    reinterpret_cast<double*>(scratch)[(size_t)seg * DP + d] = t;
    reinterpret_cast<float*>(scratch + (size_t)nseg * DP * sizeof(double))[(size_t)seg * DP + d] = mx;
  }
}

// One workgroup per (b, h): kFinalThreads / DP runs of consecutive segments per
// channel side by side, then the runs in order.  Bound by latency (109 segments
// one after the other took 48 us).
template <int D>
__global__ __launch_bounds__(kFinalThreads) void fp8_stats_final_kernel(Fp8QuantArgs a, int nseg) {
  constexpr int DP = (D + 63) / 64 * 64;
  constexpr int NG = kFinalThreads / DP;
  __shared__ double run_s[NG][DP];
  __shared__ float run_m[NG][DP];
  const int bh = blockIdx.x, d = threadIdx.x % DP, g = threadIdx.x / DP;
  const unsigned char* scratch = a.k8 + (size_t)bh * a.Np * DP;
  const double* ps = reinterpret_cast<const double*>(scratch);
  const float* pm = reinterpret_cast<const float*>(scratch + (size_t)nseg * DP * sizeof(double));
  const int g0 = (int)((int64_t)nseg * g / NG), g1 = (int)((int64_t)nseg * (g + 1) / NG);
  double t = 0.0;
  float mx = 0.0f;
#pragma unroll 8
  for (int i = g0; i < g1; ++i) {            // segment order: deterministic
    t += ps[(size_t)i * DP + d];
    mx = fmaxf(mx, pm[(size_t)i * DP + d]);
  }
  run_s[g][d] = t;
  run_m[g][d] = mx;
  __syncthreads();
  if (g != 0) return;
  for (int i = 1; i < NG; ++i) {
    t += run_s[i][d];
    mx = fmaxf(mx, run_m[i][d]);
  }
  if (d < D) a.k_mean[(size_t)bh * D + d] = round_bf16_bits(t / (double)a.N);
  a.v_exp[(size_t)bh * DP + d] = scale_exp(mx);     // padding channels: 0
}

// Q or smoothed K of one block
template <int D, int S, bool NT>
__device__ __forceinline__ void quant_qk_block(const Fp8QuantArgs& a, int row, bool is_k, float* red) {
  constexpr int DP = (D + 63) / 64 * 64;
  constexpr int TPR = DP / 8;
  constexpr int RPP = kThreads / TPR;
  constexpr int NP = S / RPP;
  const int nB = a.nB, N = a.N, Np = a.Np;
  const int bh = row / nB;
  const int i = row - bh * nB;
  const int valid = min(S, N - i * S);
  const uint16_t* src = (is_k ? a.k : a.q) + ((size_t)bh * N + (size_t)i * S) * D;
  uint8_t* dst = (is_k ? a.k8 : a.q8) + ((size_t)bh * Np + (size_t)i * S) * DP;
  const int r0 = threadIdx.x / TPR, c = threadIdx.x % TPR;
  const bool live = c < D / 8;                // padding lanes write zero codes
  float sub[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const float mul = is_k ? 1.0f : a.q_mul;
  if (is_k && live) {
    const uint4 mw = *reinterpret_cast<const uint4*>(a.k_mean + (size_t)bh * D + c * 8);
    const float mv[8] = {lo16(mw.x), hi16(mw.x), lo16(mw.y), hi16(mw.y), lo16(mw.z), hi16(mw.z), lo16(mw.w), hi16(mw.w)};
#pragma unroll
    for (int e = 0; e < 8; ++e) sub[e] = mv[e];
  }
  float x[NP][8];
  float amax = 0.0f;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = r0 + p * RPP;
    uint4 w = make_uint4(0, 0, 0, 0);
    if (live && r < valid) w = load16<NT>(src + (size_t)r * D + c * 8);
    const float v[8] = {lo16(w.x), hi16(w.x), lo16(w.y), hi16(w.y), lo16(w.z), hi16(w.z), lo16(w.w), hi16(w.w)};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // K: float32 difference (sub is zero for Q); Q: float32 product (mul is 1 for K)
      x[p][e] = (live && r < valid) ? __builtin_fmaf(v[e], mul, -sub[e]) : 0.0f;
      amax = fmaxf(amax, fabsf(x[p][e]));
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = amax;
  __syncthreads();
  float bmax = red[0];
#pragma unroll
  for (int w = 1; w < kThreads / 64; ++w) bmax = fmaxf(bmax, red[w]);
  const int e = scale_exp(bmax);
  if (threadIdx.x == 0) (is_k ? a.k_exp : a.q_exp)[row] = e;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = r0 + p * RPP;
    uint2 o;
    o.x = pack4_e4m3(ldexpf(x[p][0], -e), ldexpf(x[p][1], -e), ldexpf(x[p][2], -e), ldexpf(x[p][3], -e));
    o.y = pack4_e4m3(ldexpf(x[p][4], -e), ldexpf(x[p][5], -e), ldexpf(x[p][6], -e), ldexpf(x[p][7], -e));
    store8<NT>(dst + (size_t)r * DP + c * 8, o);             // rows past N, padding: zeros
  }
}

// 4 x 4 bytes transposed: byte j of x[i] -> byte i of y[j]
__device__ __forceinline__ void transpose4(const uint32_t (&x)[4], uint32_t (&y)[4]) {
  const uint32_t ab_lo = __builtin_amdgcn_perm(x[1], x[0], 0x05010400), ab_hi = __builtin_amdgcn_perm(x[1], x[0], 0x07030602);
  const uint32_t cd_lo = __builtin_amdgcn_perm(x[3], x[2], 0x05010400), cd_hi = __builtin_amdgcn_perm(x[3], x[2], 0x07030602);
  y[0] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x05040100);
  y[1] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x07060302);
  y[2] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x05040100);
  y[3] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x07060302);
}

// V of one block, transposed into 64-key tiles.  Rows are coded as they are
// read (a lane keeps its 8 channels' exponents), and the transpose moves codes,
// four channels x eight tokens per thread: 4-byte LDS reads without conflicts
// (pitch DP + 4: eight token groups x eight channel groups on 64 banks) and
// whole 64-byte rows per store instruction.  Transposing the 16-bit inputs
// through 2-byte LDS reads, with stores 64 bytes apart, took 72 us for 20 heads
// of 32,760 x 112 (3.2 TB/s), and Q and K in a kernel of their own 72 us more;
// together they now take 100 us, 6.9 TB/s of reads and writes.
template <int D, int S, bool NT>
__device__ __forceinline__ void quant_v_block(const Fp8QuantArgs& a, int row, unsigned char* tile) {
  constexpr int DP = (D + 63) / 64 * 64;
  constexpr int TPR = DP / 8;
  constexpr int RPP = kThreads / TPR;
  constexpr int NP = S / RPP;
  constexpr int P = DP + 4;                   // tile row pitch, bytes
  const int nB = a.nB, N = a.N, Np = a.Np;
  const int bh = row / nB;
  const int i = row - bh * nB;
  const int valid = min(S, N - i * S);
  const uint16_t* src = a.v + ((size_t)bh * N + (size_t)i * S) * D;
  const int r0 = threadIdx.x / TPR, c = threadIdx.x % TPR;
  const bool live = c < D / 8;                // padding channels: zero codes
  uint4 w[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = r0 + p * RPP;
    w[p] = make_uint4(0, 0, 0, 0);
    if (live && r < valid) w[p] = load16<NT>(src + (size_t)r * D + c * 8);
  }
  int e[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) e[k] = a.v_exp[(size_t)bh * DP + c * 8 + k];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = r0 + p * RPP;
    uint32_t* o = reinterpret_cast<uint32_t*>(tile + r * P + c * 8);
    o[0] = pack4_e4m3(ldexpf(lo16(w[p].x), -e[0]), ldexpf(hi16(w[p].x), -e[1]), ldexpf(lo16(w[p].y), -e[2]),
                      ldexpf(hi16(w[p].y), -e[3]));
    o[1] = pack4_e4m3(ldexpf(lo16(w[p].z), -e[4]), ldexpf(hi16(w[p].z), -e[5]), ldexpf(lo16(w[p].w), -e[6]),
                      ldexpf(hi16(w[p].w), -e[7]));
  }
  __syncthreads();
  // item: tokens tok .. tok+7 of channels d .. d+3; eight consecutive threads
  // take the eight token groups of a 64-key tile
  uint8_t* dst = a.v8 + ((size_t)bh * (Np / 64) + (size_t)i * (S / 64)) * DP * 64;
  for (int u = threadIdx.x; u < DP / 4 * (S / 8); u += kThreads) {
    const int t8 = u % 8, d = u / 8 % (DP / 4) * 4, tt = u / (2 * DP);
    uint32_t lo[4], hi[4], x[4], y[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      lo[k] = *reinterpret_cast<const uint32_t*>(tile + (tt * 64 + t8 * 8 + k) * P + d);
      hi[k] = *reinterpret_cast<const uint32_t*>(tile + (tt * 64 + t8 * 8 + 4 + k) * P + d);
    }
    transpose4(lo, x);
    transpose4(hi, y);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      store8<NT>(dst + ((size_t)tt * DP + d + k) * 64 + t8 * 8, make_uint2(x[k], y[k]));
  }
}

// One workgroup per block of each tensor.  V and K blocks come first, in turns
// and from the last head back, so that what the statistics read last is read
// again while it is still in the 256 MB memory-side cache; then Q.
template <int D, int S, bool NT>
__global__ __launch_bounds__(kThreads) void fp8_quant_kernel(Fp8QuantArgs a) {
  constexpr int DP = (D + 63) / 64 * 64;
  __shared__ __attribute__((aligned(16))) unsigned char tile[S * (DP + 4)];
  __shared__ float red[kThreads / 64];
  const unsigned u = blockIdx.y * (unsigned)a.n_rows + blockIdx.x;
  if (u >= 2u * a.n_rows) quant_qk_block<D, S, NT>(a, u - 2u * a.n_rows, false, red);
  else if (u & 1) quant_qk_block<D, S, NT>(a, a.n_rows - 1 - (int)(u / 2), true, red);
  else quant_v_block<D, S, NT>(a, a.n_rows - 1 - (int)(u / 2), tile);
}

// By the bytes of K and V (whole quantiser, us, plain / non-temporal): 32 MB 34.0 /
// 35.4, 128 MB 81.2 / 73.3, 294 MB 181 / 160 (stores alone 164).
bool streams_past_caches(const Fp8QuantArgs& a, int BH, int D) { return (int64_t)BH * a.N * D * 4 >= (64 << 20); }

template <int D, int S>
void launch_quant_ds(const Fp8QuantArgs& a, int BH, hipStream_t stream) {
  const int nseg = (a.N + kStatRows - 1) / kStatRows;
  hipLaunchKernelGGL((fp8_stats_partial_kernel<D>), dim3(nseg, BH), dim3(kThreads), 0, stream, a);
  hipLaunchKernelGGL((fp8_stats_final_kernel<D>), dim3(BH), dim3(kFinalThreads), 0, stream, a, nseg);
  if (streams_past_caches(a, BH, D))
    hipLaunchKernelGGL((fp8_quant_kernel<D, S, true>), dim3(a.n_rows, 3), dim3(kThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((fp8_quant_kernel<D, S, false>), dim3(a.n_rows, 3), dim3(kThreads), 0, stream, a);
}

}  // namespace

hipError_t launch_quantize_fp8(const Dims& d, const Fp8QuantArgs& args, hipStream_t stream) {
  Fp8QuantArgs a = args;
  a.N = d.N;
  a.nB = d.nB;
  a.Np = d.nB * d.S;
  a.n_rows = d.B * d.H * d.nB;
  const int BH = d.B * d.H;
  switch (d.D * 1000 + d.S) {
    case 64064: launch_quant_ds<64, 64>(a, BH, stream); break;
    case 64128: launch_quant_ds<64, 128>(a, BH, stream); break;
    case 112064: launch_quant_ds<112, 64>(a, BH, stream); break;
    case 112128: launch_quant_ds<112, 128>(a, BH, stream); break;
    case 128064: launch_quant_ds<128, 64>(a, BH, stream); break;
    case 128128: launch_quant_ds<128, 128>(a, BH, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace sva
