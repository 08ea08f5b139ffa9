// Block mean-pooling of Q and K (the block summaries the routing score compares;
// Section 4.2.2 "block-wise similarity", Appendix A.2.2 "score-based routing").
//
// One workgroup per (tensor, b, h, block).  A token row is owned by 16 lanes (8
// when D = 64) of 8 columns each, so the rows of a block divide evenly among the
// workgroup at every D and all of a lane's 16-byte loads (S / 16 of them, or S /
// 32) are in flight before the first is used; rows past the end load the last
// one and add zeros.  Float64 partial sums meet in LDS, and D threads finish the
// mean over the block's valid tokens and round once to float32.  The kernel is
// bound by HBM reads: 2*S*D bytes in, 4*D bytes out per block.
//
// With D / 8 lanes per row and a loop whose trip count the loads waited on, 20 heads
// of 32,760 x 112 at S = 64 took 70.7 us (4.15 TB/s), now 52.7 (5.57); 24 heads of
// 75,600 x 64 98.0, now 86.4 (5.37); D = 128, whose rows divided evenly, 182.7 and
// 181.6 (32 heads of 63,240, 5.71 TB/s).
#include "sva_internal.h"

namespace sva {
namespace {

constexpr int kPoolThreads = 256;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

template <int D, int S>
__global__ __launch_bounds__(kPoolThreads) void pool_kernel(const uint16_t* __restrict__ q,
                                                            const uint16_t* __restrict__ k,
                                                            float* __restrict__ q_pool,
                                                            float* __restrict__ k_pool, int N,
                                                            int nB, int n_rows) {
  constexpr int TPR = (D == 64) ? 8 : 16;           // lanes per token row
  constexpr int RPP = kPoolThreads / TPR;           // rows per pass
  constexpr int NP = S / RPP;                       // loads per lane
  __shared__ double part[RPP][D];

  const int row = xcd_remap(blockIdx.x, n_rows);    // (b*H + h)*nB + i
  const uint16_t* src = blockIdx.y ? k : q;
  float* dst = blockIdx.y ? k_pool : q_pool;
  const int bh = row / nB;
  const int i = row - bh * nB;
  const int start = i * S;
  const int valid = min(S, N - start);
  const uint16_t* base = src + ((size_t)bh * N + start) * D;

  const int t = threadIdx.x;
  const int r0 = t / TPR;
  const int c = t % TPR;
  if (c < D / 8) {                                  // D = 112: lanes 14, 15 hold nothing
    uint4 w[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p)
      w[p] = *reinterpret_cast<const uint4*>(base + (size_t)min(r0 + p * RPP, valid - 1) * D + c * 8);
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (r0 + p * RPP >= valid) w[p] = make_uint4(0, 0, 0, 0);
      acc[0] += bf16_lo(w[p].x); acc[1] += bf16_hi(w[p].x);
      acc[2] += bf16_lo(w[p].y); acc[3] += bf16_hi(w[p].y);
      acc[4] += bf16_lo(w[p].z); acc[5] += bf16_hi(w[p].z);
      acc[6] += bf16_lo(w[p].w); acc[7] += bf16_hi(w[p].w);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) part[r0][c * 8 + e] = acc[e];
  }
  __syncthreads();
  if (t < D) {
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < RPP; ++r) s += part[r][t];
    dst[(size_t)row * D + t] = (float)(s / (double)valid);
  }
}

template <int D>
void launch_d(const Dims& d, const uint16_t* q, const uint16_t* k, float* q_pool, float* k_pool, hipStream_t stream) {
  const int n_rows = d.B * d.H * d.nB;
  if (d.S == 64)
    hipLaunchKernelGGL((pool_kernel<D, 64>), dim3(n_rows, 2), dim3(kPoolThreads), 0, stream, q, k, q_pool, k_pool, d.N,
                       d.nB, n_rows);
  else
    hipLaunchKernelGGL((pool_kernel<D, 128>), dim3(n_rows, 2), dim3(kPoolThreads), 0, stream, q, k, q_pool, k_pool, d.N,
                       d.nB, n_rows);
}

}  // namespace

hipError_t launch_pool(const Dims& d, const uint16_t* q, const uint16_t* k, float* q_pool,
                       float* k_pool, hipStream_t stream) {
  if (d.S != 64 && d.S != 128) return hipErrorInvalidValue;
  switch (d.D) {
    case 64: launch_d<64>(d, q, k, q_pool, k_pool, stream); break;
    case 112: launch_d<112>(d, q, k, q_pool, k_pool, stream); break;
    case 128: launch_d<128>(d, q, k, q_pool, k_pool, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace sva
