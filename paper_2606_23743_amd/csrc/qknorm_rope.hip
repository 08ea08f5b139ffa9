// Fused QK RMSNorm + 3-D RoPE + block pooling: the producer of the Q and K the
// sparse path consumes, with the block summaries of Section 4.2.2 taken in the
// same pass (Section 4.2.5 names "fused RoPE + norm"; Appendix A.2.2 lists
// fused QKNorm+RoPE in the LTX-2.3 stack).
//
// Per token (head dimension D):
//   y = x / sqrt(mean(x^2) + eps) * gamma
//   pair p = (y[2p], y[2p+1]) turns by pos_a * base^(-i/n_a), where the D/2
//   pairs form contiguous groups for the t, y, x axes (n_y = n_x = D/6 rounded
//   down, n_t the rest), i is the pair's index in its group and pos_a the
//   token's coordinate on that axis (t-major raster order)
//   the result is rounded once to bf16 and written; the block summary is the
//   mean of the rounded outputs over the block's valid tokens.
//
// One workgroup per (tensor, b, h, block), or per block of both (below).  A token row is owned by TPR lanes
// (16, or 8 when D = 64), each holding 8 consecutive elements (4 pairs): one
// 16-byte load, the sum of squares reduced over the row's lanes, the pair
// rotations, one 16-byte store.  A rotation angle is formed and reduced
// modulo one turn in float64 (integer position times a float64 frequency),
// then the hardware sine and cosine (which take turns) give it in float32
// within 3e-7.  A pair's angle depends on one coordinate
// only, so the workgroup first tabulates (cos, sin) in LDS for the t, y and x
// values its block covers (about 1.8k entries for a 45 x 80 frame), and the
// token loop reads them; a block whose ranges would overflow the table takes
// its angles directly.  Block sums of the rounded outputs are
// kept in float64 (exact for bf16 values), so the summaries equal those the
// pooling kernel would compute from the written tensors.  The kernel is bound
// by HBM (2*S*D bytes read and written per tensor and block) and, next to it, by
// its vector instructions: with lane moves for the row sums, the hardware's
// reciprocal root, one table offset per token and axis and no waits between the
// rows, 32 heads of 63,240 x 128 take 353 us instead of 468 (5.9 TB/s instead of
// 4.4), 48 of 111,600 x 128 0.90-0.94 ms instead of 1.08 (5.9-6.1 TB/s instead of
// 5.1; the first twenty calls after a pause 1.02-1.11 on average).
#include <type_traits>

#include "sva_internal.h"

namespace sva {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ float lo16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

typedef __attribute__((ext_vector_type(2))) float float2v;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

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

// the sum over a token row's TPR lanes, in each of them (DPP lane moves)
template <int TPR>
__device__ __forceinline__ float row_sum(float x) {
  auto add = [&](auto ctrl) {
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  if constexpr (TPR == 16) {                   // rotations of the 16 lanes by 8, 4, 2, 1
    add(std::integral_constant<int, 0x128>{});
    add(std::integral_constant<int, 0x124>{});
    add(std::integral_constant<int, 0x122>{});
    add(std::integral_constant<int, 0x121>{});
  } else {                                     // pairs, quads, then the mirrored eight lanes
    static_assert(TPR == 8, "eight or sixteen lanes");
    add(std::integral_constant<int, 0xB1>{});
    add(std::integral_constant<int, 0x4E>{});
    add(std::integral_constant<int, 0x141>{});
  }
  return x;
}

// ss / D: a product where D is a power of two, else with the quotient's residual
// (a sum that overflowed has none and stays infinite: its row becomes zero)
template <int D>
__device__ __forceinline__ float mean_of(float ss) {
  constexpr float r = 1.0f / (float)D;
  const float q = ss * r;
  if constexpr ((D & (D - 1)) == 0) return q;
  return q < INFINITY ? fmaf(fmaf(-(float)D, q, ss), r, q) : q;
}

// 1 / sqrt(a), the hardware's (1 ulp); it may not take subnormal a
__device__ __forceinline__ float inv_root(float a) {
  return a < 0x1p-100f ? 1.0f / sqrtf(a) : __builtin_amdgcn_rsqf(a);
}

// NX tensors per workgroup: Q and K one after the other on one table, or one of them
template <int D, int S, int NX, bool NT>
__global__ __launch_bounds__(kThreads) void qknorm_rope_pool_kernel(RopeArgs a) {
  constexpr int TPR = (D == 64) ? 8 : 16;     // lanes per token row
  constexpr int NCH = D / 8;                  // chunks of 8 elements holding data
  constexpr int RPP = kThreads / TPR;         // token rows per pass
  constexpr int NP = S / RPP;                 // passes: rows each lane handles
  constexpr int NYX = D / 6;                  // rotation pairs of the y and of the x axis
  constexpr int NTA = D / 2 - 2 * NYX;         // rotation pairs of the t axis
  constexpr int kTab = 3072;                  // (cos, sin) entries of the per-block table
  static_assert(RPP * D * sizeof(double) <= kTab * sizeof(float2), "partial sums fit the table");
  // the (cos, sin) table during the token loop, the partial block sums after it
  __shared__ __attribute__((aligned(16))) unsigned char shared_buf[kTab * sizeof(float2)];
  float2* tab = reinterpret_cast<float2*>(shared_buf);
  double (*part)[D] = reinterpret_cast<double (*)[D]>(shared_buf);
  __shared__ double freq_s[D / 2];
  __shared__ int4 tok_pos[S];                  // per token: (t, y, x), as byte offsets into the table if there is one

  const int row = xcd_remap(blockIdx.x, a.n_rows);   // (b*H + h)*nB + i
  const bool only_k = NX == 1 && blockIdx.y != 0;
  const int N = a.N, nB = a.nB;
  const int bh = row / nB;
  const int i = row - bh * nB;
  const int start = i * S;
  const int valid = min(S, N - start);
  const size_t base = ((size_t)bh * N + start) * D;
  const int W = a.grid_w, H = a.grid_h, HW = H * W;

  const int r0 = threadIdx.x / TPR;
  const int c = threadIdx.x - r0 * TPR;
  const bool live = c < NCH;                  // D = 112: chunks 14, 15 hold nothing

  // every row this lane handles is loaded first; the table below is built while
  // the loads are in flight.  Rows past the end and dead lanes load some other
  // piece of the block: a load under a condition made the compiler wait for it.
  u32x4 w[NX][NP];
#pragma unroll
  for (int x = 0; x < NX; ++x) {
    const uint16_t* src = x || only_k ? a.k_in : a.q_in;
#pragma unroll
    for (int k = 0; k < NP; ++k)
      w[x][k] = load16<NT>(src + base + (size_t)min(r0 + k * RPP, valid - 1) * D + (live ? c : 0) * 8);
  }

  constexpr double kTwoPi = 6.283185307179586476925286766559;
  // pair frequencies base^(-i/n) in float64, once per workgroup
  if (threadIdx.x < D / 2) {
    const int p = threadIdx.x;
    int idx, n;
    if (p < NTA) { idx = p; n = NTA; }
    else if (p < NTA + NYX) { idx = p - NTA; n = NYX; }
    else { idx = p - NTA - NYX; n = NYX; }
    freq_s[p] = pow(a.base, -(double)idx / (double)n) * (1.0 / kTwoPi);   // turns per unit
  }
  // the coordinate ranges the block covers: t0..t1, y over one frame or all
  // rows, x over one row or the whole width
  const int t0 = start / HW, t1 = (start + valid - 1) / HW;
  const int y0 = (start - t0 * HW) / W, y1 = (start + valid - 1 - t1 * HW) / W;
  const int x0 = start - t0 * HW - y0 * W, x1 = start + valid - 1 - t1 * HW - y1 * W;
  const int ylo = (t0 == t1) ? y0 : 0, yhi = (t0 == t1) ? y1 : H - 1;
  const int xlo = (t0 == t1 && y0 == y1) ? x0 : 0, xhi = (t0 == t1 && y0 == y1) ? x1 : W - 1;
  const int ct = t1 - t0 + 1, cy = yhi - ylo + 1, cx = xhi - xlo + 1;
  const int off_y = ct * NTA, off_x = off_y + cy * NYX;
  const int n_tab = off_x + cx * NYX;
  const bool use_tab = n_tab <= kTab;          // uniform
  // coordinates of the block's tokens, once per token
  if (threadIdx.x < valid) {
    const int n = start + threadIdx.x;
    const int t = n / HW;
    const int rem = n - t * HW;
    const int yy = rem / W;
    const int xx = rem - yy * W;
    constexpr int E = sizeof(float2);
    tok_pos[threadIdx.x] = use_tab ? make_int4((t - t0) * NTA * E, (yy - ylo) * NYX * E, (xx - xlo) * NYX * E, 0)
                                   : make_int4(t, yy, xx, 0);
  }
  __syncthreads();                             // freq_s and tok_pos ready
  // the angle pos * f in turns (f / 2pi held in float64), reduced to
  // [-1/2, 1/2] in float64; the hardware sin and cos take turns
  auto turn = [&](int pos, double f_turns, float& sn, float& cs) {
    double rev = (double)pos * f_turns;
    rev -= rint(rev);
    sn = __builtin_amdgcn_sinf((float)rev);
    cs = __builtin_amdgcn_cosf((float)rev);
  };
  if (use_tab) {
    for (int e = threadIdx.x; e < n_tab; e += kThreads) {
      int pos, p;
      if (e < off_y) { pos = t0 + e / NTA; p = e % NTA; }
      else if (e < off_x) { const int u = e - off_y; pos = ylo + u / NYX; p = NTA + u % NYX; }
      else { const int u = e - off_x; pos = xlo + u / NYX; p = NTA + NYX + u % NYX; }
      float sn, cs;
      turn(pos, freq_s[p], sn, cs);
      tab[e] = make_float2(cs, sn);
    }
    __syncthreads();
  }

  // this lane's 4 pairs' axes, table entries and frequencies;
  // at most two axes (a group is ten pairs or more): the first pair's and the last's
  int axis[4], entry[4];                       // entry: byte offset at coordinate zero
  double freq[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int p = min(c * 4 + e, D / 2 - 1);
    axis[e] = p < NTA ? 0 : (p < NTA + NYX ? 1 : 2);
    entry[e] = (axis[e] == 0 ? p : (axis[e] == 1 ? off_y + p - NTA : off_x + p - NTA - NYX)) * (int)sizeof(float2);
    freq[e] = freq_s[p];
  }
  const int* pos_a = reinterpret_cast<const int*>(tok_pos) + axis[0];
  const int* pos_b = reinterpret_cast<const int*>(tok_pos) + axis[3];

  float g[NX][8];                              // this lane's 8 weights
  double acc[NX][8];
#pragma unroll
  for (int x = 0; x < NX; ++x) {
    const float* gamma = x || only_k ? a.gamma_k : a.gamma_q;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      g[x][e] = gamma[(live ? c : 0) * 8 + e];
      acc[x][e] = 0.0;
    }
  }
  // the weights have landed here: without this use the compiler waits for them
  // again in every row, and with them for the row's stores before it
#pragma unroll
  for (int x = 0; x < NX; ++x)
#pragma unroll
    for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(g[x][e]));
#pragma unroll
  for (int x = 0; x < NX; ++x) {
    uint16_t* dst = x || only_k ? a.k_out : a.q_out;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int r = r0 + k * RPP;
      if (r >= valid) break;                   // rows are shared by a row's lanes
      u32x4 wk = w[x][k];
      if constexpr (NCH != TPR) wk = live ? wk : u32x4{};
      float y[8] = {lo16(wk[0]), hi16(wk[0]), lo16(wk[1]), hi16(wk[1]), lo16(wk[2]), hi16(wk[2]), lo16(wk[3]), hi16(wk[3])};
      float ss = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) ss = fmaf(y[e], y[e], ss);
      const float inv = inv_root(mean_of<D>(row_sum<TPR>(ss)) + a.eps);

      const int pa = pos_a[4 * r], pb = pos_b[4 * r];
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float sn, cs;
        const int at = axis[e] == axis[0] ? pa : pb;
        if (use_tab) {
          const float2 v = *reinterpret_cast<const float2*>(shared_buf + entry[e] + at);
          cs = v.x;
          sn = v.y;
        } else {
          turn(at, freq[e], sn, cs);
        }
        const float u = y[2 * e] * inv * g[x][2 * e];
        const float v = y[2 * e + 1] * inv * g[x][2 * e + 1];
        const float2v f2 = {u * cs - v * sn, u * sn + v * cs};
        const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2, bf16x2));  // RNE
        o[e] = b;
        acc[x][2 * e] += lo16(b);
        acc[x][2 * e + 1] += hi16(b);
      }
      if (live) store16<NT>(dst + base + (size_t)r * D + c * 8, o);
    }
  }
#pragma unroll
  for (int x = 0; x < NX; ++x) {
    __syncthreads();                           // every lane is done with the table (or the other tensor's sums)
    if (live) {
#pragma unroll
      for (int e = 0; e < 8; ++e) part[r0][c * 8 + e] = acc[x][e];
    }
    __syncthreads();
    if (threadIdx.x < D) {
      float* pool = x || only_k ? a.k_pool : a.q_pool;
      double s = 0.0;
      for (int rr = 0; rr < RPP; ++rr) s += part[rr][threadIdx.x];
      pool[(size_t)row * D + threadIdx.x] = (float)(s / (double)valid);
    }
  }
}

}  // namespace

template <int D, int S>
void launch_ds(const RopeArgs& a, hipStream_t stream) {
  // Tensors past the caches are streamed, and at S = 64 Q and K share a workgroup:
  // a table of about 1,300 angles is a third of the work for 64 rows and few
  // workgroups would be left without a table to share.  us, one tensor / two per
  // workgroup: 32 heads of 63,240 x 128 374 / 353, 20 of 32,760 x 112 114 / 109, 24
  // of 75,600 x 64 219 / 178; 8 of 7,800 x 128 16.8 / 17.5; at S = 128, 48 of
  // 111,600 x 128, 900 / 926.  Plain / non-temporal: 387 / 376 (the first shape),
  // 941 / 908 (the last).
  if ((int64_t)a.n_rows * S * D * 2 >= (64 << 20)) {
    constexpr int NX = S == 64 ? 2 : 1;
    hipLaunchKernelGGL((qknorm_rope_pool_kernel<D, S, NX, true>), dim3(a.n_rows, 2 / NX), dim3(kThreads), 0, stream, a);
  } else {
    hipLaunchKernelGGL((qknorm_rope_pool_kernel<D, S, 1, false>), dim3(a.n_rows, 2), dim3(kThreads), 0, stream, a);
  }
}

hipError_t launch_qknorm_rope_pool(const Dims& d, const RopeArgs& args, hipStream_t stream) {
  RopeArgs a = args;
  a.n_rows = d.B * d.H * d.nB;
  a.N = d.N;
  a.nB = d.nB;
  a.S = d.S;
  switch (d.D * 1000 + d.S) {
    case 64064: launch_ds<64, 64>(a, stream); break;
    case 64128: launch_ds<64, 128>(a, stream); break;
    case 112064: launch_ds<112, 64>(a, stream); break;
    case 112128: launch_ds<112, 128>(a, stream); break;
    case 128064: launch_ds<128, 64>(a, stream); break;
    case 128128: launch_ds<128, 128>(a, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace sva
