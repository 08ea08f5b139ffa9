// Dispatch of bf16 attention (Section 4.2.2: the kept blocks are computed
// exactly; Appendix A.2.2: FlashAttention dense fallback) to the kernels in
// attention_q16.hip and attention_pair.hip.
#include "sva_internal.h"

namespace sva {
namespace {

// Calls whose query blocks leave wave slots empty run with 16 queries per wave
// (attention_q16.hip).  The chip holds 1024 64-query workgroups of two waves (256
// CUs, two waves per SIMD), so at most half as many leave room for four waves
// each.  Measured (us, 32 / 16 queries per wave, D = 128): 5 tiles x 4 chunks 8.0 /
// 6.7, 32 x 64 41.0 / 30.6, 128 x 16 15.8 / 13.0, 256 x 8 11.0 / 9.3, 256 x 32 24.2
// / 18.8, 302 x 302 177 / 152, 500 x 16 21.9 / 18.7, 500 x 50 50.0 / 38.1, 500 x 100
// 90.6 / 70.3, 512 x 256 150.7 / 150.5; above 512 tiles the block size decides:
// 576 x 48 50.2 / 45.5 at S = 64 and 47.6 / 55.6 at S = 128, 752 x 32 (S = 128)
// 38.2 / 43.5, 1024 x 64 (S = 64) 77 / 93.  D = 64 and 112 stand alike.
bool few_query_tiles(const Dims& d) { return (int64_t)d.B * d.H * ((d.N + 63) / 64) <= 512; }

}  // namespace

hipError_t launch_attention(const Dims& d, bool sparse, const uint16_t* q, const uint16_t* k,
                            const uint16_t* v, const int32_t* kv_idx, const int32_t* kv_count,
                            int kmax, void* out, float* lse, hipStream_t stream) {
  const bool narrow = few_query_tiles(d);
  // Dense attention does not depend on the block size: at S = 64 it runs as
  // 128-token query tiles (four waves share every staged key chunk instead of
  // two; the same keys, in the same 32-key chunks and order).
  Dims dd = d;
  if (!sparse && d.S == 64) {
    dd.S = 128;
    dd.nB = (d.N + 127) / 128;
  }
  AttnArgs a;
  a.q = q;
  a.k = k;
  a.v = v;
  a.kv_idx = kv_idx;
  a.kv_count = kv_count;
  a.out = out;
  a.lse = lse;
  a.N = dd.N;
  a.nB = dd.nB;
  a.kmax = kmax;
  a.n_rows = dd.B * dd.H * dd.nB;
  a.scale_log2 = (float)(dd.scale * 1.4426950408889634);
  const int64_t fb = ((int64_t)dd.frame_tokens + dd.S / 2) / dd.S;
  a.frame_blocks = fb < 1 ? 1 : (fb > dd.nB ? dd.nB : (int)fb);
  if (sparse && !narrow && pair_attention_fits(dd, kmax)) return launch_attention_pair(dd, a, stream);
  return launch_attention_q16(dd, sparse, narrow, a, stream);
}

}  // namespace sva
