// Dispatch of bf16 attention (Section 4.2.2: the kept blocks are computed
// exactly; Appendix A.2.2: FlashAttention dense fallback) to the kernels in
// attention_q16.hip, attention_pair.hip and attention_split.hip.
#include "sva_internal.h"

namespace sva {
namespace {

// Key groups for a call with few query blocks (attention_split.hip), or 1.
// The chip holds 1024 64-query workgroups of two waves (256 CUs, two waves per
// SIMD); a call with at most half as many tiles leaves wave slots for two
// groups per tile, one with at most a quarter for four.  What a split costs,
// the longer prologue and the merge, is about 4 chunks for two groups and 12
// for four.  Measured (us, unsplit / 2 / 4 groups; D = 128): 32 tiles x 32
// chunks 24.7 / 18.2 / 17.3, 256 x 64 45.5 / 32.9 / 29.0, 128 x 28 23.3 / 18.8
// / 17.8, 256 x 16 17.2 / 14.0 / 14.6, 256 x 8 11.5 / 10.7 / 12.2 (shorter
// rows are left alone: 4 chunks 8.6 / 8.8 / 10.7); 500 x 50 52.9 / 37.5 / 48.9,
// 500 x 16 24.3 / 19.7 / 27.4, 336 x 6 11.9 / 12.0 / 21.2; above 512 tiles 576
// x 48 48.8 / 55.7 / 64.8, 1024 x 64 66.6 / 79.6 / 103.
int split_groups(const Dims& d, bool sparse, int kmax) {
  const int64_t tiles = (int64_t)d.call_pairs * ((d.N + 63) / 64);
  const int64_t chunks = (int64_t)(sparse ? (kmax < d.nB ? kmax : d.nB) : d.nB) * (d.S / 32);
  if (tiles > 512 || chunks < 16 || (sparse && kmax > kSplitMaxList)) return 1;
  return tiles <= 256 && chunks >= 24 ? 4 : 2;
}

}  // namespace

hipError_t launch_attention(const Dims& d, bool sparse, const uint16_t* q, const uint16_t* k,
                            const uint16_t* v, const int32_t* kv_idx, const int32_t* kv_count,
                            int kmax, void* out, float* lse, hipStream_t stream) {
  const int groups = split_groups(d, sparse, kmax);
  // Dense attention does not depend on the block size: at S = 64 it runs as
  // 128-token query tiles (four waves share every staged key chunk instead of
  // two; the same keys, in the same 32-key chunks and order).
  Dims dd = d;
  if (!sparse && d.S == 64 && groups == 1) {
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
  if (groups > 1) return launch_attention_split(dd, groups, sparse, a, stream);
  if (sparse && pair_attention_fits(dd, kmax)) return launch_attention_pair(dd, a, stream);
  return launch_attention_q16(dd, sparse, a, stream);
}

}  // namespace sva
