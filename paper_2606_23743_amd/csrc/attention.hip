// Dispatch of bf16 attention (Section 4.2.2: the kept blocks are computed
// exactly; Appendix A.2.2: FlashAttention dense fallback) to the kernels in
// attention_q16.hip and attention_pair.hip.
#include "sva_internal.h"

namespace sva {

hipError_t launch_attention(const Dims& d, bool sparse, const uint16_t* q, const uint16_t* k,
                            const uint16_t* v, const int32_t* kv_idx, const int32_t* kv_count,
                            int kmax, void* out, float* lse, hipStream_t stream) {
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
  if (sparse && pair_attention_fits(dd, kmax)) return launch_attention_pair(dd, a, stream);
  return launch_attention_q16(dd, sparse, a, stream);
}

}  // namespace sva
