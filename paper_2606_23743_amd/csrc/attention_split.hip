// Block-sparse (and dense) attention for calls with few query blocks: the keys
// of a query tile are divided among KG groups of waves of one workgroup
// (Section 4.2.2: kept blocks computed exactly; Appendix A.2.2: dense
// fallback).
//
// What bounds these calls is not the chip but one wave's chain: a 32-key step
// (S products, softmax, PV products, the waits between them) takes about 1 us
// whether one or two waves share a SIMD, so a query block walks its list at
// that pace however idle the rest of the chip is.  Here a workgroup takes 64
// queries with 2*KG waves: group kg (two waves of 32 queries) walks chunks
// [G*kg/KG, G*(kg+1)/KG) of the tile's G 32-key chunks with LDS stages, a
// reference maximum and sums of its own, and group 0 merges the KG partial
// results in float32 at the end.  The walk is KG times shorter; the workgroup
// takes KG times the wave slots.  split_groups (attention.hip) says when that
// is the shorter of the two.
//
// The per-chunk arithmetic (attn_w16.h) and the two-stage pipeline (K two
// chunks, V one chunk ahead) are those of the 64-token kernel.  All groups pass
// the same number of barriers: ceil(G / KG) steps, the last of which a group
// with one chunk fewer sits out.
#include "attn_w16.h"

namespace sva {
namespace {

using namespace attn;

template <int D, int S, bool SPARSE, bool OUT_F32, int KG>
__global__ __launch_bounds__(128 * KG) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_split_kernel(AttnArgs a, int tiles_per_head, int n_tiles) {
  using G = Geo<D>;
  using G16 = Geo16<D>;
  constexpr int CK = 32;                     // keys per staged chunk
  constexpr int NCK = S / CK;                // chunks per key block
  constexpr int CT = CK * G::RB;             // bytes of one chunk tile (K or V)
  constexpr int NUW = CT / 1024 / 2;         // direct-load pieces per wave per tile
  constexpr int OB = G16::DT * 2 * 1024;     // bytes of one wave's O^T partial
  static_assert(NUW >= 1 && 2 * OB <= 4 * CT, "a group's partials fit its stages");

  // per group: two K stages, then two V stages; after the walk, its O^T partial
  __shared__ __attribute__((aligned(1024))) unsigned char stages[KG][4 * CT];
  __shared__ int list[SPARSE ? kSplitMaxList : 1];
  __shared__ __attribute__((aligned(16))) float part_ml[KG][2][64][4];   // m, l of each query tile
  __shared__ int n_list, wg_bad;

  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wv >> 1, w = wv & 1;        // key group; half of the query tile
  const int N = a.N, nB = a.nB;
  const float sl2 = a.scale_log2;

  const int tl = __builtin_amdgcn_readfirstlane(xcd_remap(blockIdx.x, n_tiles));
  const int bh = tl / tiles_per_head;
  const int tile = tl - bh * tiles_per_head;
  const int i = tile * 64 / S;               // the query block the tile belongs to
  const int row = bh * nB + i;
  const size_t head = (size_t)bh * N * D;
  const uint16_t* Qh = a.q + head;

  const int qbase = tile * 64 + w * 32;
  bf16x8 qop[2][G16::KS];
  load_q16<D>(qop, Qh, qbase, N, lane);

  // ---- the kept-block list, entries outside [0, nB) dropped ----
  if (threadIdx.x == 0) wg_bad = 0;
  if constexpr (SPARSE) {
    if (wv == 0) {
      const int count = min(max(a.kv_count[row], 0), a.kmax);
      const int32_t* idx = a.kv_idx + (size_t)row * a.kmax;
      int n = 0;
      for (int t0 = 0; t0 < count; t0 += 64) {
        const int t = t0 + lane;
        const int j = t < count ? idx[t] : -1;
        const bool ok = j >= 0 && j < nB;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(ok);
        const int pos = n + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
        if (ok) list[pos] = j;               // pos < count <= kmax <= kSplitMaxList
        n += __builtin_popcountll(m);
      }
      if (lane == 0) n_list = n;
    }
    __syncthreads();
  }
  const int total = (SPARSE ? __builtin_amdgcn_readfirstlane(n_list) : nB) * NCK;   // chunks of the tile
  const int c0 = total * kg / KG;            // this group's chunks [c0, c1)
  const int c1 = total * (kg + 1) / KG;
  const int steps = (total + KG - 1) / KG;   // of the longest group
  auto block_of = [&](int c) -> int {        // chunk c's key block; past the group's end: 0
    return c >= c1 ? 0 : (SPARSE ? list[c / NCK] : c / NCK);
  };
  auto key_of = [&](int block, int c) -> int {   // first key of chunk c; past the end: 0, in bounds
    return __builtin_amdgcn_readfirstlane(c >= c1 ? 0 : block * S + (c % NCK) * CK);
  };

  unsigned char* const ks = stages[kg];
  unsigned char* const vs = stages[kg] + 2 * CT;
  ChunkLoader<D, NUW, CT, true> ld;
  loader_init(ld, a.k + head, a.v + head, N, ks, vs, w, lane);
  int koff[G16::KS], voff[G16::DT];
  operand_offsets16<D>(lane, koff, voff);

  float m_ref[2] = {0.0f, 0.0f};     // reference max (log2 units) per query tile
  float l_part[2] = {0.0f, 0.0f};    // this lane's quarter of each row sum
  bool ref_set = false;              // wave-uniform
  f32x4 oacc[G16::DT][2];
#pragma unroll
  for (int dt = 0; dt < G16::DT; ++dt) oacc[dt][0] = oacc[dt][1] = f32x4{};
  f32x4 sacc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x) sacc[x][0] = sacc[x][1] = f32x4{};

  // keys of the current chunk and of the two after it
  int kc = key_of(block_of(c0), c0), kn = key_of(block_of(c0 + 1), c0 + 1), kn2 = key_of(block_of(c0 + 2), c0 + 2);
  if (steps > 0) {
    load_tile<true, false>(ld, 0, kc);
    load_tile<false, false>(ld, 0, kc);
    load_tile<true, false>(ld, 1, kn);
    wait_vmcnt<0>();
    wg_barrier();
    qk16<D>(sacc, ks, koff, qop);
    if (N - kc < CK) mask_tail16(sacc, N - kc, lane);
  }
  // Step c: K of chunk c+1 and V of chunk c have landed; after the barrier the
  // K stage of chunk c (read by the S products of step c-1) receives chunk
  // c+2 and the V stage of chunk c-1 receives chunk c+1.  Every step issues
  // both loads (past the end: key 0, in bounds) and waits for the previous
  // step's.  A chunk wholly past the sequence's end (the last block's) and a
  // step past the group's end compute nothing.
  for (int s0 = 0; s0 < steps; s0 += 2) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int c = c0 + s0 + p;
      wait_vmcnt_lds_idle<0>();
      wg_barrier();
      load_tile<true, false>(ld, p, kn2);
      load_tile<false, false>(ld, 1 - p, kn);
      const int block3 = block_of(c + 3);    // an LDS read: used at the end of the step
      f32x4 snext[2][2];
      qk16<D>(snext, ks + (1 - p) * CT, koff, qop);
      if (c < c1 && kc < N) {
        if (!ref_set) {                      // the group's first chunk with a valid key
          chunk_reference16(sacc, sl2, m_ref);
          ref_set = true;
        }
        bf16x8 pop[2];
        softmax16(sacc, pop, l_part, m_ref, sl2);
        pv16<D>(pop, vs + p * CT, voff, oacc);
      }
      if (N - kn < CK) {
        asm volatile("");        // keep this a real (rarely taken) branch, not select code
        mask_tail16(snext, N - kn, lane);
      }
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        sacc[x][0] = snext[x][0];
        sacc[x][1] = snext[x][1];
      }
      kc = kn;
      kn = kn2;
      kn2 = key_of(block3, c + 3);
      if (s0 + p + 1 == steps) break;        // uniform over the workgroup
    }
    rescale_if_large16<D>(l_part, m_ref, oacc);
  }
  wait_vmcnt<0>();           // no load may still target this workgroup's LDS

  // ---- overflow check, then the merge of the groups ----
  float l_tot[2];
  l_tot[0] = quad_sum(l_part[0]);
  l_tot[1] = quad_sum(l_part[1]);
  const bool bad = overflowed16<D>(l_tot, oacc);
  __syncthreads();                           // every wave is done with the stages
  if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) atomicOr(&wg_bad, 1);
  float* const ml = part_ml[kg][w][lane];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    ml[qt] = m_ref[qt];
    ml[2 + qt] = l_tot[qt];
  }
  if (kg > 0) {
    f32x4* const o = reinterpret_cast<f32x4*>(stages[kg] + w * OB);
#pragma unroll
    for (int dt = 0; dt < G16::DT; ++dt) {
      o[(dt * 2 + 0) * 64 + lane] = oacc[dt][0];
      o[(dt * 2 + 1) * 64 + lane] = oacc[dt][1];
    }
  }
  __syncthreads();
  if (wg_bad) {                              // the whole list again, by the first group
    if (kg > 0) return;
    general_walk16<D, S, OUT_F32>(a, ld, ks, vs, koff, voff, bh, qbase, total / NCK,
                                  [&](int t) { return __builtin_amdgcn_readfirstlane(SPARSE ? list[t] : t); }, true);
    return;
  }
  if (kg > 0) return;
  // A group that attended to nothing has l = 0 and takes no part in the
  // maximum; the others are brought to the largest reference.
  float m_all[2] = {m_ref[0], m_ref[1]}, l_all[2];
  bool has[2];
  float f[KG][2];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    has[qt] = l_tot[qt] > 0.0f;
#pragma unroll
    for (int g = 1; g < KG; ++g) {
      const float mg = part_ml[g][w][lane][qt], lg = part_ml[g][w][lane][2 + qt];
      if (lg > 0.0f) {
        m_all[qt] = has[qt] ? fmaxf(m_all[qt], mg) : mg;
        has[qt] = true;
      }
    }
    l_all[qt] = 0.0f;
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      const float mg = g == 0 ? m_ref[qt] : part_ml[g][w][lane][qt];
      const float lg = g == 0 ? l_tot[qt] : part_ml[g][w][lane][2 + qt];
      f[g][qt] = lg > 0.0f ? __builtin_amdgcn_exp2f(mg - m_all[qt]) : 0.0f;
      l_all[qt] = __builtin_fmaf(lg, f[g][qt], l_all[qt]);
    }
  }
#pragma unroll
  for (int dt = 0; dt < G16::DT; ++dt)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      f32x4 o = oacc[dt][qt];
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] *= f[0][qt];
#pragma unroll
      for (int g = 1; g < KG; ++g) {
        const f32x4 og = reinterpret_cast<const f32x4*>(stages[g] + w * OB)[(dt * 2 + qt) * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = __builtin_fmaf(og[r], f[g][qt], o[r]);
      }
      oacc[dt][qt] = o;
    }
  store_query16<D, OUT_F32>(a.out, a.lse, head, (size_t)bh * N, qbase, N, oacc, l_all, m_all, has, lane);
}

template <int D, int S, int KG>
hipError_t launch_split(bool sparse, bool out_f32, const AttnArgs& a, hipStream_t stream) {
  const int tiles_per_head = (a.N + 63) / 64;
  const int n_tiles = a.n_rows / a.nB * tiles_per_head;
  dim3 grid(n_tiles), block(128 * KG);
  if (sparse) {
    if (out_f32) hipLaunchKernelGGL((attn_split_kernel<D, S, true, true, KG>), grid, block, 0, stream, a, tiles_per_head, n_tiles);
    else hipLaunchKernelGGL((attn_split_kernel<D, S, true, false, KG>), grid, block, 0, stream, a, tiles_per_head, n_tiles);
  } else {
    if (out_f32) hipLaunchKernelGGL((attn_split_kernel<D, S, false, true, KG>), grid, block, 0, stream, a, tiles_per_head, n_tiles);
    else hipLaunchKernelGGL((attn_split_kernel<D, S, false, false, KG>), grid, block, 0, stream, a, tiles_per_head, n_tiles);
  }
  return hipGetLastError();
}

template <int D, int S>
hipError_t launch_split_groups(int groups, bool sparse, bool out_f32, const AttnArgs& a, hipStream_t stream) {
  return groups == 2 ? launch_split<D, S, 2>(sparse, out_f32, a, stream)
                     : launch_split<D, S, 4>(sparse, out_f32, a, stream);
}

}  // namespace

hipError_t launch_attention_split(const Dims& d, int groups, bool sparse, const AttnArgs& a, hipStream_t stream) {
  switch (d.D * 1000 + d.S) {
    case 64128: return launch_split_groups<64, 128>(groups, sparse, d.out_f32, a, stream);
    case 112128: return launch_split_groups<112, 128>(groups, sparse, d.out_f32, a, stream);
    case 128128: return launch_split_groups<128, 128>(groups, sparse, d.out_f32, a, stream);
    case 64064: return launch_split_groups<64, 64>(groups, sparse, d.out_f32, a, stream);
    case 112064: return launch_split_groups<112, 64>(groups, sparse, d.out_f32, a, stream);
    case 128064: return launch_split_groups<128, 64>(groups, sparse, d.out_f32, a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sva
