// Decode attention for batches of response groups that share a prompt (the
// GRPO groups of the paper's rollouts: several responses sampled per prompt,
// App. B).  Within a group the members' block tables start with the same page
// ids for the prompt's full pages.  Those shared pages are read from HBM once
// per group instead of once per member.  Everything is planned on the device
// from the block tables, so a call makes no host round trip:
//
//   prefix   one workgroup per (group, KV head, chunk of the group's shared
//            pages).  It finds the group's shared prefix S (leading page ids
//            equal in every member's row, full pages of every member), then
//            its waves load the pages' K and V tiles into MFMA operands and
//            apply them to the group's (member, query head) columns, two tiles
//            of 16 per wave, and it writes an unnormalised partial (o, running
//            max, sum) per column.
//   suffix   the decode kernel over each member's pages past S, writing fp32
//            rows and their log-sum-exp for the segments it finishes whole;
//            its combine merges the cut ones and folds every row with the
//            chunk partials of its group's prefix into the bf16 output.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "decode_core.h"
#include "dora_internal.h"

namespace dora {

// Steps of an item whose waves are not worth a merge (see prefix_kernel).
constexpr int kAloneSteps = 4;

// Shared prefix of group k (all threads of the workgroup get it): the number
// of leading pages that every member holds in full (floor(len / P), at most
// the table's width) and whose page id equals the leader's; a group of one
// shares nothing.  Returns early, with a value <= `enough`, once every
// member's full pages number at most `enough`.
//   The loads of the common case (at most kDetectBatch members) issue at
// once, so that the detection costs one round trip: each thread reads the
// members' lengths itself (the same few lines for all threads: the cap needs
// no barrier and no atomics), then the entries j = threadIdx.x of every
// member's row (entries past a member's pages are read and ignored: the rows
// are stride wide).  The lengths go first, so a workgroup whose chunk lies
// past the cap leaves as soon as they arrive.  More members, and prefixes
// longer than the workgroup, are compared in further passes.
constexpr int kDetectBatch = 16;
template <int P>
__device__ int shared_prefix(const GroupedParams& p, int k, int enough) {
  __shared__ int s_min;
  const int M = p.group_size, stride = p.stride;
  const int64_t b0 = (int64_t)k * M;
  if (M == 1) return 0;
  const int32_t* __restrict__ bt = p.block_table + b0 * stride;
  const int j = (int)threadIdx.x < stride ? (int)threadIdx.x : stride - 1;
  int L[kDetectBatch];
  int32_t e[kDetectBatch];
#pragma unroll
  for (int i = 0; i < kDetectBatch; ++i) L[i] = p.seq_lens[b0 + (i < M ? i : M - 1)];
  const int32_t lead = bt[j];
#pragma unroll
  for (int i = 0; i < kDetectBatch; ++i) e[i] = bt[(int64_t)(i < M ? i : M - 1) * stride + j];
  int cap = stride;
#pragma unroll
  for (int i = 0; i < kDetectBatch; ++i) cap = min(cap, L[i] > 0 ? L[i] / P : 0);
  for (int m = kDetectBatch; m < M; ++m) {
    const int Lm = p.seq_lens[b0 + m];
    cap = min(cap, Lm > 0 ? Lm / P : 0);
  }
  if (cap <= enough) return cap;  // uniform: every thread read the same lengths
  bool diff = false;
#pragma unroll
  for (int i = 0; i < kDetectBatch; ++i) diff |= e[i] != lead;
  for (int m = kDetectBatch; m < M; ++m) diff |= bt[(int64_t)m * stride + j] != lead;
  if (threadIdx.x == 0) s_min = cap;
  __syncthreads();
  int first = diff && (int)threadIdx.x < cap ? (int)threadIdx.x : cap;  // smallest mismatch
  // (a thread's later entries cannot be a smaller mismatch than its first)
  for (int jj = threadIdx.x + blockDim.x; jj < first; jj += blockDim.x) {
    const int32_t ld = bt[jj];
    bool d = false;
    for (int m = 1; m < M; ++m) d |= bt[(int64_t)m * stride + jj] != ld;
    if (d) first = jj;
  }
  if (first < cap) atomicMin(&s_min, first);
  __syncthreads();
  return s_min;
}

// One step of a wave is 32 shared tokens (load_step), whatever the page size;
// its registers become the bf16 operands of a 32-token page.
template <int D, bool FP8>
__device__ __forceinline__ PageRegs<D, 32, false> widen(const PageRegs<D, 32, FP8>& r) {
  if constexpr (!FP8) {
    return r;
  } else {
    PageRegs<D, 32, false> o;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int s = 0; s < D / 64; ++s) {
        const u32x4 w = r.k[t * (D / 64) + s];
        o.k[t * (D / 32) + 2 * s] = __builtin_bit_cast(u32x4, fp8x8_to_bf16(w[0], w[1]));
        o.k[t * (D / 32) + 2 * s + 1] = __builtin_bit_cast(u32x4, fp8x8_to_bf16(w[2], w[3]));
      }
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
      o.v[i] = __builtin_bit_cast(u32x4, fp8x8_to_bf16(r.v[i][0], r.v[i][1]));
    return o;
  }
}

// The step's scores, softmax weights and weighted values for NC tiles of 16
// columns.  ksc, vsc: score scale and V scale of this lane's tokens; bias: 0,
// or -inf in lanes whose tokens are past the prefix.
template <int D, int NC>
__device__ __forceinline__ void apply_step(const PageRegs<D, 32, false>& r, float ksc, float vsc,
                                           float bias, const bf16x8 (&q)[NC][D / 32],
                                           f32x4 (&acc)[NC][D / 16], float (&m_run)[NC],
                                           float (&l_run)[NC]) {
  f32x4 sc[NC][2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int c = 0; c < NC; ++c) sc[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        sc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, r.k[t * (D / 32) + ks]), q[c][ks], sc[c][t], 0, 0, 0);
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    float mx = -__builtin_inff();
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sc[c][t][i] = __builtin_fmaf(sc[c][t][i], ksc, bias);
        mx = fmaxf(mx, sc[c][t][i]);
      }
    mx = max_xor32(max_xor16(mx));
    if (__ballot(mx > m_run[c])) {  // some column's running maximum grows: rescale the tile
      const float m_new = fmaxf(m_run[c], mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run[c] - m_new);
      m_run[c] = m_new;
      l_run[c] *= alpha;
#pragma unroll
      for (int i = 0; i < D / 16; ++i) acc[c][i] *= alpha;
    }
  }
  bf16x8 pb[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    float psum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = __builtin_amdgcn_exp2f(sc[c][t][i] - m_run[c]);
        psum += e;
        pb[c][4 * t + i] = (__bf16)(e * vsc);
      }
    l_run[c] += psum;
  }
#pragma unroll
  for (int i = 0; i < D / 16; ++i)
#pragma unroll
    for (int c = 0; c < NC; ++c)
      acc[c][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.v[i]), pb[c],
                                                          acc[c][i], 0, 0, 0);
}

// One workgroup of WAVES waves per item (group k, KV head g, chunk c).  The group's
// (member, query head) columns form CP pairs of 16-column tiles; wave w holds
// pair w % CP and takes every SP-th step of the chunk, SP = WAVES / CP.  A wave
// loads its step straight into MFMA operand registers (as the decode kernel
// does; the CP waves of a step share its lines in the caches), so nothing is
// staged in LDS and no barrier sits between steps, and each pair gives its wave
// two independent chains of MFMA and softmax.  At the end the SP partial
// results of each pair are merged through LDS.  More columns per wave would
// load and convert a step fewer times, but the accumulators of four tiles of
// head dim 128 do not leave room for the next step's loads at two waves per
// SIMD, and with eight tiles the registers spill.
//   What bounds it: long fp8 chunks by the vector instructions of a step (64
// half-rate conversions and about 170 others per pair, 1,370 cycles, beside 512
// of MFMA) at two waves per SIMD; short chunks by what surrounds the steps
// (detection 5 us, page ids 1 us, merge and partials 5 us).  Before (every step
// staged in LDS between barriers for 8 waves of one tile each): 16 groups of
// 16, 64 / 8 heads, fp8, 68.6 -> 52.3 us; 4 groups of 16, 28 / 4 heads, bf16,
// 18.7 us both.  Moving a column's maximum only when a score exceeds it by 2^8
// (fewer rescales): 48 and 18.0 us, but it rounds the largest weight of a column,
// 0.8% more error against 64 bits: not taken.
//   An item of at most kAloneSteps steps has no merge: one wave takes all steps
// of a pair, or of one tile of a pair while there are waves for it (CP <= 2), and
// writes its partial from registers; the others leave.  Whole calls, 4 groups of
// 4, 28 / 4 heads, bf16, prompts of 32 / 64 / 128 tokens: 22.8 / 23.0 / 23.4 us
// with the merge, 19.4 / 20.1 / 21.2 without (8 steps: 24.2 / 25.4).
//   Waves (prefix_waves): 8, and one item per CU, up to 128 (group, KV head) pairs;
// beyond, where pairs times whole chunks would leave CUs idle or take two rounds,
// 4, and two items per CU: 212 pairs (53 groups of 5, 28 / 4 heads, fp8, prompts of
// 350 tokens) 62.9 -> 57.1 us a call, 472 pairs (59 groups of 2, 128 / 8 heads, fp8)
// with prompts of 32 / 256 / 3,000 tokens 38.2 / 47.8 / 116 -> 33.5 / 39.0 / 108.
// Up to 128 pairs 4 waves lose: the prefix kernels of the two batches above take
// 53.6 and 19.1 us.
template <int D, int P, bool FP8, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void prefix_kernel(GroupedParams p) {
  constexpr int PAIR = 32 / P;  // pages per step
  constexpr int KSTEPS = D / 32, DBLK = D / 16;
  constexpr int TILE = P * D * (FP8 ? 1 : 2);  // bytes of one (page, KV head) K tile; V's is the same
  constexpr int ROW = D + 4;       // floats per column in the merge buffer (spreads the banks)
  typedef PageRegs<D, 32, FP8> R;
  typedef PageRegs<D, 32, false> W;
  __shared__ __align__(16) float s_o[WAVES][16][ROW];  // merge: a tile of every wave
  __shared__ float s_m[WAVES][32], s_l[WAVES][32];
  __shared__ int s_pid[kPrefixMaxChunk];
  __shared__ float s_ksc[FP8 ? kPrefixMaxChunk : 1], s_vsc[FP8 ? kPrefixMaxChunk : 1];

  // chunk-major order: the blocks that have work (low chunk indices) come
  // first and are dispatched first
  const int KH = p.num_seqs / p.group_size * p.num_kv_heads;
  const int c = blockIdx.x / KH, kg = blockIdx.x - c * KH;
  const int k = kg / p.num_kv_heads, g = kg - k * p.num_kv_heads;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int G = p.group, MG = p.group_size * G;
  const int CP = (MG + 31) / 32, SP = WAVES / CP;
  const int pr = wave % CP, phase = wave / CP;  // waves with phase >= SP hold nothing

  // Query operands (issued first: they do not depend on the prefix).
  bf16x8 q[2][KSTEPS];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int cg = pr * 32 + h * 16 + col;  // column among (member, head) pairs
    const int m = cg < MG ? cg / G : 0, n = cg < MG ? cg - m * G : 0;
    const int64_t b = (int64_t)k * p.group_size + m;
    load_q_operand<D, FP8>(q[h], p.q + (b * p.num_q_heads + (int64_t)g * G + n) * D, cg < MG);
  }

  // The group's shared prefix; the first workgroup of each group publishes it
  // for the suffix decode and its combine.  A chunk that starts past every
  // member's full pages has no work whatever the prefix is.
  const int S = shared_prefix<P>(p, k, c * kPrefixMinChunk);
  if (c == 0 && g == 0 && threadIdx.x == 0) {
    p.group_shared[k] = S;
    if (p.shared_out) p.shared_out[k] = S;
  }
  const int chunk = prefix_chunk_of(S, p.chunks_wanted);
  const int j0 = c * chunk;
  if (j0 >= S) return;  // uniform: this chunk is past the group's prefix
  const int n_pages = (j0 + chunk < S ? j0 + chunk : S) - j0;
  // The item's page ids (and fp8 scales) go to LDS first: a page load that
  // waited on a block-table load would wait on every load issued before it.
  const int32_t* bt = p.block_table + (int64_t)k * p.group_size * p.stride;  // the leader's row
  for (int t = threadIdx.x; t < n_pages; t += 64 * WAVES) {
    const int pid = bt[j0 + t];
    s_pid[t] = pid;
    if constexpr (FP8) {
      s_ksc[t] = p.scale_log2 * p.k_scales[pid];
      s_vsc[t] = p.v_scales[pid];
    }
  }
  __syncthreads();

  // Per-lane byte offsets inside a (page, KV head) tile.
  const uint32_t koff = step_koff<D, P, 32>(col, grp), voff = step_voff<D, P, FP8, 32>(col, grp);
  const int n_steps = (n_pages + PAIR - 1) / PAIR;
  // Loads are never skipped, so the compiler's in-order wait counts stay exact
  // (a load under a branch makes it wait for everything): a step past the end
  // re-reads the last one, a missing second page the first.  Neither reaches a
  // score: the step is not applied, the page's lanes are masked.
  auto fetch = [&](R& r, int u) {
    const int t0 = (u < n_steps ? u : n_steps - 1) * PAIR;
    const int t1 = PAIR == 2 && t0 + 1 < n_pages ? t0 + 1 : t0;
    const int p0 = __builtin_amdgcn_readfirstlane(s_pid[t0]);
    const int p1 = __builtin_amdgcn_readfirstlane(s_pid[t1]);
    load_step<D, P, FP8, 32, false>(r, p.k_pages, p.v_pages,
                                (int64_t)p0 * p.page_bytes + (int64_t)g * TILE,
                                (int64_t)p1 * p.page_bytes + (int64_t)g * TILE, koff, voff);
  };
  // Steps first, first + by, ... (first < n_steps) over the NC column tiles of q.
  auto stream = [&](int first, int by, const auto& q, auto& acc, auto& m_run, auto& l_run) {
    constexpr int NC = sizeof(m_run) / sizeof(float);
    auto apply = [&](W r, int u) {
      float ksc = p.scale_log2, vsc = 1.f, bias = 0.f;
      if constexpr (PAIR == 2) {
        if (u * PAIR + 1 >= n_pages) {  // uniform: the last step has one page
#pragma unroll
          for (int i = 0; i < W::NK; ++i) r.k[i] = col >= 8 ? u32x4{0u, 0u, 0u, 0u} : r.k[i];
#pragma unroll
          for (int i = 0; i < DBLK; ++i) r.v[i] = grp >= 2 ? u32x4{0u, 0u, 0u, 0u} : r.v[i];
          bias = grp >= 2 ? -__builtin_inff() : 0.f;
        }
      }
      if constexpr (FP8) {
        int t = u * PAIR + (PAIR == 2 && grp >= 2 ? 1 : 0);
        t = t < n_pages ? t : n_pages - 1;
        ksc = s_ksc[t];
        vsc = s_vsc[t];
      }
      apply_step<D, NC>(r, ksc, vsc, bias, q, acc, m_run, l_run);
    };
#pragma unroll
    for (int h = 0; h < NC; ++h) {
#pragma unroll
      for (int i = 0; i < DBLK; ++i) acc[h][i] = f32x4{0.f, 0.f, 0.f, 0.f};
      m_run[h] = kNoMax;
      l_run[h] = 0.f;
    }
    if (first >= n_steps) return;
    R ra, rb;
    int u = first;
    fetch(ra, u);
    while (true) {
      fetch(rb, u + by);
      apply(widen<D, FP8>(ra), u);
      if ((u += by) >= n_steps) break;
      fetch(ra, u + by);
      apply(widen<D, FP8>(rb), u);
      if ((u += by) >= n_steps) break;
    }
  };
  const int64_t slot0 = ((int64_t)kg * p.cmax + c) * MG;
  // The partial of NC tiles from column c0, straight from the registers.
  auto store = [&](int c0, const auto& acc, const auto& m_run, const auto& l_run) {
    constexpr int NC = sizeof(m_run) / sizeof(float);
#pragma unroll
    for (int h = 0; h < NC; ++h) {
      const float l = sum_xor32(sum_xor16(l_run[h]));
      const int cg = c0 + h * 16 + col;
      if (cg >= MG) continue;
#pragma unroll
      for (int i = 0; i < DBLK; ++i)
        *(f32x4*)(p.part_o + (slot0 + cg) * D + 16 * i + 4 * grp) = acc[h][i];
      if (grp == 0) p.part_ml[slot0 + cg] = make_float2(m_run[h], l);
    }
  };
  const bool alone = n_steps <= kAloneSteps;  // uniform
  if (alone && CP <= 2) {                     // SP >= 2: a wave for each tile
    if (phase >= 2) return;
    bf16x8 q1[1][KSTEPS];
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) q1[0][s] = phase ? q[1][s] : q[0][s];
    f32x4 acc[1][DBLK];
    float m_run[1], l_run[1];
    stream(0, 1, q1, acc, m_run, l_run);
    store(pr * 32 + phase * 16, acc, m_run, l_run);
    return;
  }
  f32x4 acc[2][DBLK];
  float m_run[2], l_run[2];
  stream(phase < (alone ? 1 : SP) ? phase : n_steps, alone ? 1 : SP, q, acc, m_run, l_run);
  if (alone) {
    if (phase == 0) store(pr * 32, acc, m_run, l_run);
    return;
  }

  // Merge of a pair's SP waves: each scales its accumulators to the columns'
  // common reference, then the sums go through LDS in a fixed order.  Wave
  // CP * s + pr holds phase s of pair pr.
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float l = sum_xor32(sum_xor16(l_run[h]));
    if (grp == 0) {
      s_m[wave][h * 16 + col] = m_run[h];
      s_l[wave][h * 16 + col] = l;
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < MG) {
    const int pc = threadIdx.x >> 5, cc = threadIdx.x & 31;
    float M = s_m[pc][cc], L = 0.f;
    for (int s = 1; s < SP; ++s) M = fmaxf(M, s_m[CP * s + pc][cc]);
    for (int s = 0; s < SP; ++s) {
      const float m = s_m[CP * s + pc][cc];
      L += s_l[CP * s + pc][cc] * (m == M ? 1.f : __builtin_amdgcn_exp2f(m - M));
    }
    p.part_ml[slot0 + threadIdx.x] = make_float2(M, L);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float M = s_m[pr][h * 16 + col];
    for (int s = 1; s < SP; ++s) M = fmaxf(M, s_m[CP * s + pr][h * 16 + col]);
    const float f = m_run[h] == M ? 1.f : __builtin_amdgcn_exp2f(m_run[h] - M);
#pragma unroll
    for (int i = 0; i < DBLK; ++i)
      *(f32x4*)&s_o[wave][col][16 * i + 4 * grp] = acc[h][i] * f;
    __syncthreads();
    for (int e = threadIdx.x; e < CP * 16 * (D / 4); e += 64 * WAVES) {
      const int cc = e / (D / 4), d4 = e - cc * (D / 4);  // column cc & 15 of pair cc >> 4
      const int pc = cc >> 4, cg = pc * 32 + h * 16 + (cc & 15);
      f32x4 o = *(const f32x4*)&s_o[pc][cc & 15][4 * d4];
      for (int s = 1; s < SP; ++s) o += *(const f32x4*)&s_o[CP * s + pc][cc & 15][4 * d4];
      if (cg < MG) *(f32x4*)(p.part_o + (slot0 + cg) * D + 4 * d4) = o;
    }
    if (h == 0) __syncthreads();
  }
}

template <int D, int P, bool FP8>
static const void* prefix_fn(int waves) {
  return waves == 8 ? (const void*)&prefix_kernel<D, P, FP8, 8>
                    : (const void*)&prefix_kernel<D, P, FP8, 4>;
}

hipError_t launch_grouped_prefix(const GroupedParams& p, int grid, bool fp8, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  const int w = prefix_waves((int64_t)(p.num_seqs / p.group_size) * p.num_kv_heads);
  const void* fn;
  if (p.head_dim == 128)
    fn = p.page_size == 16 ? (fp8 ? prefix_fn<128, 16, true>(w) : prefix_fn<128, 16, false>(w))
                           : (fp8 ? prefix_fn<128, 32, true>(w) : prefix_fn<128, 32, false>(w));
  else
    fn = p.page_size == 16 ? (fp8 ? prefix_fn<64, 16, true>(w) : prefix_fn<64, 16, false>(w))
                           : (fp8 ? prefix_fn<64, 32, true>(w) : prefix_fn<64, 32, false>(w));
  GroupedParams arg = p;
  void* args[] = {(void*)&arg};
  return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(64 * w), args, 0, s);
}

}  // namespace dora
