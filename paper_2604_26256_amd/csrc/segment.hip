// Decode attention of small batches: a workgroup per (sequence, KV head) segment,
// or per chunk of it, in place of the stream-K decode (decode.hip), with the same
// per-page step, and the combine of a segment's chunks.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "decode_core.h"
#include "dora_internal.h"
#include "merge_core.h"

namespace dora {

// One workgroup of kSegWaves waves per (sequence, KV head) segment, or per chunk
// of p.seg_pages pages of it, for batches whose block tables bound the work (the
// rule is at segment_split).  Wave w takes the pages w, w + kSegWaves, ... of its
// workgroup; the waves' results are merged in LDS, and the workgroup writes the
// output rows, or, where the segment has further chunks, one partial for the
// combine.  Nothing is planned on the device: there is no page prefix, and the
// chain before the first page is one memory round trip, since a wave's table
// entries (lane u holds its u-th page) do not wait for the length.
//   What bounds it: latency.  8 sequences, 2 KV heads of 64, 256 tokens at the
// median: 12.0 us by stream-K (two launches), 6.0 here (one); 3 sequences of 6,000
// fp8 tokens, 8 KV heads of 128: 22.6 by stream-K, 15.4 here, with the combine.
//   Two page buffers, four waves: a third buffer costs loads past the end that
// short segments wait for, one is slower for long ones (8 segments of 24 / 96
// pages of 16 bf16 tokens: 5.7 / 13.9 us with two; geometric mean over 700
// batches 1.73x the stream-K call with two, 1.66x with one).  8 waves are
// level for few segments and slower for many (1,024 segments of 2 / 24 pages:
// 7.5 / 33.1 us with four, 11.4 / 39.4 with eight); 16 spill.
template <int D, int P, bool FP8, int T>
__global__ __launch_bounds__(64 * kSegWaves, 2) void segment_kernel(SegmentParams p) {
  constexpr int PAIR = T / P;  // pages per step
  constexpr int KSTEPS = D / 32, DBLK = D / 16;
  constexpr int TILE_BYTES = P * D * (FP8 ? 1 : 2);
  constexpr int ROW = D + 4;                          // floats per row in LDS (spreads the banks)
  __shared__ __align__(16) float s_o[kSegWaves][16][ROW];
  __shared__ float2 s_ml[kSegWaves][16];              // running max, sum

  const int lane = threadIdx.x & 63, wave = uni((int)threadIdx.x >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int Hkv = p.num_kv_heads, G = p.group;
  // Chunk-major: the workgroups that have work come first.
  const int c = (int)blockIdx.y;
  int b = (int)blockIdx.x / Hkv;
  const int g = (int)blockIdx.x - b * Hkv;
  if (p.rotate) b = (b + c + (c >> 2)) % p.num_seqs;
  const int seg = b * Hkv + g;
  const int64_t row0 = (int64_t)b * p.num_q_heads + (int64_t)g * G;
  const int L = min(p.seq_lens[b], p.stride * P);  // a contract violation stays in bounds
  const int j0 = c * p.seg_pages;  // < stride
  // this lane's step of the wave: its pages (the row's last entry past its end)
  const int jl = j0 + PAIR * (wave + kSegWaves * lane);
  const int32_t* row = p.block_table + (int64_t)b * p.stride;
  int pid0 = row[jl < p.stride ? jl : p.stride - 1];
  int pid1 = PAIR == 2 ? row[jl + 1 < p.stride ? jl + 1 : p.stride - 1] : 0;
  bf16x8 qop[KSTEPS];
  load_q_operand<D, FP8>(qop, p.q + (row0 + col) * D, col < G);

  const int n_seg = uni(pages_of(L, P, p.stride));
  if (c > 0 && j0 >= n_seg) return;  // uniform: the segment ends before this chunk
  const int n = n_seg - j0 < p.seg_pages ? n_seg - j0 : p.seg_pages;
  const int n_steps = (n + PAIR - 1) / PAIR;  // of the workgroup
  f32x4 acc[DBLK];
#pragma unroll
  for (int i = 0; i < DBLK; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = kNoMax, l_run = 0.f;
  const int steps = (n_steps - wave + kSegWaves - 1) / kSegWaves;  // <= 0: none for this wave
  if (steps > 0) {
    const uint32_t koff = step_koff<D, P, T>(col, grp), voff = step_voff<D, P, FP8, T>(col, grp);
    PageRegs<D, T, FP8> buf[2];
    float s_ks[2], s_vs[2];
    auto prefetch = [&](int r, int u) {
      // past the last step the loads still issue, one line each
      const bool past = u >= steps;
      u = past ? steps - 1 : u;
      const int p0 = __builtin_amdgcn_readlane(pid0, u);
      int p1 = p0;
      if constexpr (PAIR == 2) {
        // a second page past the sequence is the first one again: its tokens are masked
        p1 = __builtin_amdgcn_readlane(pid1, u);
        p1 = PAIR * (wave + kSegWaves * u) + 1 < n ? p1 : p0;
      }
      if constexpr (FP8) {
        s_ks[r] = (PAIR == 2 && grp >= 2 ? p.k_scales[p1] : p.k_scales[p0]) * p.scale_log2;
        s_vs[r] = PAIR == 2 && grp >= 2 ? p.v_scales[p1] : p.v_scales[p0];
      } else {
        s_ks[r] = p.scale_log2;
        s_vs[r] = 1.f;
      }
      load_step<D, P, FP8, T, true>(buf[r], p.k_pages, p.v_pages,
                                    (int64_t)p0 * p.page_bytes + (int64_t)g * TILE_BYTES,
                                    (int64_t)p1 * p.page_bytes + (int64_t)g * TILE_BYTES,
                                    past ? 0u : koff, past ? 0u : voff);
    };
    // The table entries are waited for here, once: a wait inside the loop would be
    // for every load in flight.
    asm volatile("" : "+v"(pid0), "+v"(pid1));
    prefetch(0, 0);
    int u = 0;
    while (true) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        prefetch(r ^ 1, u + 1);
        int nv = L - j0 * P - T * (wave + kSegWaves * u);
        nv = nv < T ? nv : T;
        consume_page<D, T, FP8>(buf[r], nv, s_ks[r], s_vs[r], qop, acc, m_run, l_run);
        if (++u >= steps) goto done;
      }
    }
  }
done:
  const float l_tot = sum_xor32(sum_xor16(l_run));
  if (col < G) {
#pragma unroll
    for (int i = 0; i < DBLK; ++i) *(f32x4*)&s_o[wave][col][16 * i + 4 * grp] = acc[i];
    if (grp == 0) s_ml[wave][col] = make_float2(m_run, l_tot);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < G * (D / 4); e += 64 * kSegWaves) {
    const int h = e / (D / 4), d4 = e - h * (D / 4);
    float M = s_ml[0][h].x, S = 0.f;
    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 1; w < kSegWaves; ++w) M = fmaxf(M, s_ml[w][h].x);
#pragma unroll
    for (int w = 0; w < kSegWaves; ++w) {
      if (w >= n_steps) break;  // uniform: waves past the pages hold nothing
      const float2 ml = s_ml[w][h];
      const float f = ml.x == M ? 1.f : __builtin_amdgcn_exp2f(ml.x - M);
      S += f * ml.y;
      o += f * *(const f32x4*)&s_o[w][h][4 * d4];
    }
    if (n_seg > p.seg_pages) {  // uniform: one of several chunks
      const int64_t slot = ((int64_t)seg * p.seg_chunks + c) * G + h;
      *(f32x4*)(p.part_o + slot * D + 4 * d4) = o;
      if (d4 == 0) p.part_ml[slot] = make_float2(M, S);
    } else {
      const float inv = n > 0 ? 1.f / S : 0.f;  // an empty sequence gives zeros
      *(bf16x4*)(p.out + (row0 + h) * D + 4 * d4) =
          bf16x4{(__bf16)(o[0] * inv), (__bf16)(o[1] * inv), (__bf16)(o[2] * inv),
                 (__bf16)(o[3] * inv)};
    }
  }
}

// The combine of the segment kernel: workgroup (seg, part) merges the chunks of a
// segment that has more than one, for the tasks part * per .. of it (all, or an
// equal share).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void combine_chunks_kernel(SegmentParams p, int per) {
  const int seg = (int)blockIdx.x;
  const int b = seg / p.num_kv_heads, g = seg - b * p.num_kv_heads;
  const int n = pages_of(p.seq_lens[b], p.page_size, p.stride);
  if (n <= p.seg_pages) return;
  const int64_t slot0 = (int64_t)seg * p.seg_chunks;
  merge_segment<THREADS>(p.part_o, p.part_ml, p.out, p.num_q_heads, p.group, p.head_dim, b, g,
                         (int)blockIdx.y * per, per, (n + p.seg_pages - 1) / p.seg_pages,
                         [=](int k) { return slot0 + k; });
}

// Tokens per step: 16-token pages go in pairs while the workgroups are at most
// two per CU.  A pair shares one softmax chain (8 sequences, 2 KV heads of 64,
// bf16: 7.6 us a call with single pages, 6.0 with pairs); beyond that, page by
// page keeps more loads moving (536 segments of 360 bf16 tokens, head dim 64:
// 11.3 us page by page, 13.4 in pairs).  bf16 pages of head dim 128 stay single:
// the registers of two 32-token buffers make the compiler copy one, and the copy
// waits for every load in flight (256 segments of up to 1,500 tokens: 18.1 us,
// 22.9 in pairs).
template <int D, int P, bool FP8>
static const void* segment_fn(int64_t grid) {
  if constexpr (P == 16 && (FP8 || D == 64))
    if (grid <= 512) return (const void*)&segment_kernel<D, P, FP8, 32>;
  return (const void*)&segment_kernel<D, P, FP8, P>;
}

hipError_t launch_segments(const SegmentParams& p, bool fp8, hipStream_t s) {
  const int64_t grid = (int64_t)p.num_seqs * p.num_kv_heads * p.seg_chunks;
  const void* fn;
  if (p.head_dim == 128)
    fn = p.page_size == 16
             ? (fp8 ? segment_fn<128, 16, true>(grid) : segment_fn<128, 16, false>(grid))
             : (fp8 ? segment_fn<128, 32, true>(grid) : segment_fn<128, 32, false>(grid));
  else
    fn = p.page_size == 16 ? (fp8 ? segment_fn<64, 16, true>(grid) : segment_fn<64, 16, false>(grid))
                         : (fp8 ? segment_fn<64, 32, true>(grid) : segment_fn<64, 32, false>(grid));
  SegmentParams arg = p;
  // Workgroups go to the 8 XCDs in turn, and there to the 4 shader engines.  With an
  // even number of sequences all chunks of a long row would be on some of these
  // only, so the sequences are rotated from chunk to chunk: by one, for the XCDs or
  // engines, and by one more every four chunks, for their combinations (4 fp8 rows of
  // 8 KV heads, one of 16,900 tokens: 28.0 -> 21.5 us; 8 bf16 rows of one KV head, one
  // of 40,500 tokens among rows of 48: 25.3 -> 19.0).  An odd number spreads by itself
  // and is only slower for it (3 fp8 rows of 8 KV heads: 17.7 -> 22.1); rows of few
  // chunks gain nothing (8 of them: 8.3 -> 8.8).  A grid padded by one sequence spreads
  // as well, but leaves CUs idle where all rows are full (13.8 -> 16.9).
  arg.rotate = p.seg_chunks > 16 && p.num_seqs % 2 == 0;
  void* args[] = {(void*)&arg};
  return hipLaunchKernel(fn,
                         dim3((unsigned)(p.num_seqs * p.num_kv_heads), (unsigned)p.seg_chunks),
                         dim3(64 * kSegWaves), args, 0, s);
}

// Few segments of many chunks: one workgroup of 512 threads would walk a segment's
// chunks in rounds of 4 x (512 / tasks), about 0.7 us each, so its tasks are shared
// out until two rounds do (or 64 tasks are left, the unit of a thread group).
hipError_t launch_combine_chunks(const SegmentParams& p, hipStream_t s) {
  const int segs = p.num_seqs * p.num_kv_heads;
  const int tasks = p.group * (p.head_dim / 4);
  int parts = 1;
  while (tasks > 64 * parts && p.seg_chunks * (tasks / parts) > 8 * 512 && 2 * parts * segs <= 1024)
    parts *= 2;
  hipLaunchKernelGGL(combine_chunks_kernel<512>, dim3((unsigned)segs, (unsigned)parts), dim3(512), 0,
                     s, p, (tasks + parts - 1) / parts);
  return hipGetLastError();
}

}  // namespace dora
