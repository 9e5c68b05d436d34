// Log-sum-exp merge of partial attention results, shared by the combine kernels.
// Included by HIP sources only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "decode_core.h"

namespace dora {

constexpr int kCombineBatch = 4;  // pieces whose loads a thread issues together

// Online log-sum-exp merge of one piece (max in log2 units, sum, unnormalised
// weighted values) into a running (M, S, acc).
__device__ __forceinline__ void merge_piece(float2 ml, f32x4 o, float& M, float& S, f32x4& acc) {
  if (ml.x > M) {
    const float sc = __builtin_amdgcn_exp2f(M - ml.x);
    acc = acc * sc + o;
    S = S * sc + ml.y;
    M = ml.x;
  } else if (ml.x > -__builtin_inff()) {
    const float w = __builtin_amdgcn_exp2f(ml.x - M);
    acc += w * o;
    S += w * ml.y;
  }
}

// Merge of np pieces of segment (b, g), piece k in slot slot_of(k), into its
// output rows: tasks task0 .. task0 + per - 1 of them, a task being a head and 4
// head-dim values.  Threads are tasks x piece groups; each folds its pieces into a
// running (max, normaliser, weighted sum) with one pass of loads, and the groups
// are merged in LDS.
template <int THREADS, typename SlotOf>
__device__ __forceinline__ void merge_segment(const float* part_o, const float2* part_ml,
                                              uint16_t* out, int num_q_heads, int G, int D, int b,
                                              int g, int task0, int per, int np, SlotOf slot_of) {
  __shared__ float sM[THREADS], sS[THREADS];
  __shared__ f32x4 sAcc[THREADS];
  const int t = threadIdx.x;
  const int tasks = G * (D / 4) - task0 < per ? G * (D / 4) - task0 : per;  // <= 0: none
  const int tasks_r = (per + 63) & ~63;
  const int groups = THREADS / tasks_r;  // >= 1 since per <= 512
  const int task = t % tasks_r, sg = t / tasks_r;
  const bool active = task < tasks && sg < groups;
  const int n = active ? (task0 + task) / (D / 4) : 0;
  const int d4 = active ? task0 + task - n * (D / 4) : 0;
  float M = -__builtin_inff(), S = 0.f;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  if (active) {
    for (int k0 = sg; k0 < np; k0 += groups * kCombineBatch) {
      float2 ml[kCombineBatch];
      f32x4 o[kCombineBatch];
#pragma unroll
      for (int i = 0; i < kCombineBatch; ++i) {  // all loads of the batch first
        const int k = k0 + i * groups;
        ml[i] = make_float2(-__builtin_inff(), 0.f);
        o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (k < np) {
          const int64_t row = slot_of(k) * G + n;
          ml[i] = part_ml[row];
          o[i] = *(const f32x4*)(part_o + row * D + 4 * d4);
        }
      }
#pragma unroll
      for (int i = 0; i < kCombineBatch; ++i) merge_piece(ml[i], o[i], M, S, acc);
    }
  }
  sM[t] = M;
  sS[t] = S;
  sAcc[t] = acc;
  __syncthreads();
  if (sg == 0 && task < tasks) {
    float Mx = M;
    for (int k = 1; k < groups; ++k) Mx = fmaxf(Mx, sM[k * tasks_r + task]);
    f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
    for (int k = 0; k < groups; ++k) {
      const int i = k * tasks_r + task;
      if (sM[i] == -__builtin_inff()) continue;  // a group with no pieces
      const float sc = __builtin_amdgcn_exp2f(sM[i] - Mx);
      num += sc * sAcc[i];
      den += sc * sS[i];
    }
    const float inv = 1.f / den;
    const int64_t row = (int64_t)b * num_q_heads + g * G + n;
    uint16_t* o = out + row * D + 4 * d4;
    *(bf16x4*)o = bf16x4{(__bf16)(num[0] * inv), (__bf16)(num[1] * inv),
                         (__bf16)(num[2] * inv), (__bf16)(num[3] * inv)};
  }
}

}  // namespace dora
