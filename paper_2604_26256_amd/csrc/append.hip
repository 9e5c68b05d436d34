// KV append: the write that precedes every decode step.  Each sequence's
// current token (counted in seq_lens, the token the next decode step attends
// with; the per-token step of Sec. 2.2) is stored into its page slot.
//
// One workgroup per sequence.  bf16 pages take a plain store.  fp8 pages keep
// one fp32 scale per page for K and one for V; the paper leaves the policy
// open, and the one taken is grow-only:
//   amax = max |x| over the token's Hkv x d values
//   fresh = max(amax / 448, 2^-126)          (always a normal number)
//   slot 0:                          s = fresh
//   slot > 0, not fresh <= s0:       s = fresh, and every earlier code c of
//                                    the page (all heads) becomes
//                                    enc((dec(c) * s0) / s)
//   otherwise:                       s = s0
// (comparing the scales, a token with the page's own maximum does not grow it;
// an unset NaN scale does grow)
//   the token's codes are enc(x / s), and the page's scale becomes s.
// All steps round in fp32 (IEEE, one operation at a time); enc is the nearest
// OCP E4M3FN code, ties to even, saturating at +-448.
//
// The work is a few KiB per sequence.  Small batches are bound by the chain of
// dependent memory round trips (length, block-table entry, page scale; the
// token does not wait for them).  Large ones are bound by the V stores: V's
// layout puts a token's values P elements apart, so each is a partial write of
// its own 32-byte row (1,024 fp8 sequences: 94 us for four calls, 49 us with
// no V store).  A page whose fp8 scale grows, about one append in ten, is
// requantised by table: as byte-wise arithmetic, one workgroup for K and V,
// that took 390 us for the same four calls.
//   Cost of the two workgroups a sequence: small bf16 batches whose pools lie in
// the caches take 0.2-0.4 us a call more than with one (four calls: 64 sequences
// of 4 heads 10.4 -> 11.2 us, 128 of 8 heads 15.3 -> 16.8; 512 of 8 heads 33.4 ->
// 32.0; fp8 at every size 3-4x faster, 64 of 4 heads 101 -> 24 us).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dora_internal.h"

namespace dora {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kAppendMaxThreads = 1024;

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) {
  return __uint_as_float((uint32_t)b << 16);
}

// Value of an E4M3FN code, exact in fp32.
__device__ __forceinline__ float e4m3_to_f32(uint32_t c) {
  const uint32_t sign = (c & 0x80u) << 24;
  const uint32_t e = (c >> 3) & 0xFu, m = c & 0x7u;
  if (e == 0xFu && m == 0x7u) return __uint_as_float(sign | 0x7FC00000u);
  if (e == 0) {  // subnormal (or zero): m * 2^-9
    const float v = (float)m * 0x1p-9f;
    return sign ? -v : v;
  }
  return __uint_as_float(sign | ((e + 120u) << 23) | (m << 20));
}

// Nearest E4M3FN code of x, ties to the even mantissa, saturating to +-448.
// Works on the fp32 bit pattern: the 20 mantissa bits below the kept 3 decide
// the rounding, and a carry out of the mantissa moves into the exponent.
__device__ __forceinline__ uint32_t f32_to_e4m3(float x) {
  const uint32_t u = __float_as_uint(x);
  const uint32_t sign = (u >> 24) & 0x80u;
  const uint32_t a = u & 0x7FFFFFFFu;
  if (a > 0x7F800000u) return sign | 0x7Fu;                 // NaN
  if (a >= 0x43E00000u) return sign | 0x7Eu;                // >= 448 (inf included)
  if (a < 0x3C800000u) {                                    // below 2^-6: steps of 2^-9
    const float m = __builtin_rintf(__uint_as_float(a) * 512.0f);  // exact scaling, RNE
    return sign | (uint32_t)m;                              // 8 -> 0x08 = 2^-6
  }
  const uint32_t keep = (a >> 20) & 0x7u, rest = a & 0xFFFFFu;
  uint32_t code = ((((a >> 23) - 120u) << 3) | keep);
  if (rest > 0x80000u || (rest == 0x80000u && (keep & 1u))) code += 1u;
  return sign | code;
}

// Byte offset of element (head h, token slot t, dim i) inside a page.
template <int E>
__device__ __forceinline__ int64_t k_offset(int d, int P, int h, int t, int i) {
  constexpr int X = 16 / E;
  return ((((int64_t)h * (d / X) + i / X) * P + t) * X + i % X) * E;
}
template <int E>
__device__ __forceinline__ int64_t v_offset(int d, int P, int h, int t, int i) {
  return (((int64_t)h * d + i) * P + t) * E;
}

// The four bf16 values of one 8-byte load.
struct Quad {
  u32x2 w;
  __device__ __forceinline__ float value(int k) const {
    return bf16_bits_to_f32((uint16_t)(w[k >> 1] >> (16 * (k & 1))));
  }
};

// K: store values 4i .. 4i+3 of the token, a quarter (bf16: half) of a 16-byte
// chunk, into slot `slot` of the page.  Each chunk is the only write to its
// 128-byte line, so the stores are non-temporal: they then do not hold L2 lines
// that the V stores of the same call need (four calls in a row, each
// over another pool: 512 bf16 sequences 46.9 -> 38.8 us, 1,024 fp8 ones 107 ->
// 94 us; after a 1 GiB read level; non-temporal V stores as well: 50 and 89 us).
template <bool FP8>
__device__ __forceinline__ void store_k(uint8_t* __restrict__ page, int P, int slot, int i, Quad x,
                                        float s) {
  if constexpr (!FP8) {
    const int chunk = i >> 1;  // 8 values
    __builtin_nontemporal_store(x.w, (u32x2*)(page + ((int64_t)chunk * P + slot) * 16 +
                                              8 * (i & 1)));
  } else {
    uint32_t q = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) q |= f32_to_e4m3(__fdiv_rn(x.value(k), s)) << (8 * k);
    const int chunk = i >> 2;  // 16 values
    __builtin_nontemporal_store(q, (uint32_t*)(page + ((int64_t)chunk * P + slot) * 16 +
                                               4 * (i & 3)));
  }
}

// V: store value `row` (head, dim) of the token into its row of the page.
template <bool FP8>
__device__ __forceinline__ void store_v(uint8_t* __restrict__ page, int P, int slot, int row,
                                        uint16_t x, float s) {
  if constexpr (!FP8)
    *(uint16_t*)(page + ((int64_t)row * P + slot) * 2) = x;
  else
    page[(int64_t)row * P + slot] = (uint8_t)f32_to_e4m3(__fdiv_rn(bf16_bits_to_f32(x), s));
}

// The 16 codes of a piece through a page's code table; byte k stays as it is
// where k >= live.
__device__ __forceinline__ u32x4 map_codes(u32x4 w, const uint8_t* lut, int live) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t out = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t c = (w[k] >> (8 * j)) & 0xFFu;
      out |= (4 * k + j < live ? (uint32_t)lut[c] : c) << (8 * j);
    }
    w[k] = out;
  }
  return w;
}

// Requantise slots [0, slot) of every head of one fp8 page.  The step from
// scale s0 to s is the same for every code of the page, so its 256 results are
// computed once and looked up; pages move in 16-byte pieces, kRequantBatch of
// them in flight per thread (with it, appends that grow scales take no longer
// than appends that don't: 107 and 106 us for the four calls above).
constexpr int kRequantBatch = 4;
template <bool IS_K>
__device__ void requantise(uint8_t* __restrict__ page, const uint8_t* lut, int n, int P, int slot) {
  // K: piece (16-dim chunk c, slot t), t < slot.  V: the row's first
  // ceil(slot / 16) pieces.
  const int per = IS_K ? slot : (slot + 15) / 16;
  const int pieces = (IS_K ? n / 16 : n) * per;
  for (int p0 = threadIdx.x; p0 < pieces; p0 += kRequantBatch * blockDim.x) {
    u32x4 w[kRequantBatch];
    u32x4* at[kRequantBatch];
    int live[kRequantBatch];
#pragma unroll
    for (int i = 0; i < kRequantBatch; ++i) {
      int x = p0 + i * blockDim.x;
      x = x < pieces ? x : p0;  // past the end: the first piece again, not stored
      const int r = x / per, t = x - r * per;
      live[i] = IS_K ? 16 : slot - 16 * t;
      at[i] = (u32x4*)(page + ((int64_t)r * P + (IS_K ? t : 0)) * (IS_K ? 16 : 1) +
                       (IS_K ? 0 : 16 * t));
      w[i] = *at[i];
    }
#pragma unroll
    for (int i = 0; i < kRequantBatch; ++i)
      if (p0 + i * (int)blockDim.x < pieces) *at[i] = map_codes(w[i], lut, live[i]);
  }
}

// One workgroup per (sequence, K or V), blockDim.x threads (a multiple of 64).
// K and V have a scale each and share no byte, so nothing crosses the two.
// Thread i holds values 4i .. 4i+3 of K; of V it holds values i, i + T, i +
// 2T, i + 3T, so that neighbouring lanes store into neighbouring rows (a
// 128-byte line holds the slots of four rows).  Values beyond 4T, for very
// wide tokens, are read again when stored.  The dependent memory rounds are:
// length (and the token, which does not wait for it), block-table entry, page
// scale.
template <bool FP8, bool IS_K>
__device__ __forceinline__ void append_side(const AppendParams& p, uint8_t* pages, float* scales,
                                            const uint16_t* token) {
  __shared__ float sred[kAppendMaxThreads / 64];
  __shared__ float sold;  // the page's scale before this token
  __shared__ uint8_t lut[256];
  const int b = blockIdx.x, T = blockDim.x, tid = threadIdx.x;
  const int P = p.page_size, n = p.num_kv_heads * p.head_dim;
  const uint16_t* x = token + (int64_t)b * n;
  Quad kq{u32x2{0u, 0u}};
  uint16_t vq[4] = {0, 0, 0, 0};
  if constexpr (IS_K) {
    if (4 * tid < n) kq.w = *(const u32x2*)(x + 4 * tid);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (tid + k * T < n) vq[k] = x[tid + k * T];
  }
  const int L = p.seq_lens[b];
  if (L <= 0) return;  // nothing to append
  const int t = L - 1, j = t / P, slot = t - j * P;
  bool ok = L <= p.stride * P;
  const int64_t page_id = ok ? (int64_t)p.block_table[(int64_t)b * p.stride + j] : -1;
  ok = ok && page_id >= 0 && page_id < p.num_pages;
  if (ok && p.page_owner && p.version_ids) ok = p.page_owner[page_id] == p.version_ids[b];
  if (!ok) {  // never write outside the pool or into another version's page
    if (tid == 0 && p.dev_status) *p.dev_status = (int32_t)DORA_ERR_DEVICE_CHECK;
    return;
  }
  uint8_t* page = pages + page_id * ((int64_t)n * P * (FP8 ? 1 : 2));
  float s = 0.f;
  if constexpr (FP8) {
    // Thread 0 reads the page's scale and publishes it in LDS before the
    // reduction's barrier; it alone stores the new one, after it.
    if (tid == 0) sold = slot > 0 ? scales[page_id] : 0.f;
    float m = 0.f;
    if constexpr (IS_K) {
#pragma unroll
      for (int k = 0; k < 4; ++k) m = fmaxf(m, fabsf(kq.value(k)));
      for (int i = tid + T; 4 * i < n; i += T) {
        const Quad y{*(const u32x2*)(x + 4 * i)};
#pragma unroll
        for (int k = 0; k < 4; ++k) m = fmaxf(m, fabsf(y.value(k)));
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) m = fmaxf(m, fabsf(bf16_bits_to_f32(vq[k])));
      for (int i = tid + 4 * T; i < n; i += T) m = fmaxf(m, fabsf(bf16_bits_to_f32(x[i])));
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((tid & 63) == 0) sred[tid >> 6] = m;
    __syncthreads();
    for (int i = 0; i < T >> 6; ++i) m = fmaxf(m, sred[i]);
    const float s0 = sold;
    const float fresh = fmaxf(__fdiv_rn(m, 448.0f), 0x1p-126f);
    const bool grow = slot > 0 && !(fresh <= s0);  // an unset (NaN) scale grows
    s = (slot == 0 || grow) ? fresh : s0;
    if (grow) {  // uniform
      for (int c = tid; c < 256; c += T)
        lut[c] = (uint8_t)f32_to_e4m3(__fdiv_rn(e4m3_to_f32((uint32_t)c) * s0, s));
      __syncthreads();
      requantise<IS_K>(page, lut, n, P, slot);
      // V: the requantised pieces hold the slot the token goes to
      if constexpr (!IS_K) __syncthreads();
    }
    if (tid == 0) scales[page_id] = s;
  }
  if constexpr (IS_K) {
    if (4 * tid < n) store_k<FP8>(page, P, slot, tid, kq, s);
    for (int i = tid + T; 4 * i < n; i += T)
      store_k<FP8>(page, P, slot, i, Quad{*(const u32x2*)(x + 4 * i)}, s);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (tid + k * T < n) store_v<FP8>(page, P, slot, tid + k * T, vq[k], s);
    for (int i = tid + 4 * T; i < n; i += T) store_v<FP8>(page, P, slot, i, x[i], s);
  }
}

template <bool FP8>
__global__ __launch_bounds__(kAppendMaxThreads) void append_kernel(AppendParams p) {
  if (blockIdx.y == 0)
    append_side<FP8, true>(p, p.k_pages, p.k_scales, p.k_new);
  else
    append_side<FP8, false>(p, p.v_pages, p.v_scales, p.v_new);
}

int append_threads(int num_kv_heads, int head_dim) {
  const int quads = num_kv_heads * head_dim / 4;
  const int t = (quads + 63) / 64 * 64;
  return t > kAppendMaxThreads ? kAppendMaxThreads : t;
}

hipError_t launch_append(const AppendParams& p, bool fp8, hipStream_t s) {
  if (p.num_seqs <= 0) return hipSuccess;
  if (p.dev_status) {
    const hipError_t e = launch_fill_i32(p.dev_status, (int32_t)DORA_OK, 1, s);
    if (e != hipSuccess) return e;
  }
  const dim3 grid(p.num_seqs, 2), block(append_threads(p.num_kv_heads, p.head_dim));
  if (fp8)
    hipLaunchKernelGGL(append_kernel<true>, grid, block, 0, s, p);
  else
    hipLaunchKernelGGL(append_kernel<false>, grid, block, 0, s, p);
  return hipGetLastError();
}

}  // namespace dora
