// KV append: the write that precedes every decode step.  Each sequence's
// current token (counted in seq_lens, the token the next decode step attends
// with; the per-token step of Sec. 2.2) is stored into its page slot.
//
// bf16 pages take a plain store, one workgroup per sequence.  fp8 pages keep one
// fp32 scale per page for K and one for V (a workgroup each); the paper leaves the
// policy open, and the one taken is grow-only:
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

// The four bf16 values of one 8-byte load.
struct Quad {
  u32x2 w;
  __device__ __forceinline__ float value(int k) const {
    return bf16_bits_to_f32((uint16_t)(w[k >> 1] >> (16 * (k & 1))));
  }
};

// fp8 K: store values 4i .. 4i+3 of the token, a quarter of a 16-byte chunk, into
// slot `slot` of the page.  Each chunk is the only write to its 128-byte line, so
// the stores are non-temporal: they then do not hold L2 lines that the V stores of
// the same call need (four calls in a row over 1,024 sequences, each over another
// pool: 107 -> 94 us; after a 1 GiB read level; non-temporal V stores as well: 89).
__device__ __forceinline__ void store_k(uint8_t* __restrict__ page, int P, int slot, int i, Quad x,
                                        float s) {
  uint32_t q = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) q |= f32_to_e4m3(__fdiv_rn(x.value(k), s)) << (8 * k);
  const int chunk = i >> 2;  // 16 values
  __builtin_nontemporal_store(q, (uint32_t*)(page + ((int64_t)chunk * P + slot) * 16 +
                                             4 * (i & 3)));
}

// fp8 V: store value `row` (head, dim) of the token into its row of the page.
__device__ __forceinline__ void store_v(uint8_t* __restrict__ page, int P, int slot, int row,
                                        uint16_t x, float s) {
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
// than appends that don't).
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

// Page and slot (in the page) of sequence b's current token; the page is -1 where
// there is nothing to append or the page may not be written (never outside the
// pool or into another version's page: reported by the first thread).
__device__ __forceinline__ int64_t locate(const AppendParams& p, int b, int& slot) {
  const int P = p.page_size, L = p.seq_lens[b];
  slot = 0;
  if (L <= 0) return -1;
  const int t = L - 1, j = t / P;
  slot = t - j * P;
  bool ok = L <= p.stride * P;
  const int64_t page_id = ok ? (int64_t)p.block_table[(int64_t)b * p.stride + j] : -1;
  ok = ok && page_id >= 0 && page_id < p.num_pages;
  if (ok && p.page_owner && p.version_ids) ok = p.page_owner[page_id] == p.version_ids[b];
  if (!ok && threadIdx.x == 0 && p.dev_status) *p.dev_status = (int32_t)DORA_ERR_DEVICE_CHECK;
  return ok ? page_id : -1;
}

// fp8: one workgroup per (sequence, K or V), blockDim.x threads (a multiple of 64).
// K and V have a scale each and share no byte, so nothing crosses the two.
// Thread i holds values 4i .. 4i+3 of K; of V it holds values i, i + T, i +
// 2T, i + 3T, so that neighbouring lanes store into neighbouring rows (a
// 128-byte line holds the slots of four rows).  Values beyond 4T, for very
// wide tokens, are read again when stored.  The dependent memory rounds are:
// length (and the token, which does not wait for it), block-table entry, page
// scale.
template <bool IS_K>
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
  int slot;
  const int64_t page_id = locate(p, b, slot);
  if (page_id < 0) return;
  uint8_t* page = pages + page_id * ((int64_t)n * P);
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
  const float s = (slot == 0 || grow) ? fresh : s0;
  if (grow) {  // uniform
    for (int c = tid; c < 256; c += T)
      lut[c] = (uint8_t)f32_to_e4m3(__fdiv_rn(e4m3_to_f32((uint32_t)c) * s0, s));
    __syncthreads();
    requantise<IS_K>(page, lut, n, P, slot);
    // V: the requantised pieces hold the slot the token goes to
    if constexpr (!IS_K) __syncthreads();
  }
  if (tid == 0) scales[page_id] = s;
  if constexpr (IS_K) {
    if (4 * tid < n) store_k(page, P, slot, tid, kq, s);
    for (int i = tid + T; 4 * i < n; i += T)
      store_k(page, P, slot, i, Quad{*(const u32x2*)(x + 4 * i)}, s);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (tid + k * T < n) store_v(page, P, slot, tid + k * T, vq[k], s);
    for (int i = tid + 4 * T; i < n; i += T) store_v(page, P, slot, i, x[i], s);
  }
}

__global__ __launch_bounds__(kAppendMaxThreads) void append_fp8_kernel(AppendParams p) {
  if (blockIdx.y == 0)
    append_side<true>(p, p.k_pages, p.k_scales, p.k_new);
  else
    append_side<false>(p, p.v_pages, p.v_scales, p.v_new);
}

// bf16: store chunk c (8 values) of the token's K and V.  K non-temporal, as above.
__device__ __forceinline__ void store_chunk(uint8_t* __restrict__ kpage,
                                            uint8_t* __restrict__ vpage, int P, int slot, int c,
                                            u32x4 k, u32x4 v) {
  __builtin_nontemporal_store(k, (u32x4*)(kpage + ((int64_t)c * P + slot) * 16));
#pragma unroll
  for (int i = 0; i < 8; ++i)
    *(uint16_t*)(vpage + ((int64_t)(8 * c + i) * P + slot) * 2) =
        (uint16_t)(v[i >> 1] >> (16 * (i & 1)));
}

// bf16: one workgroup per sequence, thread i with chunk i of K and of V (of very wide
// tokens every blockDim.x-th).  Nothing crosses the values, so the fewest waves that
// hold the token are the fastest: with a workgroup for each side and twice the threads,
// as for fp8, calls of up to 512 sequences took 4-17% longer than with the token loaded
// after its page is known and plain stores, this way 8-14% less (512 sequences of 8
// heads, four calls in a row, each over another pool: 45.6 us that way, 38.9 by two
// workgroups, 36.0 so).
__global__ __launch_bounds__(kAppendMaxThreads) void append_bf16_kernel(AppendParams p) {
  const int b = blockIdx.x, c0 = threadIdx.x;
  const int P = p.page_size, n = p.num_kv_heads * p.head_dim, chunks = n / 8;
  const u32x4* k_new = (const u32x4*)(p.k_new + (int64_t)b * n);
  const u32x4* v_new = (const u32x4*)(p.v_new + (int64_t)b * n);
  u32x4 k{0u, 0u, 0u, 0u}, v{0u, 0u, 0u, 0u};
  if (c0 < chunks) {
    k = k_new[c0];
    v = v_new[c0];
  }
  int slot;
  const int64_t page_id = locate(p, b, slot);
  if (page_id < 0) return;
  uint8_t* kpage = p.k_pages + page_id * ((int64_t)n * P * 2);
  uint8_t* vpage = p.v_pages + page_id * ((int64_t)n * P * 2);
  if (c0 < chunks) store_chunk(kpage, vpage, P, slot, c0, k, v);
  for (int c = c0 + blockDim.x; c < chunks; c += blockDim.x)
    store_chunk(kpage, vpage, P, slot, c, k_new[c], v_new[c]);
}

// Threads (a multiple of 64) that hold `per` values of a token each.
static dim3 append_threads(const AppendParams& p, int per) {
  const int t = (p.num_kv_heads * p.head_dim / per + 63) / 64 * 64;
  return dim3(t > kAppendMaxThreads ? kAppendMaxThreads : t);
}

hipError_t launch_append(const AppendParams& p, bool fp8, hipStream_t s) {
  if (p.num_seqs <= 0) return hipSuccess;
  if (p.dev_status) {
    const hipError_t e = launch_fill_i32(p.dev_status, (int32_t)DORA_OK, 1, s);
    if (e != hipSuccess) return e;
  }
  if (fp8)
    hipLaunchKernelGGL(append_fp8_kernel, dim3(p.num_seqs, 2), append_threads(p, 4), 0, s, p);
  else
    hipLaunchKernelGGL(append_bf16_kernel, dim3(p.num_seqs), append_threads(p, 8), 0, s, p);
  return hipGetLastError();
}

}  // namespace dora
