// Whole-page KV gather (pack) and scatter (unpack) for same-version request
// migration: the KV-data phase of the paper's two-phase state transfer
// (Sec. 3.4).  Pages are moved as raw bytes, so the copy is bit-exact and the
// destination decodes exactly as the source did.
//
// Both kernels are HBM-bound streaming copies: each workgroup moves one 8 KiB
// chunk of one page (K or V) with 16-byte loads, all loads issued before the
// stores.  Every byte is read once, so the loads are non-temporal.  The stores are
// too, except where what is written and what it is written from fit the 256 MB
// last-level cache about once (32 to 300 MB one way) and are more than the L2s hold:
// there plain stores leave the packed buffer for the unpack.  Pack and unpack, 32 KiB
// pages, over new buffers each time / over the same ones, plain loads and stores in
// 16 KiB chunks, all non-temporal, non-temporal loads: 16 MB one way 17.0 / 13.4 us,
// 15.7 / 11.4, 15.2 / 12.8; 64 MB 49.7 / 39.6, 48.2 / 46.0, 46.6 / 43.4; 192 MB 151 /
// 150, 135 / 134, 128 / 120; 512 MB 392 / 394, 360 / 358, 390 / 389.  To and from pinned
// host memory level (54 and 56 GB/s).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include "dora_internal.h"

namespace dora {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kCopyThreads = 256;
constexpr int kCopyUnroll = 2;
constexpr int kChunkBytes = kCopyThreads * kCopyUnroll * 16;  // 8 KiB
constexpr int kGridPages = 32768;  // pages per grid layer, at most

void make_pack_header(const dora_pack_desc& d, int64_t n_pages, PackHeader* h) {
  memset(h, 0, sizeof *h);
  const int e = d.kv_dtype == DORA_KV_BF16 ? 2 : 1;
  const int64_t page_bytes = (int64_t)d.num_kv_heads * d.page_size * d.head_dim * e;
  uint8_t* p = (uint8_t*)h->words;
  memcpy(p + 0, "DORAKV01", 8);
  int32_t v32;
  v32 = 1;                memcpy(p + 8, &v32, 4);
  v32 = d.policy_version; memcpy(p + 12, &v32, 4);
  v32 = d.kv_dtype;       memcpy(p + 16, &v32, 4);
  v32 = d.page_size;      memcpy(p + 20, &v32, 4);
  v32 = d.num_kv_heads;   memcpy(p + 24, &v32, 4);
  v32 = d.head_dim;       memcpy(p + 28, &v32, 4);
  memcpy(p + 32, &n_pages, 8);
  memcpy(p + 40, &page_bytes, 8);
  v32 = d.n_seqs;         memcpy(p + 48, &v32, 4);
}

__host__ __device__ inline int chunks_per_page(const PackParams& p) {
  return (int)((p.page_bytes + kChunkBytes - 1) / kChunkBytes);
}

// Copy `bytes` (multiple of 16) from src to dst, this workgroup's chunk only.
template <bool NT>
__device__ __forceinline__ void copy_chunk(uint8_t* __restrict__ dst,
                                           const uint8_t* __restrict__ src, int64_t bytes) {
  u32x4 r[kCopyUnroll];
#pragma unroll
  for (int i = 0; i < kCopyUnroll; ++i) {
    const int64_t o = ((int64_t)i * kCopyThreads + threadIdx.x) * 16;
    if (o < bytes) r[i] = __builtin_nontemporal_load((const u32x4*)(src + o));
  }
#pragma unroll
  for (int i = 0; i < kCopyUnroll; ++i) {
    const int64_t o = ((int64_t)i * kCopyThreads + threadIdx.x) * 16;
    if (o < bytes) {
      if constexpr (NT)
        __builtin_nontemporal_store(r[i], (u32x4*)(dst + o));
      else
        *(u32x4*)(dst + o) = r[i];
    }
  }
}

__device__ __forceinline__ void zero_chunk(uint8_t* __restrict__ dst, int64_t bytes) {
#pragma unroll
  for (int i = 0; i < kCopyUnroll; ++i) {
    const int64_t o = ((int64_t)i * kCopyThreads + threadIdx.x) * 16;
    if (o < bytes) *(u32x4*)(dst + o) = u32x4{0u, 0u, 0u, 0u};
  }
}

// One workgroup per chunk: grid.x = K's chunks of a page, then V's; (y, z) = the
// page, so that no index is divided by more than that and every dimension stays
// in its limits.  The first workgroup also writes the header.  fp8: the first
// chunk's workgroup of a page's K (V) moves that scale along (as one loop in a
// workgroup of its own, the last one, the scales took two dependent loads per 256
// pages after the copies: with the above, 16,384 pages of 8 KiB, pack 147 -> 92
// us, unpack 182 -> 101).
template <bool NT>
__global__ __launch_bounds__(kCopyThreads) void pack_kernel(PackParams p) {
  const int cpp = chunks_per_page(p);
  const int which = (int)blockIdx.x >= cpp ? 1 : 0;  // 0: K, 1: V
  const int c = (int)blockIdx.x - which * cpp;
  const int64_t j = (int64_t)blockIdx.z * p.layer + blockIdx.y;
  const bool first = blockIdx.x == 0 && j == 0;
  uint8_t* body = p.packed + 256;
  if (first && threadIdx.x < 64)
    ((uint32_t*)p.packed)[threadIdx.x] = p.hdr.words[threadIdx.x];
  if (j >= p.n_pages) return;
  const int64_t off = (int64_t)c * kChunkBytes;
  const int64_t bytes = p.page_bytes - off < kChunkBytes ? p.page_bytes - off : kChunkBytes;
  uint8_t* dst = body + ((int64_t)which * p.n_pages + j) * p.page_bytes + off;
  const int32_t pid = p.pages[j];
  const bool ok = pid >= 0 && pid < p.num_pages;
  if (p.has_scales && c == 0 && threadIdx.x == 0) {
    float* scales = (float*)(body + 2 * p.n_pages * p.page_bytes);  // K's, then V's
    scales[which * p.n_pages + j] = ok ? (which ? p.v_scales : p.k_scales)[pid] : 0.f;
  }
  if (!ok) {  // out-of-contract id: stay in bounds
    zero_chunk(dst, bytes);
    return;
  }
  const uint8_t* src = (which ? p.v_pages : p.k_pages) + (int64_t)pid * p.page_bytes + off;
  copy_chunk<NT>(dst, src, bytes);
}

// Every workgroup checks the header first; on any mismatch nothing is written
// and the first workgroup reports the status.  (Workgroups past the last page, fewer
// pages' than the grid has layers, read it too: an exit before it costs the others
// 0.3% at 475 MB.)
template <bool NT>
__global__ __launch_bounds__(kCopyThreads) void unpack_kernel(PackParams p) {
  __shared__ int bad;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  if (threadIdx.x < 64) {
    const uint32_t w = ((const uint32_t*)p.packed_in)[threadIdx.x];
    // word 12 (n_seqs) is informational; word 3 holds the policy version
    if (threadIdx.x != 12 && w != p.hdr.words[threadIdx.x]) {
      atomicOr(&bad, threadIdx.x == 3 ? 2 : 1);
    }
  }
  __syncthreads();
  const int cpp = chunks_per_page(p);
  const int which = (int)blockIdx.x >= cpp ? 1 : 0;  // 0: K, 1: V
  const int c = (int)blockIdx.x - which * cpp;
  const int64_t j = (int64_t)blockIdx.z * p.layer + blockIdx.y;
  const bool first = blockIdx.x == 0 && j == 0;
  if (first && threadIdx.x == 0 && p.dev_status)
    *p.dev_status = !bad      ? (int32_t)DORA_OK
                    : bad & 1 ? (int32_t)DORA_ERR_INVALID_ARG
                              : (int32_t)DORA_ERR_VERSION_MISMATCH;
  if (bad || j >= p.n_pages) return;
  const uint8_t* body = p.packed_in + 256;
  const int64_t off = (int64_t)c * kChunkBytes;
  const int64_t bytes = p.page_bytes - off < kChunkBytes ? p.page_bytes - off : kChunkBytes;
  const int32_t pid = p.pages[j];
  if (pid < 0 || pid >= p.num_pages) return;  // out-of-contract id: skip
  if (p.has_scales && c == 0 && threadIdx.x == 0) {
    const float* scales = (const float*)(body + 2 * p.n_pages * p.page_bytes);  // K's, then V's
    (which ? p.vs_out : p.ks_out)[pid] = scales[which * p.n_pages + j];
  }
  const uint8_t* src = body + ((int64_t)which * p.n_pages + j) * p.page_bytes + off;
  uint8_t* dst = (which ? p.v_out : p.k_out) + (int64_t)pid * p.page_bytes + off;
  copy_chunk<NT>(dst, src, bytes);
}

// The copy's grid; sets p.layer (from the arguments both it and the chunks of a page
// are known sooner than from the grid's own dimensions).
static dim3 copy_grid(PackParams& p) {
  const int64_t n = p.n_pages > 0 ? p.n_pages : 1;
  const int64_t z = (n + kGridPages - 1) / kGridPages;
  p.layer = (int32_t)((n + z - 1) / z);
  return dim3((unsigned)(2 * chunks_per_page(p)), (unsigned)p.layer, (unsigned)z);
}

// Whether the stores are non-temporal (the figures are at the top).
static bool nt_stores(const PackParams& p) {
  const int64_t one_way = 2 * p.n_pages * p.page_bytes;
  return one_way <= 32000000 || one_way > 300000000;
}

hipError_t launch_pack(const PackParams& params, hipStream_t s) {
  PackParams p = params;
  const dim3 grid = copy_grid(p);
  if (nt_stores(p))
    hipLaunchKernelGGL(pack_kernel<true>, grid, dim3(kCopyThreads), 0, s, p);
  else
    hipLaunchKernelGGL(pack_kernel<false>, grid, dim3(kCopyThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_unpack(const PackParams& params, hipStream_t s) {
  PackParams p = params;
  const dim3 grid = copy_grid(p);
  if (nt_stores(p))
    hipLaunchKernelGGL(unpack_kernel<true>, grid, dim3(kCopyThreads), 0, s, p);
  else
    hipLaunchKernelGGL(unpack_kernel<false>, grid, dim3(kCopyThreads), 0, s, p);
  return hipGetLastError();
}

}  // namespace dora
