// Park (swap-out) and resume (swap-in) of KV blocks for requests paused on
// external calls (Swap policy of the paper's context-handling policies,
// Appendix B; the swapped queue of Algorithm 1, step (2)).
//
// One (block, all KV heads) of the pool is contiguous: K[block] is
// num_kv_heads * 16 * head_dim elements, likewise V[block]. A parked record
// is K[block] | V[block] | k_scale[block] | v_scale[block] (scales for fp8
// caches only). Park gathers the listed blocks' records into a contiguous
// device staging buffer with one kernel (16-byte loads and stores, four
// workgroups per block) and drains it to pinned host memory with one
// asynchronous copy (the DMA engine), chunk by chunk when staging is smaller
// than the whole image; resume runs the same two steps backwards and
// scatters into the (new) destination blocks. Small images skip staging and
// the engine: the kernels then reach the pinned buffer over the host link
// themselves. The bytes are moved, never reinterpreted, so the round trip is
// exact.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "aug.h"
#include "checks.h"
#include "status.h"

namespace {

constexpr int kThreads = 256;
// Workgroups per record (2 * num_kv_heads * 16 * head_dim elements: 64 KiB for
// eight KV heads of 128 in bf16): a few blocks alone must still keep the host
// link's long round trips full.
constexpr int kSlices = 4;

struct RecordGeom {
  int64_t kv_bytes;     // bytes of K[block] (and of V[block])
  int64_t scale_bytes;  // bytes of k_scale[block] (and of v_scale[block]); 0 unless fp8
  int64_t rec_bytes;
};

RecordGeom geom(const aug_attn_shape& s) {
  const int64_t elem = s.kv_dtype == AUG_F32 ? 4 : s.kv_dtype == AUG_BF16 ? 2 : 1;
  RecordGeom g{};
  g.kv_bytes = static_cast<int64_t>(s.num_kv_heads) * s.block_size * s.head_dim * elem;
  g.scale_bytes = s.kv_dtype == AUG_FP8_E4M3FN ? static_cast<int64_t>(s.num_kv_heads) * 4 : 0;
  g.rec_bytes = 2 * g.kv_bytes + 2 * g.scale_bytes;
  return g;
}

// Copy `bytes` (a multiple of 4) between two buffers with the widest aligned
// vector width, cooperatively across the workgroup.
__device__ __forceinline__ void wg_copy(char* dst, const char* src, int64_t bytes) {
  const bool a16 = ((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src) | bytes) & 15) == 0;
  if (a16) {
    const int64_t n = bytes / 16;
    const uint4* s = reinterpret_cast<const uint4*>(src);
    uint4* d = reinterpret_cast<uint4*>(dst);
    // four loads in flight a thread: over the host link each takes microseconds
    int64_t i = threadIdx.x;
    for (; i + 3 * kThreads < n; i += 4 * kThreads) {
      uint4 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = s[i + k * kThreads];
#pragma unroll
      for (int k = 0; k < 4; ++k) d[i + k * kThreads] = v[k];
    }
    for (; i < n; i += kThreads) d[i] = s[i];
  } else {
    const int64_t n = bytes / 4;
    const uint32_t* s = reinterpret_cast<const uint32_t*>(src);
    uint32_t* d = reinterpret_cast<uint32_t*>(dst);
    for (int64_t i = threadIdx.x; i < n; i += kThreads) d[i] = s[i];
  }
}

// Zero `bytes` (a multiple of 4) cooperatively across the workgroup.
__device__ __forceinline__ void wg_zero(char* dst, int64_t bytes) {
  uint32_t* d = reinterpret_cast<uint32_t*>(dst);
  for (int64_t i = threadIdx.x; i < bytes / 4; i += kThreads) d[i] = 0u;
}

// One workgroup per (listed block, slice of its record): slice y of kSlices
// takes that part of K and of V, slice 0 the scales as well.
__global__ __launch_bounds__(kThreads) void gather_kernel(
    const char* k_cache, const char* v_cache, const char* k_scale, const char* v_scale,
    const int32_t* ids, int32_t first, int32_t num_pool_blocks, RecordGeom g, char* staging) {
  const int32_t bid = ids[first + blockIdx.x];
  char* rec = staging + static_cast<int64_t>(blockIdx.x) * g.rec_bytes;
  const int64_t part = g.kv_bytes / kSlices, at = blockIdx.y * part;
  const bool scales = g.scale_bytes && blockIdx.y == 0;
  if (static_cast<uint32_t>(bid) >= static_cast<uint32_t>(num_pool_blocks)) {
    // never dereferenced; the record reads as zero bytes rather than stale staging
    wg_zero(rec + at, part);
    wg_zero(rec + g.kv_bytes + at, part);
    if (scales) wg_zero(rec + 2 * g.kv_bytes, 2 * g.scale_bytes);
    return;
  }
  wg_copy(rec + at, k_cache + static_cast<int64_t>(bid) * g.kv_bytes + at, part);
  wg_copy(rec + g.kv_bytes + at, v_cache + static_cast<int64_t>(bid) * g.kv_bytes + at, part);
  if (scales) {
    wg_copy(rec + 2 * g.kv_bytes, k_scale + static_cast<int64_t>(bid) * g.scale_bytes, g.scale_bytes);
    wg_copy(rec + 2 * g.kv_bytes + g.scale_bytes, v_scale + static_cast<int64_t>(bid) * g.scale_bytes,
            g.scale_bytes);
  }
}

__global__ __launch_bounds__(kThreads) void scatter_kernel(
    char* k_cache, char* v_cache, char* k_scale, char* v_scale, const int32_t* ids, int32_t first,
    int32_t num_pool_blocks, RecordGeom g, const char* staging) {
  const int32_t bid = ids[first + blockIdx.x];
  if (static_cast<uint32_t>(bid) >= static_cast<uint32_t>(num_pool_blocks)) return;
  const char* rec = staging + static_cast<int64_t>(blockIdx.x) * g.rec_bytes;
  const int64_t part = g.kv_bytes / kSlices, at = blockIdx.y * part;
  wg_copy(k_cache + static_cast<int64_t>(bid) * g.kv_bytes + at, rec + at, part);
  wg_copy(v_cache + static_cast<int64_t>(bid) * g.kv_bytes + at, rec + g.kv_bytes + at, part);
  if (g.scale_bytes && blockIdx.y == 0) {
    wg_copy(k_scale + static_cast<int64_t>(bid) * g.scale_bytes, rec + 2 * g.kv_bytes, g.scale_bytes);
    wg_copy(v_scale + static_cast<int64_t>(bid) * g.scale_bytes, rec + 2 * g.kv_bytes + g.scale_bytes,
            g.scale_bytes);
  }
}

// The device address of pinned host memory [p, p + bytes), or NULL where the
// kernels cannot reach all of it (memory that HIP does not know as pinned): the
// copy engine takes such a buffer. Both ends are looked up, so a range that
// leaves its allocation is not taken for one inside it.
char* device_view(const void* p, size_t bytes) {
  if (reinterpret_cast<uintptr_t>(p) & 15) return nullptr;   // the kernels move 16-byte words
  char* at[2];
  const char* ends[2] = {static_cast<const char*>(p), static_cast<const char*>(p) + bytes - 1};
  for (int i = 0; i < 2; ++i) {
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, ends[i]) != hipSuccess || a.type != hipMemoryTypeHost ||
        a.devicePointer == nullptr || a.hostPointer == nullptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    at[i] = static_cast<char*>(a.devicePointer) + (ends[i] - static_cast<const char*>(a.hostPointer));
  }
  return at[1] - at[0] == static_cast<std::ptrdiff_t>(bytes - 1) ? at[0] : nullptr;
}

// Records of up to this many bytes in all go straight between the pool and the
// pinned host buffer: the same kernels with the buffer in the place of staging.
// A copy-engine transfer costs about 15 us beside its kernel whatever its size,
// and gather and copy run one after the other; a kernel on the link does not
// quite reach the engine's rate on long transfers and holds compute units.
// Park and resume of the same 64 KiB records, through the engine and direct: 1
// block 39 / 14 us, 8 blocks 57 / 24, 32 blocks (2 MiB) 112 / 81, 128 blocks
// (8 MiB) 336 / 308, 256 blocks 633 / 637, 2048 blocks 4837 / 4885.
constexpr int64_t kDirectBytes = int64_t{8} << 20;

aug_status check_common(const char* who, const aug_attn_shape* s, const void* k, const void* v,
                        const void* ks, const void* vs, const int32_t* ids_dev,
                        const int32_t* ids_host, int32_t n_blocks, int32_t num_pool_blocks,
                        const void* host, size_t host_bytes, const void* staging,
                        size_t staging_bytes, RecordGeom* g) {
  if (aug_status st = aug::check_shape(s, who); st != AUG_OK) return st;
  if (n_blocks < 0) return aug::fail(AUG_ERR_INVALID, "%s: n_blocks %d < 0", who, n_blocks);
  if (num_pool_blocks < 1) return aug::fail(AUG_ERR_INVALID, "%s: empty pool", who);
  *g = geom(*s);
  if (n_blocks == 0) return AUG_OK;
  if (!k || !v || !ids_dev || !host || !staging)
    return aug::fail(AUG_ERR_INVALID, "%s: NULL pointer", who);
  if (s->kv_dtype == AUG_FP8_E4M3FN && (!ks || !vs))
    return aug::fail(AUG_ERR_INVALID, "%s: fp8 KV needs scale arrays", who);
  if (host_bytes < static_cast<size_t>(g->rec_bytes) * static_cast<size_t>(n_blocks))
    return aug::fail(AUG_ERR_NO_SPACE, "%s: host buffer %zu < %lld bytes", who, host_bytes,
                     (long long)(g->rec_bytes * n_blocks));
  if (staging_bytes < static_cast<size_t>(g->rec_bytes))
    return aug::fail(AUG_ERR_NO_SPACE, "%s: staging %zu < one record (%lld bytes)", who,
                     staging_bytes, (long long)g->rec_bytes);
  if (!ids_host) return aug::fail(AUG_ERR_INVALID, "%s: block_ids_host is required", who);
  {
    for (int32_t i = 0; i < n_blocks; ++i)
      if (ids_host[i] < 0 || ids_host[i] >= num_pool_blocks)
        return aug::fail(AUG_ERR_INVALID, "%s: block id %d (entry %d) outside a pool of %d", who,
                         ids_host[i], i, num_pool_blocks);
  }
  return AUG_OK;
}

}  // namespace

extern "C" size_t aug_kv_record_bytes(const aug_attn_shape* s) {
  if (!s || aug::check_shape(s, "aug_kv_record_bytes") != AUG_OK) return 0;
  return static_cast<size_t>(geom(*s).rec_bytes);
}

extern "C" aug_status aug_kv_park(const aug_attn_shape* s, const void* k_cache, const void* v_cache,
                                  const float* k_scale, const float* v_scale,
                                  const int32_t* ids_dev, const int32_t* ids_host, int32_t n_blocks,
                                  int32_t num_pool_blocks, void* host_dst, size_t host_bytes,
                                  void* staging, size_t staging_bytes, void* stream) {
  RecordGeom g{};
  if (aug_status st = check_common("aug_kv_park", s, k_cache, v_cache, k_scale, v_scale, ids_dev,
                                   ids_host, n_blocks, num_pool_blocks, host_dst, host_bytes,
                                   staging, staging_bytes, &g);
      st != AUG_OK || n_blocks == 0)
    return st;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const auto gather = [&](int64_t first, int64_t cnt, char* to) {
    hipLaunchKernelGGL(gather_kernel, dim3(static_cast<uint32_t>(cnt), kSlices), dim3(kThreads), 0, st,
                       static_cast<const char*>(k_cache), static_cast<const char*>(v_cache),
                       reinterpret_cast<const char*>(k_scale), reinterpret_cast<const char*>(v_scale),
                       ids_dev, static_cast<int32_t>(first), num_pool_blocks, g, to);
    if (hipError_t e = hipGetLastError(); e != hipSuccess)
      return aug::fail(AUG_ERR_HIP, "aug_kv_park: gather launch: %s", hipGetErrorString(e));
    return AUG_OK;
  };
  if (n_blocks * g.rec_bytes <= kDirectBytes)
    if (char* to = device_view(host_dst, static_cast<size_t>(n_blocks * g.rec_bytes))) return gather(0, n_blocks, to);
  const int64_t per_chunk = static_cast<int64_t>(staging_bytes) / g.rec_bytes;
  for (int64_t first = 0; first < n_blocks; first += per_chunk) {
    const int64_t cnt = std::min<int64_t>(per_chunk, n_blocks - first);
    if (aug_status ls = gather(first, cnt, static_cast<char*>(staging)); ls != AUG_OK) return ls;
    if (hipError_t e = hipMemcpyAsync(static_cast<char*>(host_dst) + first * g.rec_bytes, staging,
                                      static_cast<size_t>(cnt * g.rec_bytes), hipMemcpyDeviceToHost, st);
        e != hipSuccess)
      return aug::fail(AUG_ERR_HIP, "aug_kv_park: copy to host: %s", hipGetErrorString(e));
  }
  return AUG_OK;
}

extern "C" aug_status aug_kv_resume(const aug_attn_shape* s, void* k_cache, void* v_cache,
                                    float* k_scale, float* v_scale, const int32_t* ids_dev,
                                    const int32_t* ids_host, int32_t n_blocks,
                                    int32_t num_pool_blocks, const void* host_src,
                                    size_t host_bytes, void* staging, size_t staging_bytes,
                                    void* stream) {
  RecordGeom g{};
  if (aug_status st = check_common("aug_kv_resume", s, k_cache, v_cache, k_scale, v_scale, ids_dev,
                                   ids_host, n_blocks, num_pool_blocks, host_src, host_bytes,
                                   staging, staging_bytes, &g);
      st != AUG_OK || n_blocks == 0)
    return st;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const auto scatter = [&](int64_t first, int64_t cnt, const char* from) {
    hipLaunchKernelGGL(scatter_kernel, dim3(static_cast<uint32_t>(cnt), kSlices), dim3(kThreads), 0, st,
                       static_cast<char*>(k_cache), static_cast<char*>(v_cache),
                       reinterpret_cast<char*>(k_scale), reinterpret_cast<char*>(v_scale), ids_dev,
                       static_cast<int32_t>(first), num_pool_blocks, g, from);
    if (hipError_t e = hipGetLastError(); e != hipSuccess)
      return aug::fail(AUG_ERR_HIP, "aug_kv_resume: scatter launch: %s", hipGetErrorString(e));
    return AUG_OK;
  };
  if (n_blocks * g.rec_bytes <= kDirectBytes)
    if (const char* from = device_view(host_src, static_cast<size_t>(n_blocks * g.rec_bytes)))
      return scatter(0, n_blocks, from);
  const int64_t per_chunk = static_cast<int64_t>(staging_bytes) / g.rec_bytes;
  for (int64_t first = 0; first < n_blocks; first += per_chunk) {
    const int64_t cnt = std::min<int64_t>(per_chunk, n_blocks - first);
    if (hipError_t e = hipMemcpyAsync(staging, static_cast<const char*>(host_src) + first * g.rec_bytes,
                                      static_cast<size_t>(cnt * g.rec_bytes), hipMemcpyHostToDevice, st);
        e != hipSuccess)
      return aug::fail(AUG_ERR_HIP, "aug_kv_resume: copy from host: %s", hipGetErrorString(e));
    if (aug_status ls = scatter(first, cnt, static_cast<const char*>(staging)); ls != AUG_OK) return ls;
  }
  return AUG_OK;
}
