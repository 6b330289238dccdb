// cascade_hosttier.hip -- KV movement between the DRAM tier (pinned host
// memory) and the HBM pool, with the host link overlapped with the on-GPU
// scatter / gather.
//
// Cascade allocates HBM only at the final DRAM->HBM hop of a restore and
// spills preempted prefills to DRAM (Section 4.4); the time of that hop is
// the DRAM link term of eq:restore_time.  A restore is two copies: DRAM ->
// contiguous staging over the host link, then staging ->
// scattered pool slots (cascade_unpack).  Here the move list is cut into
// batches: the link copy of batch k+1 runs on the copy stream while batch k is
// unpacked on the compute stream, each batch's unpack waiting on an event
// recorded after its link copy.  A spill runs the mirror image (pack batch k,
// then its link copy to DRAM while batch k+1 is packed).  Streams and events
// are the caller's.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "cascade.h"
#include "copy_range.h"

namespace {

bool args_ok(const cascade_kv_pool_t *pool, const void *staging, const void *host,
             const int64_t *host_offsets, const cascade_move_t *moves_dev,
             const int32_t *n_dev, int32_t n_moves, int32_t batch, void *const *events,
             int32_t n_events) {
  if (!pool || !staging || !moves_dev || !n_dev || n_moves < 0 || batch < 1) return false;
  if (n_moves > 0 && (!host || !host_offsets || !events || n_events < 1)) return false;
  for (int32_t e = 0; e < n_events && n_moves > 0; ++e)
    if (!events[e]) return false;
  return pool->num_layers >= 1 && pool->chunk_bytes >= 16;
}

constexpr int kBlock = 256;
constexpr int kUnroll = 8;
constexpr int kLinkBlocks = 128;  // blocks of one link launch
constexpr int kLinkGrid = 128;

typedef int v4i __attribute__((ext_vector_type(4)));

struct LinkPlan {
  long long off[kLinkBlocks];  // host byte offset of each block
};

// The link copy of a batch in one launch: block m between dev + m * bytes and
// host + plan.off[m], 32 KiB per workgroup and round.  A copy command per block
// is itself a launch, with 12 us between two of them against 38 us for the
// 2 MiB that each moves (55.6 GB/s): spilling and restoring 64 blocks took 6.1
// ms alone and 8.3 ms call after call.  The link needs about 0.1 MB in flight;
// kLinkGrid workgroups keep 4 MB and leave most of the GPU to the kernels
// beside them.
template <bool kToDevice>
__global__ __launch_bounds__(kBlock) void host_link_kernel(char *dev, char *host, LinkPlan plan,
                                                           int count, long long bytes) {
  constexpr int kUnit = kBlock * kUnroll;
  const long long vecs = bytes >> 4, per = (vecs + kUnit - 1) / kUnit, total = count * per;
  for (long long i = blockIdx.x; i < total; i += gridDim.x) {
    const int m = (int)(i / per);
    const long long v0 = (i - m * per) * kUnit + threadIdx.x;
    v4i *d = reinterpret_cast<v4i *>(dev + m * bytes);
    v4i *h = reinterpret_cast<v4i *>(host + plan.off[m]);
    const v4i *src = kToDevice ? h : d;
    v4i *dst = kToDevice ? d : h;
    v4i t[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const long long v = v0 + u * kBlock;
      t[u] = __builtin_nontemporal_load(src + (v < vecs ? v : 0));
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const long long v = v0 + u * kBlock;
      if (v < vecs) __builtin_nontemporal_store(t[u], dst + v);
    }
  }
}

// Whether kernels may read and write the moves' host blocks: pinned memory at
// its own address, every block inside the one allocation that host points
// into, and 16-byte aligned on both sides.  Anything else (pageable memory, an
// offset outside) goes through copy commands, which check it.
bool link_mapped(const void *staging, const void *host, const int64_t *host_offsets,
                 int64_t block, int32_t n_moves) {
  if ((((uintptr_t)staging | (uintptr_t)host | (uintptr_t)block) & 15) != 0) return false;
  int64_t lo = host_offsets[0], hi = lo, bits = 0;
  for (int32_t m = 0; m < n_moves; ++m) {
    lo = std::min(lo, host_offsets[m]);
    hi = std::max(hi, host_offsets[m]);
    bits |= host_offsets[m];
  }
  if ((bits & 15) != 0 || lo < 0) return false;
  hipPointerAttribute_t at = {};
  void *start = nullptr;
  size_t size = 0;
  hipDeviceptr_t p = const_cast<void *>(host);
  if (hipPointerGetAttributes(&at, host) != hipSuccess || at.type != hipMemoryTypeHost ||
      at.devicePointer != host ||
      hipPointerGetAttribute(&start, HIP_POINTER_ATTRIBUTE_RANGE_START_ADDR, p) != hipSuccess ||
      hipPointerGetAttribute(&size, HIP_POINTER_ATTRIBUTE_RANGE_SIZE, p) != hipSuccess) {
    (void)hipGetLastError();  // the query's, not the copies'
    return false;
  }
  const size_t at_byte = (size_t)(static_cast<const char *>(host) - static_cast<char *>(start));
  return start <= host && at_byte <= size && (uint64_t)hi <= size - at_byte &&
         (uint64_t)block <= size - at_byte - (uint64_t)hi;
}

// Whether any two of up to kLinkBlocks blocks overlap in host memory: their
// order matters then, which one launch does not keep.
bool blocks_overlap(const int64_t *host_offsets, int32_t count, int64_t block) {
  int64_t off[kLinkBlocks];
  std::copy(host_offsets, host_offsets + count, off);
  std::sort(off, off + count);
  for (int32_t k = 1; k < count; ++k)
    if (off[k] - off[k - 1] < block) return true;
  return false;
}

// The link copy of moves [m0, m1): staging slot m <-> host bytes at
// host_offsets[m].  By copy commands, moves whose slots and host blocks are
// both consecutive go as one.
hipError_t link_range(char *staging, char *host, const int64_t *host_offsets, int64_t block,
                      int32_t m0, int32_t m1, bool to_device, bool mapped, hipStream_t s) {
  int32_t m = m0;
  while (m < m1 && mapped) {
    const int32_t count = std::min(m1 - m, (int32_t)kLinkBlocks);
    if (!to_device && blocks_overlap(host_offsets + m, count, block)) break;
    LinkPlan plan;
    for (int32_t k = 0; k < kLinkBlocks; ++k) plan.off[k] = k < count ? host_offsets[m + k] : 0;
    const int64_t units = count * ((block / 16 + kBlock * kUnroll - 1) / (kBlock * kUnroll));
    hipLaunchKernelGGL(to_device ? host_link_kernel<true> : host_link_kernel<false>,
                       dim3((unsigned)std::min<int64_t>(units, kLinkGrid)), dim3(kBlock), 0, s,
                       staging + (int64_t)m * block, host, plan, count, (long long)block);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    m += count;
  }
  while (m < m1) {
    int32_t e = m + 1;
    while (e < m1 && host_offsets[e] == host_offsets[e - 1] + block) ++e;
    char *dev = staging + (int64_t)m * block;
    char *hst = host + host_offsets[m];
    const size_t bytes = (size_t)(e - m) * (size_t)block;
    const hipError_t err = to_device ? hipMemcpyAsync(dev, hst, bytes, hipMemcpyHostToDevice, s)
                                     : hipMemcpyAsync(hst, dev, bytes, hipMemcpyDeviceToHost, s);
    if (err != hipSuccess) return err;
    m = e;
  }
  return hipSuccess;
}

}  // namespace

extern "C" int cascade_restore_from_host(const cascade_kv_pool_t *pool, void *staging,
                                         int32_t staging_slots, const void *host_blocks,
                                         const int64_t *host_offsets,
                                         const cascade_move_t *moves_dev,
                                         const int32_t *n_moves_dev, int32_t n_moves,
                                         int32_t batch_moves, int32_t *status_dev,
                                         void *copy_stream, void *compute_stream,
                                         void *const *events, int32_t n_events) {
  if (!args_ok(pool, staging, host_blocks, host_offsets, moves_dev, n_moves_dev, n_moves,
               batch_moves, events, n_events))
    return CASCADE_EINVAL;
  if (n_moves > staging_slots) return CASCADE_ENOSPC;
  const int64_t block = 2 * (int64_t)pool->num_layers * pool->chunk_bytes;
  hipStream_t cs = static_cast<hipStream_t>(copy_stream);
  hipStream_t ks = static_cast<hipStream_t>(compute_stream);
  if (n_moves == 0) return CASCADE_OK;
  const bool mapped = link_mapped(staging, host_blocks, host_offsets, block, n_moves);
  // the host-to-staging copies start after everything enqueued so far on
  // the compute stream (the step that wrote the move list, earlier use of
  // the staging buffer)
  {
    hipEvent_t ev = static_cast<hipEvent_t>(events[0]);
    if (hipEventRecord(ev, ks) != hipSuccess || hipStreamWaitEvent(cs, ev, 0) != hipSuccess)
      return CASCADE_EHIP;
  }
  for (int32_t k = 0, m0 = 0; m0 < n_moves; ++k, m0 += batch_moves) {
    const int32_t m1 = std::min(n_moves, m0 + batch_moves);
    hipEvent_t ev = static_cast<hipEvent_t>(events[k % n_events]);
    if (link_range(static_cast<char *>(staging),
                   const_cast<char *>(static_cast<const char *>(host_blocks)), host_offsets,
                   block, m0, m1, true, mapped, cs) != hipSuccess ||
        hipEventRecord(ev, cs) != hipSuccess || hipStreamWaitEvent(ks, ev, 0) != hipSuccess)
      return CASCADE_EHIP;
    // moves [m0, m1) of the list, as far as the device count reaches
    const int rc = cascade::copy_range(false, pool, staging, staging_slots, moves_dev,
                                       n_moves_dev, m0, m1 - m0, status_dev, ks);
    if (rc != CASCADE_OK) return rc;
  }
  return CASCADE_OK;
}

extern "C" int cascade_spill_to_host(const cascade_kv_pool_t *pool, void *staging,
                                     int32_t staging_slots, void *host_blocks,
                                     const int64_t *host_offsets, const cascade_move_t *moves_dev,
                                     const int32_t *n_moves_dev, int32_t n_moves,
                                     int32_t batch_moves, int32_t *status_dev, void *copy_stream,
                                     void *compute_stream, void *const *events,
                                     int32_t n_events) {
  if (!args_ok(pool, staging, host_blocks, host_offsets, moves_dev, n_moves_dev, n_moves,
               batch_moves, events, n_events))
    return CASCADE_EINVAL;
  if (n_moves > staging_slots) return CASCADE_ENOSPC;
  const int64_t block = 2 * (int64_t)pool->num_layers * pool->chunk_bytes;
  hipStream_t cs = static_cast<hipStream_t>(copy_stream);
  hipStream_t ks = static_cast<hipStream_t>(compute_stream);
  const bool mapped =
      n_moves > 0 && link_mapped(staging, host_blocks, host_offsets, block, n_moves);
  for (int32_t k = 0, m0 = 0; m0 < n_moves; ++k, m0 += batch_moves) {
    const int32_t m1 = std::min(n_moves, m0 + batch_moves);
    hipEvent_t ev = static_cast<hipEvent_t>(events[k % n_events]);
    const int rc = cascade::copy_range(true, pool, staging, staging_slots, moves_dev,
                                       n_moves_dev, m0, m1 - m0, status_dev, ks);
    if (rc != CASCADE_OK) return rc;
    if (hipEventRecord(ev, ks) != hipSuccess || hipStreamWaitEvent(cs, ev, 0) != hipSuccess ||
        link_range(static_cast<char *>(staging), static_cast<char *>(host_blocks), host_offsets,
                   block, m0, m1, false, mapped, cs) != hipSuccess)
      return CASCADE_EHIP;
  }
  return CASCADE_OK;
}
