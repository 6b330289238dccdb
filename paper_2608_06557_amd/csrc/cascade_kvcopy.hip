// cascade_kvcopy.hip -- paged-KV block gather / scatter on gfx950.
//
// Cascade restores prefix KV into HBM only at the final DRAM->HBM hop and
// spills preempted prefill state to DRAM (Section 4.4).  On the GPU side both
// are byte-exact copies of every (layer, K/V) chunk of a KV block between the
// paged HBM pool, where a block's chunks are scattered over per-layer caches,
// and a contiguous staging buffer that the host-side DMA reads or fills.
//
// The copy is HBM-bound: one workgroup moves 32 KiB per iteration with
// 16-byte loads and stores, all loads of a thread issued before its stores so
// that every lane keeps kUnroll requests in flight; nontemporal loads and
// stores stream past the caches.  The grid strides over the blocks'
// 32 KiB units with up to kMaxGrid workgroups (about 32 per CU): measured on MI355X,
// a plain copy peaks near that occupancy.  The move count is read on the
// device, so the step's output count drives the copy without a host sync.
//
// The fused entry point interleaves the chunks of both lists.  On MI355X a
// stream of scattered pool reads (spill) and one of scattered pool writes
// (restore) sharing the chip move more bytes per second than either alone,
// and one launch has one tail instead of two.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "cascade.h"
#include "copy_range.h"

namespace {

constexpr int kBlock = 256;
constexpr int kUnroll = 8;
constexpr long long kMaxGrid = 8192;
constexpr int kWhole = -1, kRun = -2;  // unit shapes besides groups of chunks

typedef int v4i __attribute__((ext_vector_type(4)));

// One chunk of vecs 16-byte vectors; thread t moves vectors t + kBlock*i, so
// a thread that copies the same chunk twice touches the same addresses.
__device__ __forceinline__ void copy_chunk(const char *src_c, char *dst_c, int vecs) {
  const v4i *src = reinterpret_cast<const v4i *>(src_c);
  v4i *dst = reinterpret_cast<v4i *>(dst_c);
  for (int base = 0; base < vecs; base += kBlock * kUnroll) {
    v4i t[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int k = base + u * kBlock + threadIdx.x;
      if (k < vecs) t[u] = __builtin_nontemporal_load(src + k);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int k = base + u * kBlock + threadIdx.x;
      if (k < vecs) __builtin_nontemporal_store(t[u], dst + k);
    }
  }
}

// A spill and the restore into the same chunk in one pass: both loads of a
// batch are issued together, then the spill's stores, then the restore's.
// Each thread stores to a pool address only after its own load of that
// address has returned (the spill's store needed the loaded value), so the
// spill reads the old bytes.  Half the unroll per stream keeps the same
// kUnroll vectors in flight and the kernel's register count at the level
// of a plain copy (full occupancy).
__device__ __forceinline__ void copy_pair(char *pool_c, char *spill_c, const char *fill_c,
                                          int vecs) {
  constexpr int kHalf = kUnroll / 2;
  v4i *pool = reinterpret_cast<v4i *>(pool_c);
  v4i *spill = reinterpret_cast<v4i *>(spill_c);
  const v4i *fill = reinterpret_cast<const v4i *>(fill_c);
  for (int base = 0; base < vecs; base += kBlock * kHalf) {
    v4i a[kHalf], b[kHalf];
#pragma unroll
    for (int u = 0; u < kHalf; ++u) {
      const int k = base + u * kBlock + threadIdx.x;
      if (k < vecs) {
        a[u] = __builtin_nontemporal_load(pool + k);
        b[u] = __builtin_nontemporal_load(fill + k);
      }
    }
#pragma unroll
    for (int u = 0; u < kHalf; ++u) {
      const int k = base + u * kBlock + threadIdx.x;
      if (k < vecs) __builtin_nontemporal_store(a[u], spill + k);
    }
#pragma unroll
    for (int u = 0; u < kHalf; ++u) {
      const int k = base + u * kBlock + threadIdx.x;
      if (k < vecs) __builtin_nontemporal_store(b[u], pool + k);
    }
  }
}

__device__ __forceinline__ char *pool_chunk(const cascade_kv_pool_t &pool, int slot, int l,
                                            int kv) {
  return static_cast<char *>(pool.base) + (long long)l * pool.layer_stride +
         (long long)kv * pool.kv_stride + (long long)slot * pool.slot_stride;
}

// Chunks r = 2*l + kv of a block, in the pool and in a staging slot (the
// staging slot's chunks are consecutive).
__device__ __forceinline__ char *pool_r(const cascade_kv_pool_t &pool, int slot, int r) {
  return pool_chunk(pool, slot, r >> 1, r & 1);
}
__device__ __forceinline__ char *stage_r(char *staging, const cascade_kv_pool_t &pool, int slot,
                                         int r) {
  return staging + ((long long)slot * 2 * pool.num_layers + r) * pool.chunk_bytes;
}

// A work item ("unit") is up to a thread batch, kBlock * kUnroll vectors of 16
// bytes (32 KiB), of one block, in the shape that its chunk size allows:
//  - chunks of 4, 8 or 16 KiB that tile the block in batches: g consecutive
//    chunks r0 .. r0+g-1, where vector slot u of a thread is vector
//    ((u & (per - 1)) * kBlock + t) of chunk r0 + (u >> lg), per = 2^lg =
//    chunk / 4 KiB;
//  - other multiples of 4 KiB from 12 KiB on, which give every thread 3 or
//    more vectors: one chunk, moved by copy_chunk (cut as below, 12 to 24 KiB
//    are 1 to 5 % slower in the fused kernel);
//  - any other size: a run.  The block's chunks one behind the other are one
//    run of vectors and a unit is the next batch of it, so that every thread
//    has kUnroll vectors in flight.  With a chunk a unit, 2 KiB chunks kept
//    half the threads idle: 138 us instead of 100 for 1069 spills and 954
//    restores of 128 KiB blocks, and 80 instead of 31 us at 1 KiB.  Larger
//    chunks, whose last batch was a short one, gain too: 11 to 17 % at
//    20 KiB + 16 B, 3 to 7 % at 34 KiB, 5 to 8 % at 66 KiB, 1 to 5 % at
//    130 KiB, 1 to 3 % at 1 MiB + 4 KiB.
struct Units {
  int g, lg, per_move;  // chunks per unit (1 but for groups), shape (groups: log2(vectors per
                        // chunk / kBlock)), units per block
  unsigned vecs;        // vectors per chunk
  double per_vec;       // 1 / vecs
};

template <int kLg>
__device__ __forceinline__ int unit_off(int u) {
  return ((u & ((1 << kLg) - 1)) * kBlock) + (int)threadIdx.x;
}

// v / vecs and the rest, below 2^48: the product is off by at most one.
__device__ __forceinline__ unsigned chunk_of(long long v, const Units &un, unsigned &off) {
  int r = (int)((double)v * un.per_vec);
  long long rest = v - (long long)r * un.vecs;
  if (rest < 0) --r, rest += un.vecs;
  else if (rest >= un.vecs) ++r, rest -= un.vecs;
  off = (unsigned)rest;
  return (unsigned)r;
}

// Where a thread's vectors of unit k of a run lie in the pool, kBlock apart,
// as byte offsets from the block's slot: chunk r, vector off in it.
struct RunWalk {
  unsigned r, off;
  __device__ __forceinline__ RunWalk(int k, const Units &un) {
    r = chunk_of((long long)k * (kBlock * kUnroll) + threadIdx.x, un, off);
  }
  __device__ __forceinline__ long long at(const cascade_kv_pool_t &pool) const {
    return (long long)(r >> 1) * pool.layer_stride + ((r & 1) ? pool.kv_stride : 0) +
           (long long)off * 16;
  }
  // The same place, which the compiler does not know to be the same: else it
  // keeps every place between the loads and the stores, in registers that the
  // fused kernel at eight waves has not got (it spilled to scratch memory; 106.9
  // -> 105.6 us for 1069 spills and 954 restores of 2 KiB chunks without).
  __device__ __forceinline__ RunWalk again() const {
    RunWalk w = *this;
    asm volatile("" : "+v"(w.r), "+v"(w.off));
    return w;
  }
  __device__ __forceinline__ void next(const Units &un, unsigned dr, unsigned doff) {
    r += dr;
    off += doff;
    if (off >= un.vecs) {
      off -= un.vecs;
      ++r;
    }
  }
};

// Vectors of unit k of a block's run: a full batch, or what is left.
__device__ __forceinline__ int run_count(const cascade_kv_pool_t &pool, int k, const Units &un) {
  const long long left =
      (long long)un.vecs * 2 * pool.num_layers - (long long)k * (kBlock * kUnroll);
  return left < kBlock * kUnroll ? (int)left : kBlock * kUnroll;
}

__device__ __forceinline__ char *pool_slot(const cascade_kv_pool_t &pool, int slot) {
  return static_cast<char *>(pool.base) + (long long)slot * pool.slot_stride;
}

// Unit k of a block's run, from pool slot to staging slot (or back).  Loads
// past the block's end read its first vector instead of sitting under a
// branch; the places are worked out again for the stores, which costs less
// than the registers to keep them (full occupancy).
template <bool kToStaging>
__device__ __forceinline__ void copy_run(const cascade_kv_pool_t &pool, int slot, char *stg,
                                         int sslot, int k, const Units &un) {
  const int count = run_count(pool, k, un), t = (int)threadIdx.x;
  const unsigned dr = kBlock / un.vecs, doff = kBlock - dr * un.vecs;
  char *pb = pool_slot(pool, slot);
  v4i *sb = reinterpret_cast<v4i *>(stage_r(stg, pool, sslot, 0)) +
            (long long)k * (kBlock * kUnroll);
  v4i x[kUnroll];
  const RunWalk start(k, un);
  RunWalk w = start;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const bool in = t + u * kBlock < count;
    x[u] = __builtin_nontemporal_load(
        kToStaging ? reinterpret_cast<const v4i *>(pb + (in ? w.at(pool) : 0ll))
                   : sb + (in ? t + u * kBlock : 0));
    w.next(un, dr, doff);
  }
  w = start.again();
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    if (t + u * kBlock < count)
      __builtin_nontemporal_store(
          x[u], kToStaging ? sb + t + u * kBlock : reinterpret_cast<v4i *>(pb + w.at(pool)));
    w.next(un, dr, doff);
  }
}

// Spill and the restore into the same unit of a run, as copy_pair: half the
// vectors per stream at a time, the spill's stores before the restore's.
__device__ __forceinline__ void copy_pair_run(const cascade_kv_pool_t &pool, int slot, char *spill,
                                              int spill_slot, char *fill, int fill_slot, int k,
                                              const Units &un) {
  constexpr int kHalf = kUnroll / 2;
  const int count = run_count(pool, k, un), t = (int)threadIdx.x;
  const unsigned dr = kBlock / un.vecs, doff = kBlock - dr * un.vecs;
  const long long v0 = (long long)k * (kBlock * kUnroll);
  char *pb = pool_slot(pool, slot);
  v4i *ob = reinterpret_cast<v4i *>(stage_r(spill, pool, spill_slot, 0)) + v0;
  const v4i *ib = reinterpret_cast<const v4i *>(stage_r(fill, pool, fill_slot, 0)) + v0;
  RunWalk w(k, un);
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    const int i0 = t + h * kHalf * kBlock;
    const RunWalk start = w;
    v4i a[kHalf], b[kHalf];
#pragma unroll
    for (int u = 0; u < kHalf; ++u) {
      const bool in = i0 + u * kBlock < count;
      a[u] = __builtin_nontemporal_load(
          reinterpret_cast<const v4i *>(pb + (in ? w.at(pool) : 0ll)));
      b[u] = __builtin_nontemporal_load(ib + (in ? i0 + u * kBlock : 0));
      w.next(un, dr, doff);
    }
#pragma unroll
    for (int u = 0; u < kHalf; ++u)
      if (i0 + u * kBlock < count) __builtin_nontemporal_store(a[u], ob + i0 + u * kBlock);
    w = start.again();
#pragma unroll
    for (int u = 0; u < kHalf; ++u) {
      if (i0 + u * kBlock < count)
        __builtin_nontemporal_store(b[u], reinterpret_cast<v4i *>(pb + w.at(pool)));
      w.next(un, dr, doff);
    }
  }
}

// one unit of g = kUnroll >> kLg chunks from pool slot to staging slot (or back)
template <bool kToStaging, int kLg>
__device__ __forceinline__ void copy_group(const cascade_kv_pool_t &pool, int slot, char *stg,
                                           int sslot, int r0) {
  v4i t[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const int r = r0 + (u >> kLg);
    const char *src = kToStaging ? pool_r(pool, slot, r) : stage_r(stg, pool, sslot, r);
    t[u] = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(src) + unit_off<kLg>(u));
  }
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const int r = r0 + (u >> kLg);
    char *dst = kToStaging ? stage_r(stg, pool, sslot, r) : pool_r(pool, slot, r);
    __builtin_nontemporal_store(t[u], reinterpret_cast<v4i *>(dst) + unit_off<kLg>(u));
  }
}

// spill and the restore into the same unit, as copy_pair: half the slots per
// stream at a time, the spill's stores before the restore's
template <int kLg>
__device__ __forceinline__ void copy_pair_group(const cascade_kv_pool_t &pool, int slot,
                                                char *spill, int spill_slot, char *fill,
                                                int fill_slot, int r0) {
  constexpr int kHalf = kUnroll / 2;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    v4i a[kHalf], b[kHalf];
#pragma unroll
    for (int u = 0; u < kHalf; ++u) {
      const int uu = h * kHalf + u, r = r0 + (uu >> kLg), k = unit_off<kLg>(uu);
      a[u] = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(pool_r(pool, slot, r)) + k);
      b[u] = __builtin_nontemporal_load(
          reinterpret_cast<const v4i *>(stage_r(fill, pool, fill_slot, r)) + k);
    }
#pragma unroll
    for (int u = 0; u < kHalf; ++u) {
      const int uu = h * kHalf + u, r = r0 + (uu >> kLg), k = unit_off<kLg>(uu);
      __builtin_nontemporal_store(a[u],
                                  reinterpret_cast<v4i *>(stage_r(spill, pool, spill_slot, r)) + k);
    }
#pragma unroll
    for (int u = 0; u < kHalf; ++u) {
      const int uu = h * kHalf + u, r = r0 + (uu >> kLg), k = unit_off<kLg>(uu);
      __builtin_nontemporal_store(b[u], reinterpret_cast<v4i *>(pool_r(pool, slot, r)) + k);
    }
  }
}

// The unit shape is a template parameter of the kernels, so each compiled
// kernel holds one copy path: kRun, kWhole, else a group of g = kUnroll >> kLg
// chunks.  `first` is the unit's number in the block's run, or its first chunk.
template <bool kToStaging, int kLg>
__device__ __forceinline__ void copy_unit(const cascade_kv_pool_t &pool, int slot, char *stg,
                                          int sslot, int first, const Units &un) {
  if constexpr (kLg == kRun)
    copy_run<kToStaging>(pool, slot, stg, sslot, first, un);
  else if constexpr (kLg == kWhole) {
    char *pc = pool_r(pool, slot, first);
    char *sc = stage_r(stg, pool, sslot, first);
    copy_chunk(kToStaging ? pc : sc, kToStaging ? sc : pc, (int)un.vecs);
  } else
    copy_group<kToStaging, kLg>(pool, slot, stg, sslot, first);
}

template <int kLg>
__device__ __forceinline__ void copy_pair_unit(const cascade_kv_pool_t &pool, int slot,
                                               char *spill, int spill_slot, char *fill,
                                               int fill_slot, int first,
                                               const Units &un) {
  if constexpr (kLg == kRun)
    copy_pair_run(pool, slot, spill, spill_slot, fill, fill_slot, first, un);
  else if constexpr (kLg == kWhole)
    copy_pair(pool_r(pool, slot, first), stage_r(spill, pool, spill_slot, first),
              stage_r(fill, pool, fill_slot, first), (int)un.vecs);
  else
    copy_pair_group<kLg>(pool, slot, spill, spill_slot, fill, fill_slot, first);
}

__device__ __forceinline__ bool move_ok(const cascade_move_t &mv, int num_slots,
                                        int staging_slots) {
  return (unsigned)mv.pool_slot < (unsigned)num_slots &&
         (unsigned)mv.staging_slot < (unsigned)staging_slots;
}

__device__ __forceinline__ void flag_bad(int *status) {
  if (threadIdx.x == 0 && status) *status = CASCADE_EINVAL;
}

template <bool kToStaging, int kLg>
__global__ __launch_bounds__(kBlock) void kvcopy_kernel(cascade_kv_pool_t pool, Units un,
                                                        char *staging, int staging_slots,
                                                        const cascade_move_t *__restrict__ moves,
                                                        const int *__restrict__ n_dev,
                                                        int first, int max_moves, int *status) {
  // moves points at entry `first` of a list of *n_dev entries
  const int nm = min(*n_dev - first, max_moves);
  if (nm <= 0) return;
  const long long total = (long long)nm * un.per_move;
  // each item's move is requested one item ahead, as in kvmove_kernel
  cascade_move_t n_mv = {0, 0, 0, 0};
  if ((long long)blockIdx.x < total) n_mv = moves[(int)(blockIdx.x / un.per_move)];
  for (long long c = blockIdx.x; c < total; c += gridDim.x) {
    const int m = (int)(c / un.per_move);
    const int r0 = (int)(c - (long long)m * un.per_move) * un.g;
    const cascade_move_t mv = n_mv;
    if (c + gridDim.x < total) n_mv = moves[(int)((c + gridDim.x) / un.per_move)];
    if (!move_ok(mv, pool.num_slots, staging_slots)) {
      flag_bad(status);
      continue;
    }
    copy_unit<kToStaging, kLg>(pool, mv.pool_slot, staging, mv.staging_slot, r0, un);
  }
}

// Pack and unpack chunks interleaved: the common range holds one pack and
// one unpack chunk per item pair, the rest belongs to the longer list.
// Unpack move m paired with pack move j (phz[j] == m and uhz[m] == j) is
// copied by the item of chunk (j, l, kv), in the same pass as the spill and
// by the same threads, each of which has read the slot's old bytes before it
// overwrites them: the wait is inside the thread, none crosses workgroups.
// The pairing test reads the same two words from both sides, so every
// unpack move is copied exactly once.
// Eight waves per SIMD: the prefetched move words would otherwise push the
// scalar registers past what eight waves can hold, and at seven the copy
// moves about 2 % fewer bytes per second (the prefetch gains about 1 % at
// eight, measured on MI355X).
template <int kLg>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void kvmove_kernel(
    cascade_kv_pool_t pool, Units un, char *pst, int pst_slots,
    const cascade_move_t *__restrict__ pm, const int *__restrict__ pn_dev, int pmax,
    const int *__restrict__ phz, char *ust, int ust_slots, const cascade_move_t *__restrict__ um,
    const int *__restrict__ un_dev, int umax, const int *__restrict__ uhz, int *status) {
  const int np = max(0, min(*pn_dev, pmax));
  const int nu = max(0, min(*un_dev, umax));
  const int per_move = un.per_move;
  const long long tp = (long long)np * per_move, tu = (long long)nu * per_move;
  const long long both = 2 * (tp < tu ? tp : tu), total = tp + tu;
  // the grid is even when it is below the item count, so c and
  // c ^ 1 fall in the same iteration: flipping the low bit on odd iterations
  // is a bijection that makes every workgroup alternate between pack and
  // unpack items, whatever share of the pack items carries a paired unpack
  const long long flip = (gridDim.x & 1) == 0 ? 1 : 0;
  // item c's list, move and chunk group
  auto item_of = [&](long long c, long long it, bool &is_pack, int &mi, int &r0) {
    long long ci;
    if (c < both) {
      const long long cc = c ^ (it & flip);
      is_pack = (cc & 1) == 0;
      ci = cc >> 1;
    } else {
      is_pack = tp > tu;
      ci = c - both + (both >> 1);
    }
    mi = (int)(ci / per_move);
    r0 = (int)(ci - (long long)mi * per_move) * un.g;
  };
  // each item's move and hazard word are requested one item ahead, while
  // the workgroup copies the item before it, so that no item starts with a
  // round trip in which the workgroup has no copy load in flight
  bool n_pack = false;
  int n_mi = 0, n_r0 = 0;
  cascade_move_t n_mv = {0, 0, 0, 0};
  int n_partner = -1;
  if ((long long)blockIdx.x < total) {
    item_of(blockIdx.x, 0, n_pack, n_mi, n_r0);
    n_mv = n_pack ? pm[n_mi] : um[n_mi];
    n_partner = n_pack ? phz[n_mi] : uhz[n_mi];
  }
  long long it = 0;
  for (long long c = blockIdx.x; c < total; c += gridDim.x, ++it) {
    const bool is_pack = n_pack;
    const int mi = n_mi, r0 = n_r0;
    const cascade_move_t mv = n_mv;
    const int partner = n_partner;
    if (c + gridDim.x < total) {
      item_of(c + gridDim.x, it + 1, n_pack, n_mi, n_r0);
      n_mv = n_pack ? pm[n_mi] : um[n_mi];
      n_partner = n_pack ? phz[n_mi] : uhz[n_mi];
    }
    if (is_pack) {
      const bool ok = move_ok(mv, pool.num_slots, pst_slots);
      if (!ok) flag_bad(status);
      bool paired = false;
      cascade_move_t mu;
      if (partner >= 0 && partner < nu) {
        mu = um[partner];
        paired = uhz[partner] == mi;
      }
      if (paired && !move_ok(mu, pool.num_slots, ust_slots)) {
        flag_bad(status);
        paired = false;  // the restore is skipped; the spill still runs
      }
      if (ok && paired && mu.pool_slot == mv.pool_slot) {
        copy_pair_unit<kLg>(pool, mv.pool_slot, pst, mv.staging_slot, ust, mu.staging_slot, r0,
                            un);
      } else {
        if (ok) copy_unit<true, kLg>(pool, mv.pool_slot, pst, mv.staging_slot, r0, un);
        if (paired) copy_unit<false, kLg>(pool, mu.pool_slot, ust, mu.staging_slot, r0, un);
      }
    } else {
      if (partner >= 0 && partner < np && phz[partner] == mi) continue;  // after its pack
      if (move_ok(mv, pool.num_slots, ust_slots))
        copy_unit<false, kLg>(pool, mv.pool_slot, ust, mv.staging_slot, r0, un);
      else
        flag_bad(status);
    }
  }
}

bool pool_ok(const cascade_kv_pool_t *p) {
  if (!p || !p->base || p->num_layers < 1 || p->num_slots < 0) return false;
  if (p->chunk_bytes < 16 || (p->chunk_bytes & 15) || p->chunk_bytes > (1ll << 30)) return false;
  if ((p->layer_stride & 15) || (p->kv_stride & 15) || (p->slot_stride & 15)) return false;
  if (p->layer_stride < 0 || p->kv_stride < 0 || p->slot_stride < 0) return false;
  return ((uintptr_t)p->base & 15) == 0;
}

bool list_ok(const void *staging, int32_t staging_slots, const cascade_move_t *moves,
             const int32_t *n_dev, int32_t max_moves) {
  if (!staging || !n_dev || max_moves < 0 || staging_slots < 0) return false;
  if (max_moves > 0 && !moves) return false;
  return ((uintptr_t)staging & 15) == 0;
}

Units units_for(const cascade_kv_pool_t *pool) {
  const long long vecs = pool->chunk_bytes >> 4;
  const int chunks = 2 * pool->num_layers;
  const int full = kBlock * kUnroll;  // vectors one thread batch covers
  for (int lg = 0; lg < 3; ++lg) {
    const int g = kUnroll >> lg;
    if (vecs == (kBlock << lg) && chunks % g == 0)
      return {g, lg, chunks / g, (unsigned)vecs, 0.0};
  }
  if (vecs % kBlock == 0 && vecs >= 3 * kBlock) return {1, kWhole, chunks, (unsigned)vecs, 0.0};
  return {1, kRun, (int)((vecs * chunks + full - 1) / full), (unsigned)vecs, 1.0 / (double)vecs};
}

int grid_for(const Units &u, long long moves) {
  const long long items = moves * u.per_move;
  long long g = std::max<long long>(1, std::min(items, kMaxGrid));
  if (g > 1 && (g & 1)) --g;  // even: the fused kernel alternates its lists by iteration
  return (int)g;
}

template <bool kToStaging>
int launch(const cascade_kv_pool_t *pool, const void *staging, int32_t staging_slots,
           const cascade_move_t *moves, const int32_t *n_dev, int32_t first, int32_t max_moves,
           int32_t *status, void *stream) {
  if (!pool_ok(pool) || !list_ok(staging, staging_slots, moves, n_dev, max_moves) || first < 0)
    return CASCADE_EINVAL;
  if (max_moves == 0) return CASCADE_OK;
  const Units u = units_for(pool);
  auto kernel = u.lg == kRun     ? kvcopy_kernel<kToStaging, kRun>
                : u.lg == kWhole ? kvcopy_kernel<kToStaging, kWhole>
                : u.lg == 0      ? kvcopy_kernel<kToStaging, 0>
                : u.lg == 1      ? kvcopy_kernel<kToStaging, 1>
                                 : kvcopy_kernel<kToStaging, 2>;
  hipLaunchKernelGGL(kernel, dim3(grid_for(u, max_moves)), dim3(kBlock), 0,
                     static_cast<hipStream_t>(stream), *pool, u,
                     const_cast<char *>(static_cast<const char *>(staging)), staging_slots,
                     moves + first, n_dev, first, max_moves, status);
  return hipGetLastError() == hipSuccess ? CASCADE_OK : CASCADE_EHIP;
}

}  // namespace

int cascade::copy_range(bool to_staging, const cascade_kv_pool_t *pool, const void *staging,
                        int32_t staging_slots, const cascade_move_t *moves,
                        const int32_t *n_moves_dev, int32_t first, int32_t max_moves,
                        int32_t *status_dev, void *stream) {
  return to_staging ? launch<true>(pool, staging, staging_slots, moves, n_moves_dev, first,
                                   max_moves, status_dev, stream)
                    : launch<false>(pool, staging, staging_slots, moves, n_moves_dev, first,
                                    max_moves, status_dev, stream);
}

extern "C" int cascade_pack(const cascade_kv_pool_t *pool, void *staging, int32_t staging_slots,
                            const cascade_move_t *moves, const int32_t *n_moves_dev,
                            int32_t max_moves, int32_t *status_dev, void *stream) {
  return launch<true>(pool, staging, staging_slots, moves, n_moves_dev, 0, max_moves,
                      status_dev, stream);
}

extern "C" int cascade_unpack(const cascade_kv_pool_t *pool, const void *staging,
                              int32_t staging_slots, const cascade_move_t *moves,
                              const int32_t *n_moves_dev, int32_t max_moves, int32_t *status_dev,
                              void *stream) {
  return launch<false>(pool, staging, staging_slots, moves, n_moves_dev, 0, max_moves,
                       status_dev, stream);
}

extern "C" int cascade_pack_unpack(const cascade_kv_pool_t *pool, void *pack_staging,
                                   int32_t pack_staging_slots, const cascade_move_t *pack_moves,
                                   const int32_t *n_pack_dev, int32_t max_pack,
                                   const int32_t *pack_hazard, const void *unpack_staging,
                                   int32_t unpack_staging_slots,
                                   const cascade_move_t *unpack_moves,
                                   const int32_t *n_unpack_dev, int32_t max_unpack,
                                   const int32_t *unpack_hazard, int32_t *status_dev,
                                   void *stream) {
  if (!pool_ok(pool) ||
      !list_ok(pack_staging, pack_staging_slots, pack_moves, n_pack_dev, max_pack) ||
      !list_ok(unpack_staging, unpack_staging_slots, unpack_moves, n_unpack_dev, max_unpack))
    return CASCADE_EINVAL;
  if ((max_pack > 0 && !pack_hazard) || (max_unpack > 0 && !unpack_hazard)) return CASCADE_EINVAL;
  if (max_pack == 0 && max_unpack == 0) return CASCADE_OK;
  const Units u = units_for(pool);
  auto kernel = u.lg == kRun     ? kvmove_kernel<kRun>
                : u.lg == kWhole ? kvmove_kernel<kWhole>
                : u.lg == 0      ? kvmove_kernel<0>
                : u.lg == 1      ? kvmove_kernel<1>
                                 : kvmove_kernel<2>;
  hipLaunchKernelGGL(kernel, dim3(grid_for(u, (long long)max_pack + max_unpack)),
                     dim3(kBlock), 0, static_cast<hipStream_t>(stream), *pool, u,
                     static_cast<char *>(pack_staging), pack_staging_slots, pack_moves,
                     n_pack_dev, max_pack, pack_hazard,
                     const_cast<char *>(static_cast<const char *>(unpack_staging)),
                     unpack_staging_slots, unpack_moves, n_unpack_dev, max_unpack, unpack_hazard,
                     status_dev);
  return hipGetLastError() == hipSuccess ? CASCADE_OK : CASCADE_EHIP;
}
