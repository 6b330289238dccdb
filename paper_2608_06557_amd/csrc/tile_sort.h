// tile_sort.h -- sorting of distinct 64-bit keys inside a wave64 and a
// workgroup, for the step's order on gfx950.  Internal to the library.
//
// A wave sorts its 64 keys in registers with a bitonic network whose lane
// exchanges are DPP moves (only the three exchanges that cross a row of 16
// lanes go through the LDS crossbar).  A workgroup then merges the sorted
// runs pairwise in LDS: every key finds its place in the other run of its
// pair by a branch-free search, so a level costs about log2(run) / 2 dependent
// LDS round trips and one barrier, whatever the keys are.  Both are bound by the
// latency of that chain, not by the number of compares.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_util.h"

namespace cascade {

enum : int {
  kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppXor3 = 0x1B,  // quad permutes
  kDppXor7 = 0x141, kDppXor15 = 0x140, kDppXor8 = 0x128  // half mirror, mirror, rotate by 8
};
template <int kCtrl>
__device__ __forceinline__ unsigned dpp_perm(unsigned x) {
  return (unsigned)__builtin_amdgcn_mov_dpp((int)x, kCtrl, 0xf, 0xf, true);
}

// The value of lane (lane ^ M).
template <int M>
__device__ __forceinline__ unsigned lane_xor(unsigned x) {
  if constexpr (M == 1) return dpp_perm<kDppXor1>(x);
  else if constexpr (M == 2) return dpp_perm<kDppXor2>(x);
  else if constexpr (M == 3) return dpp_perm<kDppXor3>(x);
  else if constexpr (M == 4) return dpp_perm<kDppXor3>(dpp_perm<kDppXor7>(x));
  else if constexpr (M == 7) return dpp_perm<kDppXor7>(x);
  else if constexpr (M == 8) return dpp_perm<kDppXor8>(x);
  else if constexpr (M == 15) return dpp_perm<kDppXor15>(x);
  else if constexpr (M == 16 || M == 31)
    return (unsigned)__builtin_amdgcn_ds_swizzle((int)x, (M << 10) | 0x1f);
  else
    return (unsigned)__shfl_xor((int)x, M, 64);
}

// Compare-exchange with lane ^ M: the lane whose top bit of M is clear keeps
// the smaller key.
template <int M>
__device__ __forceinline__ void exchange(unsigned long long &k) {
  constexpr int kTop = M >= 32 ? 32 : M >= 16 ? 16 : M >= 8 ? 8 : M >= 4 ? 4 : M >= 2 ? 2 : 1;
  const unsigned long long o = ((unsigned long long)lane_xor<M>((unsigned)(k >> 32)) << 32) |
                               lane_xor<M>((unsigned)k);
  const bool low = (lane_id() & kTop) == 0;
  k = (o < k) == low ? o : k;
}

// Ascending sort of the wave's 64 keys, one per lane.  Each merge of two
// ascending runs starts with a mirrored exchange (lane ^ (2L - 1)), so every
// run stays ascending.  Equal keys (padding) are allowed here.
__device__ __forceinline__ void wave_sort(unsigned long long &k) {
  exchange<1>(k);
  exchange<3>(k), exchange<1>(k);
  exchange<7>(k), exchange<2>(k), exchange<1>(k);
  exchange<15>(k), exchange<4>(k), exchange<2>(k), exchange<1>(k);
  exchange<31>(k), exchange<8>(k), exchange<4>(k), exchange<2>(k), exchange<1>(k);
  exchange<63>(k), exchange<16>(k), exchange<8>(k), exchange<4>(k), exchange<2>(k),
      exchange<1>(k);
}

// Where each of K keys, key[k] at place q[k] of m keys in sorted runs of L (a
// power of two; the last run may be short), goes when the runs are merged in
// pairs.  With kWide the search reads three keys per round trip, which halves
// the chain of a binary one; the K searches advance together.
template <int K, bool kWide>
__device__ __forceinline__ void merge_place(const unsigned long long *run, const int (&q)[K],
                                            int L, int m, const unsigned long long (&key)[K],
                                            int (&place)[K]) {
  int other[K], len[K], below[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    place[k] = q[k] & ~(2 * L - 1);
    other[k] = place[k] + ((q[k] & L) ? 0 : L);
    len[k] = min(L, m - other[k]);  // of the other run, below 1 past the end
    below[k] = 0;
  }
  auto less = [&](int k, int mid) {  // is the run's mid-th key (from 1) below key k?
    const bool in = mid <= len[k];
    const unsigned long long o = run[in ? other[k] + mid - 1 : q[k]];
    return in && o < key[k];
  };
  int h = L;
  if (!kWide) {
    for (; h > 0; h >>= 1) {
#pragma unroll
      for (int k = 0; k < K; ++k) below[k] += less(k, below[k] + h) ? h : 0;
    }
  } else if (__builtin_ctz(L) % 2 == 0) {  // an odd number of binary steps L, L/2, .., 1
#pragma unroll
    for (int k = 0; k < K; ++k) below[k] = less(k, L) ? L : 0;
    h = L / 2;
  }
  for (h >>= 1; h > 0; h >>= 2) {
    bool c1[K], c2[K], c3[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      c1[k] = less(k, below[k] + h);
      c2[k] = less(k, below[k] + 2 * h);
      c3[k] = less(k, below[k] + 3 * h);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) below[k] += c3[k] ? 3 * h : (c2[k] ? 2 * h : (c1[k] ? h : 0));
  }
#pragma unroll
  for (int k = 0; k < K; ++k) place[k] += (q[k] & (L - 1)) + below[k];
}

// Merges m distinct keys in sorted runs of 64 in a[0, m) into one, between
// the buffers a and b; called by all N threads of the workgroup, returns the
// buffer that holds the result (complete for every thread).  A thread takes
// two keys at a time where its wave has two.  Up to 8 waves wait on the chain
// of searches, so they search three keys wide; 16 waves keep the LDS busy, and
// the binary search reads fewer keys.
template <int N>
__device__ __forceinline__ unsigned long long *merge_runs(unsigned long long *a,
                                                          unsigned long long *b, int m) {
  __syncthreads();
  for (int L = 64; L < m; L <<= 1) {
    for (int q0 = threadIdx.x; q0 < m; q0 += 2 * N) {
      if (q0 - lane_id() + N < m) {
        const int q[2] = {q0, min(q0 + N, m - 1)};
        const unsigned long long key[2] = {a[q[0]], a[q[1]]};
        int place[2];
        merge_place<2, (N <= 512)>(a, q, L, m, key, place);
        b[place[0]] = key[0];
        b[place[1]] = key[1];  // the last key again from the lanes past it
      } else {
        const int q[1] = {q0};
        const unsigned long long key[1] = {a[q0]};
        int place[1];
        merge_place<1, (N <= 512)>(a, q, L, m, key, place);
        b[place[0]] = key[0];
      }
    }
    __syncthreads();
    unsigned long long *x = a;
    a = b;
    b = x;
  }
  return a;
}

}  // namespace cascade
