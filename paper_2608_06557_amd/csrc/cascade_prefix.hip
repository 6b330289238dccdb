// cascade_prefix.hip -- prefix-hit lookup on gfx950 (Section 4.4, prefix hit
// detection).
//
// On top of per-block prefix hashing, an index records for every cached KV
// block the tiers holding it, of which the lookup reads the deepest (per-tier
// reclamation removes a tier's copy: cascade_reclaim.hip).  A request's
// prefix-hit profile is the longest run of its leading blocks present in the
// index (capped so that at least one prompt token is computed) and the
// deepest tier over that run: the n_prefix / prefix_tier inputs of the
// scheduling step.
//
// The index is an open-addressing hash table of 16-byte slots (key, set of
// tiers holding the block) in device memory (index_table.h); key 0 marks an
// empty slot.  Insert claims a slot with a 64-bit CAS on the key and adds the
// tier to the set; the block's deepest tier is the highest tier in its set.
// The probe gives each request one wave, which looks up its leading blocks
// in windows that grow while every block hits; a ballot finds the first miss
// (a block absent, or whose set is empty), and the wave stops there.  Very long
// runs, and every request of a short queue, have several waves, whose windows
// lie side by side.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include <algorithm>

#include "cascade.h"
#include "device_util.h"
#include "index_table.h"

namespace cascade {
namespace {

__global__ __launch_bounds__(kBlock) void index_clear_kernel(uint4 *slots, long long n_vec) {
  for (long long j = (long long)blockIdx.x * kBlock + threadIdx.x; j < n_vec;
       j += (long long)gridDim.x * kBlock)
    slots[j] = make_uint4(0, 0, 0, 0);
}

// One thread per (hash, tier) fact.  A new block claims its slot by a CAS on the
// key and then stores its tier: nobody else writes a claimed slot's set before
// that store is there, so it needs no atomic.  The others that find the key add
// their tier with atomicOr once the set holds a tier (no insert takes one out) or
// the slot has the mark of a reclamation, and look again until then.  A wave's
// claims are stored before any of its lanes waits for a tier, and none waits on
// the way to its slot, so every wait ends.
// Random device atomics run at about 25 G a second, reads at 50 G, and a second
// atomic on a slot is dearer than the first, since by then hundreds of thousands
// of other lines have passed through the L2s.  So many facts (kLook) read a slot
// before they claim it, and a known fact costs the read alone: 1.85 M facts into
// an empty index, 30 % of them second tiers, 140 us (CAS then atomicOr 200), when
// all are known 41 (197).  Few facts are bound by the chain of round trips and
// claim at once, their tiers stored behind the chain, which would wait for them:
// into an empty index of twice their number and one of 4 M slots, 1000 facts take
// 7.4 and 5.4 us (reading first 11.4 and 5.7, CAS then atomicOr 6.8 and 5.1), 8400
// 5.6 and 5.8 (7.8, 5.7; 5.3, 5.2), 115000 18.3 and 10.9 (22.7, 14.7; 19.4, 12.4),
// 300000 21.3 and 23.4 (26.7, 33.8; 30.3, 28.5).  Both ways may work on one index
// at the same time.
template <bool kLook>
__global__ __launch_bounds__(kBlock) void index_insert_kernel(IndexSlot *slots, unsigned mask,
                                                              const unsigned long long *hashes,
                                                              const uint8_t *tiers, int n,
                                                              int *status) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  const bool in = i < n;
  const unsigned long long h = in ? hashes[i] : 0ull;
  const unsigned t = in ? tiers[i] : 0u;
  bool done = h == 0 || t > CASCADE_KV_NVME;
  if (in && done && status) store_agent(status, (int)CASCADE_EINVAL);
  const unsigned bit = done ? 0u : 1u << t;
  unsigned s = (unsigned)fmix64(h) & mask, p = 0, polls = 0;
  unsigned long long set = 0ull;  // of the slot whose key is h, as far as known
  bool claimed = false;
  while (!done) {  // to the key's slot: no lane waits for another here
    IndexSlot *e = slots + s;
    unsigned long long k = 0ull;
    if (kLook) {
      k = load_agent(&e->key);
      set = load_agent(&e->set_word);
    }
    if (k == 0ull) {
      k = atomicCAS(&e->key, 0ull, h);
      claimed = k == 0ull;
      set = 0ull;
      if (kLook && claimed) store_agent(&e->tiers, bit);
    }
    if (claimed || k == h) break;
    if (p == mask) {  // every slot holds another key
      if (status) store_agent(status, (int)CASCADE_ENOSPC);
      done = true;
    }
    ++p;
    s = (s + 1) & mask;
  }
  IndexSlot *e = slots + s;
  if (claimed) {
    if (!kLook) store_agent(&e->tiers, bit);
    done = true;
  }
  while (__ballot(!done) != 0) {  // uniform over the wave: its own claims are stored
    if (!done) {
      if ((unsigned)set & bit) {
        done = true;
      } else if (set != 0ull || ++polls > kSpinLimit) {
        // the bound is for index memory whose emptied slots have no mark
        atomicOr(&e->tiers, bit);
        done = true;
      } else {
        set = kLook ? load_agent(&e->set_word) : atomicCAS(&e->set_word, 0ull, 0ull);
      }
    }
  }
}

// Facts from which on the slot is read first; half as many in an index of less than
// four slots a fact, as one built anew has.  Facts that are all known already are
// faster so from a few thousand on (115000: 4.7 against 11.4 us), new ones where they
// are many second tiers or fill the index: into an index of twice their number,
// without and with 30 % second tiers, 262144 facts take 35.7 and 28.6 us (claiming at
// once 33.7 and 28.9, CAS then atomicOr 39.9 and 29.9), 460000 44.2 and 36.3 (46.8
// and 49.0; 60.2 and 50.1); into 4 M slots 262144 take 27.2 and 25.0 (20.1 and 22.5;
// 24.7 and 24.4), 524287 53.2 and 47.4 (40.8 and 46.6; 53.4 and 51.9).  So from here
// on neither is slower than CAS then atomicOr.
constexpr int kLookFacts = 1 << 19;

// Lookups per lane in a probe window, at most: the window doubles from 64
// blocks (one per lane) up to 64 * kProbeMaxK.
constexpr int kProbeMaxK = 4;
// Whether a lookup also requests the slot after its home slot when both lie
// in one 128-byte line (8 slots): that read costs no extra line and decides
// most keys that sit one past their home.
constexpr bool kProbePair = true;

// Examines slot v for key h when go: returns true when that decides the
// lookup (key found, or an empty slot ends the probe sequence), and then sets
// hit (the key is there and its tier set is not empty) and t (its deepest
// tier).  Branch-free, so that the compiler keeps each slot a single load.
__device__ __forceinline__ bool examine_slot(const uint4 &v, unsigned long long h, bool go,
                                             bool &hit, unsigned &t) {
  const unsigned long long k = (unsigned long long)v.x | ((unsigned long long)v.y << 32);
  const bool match = go && k == h;
  hit = match ? v.z != 0u : hit;
  t = (match && v.z != 0u) ? 31u - (unsigned)__builtin_clz(v.z | 1u) : t;
  return go && (k == h || k == 0ull);
}

// One wave's window of a request's lookup: 64 * K leading blocks from `base`,
// K per lane (lane l, item u: block base + 64 u + l), whose hashes h[0..K) the
// previous window requested.  Every home slot is requested at once (and, with
// kProbePair, the slot after it when both lie in one line), then the hashes of
// the wave's next window, which starts at nbase, before any slot is examined;
// the keys past what was read continue slot by slot, all together.  Every load
// is issued and none under a branch, so that they are all in flight together:
// the unwanted ones read the anchor, the slot that lane 0 looks up first (one
// line per wave, requested anyway), and are ignored.  A ballot per item finds
// the window's first miss (a block absent, or whose set is empty), returned as
// its position in the window (64 * K: none).  deepest takes in the deepest tier
// before it, zero gets bit u where the lane's item u has hash 0 (reserved for
// empty slots: a miss); h then holds the next window's hashes.
template <int K, int KM>
__device__ __forceinline__ int probe_window(const uint4 *__restrict__ sl, unsigned mask,
                                            const unsigned long long *__restrict__ hb, int lim,
                                            int base, int nbase, int lane,
                                            unsigned long long (&h)[KM], unsigned &deepest,
                                            unsigned &zero) {
  constexpr int KN = K < KM ? 2 * K : KM;  // items per lane of the next window
  constexpr int win = 64 * K;
  unsigned long long hc[K];
  bool want[K], look[K], pair[K], hit[K];
  unsigned s[K], t[K];
  uint4 v[K], w[K];
#pragma unroll
  for (int u = 0; u < K; ++u) {
    hc[u] = h[u];
    want[u] = base + u * 64 + lane < lim;
    look[u] = want[u] && hc[u] != 0ull;
    zero |= (want[u] && !look[u]) ? 1u << u : 0u;
    s[u] = (unsigned)fmix64(hc[u]) & mask;
  }
  const unsigned anchor = (unsigned)__builtin_amdgcn_readfirstlane((int)s[0]);
#pragma unroll
  for (int u = 0; u < K; ++u) {
    v[u] = sl[look[u] ? s[u] : anchor];
    pair[u] = kProbePair && look[u] && (s[u] & 7u) != 7u;  // s + 1 <= mask then
    if (kProbePair) w[u] = sl[pair[u] ? s[u] + 1u : anchor];
  }
#pragma unroll
  for (int u = 0; u < KN; ++u) {
    const int j = nbase + u * 64 + lane;
    h[u] = j < lim ? hb[j] : 0ull;
  }
  unsigned pend = 0u;
#pragma unroll
  for (int u = 0; u < K; ++u) {
    hit[u] = false;
    t[u] = 0u;
    const bool d1 = examine_slot(v[u], hc[u], look[u], hit[u], t[u]);
    const bool go2 = pair[u] && !d1;
    const bool d2 = kProbePair && examine_slot(w[u], hc[u], go2, hit[u], t[u]);
    s[u] = go2 ? s[u] + 1u : s[u];
    pend |= (look[u] && !d1 && !d2) ? 1u << u : 0u;
  }
  for (unsigned p = 1; p <= mask && __ballot(pend != 0u) != 0; ++p) {  // mask + 1 slots
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const bool go = (pend >> u) & 1u;
      s[u] = go ? (s[u] + 1u) & mask : s[u];
      v[u] = sl[go ? s[u] : anchor];
    }
    unsigned left = pend;
#pragma unroll
    for (int u = 0; u < K; ++u)
      left &= examine_slot(v[u], hc[u], (pend >> u) & 1u, hit[u], t[u]) ? ~(1u << u) : ~0u;
    pend = left;
  }
  // a lookup still pending has visited every slot: the key is absent
  int first = win;  // window position of the first miss
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const uint64_t miss = __ballot(want[u] && !hit[u]);
    if (first == win && miss) first = u * 64 + __builtin_ctzll(miss);
  }
  unsigned tm = 0u;
#pragma unroll
  for (int u = 0; u < K; ++u)
    tm = (want[u] && hit[u] && u * 64 + lane < first && t[u] > tm) ? t[u] : tm;
  deepest = max(deepest, (unsigned)wave_max((unsigned long long)tm));
  return first;
}

// The CSR bounds of request i: its hashes' first index and how many of them
// count (0 with bad set when the request is invalid).  Every read of a hash
// stays in [0, offsets[n]), the caller's array, even when another request's
// offsets are out of order.
__device__ __forceinline__ int request_limit(int i, int n, const int *__restrict__ offsets,
                                             const int *__restrict__ n_in, int bt, int &b0,
                                             bool &bad) {
  const int b1 = offsets[i + 1], total = offsets[n], nin = n_in[i];
  b0 = offsets[i];
  bad = b0 < 0 || b1 < b0 || b1 > total || nin < 1 || (i == 0 && b0 != 0);
  if (bad) b0 = 0;
  const int have = bad ? 0 : b1 - b0, cap = bad ? 0 : (nin - 1) / bt;
  return have < cap ? have : cap;
}

// A wave's windows start at blocks 0, 64, 192, 448, 704, ...: the end of the
// window that block b lies in.  A hash 0 is reported when it lies before the
// end of the window that holds the run's first miss, whichever kernel finds it.
__device__ __forceinline__ int window_end(int b) {
  return b < 64 ? 64 : b < 192 ? 192 : 448 + (b < 448 ? 0 : (b - 448) / 256 * 256 + 256);
}

// Lookups of one request by `nw` waves of a workgroup (`g0` the first of them),
// from block `base` (a window's start, every earlier block cached): rounds of nw
// adjacent windows of 64 * kProbeMaxK blocks, one per wave, until a round holds
// a miss or the request ends.  Every wave of the workgroup calls it (lim 0: no
// request), and a round's one barrier is also what ends the loop for all of them
// at once; with kOne they share one request, and its last round ends it.  Returns
// the run's length; s_round holds the answers of two rounds.  bad (a hash 0 that
// counts) is complete in the first wave, which reports it.
struct WaveAnswer {
  int miss, zero;  // first missing block, first hash 0 (INT_MAX: none)
  unsigned deepest;
  int active;      // the wave's request was not decided before this round
};
// The answer of a wave's window of K items per lane from block `at`.
template <int K>
__device__ __forceinline__ WaveAnswer wave_answer(int at, int first, unsigned z, unsigned deepest,
                                                  bool active) {
  int zero = INT_MAX;
  if (__ballot(z != 0u)) {  // invalid input
#pragma unroll
    for (int u = K - 1; u >= 0; --u) {
      const uint64_t m = __ballot((z >> u) & 1u);
      if (m) zero = at + u * 64 + __builtin_ctzll(m);
    }
  }
  return {first < 64 * K ? at + first : INT_MAX, zero, deepest, (int)active};
}

template <bool kOne>
__device__ __forceinline__ int probe_wide(const uint4 *__restrict__ sl, unsigned mask,
                                          const unsigned long long *__restrict__ hb, int lim,
                                          int base, int g0, int nw,
                                          WaveAnswer (&s_round)[2][kWaves], unsigned &deepest,
                                          bool &bad) {
  constexpr int K = kProbeMaxK, win = 64 * K;
  const int lane = lane_id(), wave = wave_id();
  unsigned long long h[K];
  int wb = base + (wave - g0) * win, run = 0, first_zero = INT_MAX;
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const int j = wb + u * 64 + lane;
    h[u] = j < lim ? hb[j] : 0ull;
  }
  bool active = base < lim;
  for (int r = 0;; r ^= 1) {  // uniform over the workgroup
    unsigned d = 0u, z = 0u;
    int first = win;
    if (active && wb < lim)  // uniform over the wave
      first = probe_window<K, K>(sl, mask, hb, lim, wb, wb + nw * win, lane, h, d, z);
    const WaveAnswer mine = wave_answer<K>(wb, first, z, d, active);
    if (lane == 0) s_round[r][wave] = mine;
    __syncthreads();
    int miss = INT_MAX, any = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const WaveAnswer a = s_round[r][w];
      any |= a.active;
      if (w < g0 || w >= g0 + nw) continue;
      if (active && miss == INT_MAX) deepest = max(deepest, a.deepest);  // none past the miss
      miss = min(miss, a.miss);
      first_zero = min(first_zero, a.zero);
    }
    if (!kOne && !any) return run;
    base += nw * win;
    wb += nw * win;
    if (active && (miss != INT_MAX || base >= lim)) {
      if (miss != INT_MAX) {
        // the miss's window may reach past the round: into the hashes that the
        // first wave holds for the next one
        const int end = min(window_end(miss), lim);
        bool z = first_zero < end;
#pragma unroll
        for (int u = 0; u < K; ++u) z = z || (wb + u * 64 + lane < end && h[u] == 0ull);
        bad = bad || __ballot(z) != 0;
      }
      run = miss != INT_MAX ? miss : lim;
      if (kOne) return run;
      active = false;
    }
  }
}

// A request of up to kWaves * 64 * K blocks in one round, a window of 64 * K
// blocks per wave: as probe_wide with kOne.
template <int K>
__device__ __forceinline__ int probe_once(const uint4 *__restrict__ sl, unsigned mask,
                                          const unsigned long long *__restrict__ hb, int lim,
                                          WaveAnswer (&s_round)[kWaves], unsigned &deepest,
                                          bool &bad) {
  const int lane = lane_id(), at = wave_id() * 64 * K;
  unsigned long long h[K];
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const int j = at + u * 64 + lane;
    h[u] = j < lim ? hb[j] : 0ull;
  }
  unsigned d = 0u, z = 0u;
  int first = 64 * K;
  if (at < lim)  // uniform over the wave
    first = probe_window<K, K>(sl, mask, hb, lim, at, lim, lane, h, d, z);
  const WaveAnswer mine = wave_answer<K>(at, first, z, d, true);
  if (lane == 0) s_round[wave_id()] = mine;
  __syncthreads();
  int miss = INT_MAX, zero = INT_MAX;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const WaveAnswer a = s_round[w];
    if (miss == INT_MAX) deepest = max(deepest, a.deepest);  // none past the miss
    miss = min(miss, a.miss);
    zero = min(zero, a.zero);
  }
  if (miss == INT_MAX) return lim;
  bad = bad || zero < min(window_end(miss), lim);
  return miss;
}

// One wave per request.  Its leading blocks are looked up in windows of
// 64 * k blocks, k doubling from 1 to kProbeMaxK while every block hits, so a
// short run (most of them) costs one small window, and the wave stops at the
// first miss: blocks past it in later windows cost nothing.
// From block kProbeTail on the workgroup's waves share the requests that are left
// among them: window after window in one wave, the longest runs (5000 blocks)
// outlast the rest of the launch.  A workgroup without a prompt that long does not
// wait for its slowest wave (16384 chat requests 25.1 us, 26.1 with that wait).
// Chat and agentic prompts, this against every request alone in its wave: 16384
// requests 75 against 103 us, 32768 139 against
// 181, 65536 191 against 208.  Starting to share at block 960 measured 70, 157
// and 184 us there, but 700 against 664 us (1984: 660) where half the prompts are
// long ones and the chip is full without it: the waves' windows past the miss
// then take the place of others' lookups.  72 registers (7 waves a SIMD) against
// 76 (6): 185 against 194 us at 65536; 64 (8) spill, 215 us.
constexpr int kProbeTail = 1984;
__global__ __launch_bounds__(kBlock, 7) void probe_kernel(const IndexSlot *__restrict__ slots,
                                                       unsigned mask, int n,
                                                       const int *__restrict__ offsets,
                                                       const unsigned long long *__restrict__ hashes,
                                                       const int *__restrict__ n_in, int bt,
                                                       int *__restrict__ n_prefix_out,
                                                       uint8_t *__restrict__ tier_out,
                                                       int *status) {
  constexpr int KM = kProbeMaxK;
  static_assert(KM == 4, "window_end");
  const int i = blockIdx.x * kWaves + wave_id();
  const int lane = lane_id();
  const uint4 *sl = reinterpret_cast<const uint4 *>(slots);
  // lane w: the workgroup's request w.  Only runs that may reach block kProbeTail
  // make the waves meet there.
  int b0 = 0, lim = 0;
  bool bad = false;
  if (lane < kWaves && i - wave_id() + lane < n)
    lim = request_limit(i - wave_id() + lane, n, offsets, n_in, bt, b0, bad);
  const bool meet = __ballot(lim > kProbeTail) != 0;  // uniform over the workgroup
  bad = (__ballot(bad) >> wave_id()) & 1;
  lim = __builtin_amdgcn_readlane(lim, __builtin_amdgcn_readfirstlane(wave_id()));
  b0 = __builtin_amdgcn_readlane(b0, __builtin_amdgcn_readfirstlane(wave_id()));
  const unsigned long long *hb = hashes + b0;
  int matched = 0;
  unsigned deepest = 0, zero = 0;
  unsigned long long h[KM];
#pragma unroll
  for (int u = 0; u < KM; ++u) h[u] = (u == 0 && lane < lim) ? hb[lane] : 0ull;
  int base = 0, k = 1;
  bool done = lim <= 0;
  while (!done && base < kProbeTail) {  // uniform over the wave
    const int nbase = base + 64 * k;
    int first;
    if (k == 1)
      first = probe_window<1, KM>(sl, mask, hb, lim, base, nbase, lane, h, deepest, zero);
    else if (k == 2)
      first = probe_window<2, KM>(sl, mask, hb, lim, base, nbase, lane, h, deepest, zero);
    else
      first = probe_window<KM, KM>(sl, mask, hb, lim, base, nbase, lane, h, deepest, zero);
    done = first < 64 * k || nbase >= lim;
    matched = first < 64 * k ? base + first : min(nbase, lim);
    base = nbase;
    k = k < KM ? 2 * k : KM;
  }
  bad = bad || __ballot(zero != 0u) != 0;
  __shared__ int s_lim[kWaves], s_b0[kWaves];
  __shared__ unsigned s_deep[kWaves];
  __shared__ WaveAnswer s_round[2][kWaves];
  if (lane == 0) {
    s_lim[wave_id()] = done ? 0 : lim;
    s_b0[wave_id()] = b0;
    s_deep[wave_id()] = deepest;
    if (done && i < n) {
      if (bad && status) store_agent(status, (int)CASCADE_EINVAL);
      n_prefix_out[i] = matched * bt;
      tier_out[i] = (uint8_t)(matched > 0 ? deepest : (unsigned)CASCADE_KV_NONE);
    }
  }
  if (!meet) return;
  __syncthreads();
  // m requests are left: the j-th of them takes (kWaves + m - 1 - j) / m waves
  int m = 0, req = -1, g0 = 0, nw = 1;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) m += s_lim[w] > 0 ? 1 : 0;
  if (m == 0) return;  // uniform over the workgroup
  int at = 0, j = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (s_lim[w] <= 0) continue;
    const int q = (kWaves + m - 1 - j) / m;
    if (wave_id() >= at && wave_id() < at + q) {
      req = w;
      g0 = at;
      nw = q;
    }
    at += q;
    ++j;
  }
  deepest = s_deep[req];
  const int run = probe_wide<false>(sl, mask, hashes + s_b0[req], s_lim[req], kProbeTail, g0,
                                    nw, s_round, deepest, bad);
  if (lane == 0 && wave_id() == g0) {
    const int o = blockIdx.x * kWaves + req;
    if (bad && status) store_agent(status, (int)CASCADE_EINVAL);
    n_prefix_out[o] = run * bt;
    tier_out[o] = (uint8_t)deepest;
  }
}

// One workgroup per request, from its first block: every wave's window at once
// costs lookups past the miss, but few requests leave the chip idle, and then
// the number of dependent rounds is the time.  Chat and agentic requests, against
// one wave each: 64 of them 16 against 21 us, 512 12 against 30, 1024 22 against
// 45, 2048 30 against 48.  Longer queues fill the chip: at 8192 short prompts 27
// against 17 us (long ones 52 against 48).  A prompt of up to 256 or 512 blocks
// takes one round of windows of 64 or 128: it need not wait for the slots of blocks
// far behind its miss.  64 chat requests 3.7 us (windows of 256 6.8, one wave each
// 4.7), 256 4.5 (8.4, 6.2), 2048 6.2 (10.3, 8.6).
__global__ __launch_bounds__(kBlock) void probe_wide_kernel(
    const IndexSlot *__restrict__ slots, unsigned mask, int n, const int *__restrict__ offsets,
    const unsigned long long *__restrict__ hashes, const int *__restrict__ n_in, int bt,
    int *__restrict__ n_prefix_out, uint8_t *__restrict__ tier_out, int *status) {
  __shared__ WaveAnswer s_round[2][kWaves];
  const int i = blockIdx.x;
  int b0;
  bool bad;
  const int lim = request_limit(i, n, offsets, n_in, bt, b0, bad);
  const uint4 *sl = reinterpret_cast<const uint4 *>(slots);
  const unsigned long long *hb = hashes + b0;
  unsigned deepest = 0u;
  int run = 0;
  if (lim > kWaves * 128)
    run = probe_wide<true>(sl, mask, hb, lim, 0, 0, kWaves, s_round, deepest, bad);
  else if (lim > kWaves * 64)
    run = probe_once<2>(sl, mask, hb, lim, s_round[0], deepest, bad);
  else if (lim > 0)
    run = probe_once<1>(sl, mask, hb, lim, s_round[0], deepest, bad);
  if (threadIdx.x == 0) {
    if (bad && status) store_agent(status, (int)CASCADE_EINVAL);
    n_prefix_out[i] = run * bt;
    tier_out[i] = (uint8_t)(run > 0 ? deepest : (unsigned)CASCADE_KV_NONE);
  }
}

constexpr int kWideReqs = 2048;  // the queues that one workgroup per request pays for

bool capacity_ok(int32_t capacity) {
  return capacity >= 64 && capacity <= (1 << 30) && (capacity & (capacity - 1)) == 0;
}

}  // namespace
}  // namespace cascade

using namespace cascade;

extern "C" size_t cascade_prefix_index_bytes(int32_t capacity) {
  return capacity_ok(capacity) ? (size_t)capacity * CASCADE_INDEX_SLOT_BYTES : 0;
}

extern "C" int cascade_prefix_index_clear(void *index, int32_t capacity, void *stream) {
  if (!index || !capacity_ok(capacity) || ((uintptr_t)index & 15)) return CASCADE_EINVAL;
  const long long n_vec = (long long)capacity;  // one 16-byte vector per slot
  const int grid = (int)std::min<long long>((n_vec + kBlock - 1) / kBlock, 4096);
  hipLaunchKernelGGL(index_clear_kernel, dim3(grid), dim3(kBlock), 0,
                     static_cast<hipStream_t>(stream), static_cast<uint4 *>(index), n_vec);
  return hipGetLastError() == hipSuccess ? CASCADE_OK : CASCADE_EHIP;
}

extern "C" int cascade_prefix_index_insert(void *index, int32_t capacity, const uint64_t *hashes,
                                           const uint8_t *tiers, int32_t n, int32_t *status_dev,
                                           void *stream) {
  if (!index || !capacity_ok(capacity) || ((uintptr_t)index & 15) || n < 0) return CASCADE_EINVAL;
  if (n == 0) return CASCADE_OK;
  if (!hashes || !tiers) return CASCADE_EINVAL;
  const bool look = n >= kLookFacts || (n >= kLookFacts / 2 && capacity / 4 < n);
  hipLaunchKernelGGL(look ? index_insert_kernel<true> : index_insert_kernel<false>,
                     dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0,
                     static_cast<hipStream_t>(stream), static_cast<IndexSlot *>(index),
                     (unsigned)(capacity - 1), reinterpret_cast<const unsigned long long *>(hashes),
                     tiers, n, status_dev);
  return hipGetLastError() == hipSuccess ? CASCADE_OK : CASCADE_EHIP;
}

extern "C" int cascade_prefix_probe(const void *index, int32_t capacity, int32_t n,
                                    const int32_t *block_offsets, const uint64_t *block_hashes,
                                    const int32_t *n_in, int32_t block_tokens,
                                    int32_t *n_prefix_out, uint8_t *prefix_tier_out,
                                    int32_t *status_dev, void *stream) {
  if (!index || !capacity_ok(capacity) || ((uintptr_t)index & 15) || n < 0 || block_tokens < 1)
    return CASCADE_EINVAL;
  if (n == 0) return CASCADE_OK;
  if (!block_offsets || !block_hashes || !n_in || !n_prefix_out || !prefix_tier_out)
    return CASCADE_EINVAL;
  const IndexSlot *slots = static_cast<const IndexSlot *>(index);
  const unsigned long long *hashes = reinterpret_cast<const unsigned long long *>(block_hashes);
  const unsigned mask = (unsigned)(capacity - 1);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (n <= kWideReqs) {
    hipLaunchKernelGGL(probe_wide_kernel, dim3(n), dim3(kBlock), 0, s, slots, mask, n,
                       block_offsets, hashes, n_in, block_tokens, n_prefix_out, prefix_tier_out,
                       status_dev);
  } else {
    hipLaunchKernelGGL(probe_kernel, dim3((n + kWaves - 1) / kWaves), dim3(kBlock), 0, s, slots,
                       mask, n, block_offsets, hashes, n_in, block_tokens, n_prefix_out,
                       prefix_tier_out, status_dev);
  }
  return hipGetLastError() == hipSuccess ? CASCADE_OK : CASCADE_EHIP;
}
