// nopfs_buffer_sim: a clairvoyant buffer of d0 bytes per worker (the
// replacement rules of the I/O Access Patterns section: discard the sample
// whose next use is furthest in the future, and never one used before the
// sample being brought in).
//
// The buffer holds samples keyed by the stream position of their next use,
// so the read at position f hits exactly when key f is held. After a read
// with a next use n the sample is (re)admitted under key n, then, while the
// held bytes exceed d0, the furthest key is discarded (possibly n itself).
// The size of the sample held under key x is that of the sample read at x,
// sizes[R[x]].
// The workers are independent. Two ways to replay one:
//
// In the order of next uses (kb_*). A discard takes the furthest keys first,
// so whether key k stays does not depend on later keys. Take the candidates
// (reads f with a next use k and a size s <= d0, held over [f, k)) by
// increasing k. Let load(t) be the bytes of the accepted earlier keys held
// after read t, and T the last time any earlier key was discarded (a key
// discarded at T takes every later key held then with it). Then k stays, and
// its read hits, exactly when f > T and load(t) + s <= d0 for every t in
// [f, k); otherwise, when f > T, it is discarded at the first t where that
// fails, which becomes T. In a shuffled stream T moves only a few times per
// epoch (18 times over the 160,000 candidates of an ImageNet-22k worker, 350
// over 5.9M at ImageNet-1k on 16 workers): in between, everything with f > T
// is accepted, thousands of candidates at a time, as long as the load provably
// stays within d0.
//   kb_init  -- hit flags to 0 (-1 in padding), previous uses to -1.
//   kb_prev  -- previous uses, prev[next[f]] = f.
//   kb_sim   -- one workgroup per worker. A batch is the candidates whose next
//               uses lie in up to 4,096 consecutive positions. Per block of
//               positions (8,192 blocks a row) U is the bytes of the accepted
//               candidates and the batch's that touch the block, kept as
//               differences in LDS: at least load(t) anywhere in it. If no U
//               after T exceeds d0 the batch is accepted. Otherwise the
//               blocks in question are looked into position by position; what
//               U is above the true maximum by is remembered with the block,
//               which settles most of them for good. A true excess is first
//               narrowed to a batch of few candidates, then found by taking
//               candidates back from the load, last to first, at every
//               position in question.
// ImageNet-22k, 5 GB: 102 ms in stream order, 9.0 in the order of next uses
// (kb_sim 6.5, kb_prev 1.5, kb_init 0.7; the rest is the gaps between them); 300,000
// samples, 10 epochs, 2 workers 620 -> 4.4; 10,000 samples, 5 epochs, 4 workers
// 2.6 -> 0.7. What bounds kb_sim: barriers and latency, not its vector units (23%
// busy). Per batch two block-wide scans and five barriers, per change of T several
// looks into blocks (about 50 us). The looks also are most of what it reads: 21.9 GB
// at ImageNet-22k with 5 GB, 9.7 with a buffer of four epochs, where nothing is
// discarded (the rows' next and previous uses 4.5, the rest the candidates' ids and
// sizes, a 128-byte line each).
//
// In stream order (bs_sim), where an epoch brings too few candidates for that or
// the buffer holds too few samples (the rule in buffer_impl), or memory for the
// previous uses is missing:
//
//   bs_sim   -- one wave per worker. Held keys in a three-level bitmap: a
//               bit per position in 64-bit words in global memory, one word
//               per batch of 64 reads, changed and read only by atomics so it
//               is always current; a bit per word that may hold keys, and a
//               bit per such level-1 word, in LDS. A batch of 64 reads
//               arrives one per lane (ids and next uses loaded two batches
//               ahead, sizes gathered and the batch's word loaded one ahead,
//               with changes to that word made meanwhile kept as set and
//               clear masks); only the reads that can change
//               anything are visited, in order: those whose key is held (a
//               hit) and those with a next use that fits (an admission). The
//               highest held keys (up to 64) live in registers, ascending
//               across the lanes with their sizes: the furthest key is
//               discarded from there, an admitted key above the lowest cached
//               one joins in order, and an admission above the highest that
//               does not fit is a bypass that touches nothing. Only when the
//               cache empties are the highest keys gathered again from the two
//               highest level-1 words, one word per lane (discards do not
//               clear level bits; words found empty clear theirs then).

#include <algorithm>
#include <climits>
#include <cmath>
#include <new>
#include <string>

#include "common.hpp"

namespace nopfs {
namespace {

constexpr int kBsMaxLog = 24;                          // positions per worker: < 2^24
constexpr int kBsW1 = (1 << kBsMaxLog) / 64 / 32;      // level-1 words: 8192
constexpr int kBsW2 = kBsW1 / 32;                      // level-2 words: 256

struct BsShape {
  int64_t F, N, B, M_max, E;
  int32_t drop_last;
};

__device__ __forceinline__ int64_t bs_row_len(const BsShape& r, int64_t i) {
  return r.E * epoch_len(r.F, r.N, r.B, r.drop_last, i);
}

__device__ __forceinline__ int64_t rl64(int64_t v, int lane) {
  const uint32_t lo = __builtin_amdgcn_readlane(uint32_t(uint64_t(v)), lane);
  const uint32_t hi = __builtin_amdgcn_readlane(uint32_t(uint64_t(v) >> 32), lane);
  return int64_t((uint64_t(hi) << 32) | lo);
}

__device__ __forceinline__ uint64_t rfl64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(v >> 32));
  return (uint64_t(hi) << 32) | lo;
}

__device__ __forceinline__ int hi_bit(uint32_t v) { return 31 - __builtin_clz(v); }

// whole-wave lane shifts: lane i takes lane i + 1 (shl1) or lane i - 1
// (shr1); the lane with no source keeps `edge`
__device__ __forceinline__ int32_t shl1(int32_t v, int32_t edge) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x130, 0xf, 0xf, false);
}
__device__ __forceinline__ int32_t shr1(int32_t v, int32_t edge) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ int64_t shl1_64(int64_t v) {
  const uint32_t lo = uint32_t(shl1(int32_t(uint32_t(uint64_t(v))), 0));
  const uint32_t hi = uint32_t(shl1(int32_t(uint32_t(uint64_t(v) >> 32)), 0));
  return int64_t((uint64_t(hi) << 32) | lo);
}
__device__ __forceinline__ int64_t shr1_64(int64_t v) {
  const uint32_t lo = uint32_t(shr1(int32_t(uint32_t(uint64_t(v))), 0));
  const uint32_t hi = uint32_t(shr1(int32_t(uint32_t(uint64_t(v) >> 32)), 0));
  return int64_t((uint64_t(hi) << 32) | lo);
}
__device__ __forceinline__ int hi_bit64(uint64_t v) { return 63 - __builtin_clzll(v); }

__device__ __forceinline__ uint64_t l0_load(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void __launch_bounds__(64)
bs_sim(BsShape r, const int32_t* __restrict__ R, const int32_t* __restrict__ next,
       const int64_t* __restrict__ sizes, int64_t d0, const uint32_t* __restrict__ in_order,
       uint64_t* __restrict__ L0, int8_t* __restrict__ hit, int64_t* __restrict__ hits) {
  __shared__ uint32_t l1[kBsW1];
  __shared__ uint32_t l2[kBsW2];
  if (in_order && *in_order == 0u) return;  // the other replay takes this call
  const int64_t i = blockIdx.x;
  const int lane = threadIdx.x;
  const int64_t Mi = bs_row_len(r, i);
  const int64_t W0 = (r.M_max + 63) >> 6;
  const int64_t W1 = (W0 + 31) >> 5;
  const int64_t W2 = (W1 + 31) >> 5;
  uint64_t* l0 = L0 + i * W0;
  const int32_t* Xr = next + i * r.M_max;
  const int32_t* Rr = R + i * r.M_max;
  // a sample's size (0 for an id outside [0, F))
  auto size_at_id = [&](int32_t k) -> int64_t {
    return (k >= 0 && k < r.F) ? sizes[k] : int64_t(0);
  };
  int8_t* hrow = hit + i * r.M_max;
  for (int64_t w = lane; w < W0; w += 64) l0[w] = 0u;
  for (int64_t w = lane; w < W1; w += 64) l1[w] = 0u;
  for (int64_t w = lane; w < W2; w += 64) l2[w] = 0u;
  __threadfence();  // the cleared words reach L2 before the atomics below
  __syncthreads();

  __shared__ int32_t kslot[64];
  int64_t used = 0, hc = 0, hb = 0;
  // the highest held keys, ascending in lanes 0..n-1, with their sizes;
  // every held key >= ck[0] is cached, and n == 0 only when nothing is held
  int32_t ck = INT32_MAX;
  int64_t cz = 0;
  int n = 0;
  int64_t nheld = 0;

  // clears the level bits above a level-0 word that has become zero
  auto word_emptied = [&](int64_t w) {
    if (lane == 0) {
      const int64_t a = w >> 5;
      const uint32_t v1 = atomicAnd(&l1[a], ~(1u << (w & 31))) & ~(1u << (w & 31));
      if (v1 == 0u) atomicAnd(&l2[a >> 5], ~(1u << (a & 31)));
    }
  };
  // the cache's lowest key leaves (it stays held in the bitmap)
  auto drop_min = [&]() {
    ck = shl1(ck, INT32_MAX);
    cz = shl1_64(cz);
    --n;
  };
  // a key above ck[0] (or into an empty cache) joins in order; a full cache
  // first lets its lowest key go
  auto cache_insert = [&](int32_t key, int64_t sz) {
    if (n == 64) drop_min();
    const int p = __builtin_popcountll(__ballot(lane < n && ck < key));
    const int32_t uk = shr1(ck, INT32_MAX);
    const int64_t uz = shr1_64(cz);
    if (lane > p && lane <= n) {
      ck = uk;
      cz = uz;
    }
    if (lane == p) {
      ck = key;
      cz = sz;
    }
    ++n;
  };
  // fills the empty cache with the highest held keys: the words of the two
  // highest level-1 words that have set bits, one word per lane, highest
  // first; level bits of words found empty (keys discarded from the cache
  // leave them set) are cleared on the way
  auto refill = [&]() {
    __builtin_amdgcn_s_waitcnt(0);  // lane 0's atomics are in L2 before other lanes load
    n = 0;
    while (n == 0 && nheld > 0) {
      int64_t w2 = -1;
      for (int64_t base = ((W2 - 1) >> 6) << 6; base >= 0; base -= 64) {
        const int64_t idx = base + lane;
        const uint32_t v = idx < W2 ? l2[idx] : 0u;
        const uint64_t bl = __ballot(v != 0u);
        if (bl) {
          w2 = base + (63 - __builtin_clzll(bl));
          break;
        }
      }
      if (w2 < 0) break;  // nothing marked (only if sizes or next uses break the precondition)
      const uint32_t v2 = l2[w2];
      const int64_t a1 = (w2 << 5) + hi_bit(v2);
      const uint32_t v1a = l1[a1];
      if (v1a == 0u) {  // a level-2 bit over an empty level-1 word
        if (lane == 0) atomicAnd(&l2[w2], ~(1u << (a1 & 31)));
        __builtin_amdgcn_s_waitcnt(0);
        continue;
      }
      // the next level-1 word with a level-2 bit, below a1
      int64_t a2 = -1;
      const uint32_t below = v2 & ((1u << (a1 & 31)) - 1u);
      if (below) {
        a2 = (w2 << 5) + hi_bit(below);
      } else {
        for (int64_t base = ((w2 - 1) >> 6) << 6; w2 > 0 && base >= 0; base -= 64) {
          const int64_t idx = base + lane;
          const uint32_t v = idx < w2 ? l2[idx] : 0u;
          const uint64_t bl = __ballot(v != 0u);
          if (bl) {
            const int64_t w2b = base + (63 - __builtin_clzll(bl));
            a2 = (w2b << 5) + hi_bit(l2[w2b]);
            break;
          }
        }
      }
      const uint32_t v1b = a2 >= 0 ? l1[a2] : 0u;
      const int jj = lane & 31;
      const uint32_t v1 = lane < 32 ? v1a : v1b;
      const int64_t a = lane < 32 ? a1 : a2;
      const bool has = a >= 0 && ((v1 >> (31 - jj)) & 1u);
      const int64_t w = a * 32 + (31 - jj);
      uint64_t v = has ? l0_load(&l0[w]) : uint64_t(0);
      if (has && v == 0u) {  // marked but empty: clear the marks
        const uint32_t m1 = 1u << (w & 31);
        const uint32_t left = atomicAnd(&l1[w >> 5], ~m1) & ~m1;
        if (left == 0u) atomicAnd(&l2[w >> 10], ~(1u << ((w >> 5) & 31)));
      }
      const uint32_t pop = uint32_t(__builtin_popcountll(v));
      const uint32_t incl = wave_inclusive_scan(pop);
      const uint32_t ex = incl - pop;
      const uint32_t sum = __builtin_amdgcn_readlane(incl, 63);
      const int total = sum < 64u ? int(sum) : 64;
      __builtin_amdgcn_s_waitcnt(0);
      if (total == 0) continue;  // only empty words: their marks are gone now
      const int k = ex >= 64u ? 0 : (int(pop) < 64 - int(ex) ? int(pop) : 64 - int(ex));
      for (int it = 0; it < 64; ++it) {
        if (!__ballot(it < k)) break;
        if (it < k) {
          const int bp = hi_bit64(v);
          v &= ~(uint64_t(1) << bp);
          kslot[total - 1 - (int(ex) + it)] = int32_t((w << 6) + bp);
        }
      }
      __builtin_amdgcn_wave_barrier();
      const int32_t key = lane < total ? kslot[lane] : INT32_MAX;
      ck = key;
      const int32_t kid = (lane < total && key >= 0 && key < Mi) ? Rr[key] : -1;
      cz = size_at_id(kid);
      n = total;
      // wait for the sizes here, once: an empty asm that takes and redefines
      // them, so no later use of the cache waits on memory (such a wait would
      // also wait for lane 0's latest atomics)
      asm volatile("" : "+v"(cz), "+v"(ck));
    }
  };
  // the batch: its index, held keys among its positions, and the changes
  // made to the next batch's word since lane 0 loaded it
  int64_t b = 0;
  uint64_t hw = 0, nset = 0, nclr = 0;
  // discards the highest key
  auto evict = [&]() -> bool {
    const int32_t x = __builtin_amdgcn_readlane(ck, n - 1);
    const int64_t sx = rl64(cz, n - 1);
    --n;
    if (x < 0 || x >= Mi) return false;  // cannot happen: cached keys are held positions
    const int64_t w = x >> 6;
    const uint64_t bx = uint64_t(1) << (x & 63);
    if (lane == 0) atomicAnd(reinterpret_cast<unsigned long long*>(&l0[w]), ~bx);
    // this batch's word or the next one's (branch-free: keeps them in registers)
    const uint64_t mb = w == b ? bx : uint64_t(0);
    const uint64_t mn = w == b + 1 ? bx : uint64_t(0);
    hw &= ~mb;
    nclr |= mn;
    nset &= ~mn;
    used -= sx;
    --nheld;
    if (n == 0 && nheld > 0) refill();
    return true;
  };

  // the next batch: sizes, next uses, lane 0's copy of its word, and the
  // changes made to that word since it was loaded
  // pipeline: ids and next uses two batches ahead, sizes one
  int32_t kN2 = 64 + lane < Mi ? Rr[64 + lane] : -1;
  int32_t nN2 = 64 + lane < Mi ? Xr[64 + lane] : -1;
  int64_t sN = size_at_id(lane < Mi ? Rr[lane] : -1);
  int32_t nN = lane < Mi ? Xr[lane] : -1;
  uint64_t hN = 0;  // every word starts empty
  for (int64_t f0 = 0; f0 < Mi; f0 += 64, ++b) {
    const int64_t f = f0 + lane;
    const int64_t s = sN;
    int32_t nx = nN;
    if (nx <= f || nx >= Mi) nx = -1;
    hw = (rfl64(hN) & ~nclr) | nset;
    const uint64_t cand = __ballot(nx >= 0 && s <= d0);
    nset = nclr = 0;
    hN = 0;
    {  // the next batches' loads, after this batch's values are in use
      sN = size_at_id(kN2);
      nN = nN2;
      const int64_t g = f + 128;
      kN2 = g < Mi ? Rr[g] : -1;
      nN2 = g < Mi ? Xr[g] : -1;
      if (lane == 0 && b + 1 < W0) hN = l0_load(&l0[b + 1]);
    }
    uint64_t mask = cand | hw;
    uint64_t hm = 0;
    while (mask) {
      const int q = __builtin_ctzll(mask);
      const uint64_t bit = uint64_t(1) << q;
      mask &= ~bit;
      const int64_t sq = rl64(s, q);
      if (hw & bit) {  // key f0 + q held: a hit, and its entry ends here
        hc += 1;
        hb += sq;
        hm |= bit;
        used -= sq;
        --nheld;
        hw &= ~bit;
        if (lane == 0) atomicAnd(reinterpret_cast<unsigned long long*>(&l0[b]), ~bit);
        if (hw == 0u) word_emptied(b);
        if (n > 0 && __builtin_amdgcn_readlane(ck, 0) == int32_t(f0 + q)) {
          drop_min();
          if (n == 0 && nheld > 0) refill();
        }
      }
      if (!(cand & bit)) continue;
      const int32_t nq = __builtin_amdgcn_readlane(nx, q);
      const int64_t top = n > 0 ? int64_t(__builtin_amdgcn_readlane(ck, n - 1)) : -1;
      if (nq > top && sq > d0 - used) continue;  // the furthest and it does not fit: bypass
      {  // admit under the next use
        const int64_t w = nq >> 6;
        const uint64_t bn = uint64_t(1) << (nq & 63);
        if (lane == 0) {
          atomicOr(reinterpret_cast<unsigned long long*>(&l0[w]), bn);
          atomicOr(&l1[w >> 5], 1u << (w & 31));
          atomicOr(&l2[w >> 10], 1u << ((w >> 5) & 31));
        }
        // a later read of this batch, or of the next one
        const uint64_t mb = w == b ? bn : uint64_t(0);
        const uint64_t mn = w == b + 1 ? bn : uint64_t(0);
        hw |= mb;
        mask |= mb;
        nset |= mn;
        nclr &= ~mn;
        if (n == 0 || nq > __builtin_amdgcn_readlane(ck, 0)) cache_insert(nq, sq);
        ++nheld;
        used += sq;
      }
      // discard the furthest while over capacity
      while (used > d0) {
        if (n == 0 || !evict()) {  // nothing held (broken precondition)
          used = 0;
          break;
        }
      }
    }
    if (f < Mi) hrow[f] = int8_t((hm >> lane) & 1u);
  }
  for (int64_t f = Mi + lane; f < r.M_max; f += 64) hrow[f] = -1;
  if (lane == 0) {
    hits[i * 2] = hc;
    hits[i * 2 + 1] = hb;
  }
}

// -- the replay in the order of next uses ---------------------------------------
constexpr int kKbThreads = 512;
constexpr int kKbWaves = kKbThreads / 64;
constexpr int kKbPer = 8;                            // positions per thread and window
constexpr int kKbWindow = kKbThreads * kKbPer;       // 4,096
constexpr int kKbList = 2048;                        // candidates per batch
constexpr int kKbBlocks = 8192;                      // time blocks
constexpr int kKbMinShift = 6;                       // of at least 64 positions
constexpr int kKbSeg = kKbBlocks / kKbThreads;       // blocks per thread in the scan
// A batch of more than kKbFew candidates is cut before its record is searched, as
// is one that puts more than kKbMany blocks over, but not below kKbMinSpan
// positions. Kernel times, us, of (a) 10,000 samples x 5 epochs x 4 workers with a
// buffer of 180 samples, (b) 300,000 x 10 x 2, (c) 32,000 x 40 x 16, (d) ImageNet-22k:
//                     (a)     (b)      (c)      (d)
//   as here           449   3,026    5,068    8,751
//   kKbFew 64         448   3,023    4,654    8,768
//   kKbFew 512      1,379   6,821   10,958   14,787
//   kKbMany 8         440   2,988    5,033    8,799
//   kKbMany 128       494   3,556    5,504    8,896
//   kKbMinSpan 128    450   2,865    5,065    8,762
//   kKbMinSpan 1024   705   7,953    6,299    9,084
constexpr uint32_t kKbFew = 128;
constexpr uint32_t kKbMany = 32;
constexpr int kKbMinSpan = 256;
constexpr double kKbMinCands = 300;  // candidates per worker and epoch
constexpr int64_t kKbMaxD0 = int64_t(1) << 50;       // sums over a block and a batch stay below 2^63
constexpr int kKbSample = 16;                        // sizes per thread whose mean is taken

// padded index: a thread's 16 consecutive blocks start on different banks
__device__ __forceinline__ int kb_slot(int b) { return b + (b >> 4); }

struct KbCand {
  int32_t f, k;  // held from its read f to its next use k
  int64_t s;
};

struct KbSmem {
  int64_t dd[kKbBlocks + kKbBlocks / 16 + 2];   // differences of U between blocks (or U itself)
  uint32_t adj[kKbBlocks + kKbBlocks / 16 + 2]; // what U is known to be above the exact maximum by
  KbCand cand[kKbList];                         // the batch's candidates
  uint16_t flag[kKbBlocks];                     // blocks to look into; bit 15: over capacity
  int64_t wtot[kKbWaves];
  uint32_t cnt[kKbWaves];
  uint32_t nflag, nviol;
  unsigned long long best;
  int64_t hc, hb;
};

// hit: 0 up to the row's length, -1 behind it; prev: -1. The first workgroup
// also chooses the replay: in stream order (*in_order = 1) when d0 is less than
// `least` sizes' worth, by the mean of up to 4,096 sizes, and one of them fits.
__global__ void __launch_bounds__(256)
kb_init(BsShape r, const int64_t* __restrict__ sizes, int64_t d0, double least,
        uint32_t* __restrict__ in_order, int32_t* __restrict__ prev, int8_t* __restrict__ hit) {
  if (in_order && blockIdx.x == 0 && blockIdx.y == 0) {
    __shared__ double part[4];
    const int64_t n = r.F < 256 * kKbSample ? r.F : 256 * kKbSample;
    double sum = 0;
    bool fits = false;
#pragma unroll
    for (int u = 0; u < kKbSample; ++u) {
      const int64_t x = u * 256 + int64_t(threadIdx.x);
      const int64_t s = sizes[x < n ? x * r.F / n : 0];  // unconditional
      sum += x < n ? double(s) : 0.0;
      fits = fits || s <= d0;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    fits = __syncthreads_or(fits);
    if (threadIdx.x == 0)
      *in_order = fits && double(d0) * double(n) < least * (part[0] + part[1] + part[2] + part[3]) ? 1u : 0u;
  }
  const int64_t i = blockIdx.y;
  const int64_t Mi = bs_row_len(r, i);
  const int64_t f0 = (int64_t(blockIdx.x) * 256 + threadIdx.x) * 16;
  int32_t* p = prev + i * r.M_max;
  int8_t* h = hit + i * r.M_max;
  // 16 positions per thread; a position at a time only at the end of the row
  if (f0 + 16 <= Mi) {
    const int4 v = make_int4(-1, -1, -1, -1);
#pragma unroll
    for (int u = 0; u < 4; ++u) __builtin_memcpy(p + f0 + 4 * u, &v, 16);
    const int4 z = make_int4(0, 0, 0, 0);
    __builtin_memcpy(h + f0, &z, 16);
    return;
  }
  for (int64_t f = f0; f < f0 + 16 && f < r.M_max; ++f) {
    p[f] = -1;
    h[f] = f < Mi ? 0 : -1;
  }
}

// prev[next[f]] = f
__global__ void __launch_bounds__(256)
kb_prev(BsShape r, const int32_t* __restrict__ next, const uint32_t* __restrict__ in_order,
        int32_t* __restrict__ prev) {
  if (in_order && *in_order != 0u) return;
  const int64_t i = blockIdx.y;
  const int64_t Mi = bs_row_len(r, i);
  const int64_t f0 = (int64_t(blockIdx.x) * 256 + threadIdx.x) * 4;
  const int32_t* x = next + i * r.M_max;
  int32_t* p = prev + i * r.M_max;
  int32_t v[4] = {-1, -1, -1, -1};
  if (f0 + 4 <= Mi) {
    __builtin_memcpy(v, x + f0, 16);
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (f0 + u < Mi) v[u] = x[f0 + u];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (v[u] > f0 + u && v[u] < Mi) p[v[u]] = int32_t(f0 + u);
}

__global__ void __launch_bounds__(kKbThreads)
kb_sim(BsShape r, const int32_t* __restrict__ R, const int32_t* __restrict__ next,
       const int64_t* __restrict__ sizes, int64_t d0, const uint32_t* __restrict__ in_order, int ash,
       int sh, const int32_t* __restrict__ prev, int8_t* __restrict__ hit, int64_t* __restrict__ hits) {
  __shared__ KbSmem m;
  const int64_t i = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool here = !in_order || *in_order == 0u;  // else the other replay takes the call
  const int32_t Mi = here ? int32_t(bs_row_len(r, i)) : 0;  // < 2^24
  const int32_t* Rr = R + i * r.M_max;
  const int32_t* Xr = next + i * r.M_max;
  const int32_t* Pr = prev + i * r.M_max;
  int8_t* hrow = hit + i * r.M_max;
  auto size_of = [&](int32_t id) -> int64_t {
    const bool in = id >= 0 && id < r.F;
    const int64_t v = sizes[in ? id : 0];  // unconditional
    return in ? v : 0;
  };
  // an interval [f, k) of s bytes joins the blocks it touches (or leaves, s < 0)
  auto join = [&](int32_t f, int32_t k, int64_t s) {
    const int b0 = f >> sh, b1 = ((k - 1) >> sh) + 1;  // f < k
    atomicAdd(reinterpret_cast<unsigned long long*>(&m.dd[kb_slot(b0)]), (unsigned long long)(s));
    if (b1 < kKbBlocks)
      atomicAdd(reinterpret_cast<unsigned long long*>(&m.dd[kb_slot(b1)]), (unsigned long long)(-s));
  };

  // windows of kKbWindow positions, eight consecutive ones per thread:
  // previous uses and ids two windows ahead, sizes one
  int32_t pv[kKbPer], pvN[kKbPer], idN[kKbPer], pvA[kKbPer], idA[kKbPer];
  int64_t sz[kKbPer], szN[kKbPer];
  auto load_ids = [&](int32_t w0, int32_t (&p)[kKbPer], int32_t (&id)[kKbPer]) {
    const int32_t at = w0 + kKbPer * tid;
    if (w0 + kKbWindow <= Mi) {
#pragma unroll
      for (int u = 0; u < kKbPer; u += 4) {
        __builtin_memcpy(&p[u], Pr + at + u, 16);
        __builtin_memcpy(&id[u], Rr + at + u, 16);
      }
    } else {
#pragma unroll
      for (int u = 0; u < kKbPer; ++u) {
        const int32_t q = at + u < Mi ? at + u : 0;
        p[u] = Pr[q];
        id[u] = Rr[q];
        if (at + u >= Mi) p[u] = -1;
      }
    }
  };
  auto load_sizes = [&](const int32_t (&p)[kKbPer], const int32_t (&id)[kKbPer], int64_t (&s)[kKbPer]) {
#pragma unroll
    for (int u = 0; u < kKbPer; ++u) s[u] = size_of(p[u] >= 0 ? id[u] : -1);
  };

  int32_t T = -1;          // starts up to T are discarded
  int32_t p0 = 0, pe = 0;  // the batch: next uses in [p0, pe)
  int32_t span = kKbWindow;
  // four steps of 64 positions, one position per lane and step: step u's at
  // p[u], of the block [bs[u], be[u]). With every candidate of the batch
  // accepted: what a position's own start adds, and that less what its own
  // end takes away.
  constexpr int kEv = 4;
  typedef int32_t Steps[kEv];
  auto events = [&](const Steps& p, const Steps& bs, const Steps& be, int64_t (&start)[kEv],
                    int64_t (&change)[kEv]) {
    int32_t q[kEv], nx[kEv], pq[kEv], id[kEv];
#pragma unroll
    for (int u = 0; u < kEv; ++u) {  // unconditional loads, all steps in flight together
      q[u] = p[u] < be[u] ? p[u] : bs[u];
      nx[u] = Xr[q[u]];
      pq[u] = Pr[q[u]];
      id[u] = Rr[q[u]];
    }
    int64_t s[kEv];
    int8_t hn[kEv], hq[kEv];
#pragma unroll
    for (int u = 0; u < kEv; ++u) {
      if (!(nx[u] > q[u] && nx[u] < Mi)) nx[u] = -1;
      s[u] = size_of(id[u]);
      hn[u] = hrow[nx[u] >= 0 ? nx[u] : q[u]];
      hq[u] = hrow[q[u]];
    }
#pragma unroll
    for (int u = 0; u < kEv; ++u) {
      const bool in = p[u] < be[u];
      const bool st = in && nx[u] >= 0 && s[u] <= d0 &&
                      (nx[u] < p0 ? hn[u] == 1 : nx[u] < pe && q[u] > T);
      const bool en = in && q[u] > bs[u] &&
                      (q[u] < p0 ? hq[u] == 1 : pq[u] > T && pq[u] >= 0 && q[u] < pe && s[u] <= d0);
      start[u] = st ? s[u] : 0;
      change[u] = start[u] - (en ? s[u] : 0);
    }
  };
  // Blocks of 64 positions are looked into four at a time, longer ones in
  // four steps at a time; x counts the flagged blocks.
  const uint32_t at_once = sh == kKbMinShift ? kEv : 1;
  struct Look {
    Steps p, bs, be, b;  // b: -1 past the last flagged block
  };
  auto look = [&](uint32_t x, uint32_t nx, int32_t y) {
    Look l;
#pragma unroll
    for (int u = 0; u < kEv; ++u) {
      const uint32_t xu = at_once == 1 ? x : x + u;
      const bool in = xu < nx;
      l.b[u] = in ? m.flag[in ? xu : 0] & 0x7FFF : -1;
      l.bs[u] = in ? l.b[u] << sh : 0;
      l.be[u] = in ? (Mi - l.bs[u] < (1 << sh) ? Mi : l.bs[u] + (1 << sh)) : 0;
      l.p[u] = l.bs[u] + y + (at_once == 1 ? 64 * u : 0) + lane;
    }
    return l;
  };
  const int32_t block = 1 << sh, stride = at_once == 1 ? 64 * kEv : block;

  for (int b = tid; b < kKbBlocks + kKbBlocks / 16 + 2; b += kKbThreads) {
    m.dd[b] = 0;
    m.adj[b] = 0;
  }
  if (tid == 0) {
    m.hc = 0;
    m.hb = 0;
  }
  int64_t hc = 0, hb = 0;
  int32_t w0 = 0;
  if (Mi > 0) {
    load_ids(0, pv, idN);
    load_sizes(pv, idN, sz);
    load_ids(kKbWindow, pvN, idN);
  }
  bool fresh = true;  // the window's loads for the ones after it are to be issued
  __syncthreads();
  while (p0 < Mi) {
    if (p0 >= w0 + kKbWindow) {
      w0 += kKbWindow;
#pragma unroll
      for (int u = 0; u < kKbPer; ++u) {
        pv[u] = pvN[u];
        sz[u] = szN[u];
        pvN[u] = pvA[u];
        idN[u] = idA[u];
      }
      fresh = true;
    }
    if (fresh) {
      load_sizes(pvN, idN, szN);
      load_ids(w0 + 2 * kKbWindow, pvA, idA);
      fresh = false;
    }
    // the batch's candidates (starts after T that fit) in order of next use
    pe = w0 + kKbWindow;
    if (p0 + span < pe) pe = p0 + span;
    if (pe > Mi) pe = Mi;
    uint32_t cand = 0;
#pragma unroll
    for (int u = 0; u < kKbPer; ++u) {
      const int32_t p = w0 + kKbPer * tid + u;
      if (p >= p0 && p < pe && pv[u] > T && pv[u] >= 0 && sz[u] <= d0) cand |= 1u << u;
    }
    const uint32_t n = __popc(cand);
    const uint32_t inc = wave_inclusive_scan(n);
    if (lane == 63) m.cnt[wave] = inc;
    if (tid == 0) {
      m.nflag = 0;
      m.nviol = 0;
      m.best = ~0ull;
    }
    __syncthreads();
    uint32_t slot = inc - n, total = 0;
#pragma unroll
    for (int w = 0; w < kKbWaves; ++w) {
      const uint32_t c = m.cnt[w];
      slot += w < wave ? c : 0u;
      total += c;
    }
    if (total > uint32_t(kKbList)) {  // uniform: half the positions
      span = (pe - p0 + 1) / 2;
      __syncthreads();
      continue;
    }
#pragma unroll
    for (int u = 0; u < kKbPer; ++u)
      if ((cand >> u) & 1u) {
        const int32_t k = w0 + kKbPer * tid + u;
        m.cand[slot++] = KbCand{pv[u], k, sz[u]};
        join(pv[u], k, sz[u]);
      }
    __syncthreads();
    // U per block: the bytes of all accepted intervals and the batch's
    // candidates that touch it, at least the exact maximum inside it plus adj.
    // Only times after T can go over.
    bool alarm = false;
    int64_t base = 0;
    const int bT = T >= 0 ? T >> sh : 0;
    if (total > 0) {
      int64_t run = 0, most = INT64_MIN;
#pragma unroll
      for (int q = 0; q < kKbSeg; ++q) {
        const int b = tid * kKbSeg + q;
        run += m.dd[kb_slot(b)];
        const int64_t over = run - (int64_t(m.adj[kb_slot(b)]) << ash);
        most = b >= bT && over > most ? over : most;
      }
      const int64_t ri = int64_t(wave_inclusive_scan64(uint64_t(run)));
      if (lane == 63) m.wtot[wave] = ri;
      __syncthreads();
      base = ri - run;
#pragma unroll
      for (int w = 0; w < kKbWaves; ++w) base += w < wave ? m.wtot[w] : 0;
      alarm = __syncthreads_or(most != INT64_MIN && base + most > d0);
    }
    uint32_t accept = total;  // of the batch's candidates
    bool record = false, retry = false;
    if (alarm) {
      // U in place of the differences; the blocks over capacity by it
      int64_t run = base;
#pragma unroll
      for (int q = 0; q < kKbSeg; ++q) {
        const int b = tid * kKbSeg + q;
        run += m.dd[kb_slot(b)];
        m.dd[kb_slot(b)] = run;
        if (b >= bT && run - (int64_t(m.adj[kb_slot(b)]) << ash) > d0)
          m.flag[atomicAdd(&m.nflag, 1u)] = uint16_t(b);
      }
      __syncthreads();
      const uint32_t nflag = m.nflag;
      // many candidates and many blocks: fewer candidates first
      retry = total > kKbFew && pe - p0 > kKbMinSpan && nflag > kKbMany;
      // the exact maximum of each after T
      for (uint32_t x = wave * at_once; x < nflag && !retry; x += kKbWaves * at_once) {
        int64_t carry = 0, started[kEv] = {}, most[kEv];
#pragma unroll
        for (int u = 0; u < kEv; ++u) most[u] = INT64_MIN;
        Look l;
        for (int32_t y = 0; y < block; y += stride) {
          l = look(x, nflag, y);
          int64_t st[kEv], ch[kEv];
          events(l.p, l.bs, l.be, st, ch);
#pragma unroll
          for (int u = 0; u < kEv; ++u) {
            int64_t v = int64_t(wave_inclusive_scan64(uint64_t(ch[u])));
            if (at_once == 1) {
              v += carry;
              carry = rl64(v, 63);
            }
            if (l.p[u] < l.be[u] && l.p[u] > T && v > most[u]) most[u] = v;
            started[u] += st[u];
          }
        }
        if (at_once == 1) {
#pragma unroll
          for (int u = 1; u < kEv; ++u) {
            most[0] = most[u] > most[0] ? most[u] : most[0];
            started[0] += started[u];
          }
        }
#pragma unroll
        for (int u = 0; u < kEv; ++u) {
          if (u > 0 && at_once == 1) break;
          const int64_t sum = int64_t(read_lane64(wave_inclusive_scan64(uint64_t(started[u])), 63));
          int64_t top = most[u];
#pragma unroll
          for (int d = 32; d >= 1; d >>= 1) {
            const int64_t o = __shfl_xor(top, d, 64);
            top = o > top ? o : top;
          }
          if (lane == 0 && l.b[u] >= 0) {
            const int64_t U = m.dd[kb_slot(l.b[u])];
            // no time after T in the block: nothing more can start in it
            const int64_t exact = top == INT64_MIN ? 0 : U - sum + top;
            if (exact > d0) {
              m.flag[x + u] = uint16_t(l.b[u] | 0x8000);
              atomicAdd(&m.nviol, 1u);
            }
            const uint64_t a = exact < U ? uint64_t(U - exact) >> ash : 0u;
            m.adj[kb_slot(l.b[u])] = a < 0xFFFFFFFFull ? uint32_t(a) : 0xFFFFFFFFu;
          }
        }
      }
      __syncthreads();
      record = retry || m.nviol != 0u;
      retry = record && total > kKbFew && pe - p0 > kKbMinSpan;
      if (record && !retry) {
        // the first candidate whose bytes exceed the capacity somewhere, and
        // the first position at which they do: from the load with the whole
        // batch, candidates are taken away from the last to the first
        for (uint32_t x = wave * at_once; x < nflag; x += kKbWaves * at_once) {
          bool over = false;
          for (uint32_t u = 0; u < at_once; ++u) over = over || (x + u < nflag && (m.flag[x + u] & 0x8000u));
          if (!over) continue;
          // the bytes before each block's first position: U less what starts inside
          int64_t before[kEv] = {};
          for (int32_t y = 0; y < block; y += stride) {
            const Look l = look(x, nflag, y);
            int64_t st[kEv], ch[kEv];
            events(l.p, l.bs, l.be, st, ch);
#pragma unroll
            for (int u = 0; u < kEv; ++u) before[u] -= st[u];
          }
          if (at_once == 1) {
#pragma unroll
            for (int u = 1; u < kEv; ++u) before[0] += before[u];
          }
#pragma unroll
          for (int u = 0; u < kEv; ++u) {
            before[u] = int64_t(read_lane64(wave_inclusive_scan64(uint64_t(before[u])), 63));
            const uint32_t xu = at_once == 1 ? x : x + u;
            if (xu < nflag) before[u] += m.dd[kb_slot(m.flag[xu] & 0x7FFF)];
          }
          int64_t carry = before[0];
          for (int32_t y = 0; y < block; y += stride) {
            const Look l = look(x, nflag, y);
            int64_t st[kEv], ch[kEv], v[kEv];
            events(l.p, l.bs, l.be, st, ch);
            bool any = false;
            int best[kEv];
#pragma unroll
            for (int u = 0; u < kEv; ++u) {
              v[u] = (at_once == 1 ? carry : before[u]) + int64_t(wave_inclusive_scan64(uint64_t(ch[u])));
              carry = rl64(v[u], 63);
              if (l.p[u] >= l.be[u] || l.p[u] <= T) v[u] = INT64_MIN;
              any = any || v[u] > d0;
              best[u] = -1;
            }
            if (!__any(any)) continue;
            for (int j = int(total) - 1; j >= 0; --j) {
              const KbCand c = m.cand[j];
#pragma unroll
              for (int u = 0; u < kEv; ++u)
                if (v[u] > d0 && c.f <= l.p[u] && l.p[u] < c.k) {
                  best[u] = j;
                  v[u] -= c.s;
                }
            }
#pragma unroll
            for (int u = 0; u < kEv; ++u)
              if (best[u] >= 0)
                atomicMin(&m.best, (static_cast<unsigned long long>(best[u]) << 32) | uint32_t(l.p[u]));
          }
        }
        __syncthreads();
        record = m.best != ~0ull;
      }
      // back to differences; where the batch does not stay whole, what was
      // found out about the blocks looked into does not hold
      {
        int64_t u[kKbSeg + 1];
        u[0] = tid > 0 ? m.dd[kb_slot(tid * kKbSeg - 1)] : 0;
#pragma unroll
        for (int q = 0; q < kKbSeg; ++q) u[q + 1] = m.dd[kb_slot(tid * kKbSeg + q)];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kKbSeg; ++q) m.dd[kb_slot(tid * kKbSeg + q)] = u[q + 1] - u[q];
      }
      if (record) {
        for (uint32_t x = tid; x < nflag; x += kKbThreads) m.adj[kb_slot(m.flag[x] & 0x7FFF)] = 0;
        accept = retry ? 0u : uint32_t(m.best >> 32);
        __syncthreads();
        for (uint32_t j = accept + tid; j < total; j += kKbThreads) {
          const KbCand c = m.cand[j];
          join(c.f, c.k, -c.s);
        }
      }
    }
    if (retry) {
      // fewer candidates, so that the search is short
      span = (pe - p0 + 3) / 4 > kKbMinSpan ? (pe - p0 + 3) / 4 : kKbMinSpan;
    } else {
      // accepted: hits at their next use
      for (uint32_t j = tid; j < accept; j += kKbThreads) {
        hrow[m.cand[j].k] = 1;
        hc += 1;
        hb += m.cand[j].s;
      }
      if (record) {
        // the candidate is discarded at t, and with it every later key that
        // starts up to t
        p0 = m.cand[accept].k + 1;
        T = int32_t(uint32_t(m.best));
      } else {
        p0 = pe;
        span = 2 * span < kKbWindow ? 2 * span : kKbWindow;
      }
    }
    __syncthreads();
  }
  // the worker's sums
  atomicAdd(reinterpret_cast<unsigned long long*>(&m.hc), (unsigned long long)(hc));
  atomicAdd(reinterpret_cast<unsigned long long*>(&m.hb), (unsigned long long)(hb));
  __syncthreads();
  if (tid == 0 && here) {
    hits[i * 2] = m.hc;
    hits[i * 2 + 1] = m.hb;
  }
}

int buffer_impl(const nopfs_job* job, const int32_t* R, const int32_t* next, const int64_t* sizes,
                int64_t d0, int8_t* hit, int64_t* hits, hipStream_t st) {
  Shape s;
  int rc = make_shape(job, &s);
  if (rc) return rc;
  if (!sizes || !hits) return fail(NOPFS_EINVAL, "sizes and hits must be non-NULL");
  if (d0 < 0) return fail(NOPFS_EINVAL, "d0 must be >= 0");
  if (s.M_max > 0 && (!R || !next || !hit)) return fail(NOPFS_EINVAL, "R, next and hit must be non-NULL");
  if (s.M_max >= (int64_t(1) << kBsMaxLog)) return fail(NOPFS_ERANGE, "M_max must be < 2^24");
  if (s.N >= (int64_t(1) << 31)) return fail(NOPFS_ERANGE, "N too large for one launch");
  BsShape r{s.F, s.N, s.B, s.M_max, s.E, s.drop_last};
  Scratch scr(st);
  // Candidates per worker and epoch of a uniform shuffle (a read has an
  // earlier one with probability 1 - (1 - p)^e in epoch e, p = L / F). The order
  // of next uses pays per change of T, a few per epoch, the stream order per
  // candidate. Measured, the least gain over buffers of 2% to 150% of an
  // epoch: 74 candidates 0.3x, 132 0.6x, 240 0.9x (2.2x typical), 480 1.6x,
  // 520 1.0x (3.0x), 780 1.3x (4.3x), 1,030 1.05x (4.6x).
  const double p = double(s.L) / double(s.F), pe = p * double(s.E);
  const double cands = s.M_max > 0 ? double(s.L) * (1.0 - (1.0 - pow(1.0 - p, double(s.E))) / pe) : 0.0;
  const bool many = cands >= kKbMinCands && d0 < kKbMaxD0 && s.N < 65536;
  // A buffer of few samples: T changes again after few candidates, and the
  // stream order has little to discard. The line lies at a capacity in samples
  // that falls with the candidates and rises with the reads between them: a
  // fit over 110 shapes of 300 to 6,000 candidates at capacities of 1 to 1,000
  // samples, where beyond it the order of next uses took at most 1.4 times the
  // other's time in all but one (355 reads, 338 candidates an epoch, 2 workers,
  // line at 17 samples: 3 samples 2.3x, 20 1.15x, 80 0.6x; 27,365 reads, 1,047
  // candidates, 64 workers, line at 30: 10 1.2x, 40 0.75x; ImageNet-22k, line at 4).
  // Only the device knows the sizes, so both replays are launched and one leaves.
  const double least = many ? 2.2e4 * pow(double(s.L), 0.6) / pow(cands, 1.83) : 0.0;
  const int64_t W0 = (s.M_max + 63) >> 6;
  uint64_t* L0 = nullptr;
  uint32_t* in_order = nullptr;
  int32_t* prev = nullptr;
  const bool either = many && least > 1.0;
  if (!many || either) {
    if ((rc = scr.alloc_n(&L0, size_t(s.N * W0) + 1))) return rc;  // and the choice
    if (either) in_order = reinterpret_cast<uint32_t*>(L0 + s.N * W0);
  }
  if (many && scr.try_alloc_n(&prev, size_t(s.N * s.M_max))) {
    int ash = 0;  // units of adj: 2^ash bytes, at most 2^26 of them in d0
    while ((d0 >> ash) >= (int64_t(1) << 26)) ++ash;
    int sh = kKbMinShift;  // time blocks of 2^sh positions
    while (((s.M_max - 1) >> sh) >= kKbBlocks) ++sh;
    if ((rc = launch("kb_init", kb_init, dim3(uint32_t(ceil_div(s.M_max, 4096)), uint32_t(s.N)),
                     dim3(256), 0, st, r, sizes, d0, least, in_order, prev, hit)))
      return rc;
    if ((rc = launch("kb_prev", kb_prev, dim3(uint32_t(ceil_div(s.M_max, 1024)), uint32_t(s.N)),
                     dim3(256), 0, st, r, next, (const uint32_t*)in_order, prev)))
      return rc;
    if ((rc = launch("kb_sim", kb_sim, dim3(uint32_t(s.N)), dim3(kKbThreads), 0, st, r, R, next, sizes,
                     d0, (const uint32_t*)in_order, ash, sh, (const int32_t*)prev, hit, hits)))
      return rc;
    if (!either) return NOPFS_OK;
  } else {
    in_order = nullptr;  // without memory for the previous uses: stream order
    if (!L0 && (rc = scr.alloc_n(&L0, size_t(s.N * W0)))) return rc;
  }
  return launch("bs_sim", bs_sim, dim3(uint32_t(s.N)), dim3(64), 0, st, r, R, next, sizes, d0,
                (const uint32_t*)in_order, L0, hit, hits);
}

}  // namespace
}  // namespace nopfs

extern "C" int nopfs_buffer_sim(const nopfs_job* job, const int32_t* R, const int32_t* next,
                                const int64_t* sizes, int64_t d0, int8_t* hit, int64_t* hits,
                                void* hip_stream) {
  try {
    return nopfs::buffer_impl(job, R, next, sizes, d0, hit, hits,
                              static_cast<hipStream_t>(hip_stream));
  } catch (const std::bad_alloc&) {
    return nopfs::fail(NOPFS_ENOMEM, "host allocation failed");
  } catch (...) {
    return nopfs::fail(NOPFS_EDEVICE, "unexpected host exception");
  }
}
