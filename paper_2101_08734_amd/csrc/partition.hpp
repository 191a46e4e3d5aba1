// Per-worker partition of the stream R by sample window, shared by the
// passes that need R grouped by sample (access frequencies and first reads,
// next uses, prefetch marks, staging sizes).
//
// For every sub-chunk of 2^14 consecutive reads of one (worker, epoch)
// segment, seg_partition counting-sorts the reads by sample window
// kb = k >> ws and writes them back in place of order, packed as
// (k - kb*W) << 14 | j (j: the read's position in the sub-chunk), with the
// window offsets of the sub-chunk. A "run" is the reads of one window inside
// one sub-chunk; tile (i, kb) walks the runs of all sub-chunks of worker i.
#pragma once

#include "common.hpp"

namespace nopfs {

constexpr int kScShift = 14;
constexpr int kSC = 1 << kScShift;  // reads per sub-chunk
constexpr uint32_t kJMask = kSC - 1;
constexpr uint32_t kMaxWindows = 8192;  // sample windows per worker

struct SegParams {
  int64_t F, N, B, L, M_max;
  int32_t E, drop_last;
  int32_t ws;     // log2 of the window width W
  uint32_t nbk;   // windows per worker: ceil(F / W)
  int32_t nsc;    // sub-chunks per (worker, epoch) segment
  int32_t ent_cap;  // next_tile fast-path capacity (reads)
  int32_t emul;   // epochs per segment: 1, or E when a row is one segment (E = 1)
};

// Reads of one segment of worker i (an epoch, or the whole row when the
// epochs are folded into one segment).
__device__ __forceinline__ int64_t seg_len(const SegParams& p, int64_t i) {
  return int64_t(p.emul) * (p.drop_last ? p.L : epoch_len(p.F, p.N, p.B, 0, i));
}

// For the passes that do not depend on the order of a run's reads: epochs of
// at most half a sub-chunk are folded into one segment per row, cut into
// sub-chunks of 2^14 positions, so that short epochs share a workgroup.
// CosmoFlow (256 reads an epoch, 1,024 workers): 40,960 workgroups of 256 reads
// become 1,024 of 10,240, seg_partition 0.27 -> 0.024, next_unpartition 0.17 ->
// 0.021 ms; ImageNet-1k on 256 workers (5,004 reads): partition 0.16 -> 0.12 ms.
// Long epochs stay as they are: folded at ImageNet-22k (55,456 reads, 3.4
// sub-chunks) the partition took 0.93 ms against 0.87 and the unpartition 1.36
// against 1.25. So do those of jobs that would be left with fewer than 64
// sub-chunks (10,000 samples on 4 workers, 5 epochs: prefetch tiles 16 -> 40 us).
// `fewest` unfolded sub-chunks at least, for passes that take longer over a
// long sub-chunk than over many short ones.
inline void fold_epochs(SegParams& p, int64_t fewest = 0) {
  const int64_t nsc = ceil_div(p.M_max, kSC);
  if (p.L > kSC / 2 || p.N * nsc < 64 || p.N * p.E * int64_t(p.nsc) < fewest) return;
  p.nsc = int32_t(nsc);
  p.emul = p.E;
  p.E = 1;
}

// Mean reads of a run for a uniform shuffle.
inline double run_mean(const SegParams& p) {
  const double seg = double(p.emul) * double(p.L);
  const double span = seg < kSC ? seg : double(kSC);
  const double win = p.F < (int64_t(1) << p.ws) ? double(p.F) : double(int64_t(1) << p.ws);
  const double m = span * win / double(p.F);
  return m > 1e-6 ? m : 1e-6;
}

__device__ __forceinline__ int64_t orow(const SegParams& p, int64_t i, int64_t e, int64_t sc) {
  return ((i * p.E + e) * p.nsc + sc) * int64_t(p.nbk + 1);
}

constexpr uint32_t kRunMap = 2048;  // reads whose run index is kept in LDS

template <int NT>
struct RunTable {
  uint32_t pref[NT + 1];
  int32_t start[NT];  // position in the row of the run's first read
  int32_t fbase[NT];  // stream position of the sub-chunk start
  uint32_t tmp[65];
  uint16_t run_of[kRunMap];  // run index of each read (when total <= kRunMap)
};

// Loads the run table of runs [r0, r0 + NT), none past `runs`, and returns the
// number of reads they hold. Leaves rt ready for lookups.
template <int NT>
__device__ __forceinline__ uint32_t load_runs(const SegParams& p, int64_t i, uint32_t kb,
                                              const uint16_t* __restrict__ OT, RunTable<NT>& rt,
                                              int64_t runs, int64_t r0) {
  const int64_t Li = seg_len(p, i);
  const int64_t R = int64_t(p.E) * p.nsc;
  const uint16_t* oa = OT + (i * (p.nbk + 1) + kb) * R;  // window kb: run starts
  const uint16_t* ob = oa + R;                            // window kb+1: run ends
  const int64_t r = r0 + threadIdx.x;
  uint32_t len = 0;
  if (r < runs) {
    const uint32_t e = uint32_t(r) / uint32_t(p.nsc), sc = uint32_t(r) - e * uint32_t(p.nsc);
    const uint32_t a = oa[r], b = ob[r];
    len = b - a;
    rt.fbase[threadIdx.x] = int32_t(e * Li + sc * kSC);
    rt.start[threadIdx.x] = int32_t(e * Li + sc * kSC + a);
  }
  uint32_t total;
  const uint32_t ex = block_exclusive_scan<false>(len, rt.tmp, &total);  // closed below
  rt.pref[threadIdx.x] = ex;
  if (total <= kRunMap) {
    if (runs - r0 > NT / 4 || total <= uint32_t(NT / 16)) {
      for (uint32_t q = 0; q < len; ++q) rt.run_of[ex + q] = uint16_t(threadIdx.x);
    } else {
      // few runs: 2^lg threads write a run's entries (one alone would write a
      // run of hundreds; for a few reads the barrier costs more: one epoch of
      // 170 reads on 2,763 workers, next-use tiles 473 us with it, 432 without)
      __syncthreads();
      int lg = 2;
      while ((runs - r0) << (lg + 1) <= NT) ++lg;
      const uint32_t run = threadIdx.x >> lg, per = 1u << lg;
      const uint32_t z = rt.pref[run + 1];
      for (uint32_t q = rt.pref[run] + (threadIdx.x & (per - 1)); q < z; q += per) rt.run_of[q] = uint16_t(run);
    }
  }
  __syncthreads();
  return total;
}

// Calls fn(pos, f_base, v, idx) for the `total` reads of the loaded runs:
// pos is the read's position in the partitioned row, f_base the stream
// position of its sub-chunk start, v the packed read and idx its running
// index in (epoch, sub-chunk, position) order. Four loads per thread are in
// flight before any is consumed.
template <int NT, typename Fn>
__device__ __forceinline__ void consume_runs(const RunTable<NT>& rt, int nr, uint32_t total,
                                             const uint32_t* __restrict__ prow, uint32_t done,
                                             Fn fn) {
  for (uint32_t t0 = threadIdx.x; t0 < total; t0 += 4 * NT) {
    int64_t pos[4], fb[4];
    uint32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t t = t0 + u * NT;
      pos[u] = -1;
      fb[u] = 0;
      if (t < total) {
        int lo;
        if (total <= kRunMap) {
          lo = rt.run_of[t];
        } else {
          lo = 0;  // last run with pref <= t
          int hi = nr - 1;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (rt.pref[mid] <= t) lo = mid; else hi = mid - 1;
          }
        }
        pos[u] = rt.start[lo] + (t - rt.pref[lo]);
        fb[u] = rt.fbase[lo];
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = pos[u] >= 0 ? prow[pos[u]] : 0u;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (pos[u] >= 0) fn(pos[u], fb[u], v[u], done + t0 + u * NT);
  }
}

// Calls fn as consume_runs does for every read of runs [lo, hi) of window kb.
template <int NT, typename Fn>
__device__ __forceinline__ void for_runs(const SegParams& p, int64_t i, uint32_t kb,
                                         const uint16_t* __restrict__ O,
                                         const uint32_t* __restrict__ prow, RunTable<NT>& rt,
                                         int64_t lo, int64_t hi, Fn fn) {
  uint32_t done = 0;
  for (int64_t r0 = lo; r0 < hi; r0 += NT) {
    const uint32_t total = load_runs(p, i, kb, O, rt, hi, r0);
    const int nr = int(hi - r0 < NT ? hi - r0 : NT);
    consume_runs(rt, nr, total, prow, done, fn);
    done += total;
    __syncthreads();
  }
}

constexpr int kRunBatch = 8;  // loads in flight per run walk

// Reads of sub-chunk sc of an epoch segment of Li reads.
__device__ __forceinline__ int64_t sub_len(int64_t Li, int64_t sc) {
  const int64_t len = Li - sc * kSC;
  return len < 0 ? 0 : (len > kSC ? kSC : len);
}

// Lanes that share a run in walk_runs: about an eighth of a run's reads
// (kRunBatch loads each), more where there are fewer runs than that many
// groups of threads.
inline int run_lanes(const SegParams& p, int threads) {
  const double m = run_mean(p);
  const int64_t runs = int64_t(p.E) * p.nsc;
  int l = 1;
  while (2 * l <= threads && (l * kRunBatch < m || (2 * l * runs <= threads && l < m))) l *= 2;
  return l;
}

// Calls fn(fb, q, v) for every read of window kb of worker i: fb is the
// stream position of the run's sub-chunk, q the read's index in the
// sub-chunk's partitioned entries (its partitioned position is fb + q) and v
// the packed read. `lanes` consecutive threads of the workgroup share a run
// (a power of two, at most NT).
template <int NT, typename Fn>
__device__ __forceinline__ void walk_runs(const SegParams& p, int64_t i, uint32_t kb,
                                          const uint32_t* __restrict__ Pk,
                                          const uint16_t* __restrict__ OT, uint32_t lanes, Fn fn) {
  const int64_t Li = seg_len(p, i);
  const int64_t runs = int64_t(p.E) * p.nsc;
  const uint16_t* oa = OT + (i * (p.nbk + 1) + kb) * runs;  // run starts in window kb
  const uint16_t* ob = oa + runs;                            // run ends
  const uint32_t* prow = Pk + i * p.M_max;
  const uint32_t nsc = uint32_t(p.nsc);
  const uint32_t sub = threadIdx.x & (lanes - 1);
  for (int64_t r = threadIdx.x / lanes; r < runs; r += NT / lanes) {
    const uint32_t ra = oa[r], rb = ob[r];
    const uint32_t e = uint32_t(r) / nsc, sc = uint32_t(r) - e * nsc;
    const int64_t fb = int64_t(e) * Li + int64_t(sc) * kSC;
    const uint32_t* src = prow + fb;
    for (uint32_t q = ra + sub; q < rb; q += kRunBatch * lanes) {
      uint32_t v[kRunBatch];
#pragma unroll
      for (int u = 0; u < kRunBatch; ++u) {
        const uint32_t y = q + u * lanes;
        v[u] = src[y < rb ? y : ra];  // unconditional
      }
#pragma unroll
      for (int u = 0; u < kRunBatch; ++u)
        if (q + u * lanes < rb) fn(fb, q + u * lanes, v[u]);
    }
  }
}

// Sub-chunk c = e * nsc + sc of worker i covers stream positions
// [e*Li + sc*kSC, + len).
struct SubChunk {
  int64_t i, c, Li, len, base;  // base: offset of its first position in [N][M_max]
};

__device__ __forceinline__ SubChunk sub_chunk(const SegParams& p, uint32_t nch, uint32_t blk) {
  SubChunk s;
  s.i = blk / nch;
  s.c = blk - s.i * nch;
  const int64_t e = s.c / p.nsc, sc = s.c - e * p.nsc;
  s.Li = seg_len(p, s.i);
  s.len = sub_len(s.Li, sc);
  s.base = s.i * p.M_max + e * s.Li + sc * kSC;
  return s;
}

// Partition parameters for windows of 2^ws samples (raised to keep at most
// kMaxWindows windows per worker).
SegParams seg_params(const Shape& s, int ws);

// Partitions R (device, [N][M_max]) into *Pk ([N][M_max], packed reads) and
// the window-major run offsets *OT, both allocated from scr.
int run_partition(const SegParams& p, const int32_t* R, Scratch& scr, uint32_t** Pk,
                  uint16_t** OT, hipStream_t st);

}  // namespace nopfs
