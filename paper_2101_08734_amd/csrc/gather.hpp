// Window-major pass over the partition of R for per-sample values: for every
// read, a value taken from its sample's window (held in LDS) is written at
// the read's place in the partitioned row. Used by the staging schedule
// (each read's size) and by the fetch model (each read's size and source).
//
// The rows are folded into one segment (E = 1 in SegParams, the epochs
// counted by emul), so run c of a row is the window's reads inside span c
// of 2^14 positions. A tile is (window, group of consecutive runs: rows in
// order, a row's spans in order); tiles are window-major, so the groups of
// one window and the tiles of neighbouring windows (whose runs adjoin in
// memory) run together on one XCD. Consecutive threads take consecutive reads
// of the tile's runs, so loads and stores go out in run-long pieces (at
// ImageNet-22k 19 reads on average in the fetch model's windows of 2^14 samples,
// 38 in the staging schedule's of 2^15) instead of one store per lane into 64
// different runs.
#pragma once

#include "partition.hpp"

namespace nopfs {

constexpr int kGatherWs = 14;                 // window: 2^14 samples of 8-byte values
constexpr int kGatherWin = 1 << kGatherWs;    // 8-byte values held in LDS (128 KB)
constexpr int kGThreads = 1024;
// A tile holds about kGReads reads (ImageNet-22k, 20 epochs, with 81,920, 163,840 and
// 327,680: the staging schedule's pass 957, 888 and 832 us, the fetch model's 2,384,
// 2,407 and 2,142; the largest was not measured on other jobs): its window's values
// (128 KB of LDS) are loaded once for all of them, which takes as long as kGLoad
// reads do (10.5 us and 0.65 ns a read: 166 tiles of 65,000 reads 53 us, 1,162 of
// 9,300 83 us). Where that makes fewer than kGRounds rounds of tiles (one at a time
// per compute unit), their number follows the last round: the cheapest of the splits
// that fill 1 to kGRounds rounds.
constexpr double kGReads = 163840, kGLoad = 16384;
constexpr int64_t kGRounds = 8, kGUnits = 256;
constexpr int kGRuns = 1024;                  // runs per pass of a tile
// Mean reads per run from which waves take whole runs. With eight reads per
// thread (staging) a wave takes 512 of a run at a time: runs of 107 reads 206 us
// so and 149 by search, of 153 123 and 112, of 199 137 and 145, of 268 93 and 111,
// of 1,342 37 and 53. With four (fetch model; each read also waits for its own
// tier, which the search's shorter steps hide): 99 reads 366 and 279 us, 210 715
// and 583, 383 137 and 120, 5,370 38 and 35, 8,950 36 and 38, 10,000 21 and 25.
template <int kPer>
constexpr uint32_t kGLongRun = kPer >= 8 ? 192 : 8192;
static_assert(kGRuns % kGThreads == 0, "gather tile shape");

// kChunk: reads per inner pass of the workgroup; each thread requests
// kChunk / kGThreads reads of the pass at once.
template <int kChunk>
struct GatherLds {
  static_assert(kChunk % kGThreads == 0, "gather tile shape");
  union {
    uint64_t win[kGatherWin];        // the window's 8-byte values
    uint32_t win4[2 * kGatherWin];   // or 4-byte values, twice as many
  };
  uint32_t pref[kGRuns + 1];  // reads before each run of the pass
  int32_t rpos[kGRuns];       // span start + run start, in the row
  uint32_t rrow[kGRuns];      // row - first row of the tile
  uint32_t tmp[65];
};

// Runs per tile of a gather pass, and from it the groups per window.
inline int64_t gather_runs(const SegParams& p) {
  const int64_t runs = p.N * p.nsc;
  const double run = run_mean(p);  // reads
  int64_t per = int64_t(kGReads / run) + 1;
  per = per < runs ? per : runs;
  if (runs < 1 || ceil_div(runs, per) * p.nbk >= kGRounds * kGUnits) return per;
  const double win = double(int64_t(1) << p.ws);
  const double load = kGLoad * (double(p.F) < win ? double(p.F) / win : 1.0);
  double best = 0;
  for (int64_t r = 1; r <= kGRounds; ++r) {
    int64_t g = r * kGUnits / p.nbk;  // groups per window that fill r rounds
    g = g < 1 ? 1 : (g < runs ? g : runs);
    const double cost = double(ceil_div(g * p.nbk, kGUnits)) * (load + run * double(runs) / double(g));
    if (best == 0 || cost < best) {
      best = cost;
      per = ceil_div(runs, g);
    }
  }
  return per;
}

// Window width (log2) of a gather pass: kGatherWs, or wider by the test
// hook's doublings (at most 4: the packed partition entries hold 18 bits of
// offset), so that small jobs take the several-pass path of larger ones.
inline int gather_ws() {
  const int64_t x = debug_value(5);
  return kGatherWs + int(x > 0 ? (x < 4 ? x : 4) : 0);
}

// Tile `tile` of the pass. value(k) gives sample k's value of type V (8 or
// 4 bytes; it is called for k in [0, F) only); emit(pos, row, x, w0, wl)
// receives kChunk / kGThreads reads of this thread at once: pos[u] the read's index in the
// row table ([N][M_max], -1 for none), row[u] its row, x[u] its sample's
// offset in the window pass starting at sample w0 (valid when x[u] < wl),
// with the window's values in L.win (V = uint64_t) or L.win4 (uint32_t).
template <typename V, int kChunk, typename Value, typename Emit>
__device__ __forceinline__ void gather_tile(const SegParams& p, const uint32_t* __restrict__ Pk,
                                            const uint16_t* __restrict__ OT, uint32_t tile,
                                            uint32_t ngroups, int64_t per, GatherLds<kChunk>& L,
                                            Value value, Emit emit) {
  constexpr int kPer = kChunk / kGThreads;
  const uint32_t kb = tile / ngroups;
  const int64_t nch = p.nsc;
  const int64_t run0 = int64_t(tile - kb * ngroups) * per;  // the tile's first run
  const int64_t i0 = run0 / nch;                            // its row
  const int64_t c0 = run0 - i0 * nch;                       // and span
  const int64_t nruns = p.N * nch - run0 < per ? p.N * nch - run0 : per;  // c0 + nruns < 2^32
  const int64_t k0 = int64_t(kb) << p.ws;
  const int64_t kend = k0 + (int64_t(1) << p.ws) < p.F ? k0 + (int64_t(1) << p.ws) : p.F;
  constexpr int kWin = int(kGatherWin * sizeof(uint64_t) / sizeof(V));  // values per pass
  V* win = sizeof(V) == 8 ? reinterpret_cast<V*>(L.win) : reinterpret_cast<V*>(L.win4);
  for (int64_t w0 = k0; w0 < kend; w0 += kWin) {  // one pass unless windows are wider
    const uint32_t wl = uint32_t(kend - w0 < kWin ? kend - w0 : kWin);
    const uint32_t xoff = uint32_t(w0 - k0);
    // the window's values, sixteen loads per thread in flight at once
    for (uint32_t x0 = 0; x0 < wl; x0 += 16 * kGThreads) {
      V v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const uint32_t x = x0 + u * kGThreads + threadIdx.x;
        v[u] = value(w0 + (x < wl ? x : 0));
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const uint32_t x = x0 + u * kGThreads + threadIdx.x;
        if (x < wl) win[x] = v[u];
      }
    }
    for (int64_t r0 = 0; r0 < nruns; r0 += kGRuns) {
      const uint32_t nr = uint32_t(nruns - r0 < kGRuns ? nruns - r0 : kGRuns);
      uint32_t len[kGRuns / kGThreads];
      uint32_t sum = 0;
#pragma unroll
      for (int m = 0; m < kGRuns / kGThreads; ++m) {
        const uint32_t r = threadIdx.x * (kGRuns / kGThreads) + m;
        // loads for runs past nr read run r0's bounds and are dropped
        const uint32_t rr = uint32_t(c0 + r0) + (r < nr ? r : 0u);
        const uint32_t il = rr / uint32_t(nch), c = rr - il * uint32_t(nch);
        const uint16_t* o = OT + ((i0 + il) * (p.nbk + 1) + kb) * nch + c;
        const uint32_t a = o[0], b = o[nch];
        len[m] = r < nr ? b - a : 0u;
        if (r < nr) {
          L.rpos[r] = int32_t((int64_t(c) << kScShift) + a);
          L.rrow[r] = il;
        }
        sum += len[m];
      }
      uint32_t total;
      uint32_t run = block_exclusive_scan<false>(sum, L.tmp, &total);  // closed below
#pragma unroll
      for (int m = 0; m < kGRuns / kGThreads; ++m) {
        L.pref[threadIdx.x * (kGRuns / kGThreads) + m] = run;
        run += len[m];
      }
      if (threadIdx.x == 0) L.pref[nr] = total;
      __syncthreads();
      if (total >= kGLongRun<kPer> * nr) {  // uniform
        // long runs: kG waves to a run (one where there are as many runs as
        // waves), each lane's loads of a step together, no lookup per read.
        constexpr uint32_t kWaves = kGThreads / 64, kStep = 64 * kPer;
        const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
        uint32_t wpr = 1;
        while (2 * wpr * nr <= kWaves) wpr *= 2;
        for (uint32_t r = wave / wpr; r < nr; r += kWaves / wpr) {
          const uint32_t rl = L.pref[r + 1] - L.pref[r];
          const int64_t rrow = i0 + L.rrow[r];
          const int64_t rbase = rrow * p.M_max + L.rpos[r];
          for (uint32_t q0 = (wave & (wpr - 1)) * kStep; q0 < rl; q0 += wpr * kStep) {
            int64_t pos[kPer], row[kPer];
            uint32_t x[kPer];
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
              const uint32_t q = q0 + u * 64 + lane;
              row[u] = rrow;
              pos[u] = q < rl ? rbase + q : -1;
            }
#pragma unroll
            for (int u = 0; u < kPer; ++u) x[u] = Pk[pos[u] >= 0 ? pos[u] : rbase];  // unconditional
#pragma unroll
            for (int u = 0; u < kPer; ++u) x[u] = pos[u] >= 0 ? (x[u] >> kScShift) - xoff : 0xFFFFFFFFu;
            emit(pos, row, x, w0, wl);
          }
        }
        __syncthreads();  // the run table is rewritten
        continue;
      }
      // short runs: each wave takes 64 * kPer consecutive reads at a time and
      // looks up each read's run in the counts before the runs (those past nr
      // hold the total): ten steps in LDS, and no barrier, so that the waves'
      // loads overlap. A map of 4,096 reads at a time, written by the runs'
      // owners between barriers, took 4.40 ms in the fetch model's pass at
      // ImageNet-22k (19 reads a run), this 3.88.
      constexpr uint32_t kSpan = 64 * kPer;
      const uint32_t lane = threadIdx.x & 63;
      for (uint32_t x0 = (threadIdx.x >> 6) * kSpan; x0 < total; x0 += kChunk) {
        uint32_t r[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) r[u] = 0;
#pragma unroll
        for (uint32_t st = kGRuns / 2; st > 0; st >>= 1)
#pragma unroll
          for (int u = 0; u < kPer; ++u)
            r[u] += L.pref[r[u] + st] <= x0 + u * 64 + lane ? st : 0u;
        int64_t pos[kPer], row[kPer];
        uint32_t x[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
          const uint32_t t = x0 + u * 64 + lane;
          pos[u] = -1;
          row[u] = i0;
          if (t < total) {
            row[u] = i0 + L.rrow[r[u]];
            pos[u] = row[u] * p.M_max + L.rpos[r[u]] + (t - L.pref[r[u]]);
          }
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) x[u] = Pk[pos[u] >= 0 ? pos[u] : 0];  // unconditional
#pragma unroll
        for (int u = 0; u < kPer; ++u) x[u] = pos[u] >= 0 ? (x[u] >> kScShift) - xoff : 0xFFFFFFFFu;
        emit(pos, row, x, w0, wl);
      }
      __syncthreads();  // the run table is rewritten
    }
    __syncthreads();
  }
}

}  // namespace nopfs
