// nopfs_fetch_model: the performance model of the Performance Modeling
// section evaluated for every read of every worker's stream, with the
// placement static (a sample is in tier j of worker i exactly when
// tier[i][k] == j).
//
// A read of sample k (s bytes) by worker i is fetched from the fastest of
// the PFS (t(gamma) / gamma per reader), another worker's tier j
// (min(b_c, r_j / p_j)) and its own tier j (r_j / p_j); on equal throughput
// its own tier wins over a remote one and a remote one over the PFS. It is
// then preprocessed and written to the staging buffer at min(beta, w0 / p0)
// per thread. With the p0 staging threads load-balanced, read f is in the
// buffer at avail(f) = (sum of the read times of reads 0..f) / p0, and the
// worker consumes it at
//   t(f) = max(avail(f), t(f-1) + s(f-1) / c) = U(f) + max over g <= f of (avail(g) - U(g)),
// U(f) = sum of s(m) / c over m < f (the recurrence unrolled): a prefix sum
// and a prefix maximum, evaluated per sub-chunk and chained along the worker's row.
//
//   fm_holders -- per sample: the best remote class among all workers'
//                 copies (highest min(b_c, r_j / p_j), lower tier on ties),
//                 packed above the sample's size. A worker's own copy may be
//                 that class: a remote copy of class j is never faster than
//                 the local copy of j, so counting it never changes a choice.
//   fm_gather  -- per (16K-sample window, group of runs) of the
//                 partition of R (rows folded into one segment of E * L_i
//                 reads, cut into spans of 2^14): each read's source from
//                 its own tier and the sample's best remote class; size and
//                 source in partitioned order.
//   fm_final   -- per span of 2^14 reads: every entry loaded once into the LDS
//                 slot of its stream position (the whole sub-chunk, 135 KB);
//                 its read-time sum, compute-time sum and maximum of
//                 avail - U are scanned and published, what enters it is
//                 chained from the spans before; source codes and consumption
//                 times in stream order.
#include <math.h>

#include <new>

#include "gather.hpp"
#include "partition.hpp"

namespace nopfs {
namespace {

constexpr int kMaxClasses = 32;
constexpr uint32_t kNoClass = 255;
constexpr int kSizeBits = 56;
constexpr uint64_t kSizeMask = (uint64_t(1) << kSizeBits) - 1;
constexpr int kFmThreads = 1024;
constexpr int kFmPer = kSC / kFmThreads;        // positions (and entries) per thread
constexpr uint32_t kFmBlocks = 256;             // workgroups in flight: one per CU
static_assert(kFmPer == 16, "16 consecutive positions stay within one pad of fm_slot");

// Source codes inside the library: 0 the PFS, 1 + j another worker's tier j,
// 1 + kMaxClasses + j the worker's own tier j.
constexpr uint32_t kOwn0 = 1 + kMaxClasses;

// Source rates, computed once on the host from the model's parameters.
struct Rates {
  double own[kMaxClasses];  // r_j / p_j
  double rem[kMaxClasses];  // min(b_c, r_j / p_j)
  double pfs;               // t(gamma) / gamma
  double wthr;              // min(beta, w0 / p0)
  double c, p0;
  // reciprocals for the per-read times (a product instead of a division:
  // within two units in the last place of the quotient)
  double inv[1 + 2 * kMaxClasses];  // by source code
  double inv_wthr, inv_c;
  int32_t J;
  uint8_t rank_cls[kMaxClasses];  // classes by remote rate, best first, lower tier on ties
  uint8_t cls_rank[kMaxClasses];  // the inverse
};

struct SharedRates {
  double own[kMaxClasses], rem[kMaxClasses];
  double inv[1 + 2 * kMaxClasses];
  uint8_t rank_cls[kMaxClasses], cls_rank[kMaxClasses];
};

__device__ __forceinline__ void load_rates(const Rates& r, SharedRates& s) {
  if (threadIdx.x < kMaxClasses) {
    s.own[threadIdx.x] = r.own[threadIdx.x];
    s.rem[threadIdx.x] = r.rem[threadIdx.x];
    s.rank_cls[threadIdx.x] = r.rank_cls[threadIdx.x];
    s.cls_rank[threadIdx.x] = r.cls_rank[threadIdx.x];
  }
  for (uint32_t x = threadIdx.x; x < 1 + 2 * kMaxClasses; x += blockDim.x) s.inv[x] = r.inv[x];
}

// ---------------------------------------------------------------- holders --
__global__ void __launch_bounds__(256)
fm_holders(int64_t F, int64_t N, const int8_t* __restrict__ tier, const int64_t* __restrict__ sizes,
           Rates rt, uint64_t* __restrict__ szb, uint64_t* __restrict__ state, int64_t nstate,
           uint32_t* __restrict__ ticket) {
  __shared__ SharedRates sr;
  load_rates(rt, sr);
  __syncthreads();
  const int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x;
  // the spans' states and the ticket of the last kernel
  for (int64_t x = k; x < nstate; x += int64_t(gridDim.x) * 256) state[x] = ~uint64_t(0);
  if (k == 0) *ticket = 0;
  if (k >= F) return;
  uint32_t best = kNoClass;  // as a rank: lower is better
  constexpr int kRows = 8;
  for (int64_t i0 = 0; i0 < N; i0 += kRows) {
    int32_t q[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) q[u] = i0 + u < N ? tier[(i0 + u) * F + k] : -1;
#pragma unroll
    for (int u = 0; u < kRows; ++u)
      if (q[u] >= 0 && q[u] < rt.J) {
        const uint32_t rk = sr.cls_rank[q[u]];
        best = rk < best ? rk : best;
      }
  }
  const uint64_t cls = best == kNoClass ? kNoClass : sr.rank_cls[best];
  szb[k] = (uint64_t(sizes[k]) & kSizeMask) | (cls << kSizeBits);
}

// ------------------------------------------------------------------ tiles --
__device__ __forceinline__ uint32_t choose(const Rates& rt, const SharedRates& sr, int32_t own,
                                           uint32_t b1) {
  double best = -1;
  uint32_t code = 0;
  if (own >= 0 && own < rt.J) {
    best = sr.own[own];
    code = kOwn0 + uint32_t(own);
  }
  if (b1 != kNoClass && sr.rem[b1] > best) {
    best = sr.rem[b1];
    code = 1 + b1;
  }
  if (rt.pfs > best) code = 0;
  return code;
}

// Each read of the tile's window and rows gets its source (choose) and its
// size, packed, at its place in the partitioned row. Four reads per thread
// and inner pass (eight, as in the staging gather, were no faster here).
constexpr int kFmGChunk = 4 * kGThreads;
constexpr int kFmGPer = kFmGChunk / kGThreads;
__global__ void __launch_bounds__(kGThreads)
fm_gather(SegParams p, const uint32_t* __restrict__ Pk, const uint16_t* __restrict__ OT,
          const int8_t* __restrict__ tier, const uint64_t* __restrict__ szb, Rates rt,
          uint64_t* __restrict__ zP, uint32_t ngroups, int64_t per, uint32_t ntiles) {
  __shared__ GatherLds<kFmGChunk> L;
  __shared__ SharedRates sr;
  const uint32_t tile = xcd_logical(blockIdx.x, gridDim.x);
  if (tile >= ntiles) return;
  load_rates(rt, sr);  // visible after the tile's first barrier
  gather_tile<uint64_t, kFmGChunk>(
      p, Pk, OT, tile, ngroups, per, L, [&](int64_t k) { return szb[k]; },
      [&](const int64_t (&pos)[kFmGPer], const int64_t (&row)[kFmGPer], const uint32_t (&x)[kFmGPer],
          int64_t w0, uint32_t wl) {
        // each read's own tier: a byte of its row's window slice (cached),
        // loads first, unconditional
        int32_t own[kFmGPer];
#pragma unroll
        for (int u = 0; u < kFmGPer; ++u) own[u] = tier[row[u] * p.F + w0 + (x[u] < wl ? x[u] : 0u)];
#pragma unroll
        for (int u = 0; u < kFmGPer; ++u)
          if (pos[u] >= 0 && x[u] < wl) {
            const uint64_t sb = L.win[x[u]];
            const uint32_t code = choose(rt, sr, own[u], uint32_t(sb >> kSizeBits));
            zP[pos[u]] = (sb & kSizeMask) | (uint64_t(code) << kSizeBits);
          }
      });
}

// ------------------------------------------------------------------ scans --
__device__ __forceinline__ double wave_incl_sum(double v) {
  const int lane = __lane_id();
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double o = __shfl_up(v, d, 64);
    if (lane >= d) v += o;
  }
  return v;
}

__device__ __forceinline__ double wave_incl_max(double v) {
  const int lane = __lane_id();
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double o = __shfl_up(v, d, 64);
    if (lane >= d) v = fmax(v, o);
  }
  return v;
}

// Exclusive prefix scans over the workgroup (blockDim.x a multiple of 64):
// two sums at once, or a maximum with -inf as identity; the totals go to
// *tot*. No closing barrier: the caller's next use of tmp comes after later
// barriers. tmp holds 65 entries.
__device__ __forceinline__ void block_excl_sum2(double a, double u, double2* tmp, double* exa,
                                                double* exu, double* tota, double* totu) {
  const int lane = __lane_id();
  const int wave = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  const double ia = wave_incl_sum(a), iu = wave_incl_sum(u);
  if (lane == 63) tmp[wave] = make_double2(ia, iu);
  __syncthreads();
  if (threadIdx.x < 64) {
    const double2 w = threadIdx.x < unsigned(nwaves) ? tmp[threadIdx.x] : make_double2(0.0, 0.0);
    const double wa = wave_incl_sum(w.x), wu = wave_incl_sum(w.y);
    const double pa = __shfl_up(wa, 1, 64), pu = __shfl_up(wu, 1, 64);
    if (threadIdx.x < unsigned(nwaves))
      tmp[threadIdx.x] = threadIdx.x == 0 ? make_double2(0.0, 0.0) : make_double2(pa, pu);
    if (threadIdx.x == 63) tmp[64] = make_double2(wa, wu);
  }
  __syncthreads();
  const double ba = __shfl_up(ia, 1, 64), bu = __shfl_up(iu, 1, 64);
  const double2 tw = tmp[wave];
  *exa = tw.x + (lane == 0 ? 0.0 : ba);
  *exu = tw.y + (lane == 0 ? 0.0 : bu);
  *tota = tmp[64].x;
  *totu = tmp[64].y;
}

__device__ __forceinline__ double block_excl_max(double v, double* tmp, double* total) {
  const int lane = __lane_id();
  const int wave = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  const double inc = wave_incl_max(v);
  if (lane == 63) tmp[wave] = inc;
  __syncthreads();
  if (threadIdx.x < 64) {
    const double w = threadIdx.x < unsigned(nwaves) ? tmp[threadIdx.x] : -INFINITY;
    const double wi = wave_incl_max(w);
    const double prev = __shfl_up(wi, 1, 64);
    if (threadIdx.x < unsigned(nwaves)) tmp[threadIdx.x] = threadIdx.x == 0 ? -INFINITY : prev;
    if (threadIdx.x == 63) tmp[64] = wi;
  }
  __syncthreads();
  const double before_lane = __shfl_up(inc, 1, 64);
  *total = tmp[64];
  return fmax(tmp[wave], lane == 0 ? -INFINITY : before_lane);
}

// LDS slot of position p: one pad per 32 positions, so the 16 consecutive
// positions each thread takes fall on distinct banks across a half-wave
__device__ __forceinline__ int fm_slot(int p) { return p + (p >> 5); }

// What enters a span of worker i: read-time sum and compute-time sum of the
// reads before it, and the largest avail(g) - U(g) over them. A span's own
// sums have the same form, relative to its start.
struct Enter {
  double a, u, m;
};

// `in` followed by a span with the sums `x`
__device__ __forceinline__ Enter fm_then(const Enter& in, const Enter& x, double inv_p0) {
  return Enter{in.a + x.a, in.u + x.u, fmax(in.m, in.a * inv_p0 - in.u + x.m)};
}

// What a span publishes: its own sums as soon as they are known, then what
// leaves it. Each word is valid by itself once it is no longer all ones (a
// NaN that no arithmetic makes), so no fence goes with it.
struct FmState {
  uint64_t own[3], out[3];
};
constexpr uint64_t kFmUnset = ~uint64_t(0);

__device__ __forceinline__ void fm_publish(uint64_t (&w)[3], const Enter& e) {
  const double d[3] = {e.a, e.u, e.m};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint64_t b = uint64_t(__double_as_longlong(d[k]));
    __hip_atomic_store(&w[k], b == kFmUnset ? b - 1 : b, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
}

__device__ __forceinline__ bool fm_read(const uint64_t (&w)[3], Enter& e) {
  uint64_t b[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    b[k] = __hip_atomic_load(&w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  e = Enter{__longlong_as_double(int64_t(b[0])), __longlong_as_double(int64_t(b[1])),
            __longlong_as_double(int64_t(b[2]))};
  return b[0] != kFmUnset && b[1] != kFmUnset && b[2] != kFmUnset;
}

// What enters span c of a row (one whole wave): lane l looks at span
// c - 1 - l; from the nearest span whose output is there, the own sums of
// those after it are added in span order, so the result is that of the
// sequential sum whichever span that was. The wait ends: every span before
// this one was taken earlier by a running workgroup, and publishes its own
// sums before it waits for anything.
__device__ Enter fm_enter(const FmState* row, int64_t c, double inv_p0) {
  const int64_t q = c - 1 - __lane_id();
  for (;;) {
    Enter own{0, 0, 0}, out{0, 0, -INFINITY};
    bool has_own = false, has_out = q == -1;  // nothing enters the row's first span
    if (q >= 0) {
      has_own = fm_read(row[q].own, own);
      has_out = fm_read(row[q].out, out);
    }
    const uint64_t mo = __ballot(has_out), mw = __ballot(has_own);
    if (mo) {
      const int f = __ffsll(static_cast<unsigned long long>(mo)) - 1;
      const uint64_t need = (uint64_t(1) << f) - 1;
      if ((mw & need) == need) {
        Enter e{__shfl(out.a, f, 64), __shfl(out.u, f, 64), __shfl(out.m, f, 64)};
        for (int l = f - 1; l >= 0; --l)
          e = fm_then(e, Enter{__shfl(own.a, l, 64), __shfl(own.u, l, 64), __shfl(own.m, l, 64)},
                      inv_p0);
        return e;
      }
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

struct FmLds {
  uint64_t sv[kSC + kSC / 32];  // the span's entries by position, then the times
  uint32_t code[kSC / 4];       // source codes by position, a byte each
  double2 tmp2[65];             // the two sum scans
  double tmpm[65];              // the maximum scan
  Enter in;
  uint32_t ticket;
  SharedRates sr;
};

// A span's entries as loaded by one thread: entries t, t + kFmThreads, ...
// of its partitioned order (packed position, size and source). The loads
// are unconditional (past the span's end they read its first entry and are
// dropped when stored), so they are in flight together.
struct FmRegs {
  uint32_t j[kFmPer];
  uint64_t v[kFmPer];
};

__device__ __forceinline__ void fm_load(const SubChunk& s, const uint32_t* __restrict__ Pk,
                                        const uint64_t* __restrict__ zP, FmRegs& g) {
  const uint32_t* pk = Pk + s.base;
  const uint64_t* z = zP + s.base;
  const uint32_t len = uint32_t(s.len);
#pragma unroll
  for (int u = 0; u < kFmPer; ++u) {
    const uint32_t q = uint32_t(u) * kFmThreads + threadIdx.x;
    g.j[u] = pk[q < len ? q : 0];
    g.v[u] = z[q < len ? q : 0];
  }
}

// Every entry of the span into the LDS slot of its stream position. Ends
// with a barrier.
__device__ __forceinline__ void fm_place(const SubChunk& s, const FmRegs& g, FmLds& L) {
#pragma unroll
  for (int u = 0; u < kFmPer; ++u)
    if (uint32_t(u) * kFmThreads + threadIdx.x < uint32_t(s.len)) L.sv[fm_slot(int(g.j[u] & kJMask))] = g.v[u];
  __syncthreads();
}

// One workgroup per CU (the span takes 135 KB of LDS) takes spans by ticket, in
// order of their place in the row (the first of every row, then the second,
// ...), so that what enters a span is mostly there when it is asked for.
// The row's times are chained by a scan with decoupled look-back (Merrill and
// Garland, Single-pass Parallel Prefix Scan with Decoupled Look-back, 2016): a span
// publishes its own sums, then its row's up to its end.
// Bound by HBM traffic (ImageNet-22k: 6.8 GB of entries in, 5.7 GB of times and
// codes out, 3.49 ms, 3.6 TB/s of a copy's 4.9) and, for what is missing to the
// copy, by the scan, when the workgroup, alone on its compute unit, has nothing in
// flight. One kernel for the spans' sums, one that chained them per row and a last one
// that read the entries again took 2.72 + 0.15 + 3.64 ms. Positions go 16 to a
// thread, so the span is scanned once (six barriers), and the next span's
// entries are requested while this one goes out; a thread's times are looked
// up by each sweep, as holding them (64 registers) spills.
__global__ void __launch_bounds__(kFmThreads)
fm_final(SegParams p, const uint32_t* __restrict__ Pk, const uint64_t* __restrict__ zP, Rates rt,
         uint32_t nch, uint32_t nblk, FmState* state, uint32_t* ticket,
         int16_t* __restrict__ src, double* __restrict__ t) {
  __shared__ FmLds L;
  static_assert(sizeof(FmLds) <= 160 * 1024, "one span fits the LDS");
  load_rates(rt, L.sr);
  const double inv_p0 = 1.0 / rt.p0;
  if (threadIdx.x == 0) L.ticket = atomicAdd(ticket, 1u);
  __syncthreads();
  uint32_t b = uint32_t(__builtin_amdgcn_readfirstlane(int(L.ticket)));
  const uint32_t rows = uint32_t(p.N);
  SubChunk s;
  FmRegs g;
  if (b < nblk) {
    s = sub_chunk(p, nch, b % rows * nch + b / rows);
    fm_load(s, Pk, zP, g);
  }
  while (b < nblk) {
    if (s.c == int64_t(nch) - 1) {
      // the row's padding past its last read
      for (int64_t f = int64_t(p.E) * s.Li + threadIdx.x; f < p.M_max; f += kFmThreads) {
        src[s.i * p.M_max + f] = -1;
        t[s.i * p.M_max + f] = -1.0;
      }
    }
    fm_place(s, g, L);
    const int x0 = int(threadIdx.x) * kFmPer;
    const int len = int(s.len);
    uint64_t* mine = L.sv + fm_slot(x0);  // its slots: consecutive (16 of 32)
    // read and compute time of a position of this thread (0 past the span's end)
    auto times = [&](int u, double& rd, double& uu) {
      const uint64_t e = mine[u];
      const double sz = x0 + u < len ? double(e & kSizeMask) : 0.0;
      const uint32_t code = x0 + u < len ? uint32_t(e >> kSizeBits) : 0u;
      rd = sz * L.sr.inv[code] + sz * rt.inv_wthr;
      uu = sz * rt.inv_c;
      return code;
    };
    double ta = 0, tu = 0;
    const int mine_n = x0 < len ? kFmPer : 0;  // threads behind the span's end take no sweep
#pragma unroll 1
    for (int u0 = 0; u0 < mine_n; u0 += 4) {
      uint32_t cw = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double rd, uu;
        cw |= times(u0 + v, rd, uu) << (8 * v);
        ta += rd;
        tu += uu;
      }
      L.code[(x0 + u0) / 4] = cw;
    }
    Enter own;
    double exa, exu;
    block_excl_sum2(ta, tu, L.tmp2, &exa, &exu, &own.a, &own.u);
    // avail - U at each position, relative to the span's start. A position's
    // sums are the thread's own (small) plus what precedes them: one rounding
    // at the sums' size per position, not one per read of the thread.
    double la = 0, lu = 0, tm = -INFINITY;
#pragma unroll 4
    for (int u = 0; u < mine_n; ++u) {
      double rd, uu;
      times(u, rd, uu);
      la += rd;
      if (x0 + u < len) tm = fmax(tm, (exa + la) * inv_p0 - (exu + lu));
      lu += uu;
    }
    double run = block_excl_max(tm, L.tmpm, &own.m);
    if (threadIdx.x < 64) {
      FmState* row = state + s.i * nch;
      if (threadIdx.x == 0) fm_publish(row[s.c].own, own);
      const Enter in = fm_enter(row, s.c, inv_p0);
      if (threadIdx.x == 0) {
        fm_publish(row[s.c].out, fm_then(in, own, inv_p0));
        L.in = in;
        L.ticket = atomicAdd(ticket, 1u);
      }
    }
    __syncthreads();
    const Enter in = L.in;
    const double base_mu = in.a * inv_p0 - in.u;
    // t at each position: U(f) + max(what entered, base + best so far), into
    // the slots this thread read its entries from
    la = lu = 0;
#pragma unroll 4
    for (int u = 0; u < mine_n; ++u) {
      double rd, uu;
      times(u, rd, uu);
      la += rd;
      const double ru = exu + lu;
      run = fmax(run, (exa + la) * inv_p0 - ru);
      mine[u] = uint64_t(__double_as_longlong((in.u + ru) + fmax(in.m, base_mu + run)));
      lu += uu;
    }
    const uint32_t b2 = uint32_t(__builtin_amdgcn_readfirstlane(int(L.ticket)));
    __syncthreads();
    // the next span's entries are requested before this one goes out
    const SubChunk d = s;
    if (b2 < nblk) {
      s = sub_chunk(p, nch, b2 % rows * nch + b2 / rows);
      fm_load(s, Pk, zP, g);
    }
    const uint8_t* code = reinterpret_cast<const uint8_t*>(L.code);
#pragma unroll 4
    for (int u = 0; u < kFmPer; ++u) {
      if (u * kFmThreads >= len) break;  // uniform
      const int x = u * kFmThreads + int(threadIdx.x);
      if (x < len) {
        const uint32_t c = code[x];
        stream_store(t + d.base + x, __longlong_as_double(int64_t(L.sv[fm_slot(x)])));
        stream_store(src + d.base + x,
                     int16_t(c == 0 ? 0u : (c < kOwn0 ? 128u + (c - 1) : 256u + (c - kOwn0))));
      }
    }
    b = b2;
    __syncthreads();
  }
}

Rates make_rates(const nopfs_model* m) {
  Rates r{};
  r.J = m->J;
  for (int32_t j = 0; j < kMaxClasses; ++j) {
    r.own[j] = j < m->J ? m->r[j] / m->p[j] : 0;
    r.rem[j] = j < m->J ? (m->b_c < r.own[j] ? m->b_c : r.own[j]) : 0;
  }
  r.pfs = m->pfs_t / m->pfs_gamma;
  const double wb = m->w0 / m->p0;
  r.wthr = m->beta < wb ? m->beta : wb;
  r.c = m->c;
  r.p0 = m->p0;
  for (int32_t j = 0; j < kMaxClasses; ++j) {
    r.inv[1 + j] = j < m->J ? 1.0 / r.rem[j] : 0;
    r.inv[kOwn0 + j] = j < m->J ? 1.0 / r.own[j] : 0;
  }
  r.inv[0] = 1.0 / r.pfs;
  r.inv_wthr = 1.0 / r.wthr;
  r.inv_c = 1.0 / r.c;
  // classes ranked by remote rate (higher first), lower tier on ties
  int32_t order[kMaxClasses];
  for (int32_t j = 0; j < m->J; ++j) order[j] = j;
  for (int32_t a = 1; a < m->J; ++a)
    for (int32_t b = a; b > 0 && r.rem[order[b]] > r.rem[order[b - 1]]; --b) {
      const int32_t x = order[b];
      order[b] = order[b - 1];
      order[b - 1] = x;
    }
  for (int32_t q = 0; q < kMaxClasses; ++q) {
    r.rank_cls[q] = q < m->J ? uint8_t(order[q]) : uint8_t(kNoClass);
    r.cls_rank[q] = uint8_t(kNoClass);
  }
  for (int32_t q = 0; q < m->J; ++q) r.cls_rank[order[q]] = uint8_t(q);
  return r;
}

int model_impl(const nopfs_job* job, const int32_t* R, const int8_t* tier, const int64_t* sizes,
               const nopfs_model* model, int16_t* src, double* t, hipStream_t st) {
  Shape s;
  int rc = make_shape(job, &s);
  if (rc) return rc;
  if ((rc = model_check(model))) return rc;
  if (!tier || !sizes) return fail(NOPFS_EINVAL, "tier and sizes must be non-NULL");
  if (s.M_max == 0) return NOPFS_OK;
  if (!R || !src || !t) return fail(NOPFS_EINVAL, "R, src and t must be non-NULL");
  const Rates rt = make_rates(model);
  // one segment per row (the E epochs folded together), cut into spans of
  // 2^14 positions, partitioned by windows of 2^14 samples
  SegParams p = seg_params(s, gather_ws());
  const uint32_t nch = uint32_t(ceil_div(s.M_max, kSC));  // spans per row
  p.emul = int32_t(s.E);
  p.E = 1;
  p.nsc = int32_t(nch);
  const int64_t per = gather_runs(p);
  const int64_t nblk = s.N * int64_t(nch);
  const uint32_t ngroups = uint32_t(ceil_div(nblk, per));
  const int64_t ntiles = int64_t(p.nbk) * ngroups;
  if (nblk >= (int64_t(1) << 31) || ntiles >= (int64_t(1) << 31))
    return fail(NOPFS_ERANGE, "job too large for one launch");
  Scratch scr(st);
  uint64_t *szb, *zP;
  uint32_t* Pk;
  uint16_t* OT;
  FmState* state;
  uint32_t* ticket;
  if ((rc = scr.alloc_n(&szb, size_t(s.F)))) return rc;
  if ((rc = run_partition(p, R, scr, &Pk, &OT, st))) return rc;
  if ((rc = scr.alloc_n(&zP, size_t(s.N * s.M_max)))) return rc;
  if ((rc = scr.alloc_n(&state, size_t(nblk)))) return rc;
  if ((rc = scr.alloc_n(&ticket, 1))) return rc;
  if ((rc = launch("fm_holders", fm_holders, dim3(uint32_t(ceil_div(s.F, 256))), dim3(256), 0, st,
                   s.F, s.N, tier, sizes, rt, szb, reinterpret_cast<uint64_t*>(state),
                   nblk * int64_t(sizeof(FmState) / 8), ticket)))
    return rc;
  if ((rc = launch("fm_gather", fm_gather, dim3(xcd_padded(uint32_t(ntiles))), dim3(kGThreads), 0,
                   st, p, (const uint32_t*)Pk, (const uint16_t*)OT, tier, (const uint64_t*)szb, rt,
                   zP, ngroups, per, uint32_t(ntiles))))
    return rc;
  const uint32_t blocks = nblk < int64_t(kFmBlocks) ? uint32_t(nblk) : kFmBlocks;
  return launch("fm_final", fm_final, dim3(blocks), dim3(kFmThreads), 0, st, p,
                (const uint32_t*)Pk, (const uint64_t*)zP, rt, nch, uint32_t(nblk), state, ticket,
                src, t);
}

}  // namespace

int model_check(const nopfs_model* m) {
  if (!m) return fail(NOPFS_EINVAL, "model is NULL");
  if (m->J < 1) return fail(NOPFS_EINVAL, "model J must be >= 1");
  if (m->J > kMaxClasses) return fail(NOPFS_ERANGE, "model J must be <= 32");
  const double v[7] = {m->c, m->beta, m->b_c, m->pfs_t, m->pfs_gamma, m->w0, m->p0};
  for (double x : v)
    if (!(x > 0) || !isfinite(x)) return fail(NOPFS_EINVAL, "model rates and counts must be positive and finite");
  for (int32_t j = 0; j < m->J; ++j)
    if (!(m->r[j] > 0) || !(m->p[j] > 0) || !isfinite(m->r[j]) || !isfinite(m->p[j]))
      return fail(NOPFS_EINVAL, "model rates and counts must be positive and finite");
  return NOPFS_OK;
}

}  // namespace nopfs

extern "C" int nopfs_fetch_model(const nopfs_job* job, const int32_t* R, const int8_t* tier,
                                 const int64_t* sizes, const nopfs_model* model, int16_t* src,
                                 double* t, void* hip_stream) {
  try {
    return nopfs::model_impl(job, R, tier, sizes, model, src, t,
                             static_cast<hipStream_t>(hip_stream));
  } catch (const std::bad_alloc&) {
    return nopfs::fail(NOPFS_ENOMEM, "host allocation failed");
  } catch (...) {
    return nopfs::fail(NOPFS_EDEVICE, "unexpected host exception");
  }
}
