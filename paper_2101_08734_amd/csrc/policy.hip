// nopfs_policy_sim: the data-loading policies of the Performance Simulator
// section, evaluated on the Performance Modeling section's model, read by
// read for every worker.
//
// For read f of a worker with size s: u(f) = s / c is its compute time,
// read(f) = fetch(f) + write(f) the time to stage it, write(f) =
// s / min(beta, w0 / p0) (preprocessing and buffer writes pipelined), and
// fetch(f) = s over the throughput of its source (the PFS, t(gamma) / gamma;
// another worker's tier j, min(b_c, r_j / p_j); the own tier j, r_j / p_j).
//   Perfect        t(0) = 0, t(f) = t(f-1) + u(f-1): never stalls.
//   Naive          t(0) = read(0), t(f) = t(f-1) + u(f-1) + read(f): one
//                  PFS read at a time, after the previous compute.
//   StagingBuffer  p0 threads stage reads in stream order from the PFS into
//   NoPFS          a buffer of d0 bytes (NoPFS: from the source the fetch
//                  model chose). Q(f) is the thread-time spent staging reads
//                  0..f; read f starts only once the reads before fill(f),
//                  its staging-schedule window, are consumed:
//                    Q(f) = max(Q(f-1), p0 t(fill(f) - 1)) + read(f),
//                    t(0) = Q(0) / p0, t(f) = max(Q(f) / p0, t(f-1) + u(f-1)).
// finish = t(last) + u(last); io sums fetch times by source class.
//
// The results are those of the definition evaluated read by read with IEEE
// doubles, bit for bit, but the chains are not stepped read by read: they are
// scanned. While the running value x of a chain stays inside one binade
// [2^E, 2^(E+1)), its values are consecutive integers (their bit patterns),
// and adding a >= 0 with rounding adds an integer that depends on a and E
// alone, round(a / ulp), unless a / ulp is exactly halfway between two
// integers (then the parity of x decides). It is read off a single addition:
// bits(2^E + a) - bits(2^E). A maximum with w is a maximum of bit patterns,
// and rounding is monotone, so each read of a chain is a link
//   x -> max(x + add, floor)    on 64-bit integers
// (Q: add from read(f), floor = bits(p0 t(fill(f) - 1)) + add; with y(f) =
// t(f) + u(f): add from u(f), floor = bits(Q(f) / p0) + add, t(f) the larger
// of y(f-1) and Q(f) / p0), and links compose into links of the same form: a
// prefix scan gives every value. The scan is exact up to the first read that
// leaves the binade, falls halfway, has an operand that is not a plain
// non-negative number, or waits for a read whose t is not known yet. Up to
// there the values are kept, that read is stepped with ordinary additions
// and maxima, and the scan resumes behind it. A row of M reads has about
// log2(M) binades, and halfway cases are rare (a / ulp has tens of fractional
// bits), so few scans are cut short.
//
//   ps_sim -- one workgroup per worker (512 threads; 256 where workers
//             outnumber the compute units), chunks of four reads per thread:
//             per-read terms (ids, sources and windows loaded two chunks
//             ahead, sizes and far waits one), the Q scan and the y scan (one
//             barrier each) and one barrier that finds the first read, if
//             any, at which the scan stops. The t of this chunk and the one
//             before stay in LDS for the waits. The first reads of a row are
//             stepped, 64 at a time, by three waves (the Q chain, the t chain
//             one batch behind, the sums). Where scans would stop early
//             (windows of less than 512 reads), one
//             wave takes the chunk in scans of 64 reads without barriers, and
//             steps reads one by one where even those stop within 8. The
//             fetch-time sums by class are sums of the same kind (no maxima,
//             only the final value needed): integer totals per chunk, and a
//             chunk in which a class leaves its binade is added up in order
//             by one wave.
//
// Stepping read by read took 37 ns a read (NoPFS, a chain of dependent
// additions per worker); ImageNet-22k (2.2M reads per worker): Perfect 36,
// Naive 56, StagingBuffer 63, NoPFS 82 ms, now NoPFS 13.0. ImageNet-1k on 256
// workers: 7.4 / 11.3 / 12.8 / 16.7 ms, now 1.4 / 1.7 / 2.4 / 2.8. Bounds:
//   many workers, a size table larger than an L2 (ImageNet-22k, 114 MB): the
//     128-byte lines that the random 8-byte gathers fetch, 73 to 81 GB a call at
//     6.6 to 6.9 TB/s at the L2s' outer side, which counts what the last-level
//     cache serves too (NoPFS without the gathers: 8.1 ms);
//   many workers, a smaller table (ImageNet-1k, 10 MB, 256 workers): Perfect and
//     Naive those lines again (7.7 and 6.3 TB/s), the staging policies the chunk's
//     barriers and latency (4.6 TB/s, vector units 32% busy, occupancy 24%: one
//     workgroup per compute unit);
//   few workers (ImageNet-1k on 16): the latency of one workgroup's chunks, on 16
//     of 256 compute units (0.4 TB/s, vector units 2.5% busy).
// 1,024 threads of two reads each: 15.3 ms (the scans' cross-lane steps double).

#include <cmath>
#include <new>
#include <type_traits>

#include "common.hpp"

namespace nopfs {
namespace {

// Threads per worker: 512 where every worker has a compute unit of its own
// (up to 256 workers), 256 where workers outnumber them, so that two
// workgroups fit a compute unit's LDS.
constexpr int kPsFew = 512, kPsMany = 256;
constexpr int64_t kPsUnits = 256;                     // compute units
constexpr int kPsPer = 4;                             // reads per thread and chunk
// Scans shorter than kPsMinStep, twice in a chunk: one wave goes on. (With 256 the
// same times; with 1,024 windows of 700 reads 7,588 us instead of 4,243, 300
// workers 584 instead of 476.)
constexpr int kPsMinStep = 512;
// Wave scans shorter than kPsMinWave: read by read. (With 4 windows of 12 reads
// 37.2 ms instead of 43.3, but of 4 reads 72.4 instead of 69.9; with 16 windows of
// 12 62.3.)
constexpr int kPsMinWave = 8;
// The first reads of a row are stepped: its values double every few reads, so
// that scans stop at once (StagingBuffer, windows longer than the row: 656 reads
// of one worker 72 us with scans from the first read, 31 stepped; 684 reads on
// 4,096 workers 714 and 338). Up to 1,024 reads (768 of Naive, whose scans are cheaper,
// 256 of Perfect: 16 workers, rows of 100, 332 and 2,600 reads 12.4, 17.8 and 28.2 us
// with none, 10.8, 15.3 and 26.7 with 256, 9.5, 13.5 and 34.2 with 768).
// Fewer where one wave would go on with short windows anyway: with 256 threads
// and windows of less than 512 reads 512 (rows of 2,048 to 4,096 reads on 300 to
// 1,024 workers 5% faster than with 1,024), with windows of less than 128, whose
// batches wait for each other, 256 (rows of 512 to 1,024 reads 20% faster). Naive
// with more than two workgroups per compute unit, which hide each other's scans
// but not the steps, 384 (1,024 workers, 2,048 and 10,240 reads: 90 and 168 us with
// 768, 79 and 155 with 384; 4,096 workers, 1,024 reads 212 and 172).
constexpr int kPsHead = 1024, kPsHeadNaive = 768, kPsHeadPerfect = 256, kPsHeadShort = 512, kPsHeadPrev = 256;
constexpr int kPsHeadNaiveMany = 384;
// Short scans of a row's first chunk before one wave goes on (of others, and of
// Perfect: 2. Rows of 332 reads on 16 workers 21.6 us with 8 for Perfect too, 17.6
// with 2; StagingBuffer's rows of 2,600 reads 90 and 110).
constexpr int kPsShortsFirst = 8, kPsShorts = 2;
constexpr int kPsMaxJ = 32;
constexpr int kPsClasses = 1 + 2 * kPsMaxJ;           // PFS, remote j, own j
constexpr int kPsCopies = 16;                         // partial sums per class in LDS

enum : int32_t { kPerfect = 0, kNaive = 1, kStaging = 2, kNoPFS = 3 };

struct PsShape {
  int64_t F, N, B, M_max, E;
  int32_t drop_last;
};

// Throughputs computed once on the host, in the model's own expressions.
struct PsRates {
  double thr[kPsClasses];  // by class: 0 the PFS, 1 + j remote tier j, 1 + J + j own tier j
  double wthr;             // min(beta, w0 / p0)
  double c, p0;
  double rthr[kPsClasses], rwthr, rc, rp0;  // their reciprocals
  int32_t J;
  int32_t rcp;             // quotients may be formed from the reciprocals
};

__device__ __forceinline__ int64_t ps_row_len(const PsShape& r, int64_t i) {
  return r.E * epoch_len(r.F, r.N, r.B, r.drop_last, i);
}

__device__ __forceinline__ uint64_t bits_of(double v) { return __builtin_bit_cast(uint64_t, v); }
__device__ __forceinline__ double double_of(uint64_t b) { return __builtin_bit_cast(double, b); }

__device__ __forceinline__ double rl_d(double v, int lane) {
  return double_of(read_lane64(bits_of(v), lane));
}

__device__ __forceinline__ uint64_t max_u64(uint64_t a, uint64_t b) { return a > b ? a : b; }

// class of a source code (0 the PFS, 128 + j remote, 256 + j own); any
// other code, and every code outside NoPFS, reads from the PFS
__device__ __forceinline__ int ps_class(int32_t policy, int32_t code, int32_t J) {
  if (policy != kNoPFS) return 0;
  if (code >= 128 && code < 128 + J) return 1 + (code - 128);
  if (code >= 256 && code < 256 + J) return 1 + J + (code - 256);
  return 0;
}

// a / b from y = 1 / b, rounded as the division is: a first quotient, one
// correction (within an ulp of a / b), and the correction with the exact
// remainder, which gives the rounded quotient when y is within half an ulp
// of 1 / b (Markstein, "Computation of elementary functions on the IBM RISC
// System/6000 processor", 1990). Five operations instead of a division's
// twelve. Valid away from overflow and underflow of any of the terms, which
// rcp_ok and the range of binade_of keep it from.
__device__ __forceinline__ double div_rcp(double a, double b, double y) {
  const double q0 = a * y;
  const double q1 = __builtin_fma(__builtin_fma(-b, q0, a), y, q0);
  return __builtin_fma(__builtin_fma(-b, q1, a), y, q1);
}

// b's quotients may be formed from y = 1 / b: y is closer to 1 / b than half
// an ulp of any number of its binade can be, and b is far from the ends of
// the exponent range.
bool rcp_ok(double b, double y) {
  return b > 0x1p-300 && b < 0x1p300 && std::fabs(std::fma(-b, y, 1.0)) < 0x1p-53;
}

// The binade of a chain's value: bit patterns of its first value and of the
// next binade's, and half its ulp. base = top = 0 (nothing can be added) when
// the value is zero, below 2^-500 or above 2^500, negative or no number.
struct Binade {
  uint64_t base, top;
  double half_ulp;
};

__device__ __forceinline__ Binade binade_of(double x) {
  const uint32_t ex = uint32_t(bits_of(x) >> 52);  // sign and exponent
  const bool ok = ex >= 1023u - 500u && ex <= 1023u + 500u;
  Binade b;
  b.base = ok ? uint64_t(ex) << 52 : 0ull;
  b.top = ok ? uint64_t(ex + 1u) << 52 : 0ull;
  b.half_ulp = double_of(uint64_t(ok ? ex - 53u : 0u) << 52);
  return b;
}

// The integer that adding a adds inside the binade; *stop is set (and the
// result 0) when a is not below 2^E, not a plain non-negative number, or
// halfway between two multiples of the ulp. 2^E + a < 2^(E+1) rounds to a
// multiple of the ulp with ties to even; its difference to 2^E and the
// rounding error a - difference are exact.
__device__ __forceinline__ uint64_t units(double a, const Binade& b, bool* stop) {
#pragma clang fp contract(off)
  const double base = double_of(b.base);
  const double z = base + a;
  const double err = a - (z - base);
  const bool bad = bits_of(a) >= b.base || __builtin_fabs(err) == b.half_ulp;
  *stop = *stop || bad;
  return bad ? 0ull : bits_of(z) - b.base;
}

// x -> max(x + add, floor). {0, 0} leaves every x as it is; where only sums
// are scanned (kMax false) floor stays 0.
struct Link {
  uint64_t add, floor;
};

template <bool kMax>
__device__ __forceinline__ Link then(const Link& a, const Link& b) {
  return Link{a.add + b.add, kMax ? max_u64(a.floor + b.add, b.floor) : 0ull};
}
template <bool kMax>
__device__ __forceinline__ uint64_t apply(uint64_t x, const Link& l) {
  return kMax ? max_u64(x + l.add, l.floor) : x + l.add;
}

// One step of a lane scan: the link of the DPP source lane goes before this
// lane's (no source: {0, 0}; floor then becomes at least add, which is below
// x + add for every x the links are applied to).
template <bool kMax, int Ctrl, int RowMask>
__device__ __forceinline__ void link_step(Link& v) {
  const Link p{dpp_move64<Ctrl, RowMask>(v.add), kMax ? dpp_move64<Ctrl, RowMask>(v.floor) : 0ull};
  v = then<kMax>(p, v);
}
template <bool kMax>
__device__ __forceinline__ Link wave_link_scan(Link v) {  // inclusive, all lanes active
  link_step<kMax, 0x111, 0xf>(v);  // row_shr:1
  link_step<kMax, 0x112, 0xf>(v);  // row_shr:2
  link_step<kMax, 0x114, 0xf>(v);  // row_shr:4
  link_step<kMax, 0x118, 0xf>(v);  // row_shr:8
  link_step<kMax, 0x142, 0xa>(v);  // row_bcast:15, rows 1 and 3
  link_step<kMax, 0x143, 0xc>(v);  // row_bcast:31, rows 2 and 3
  return v;
}
template <bool kMax>
__device__ __forceinline__ Link wave_link_shift(const Link& v) {  // the lane below's, {0, 0} in lane 0
  return Link{dpp_move64<0x138, 0xf>(v.add), kMax ? dpp_move64<0x138, 0xf>(v.floor) : 0ull};
}

// The chain's value before this wave's reads and after the whole chunk's,
// from the waves' links in LDS (every wave computes both).
template <bool kMax, int kWaves>
__device__ __forceinline__ void block_links(const Link* tot, int wave, int lane, uint64_t x,
                                            uint64_t* before, uint64_t* after) {
  static_assert(kWaves == 4 || kWaves == 8, "lanes 0 to 7 of a row of 16");
  Link v = tot[lane & (kWaves - 1)];
  link_step<kMax, 0x111, 0xf>(v);
  link_step<kMax, 0x112, 0xf>(v);
  if (kWaves == 8) link_step<kMax, 0x114, 0xf>(v);
  auto lane_link = [&](int l) {
    return Link{read_lane64(v.add, l), kMax ? read_lane64(v.floor, l) : 0ull};
  };
  *before = wave > 0 ? apply<kMax>(x, lane_link(wave - 1)) : x;
  *after = apply<kMax>(x, lane_link(kWaves - 1));
}

template <int32_t kPolicy, int kPsThreads>
__global__ void __launch_bounds__(kPsThreads)
ps_sim(PsShape r, const int32_t* __restrict__ R, const int64_t* __restrict__ sizes,
       const int16_t* __restrict__ src, const int32_t* __restrict__ fill, PsRates rt,
       double* __restrict__ t, double* __restrict__ finish, double* __restrict__ io) {
#pragma clang fp contract(off)
  constexpr bool kStaged = kPolicy == kStaging || kPolicy == kNoPFS;
  constexpr bool kIo = kPolicy != kPerfect;
  constexpr int kPsWaves = kPsThreads / 64;
  constexpr int kPsChunk = kPsThreads * kPsPer;
  constexpr int kRing = kStaged ? 2 * kPsChunk : kPsChunk;
  constexpr int kCls = kPolicy == kNoPFS ? kPsClasses : 1;
  __shared__ double ring[kRing];                   // t of position f at [f % kRing]
  __shared__ double st_u[kPsChunk];                // a chunk's terms, where one wave needs them all
  __shared__ double st_rd[kIo ? kPsChunk : 1];
  __shared__ double st_w[kStaged ? kPsChunk : 1];
  __shared__ int32_t st_g[kStaged ? kPsChunk : 1];
  __shared__ double st_f[kIo ? kPsChunk : 1];      // a chunk's fetch times and classes
  __shared__ uint8_t st_c[kPolicy == kNoPFS ? kPsChunk : 1];
  __shared__ uint64_t io_x[kCls];                  // bits of each class's sum
  __shared__ uint64_t io_acc[kCls * kPsCopies];    // this chunk's units, in partial sums
  __shared__ uint32_t io_bad[kCls];                // a read of this chunk the units do not cover
  __shared__ uint32_t s_io_slow;
  __shared__ double thr[kPsClasses], rthr[kPsClasses];
  __shared__ Link s_q[kPsWaves], s_y[kPsWaves];
  __shared__ uint32_t s_stop[kPsWaves];
  __shared__ double s_Q, s_Y;
  __shared__ int32_t s_pos;
  __shared__ uint32_t s_near[2];  // of chunks (even, odd): reads wait for reads of the chunk
  const int64_t i = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t Mi = ps_row_len(r, i);
  const int64_t M = r.M_max;
  const int32_t* Rr = R + i * M;
  const int16_t* Sr = kPolicy == kNoPFS ? src + i * M : nullptr;
  const int32_t* Fr = kStaged ? fill + i * M : nullptr;
  double* tr = t + i * M;
  const int K = 1 + 2 * rt.J;
  for (int c = tid; c < kPsClasses; c += kPsThreads) {
    thr[c] = rt.thr[c];
    rthr[c] = rt.rthr[c];
  }
  if (kIo) {
    for (int c = tid; c < kCls; c += kPsThreads) {
      io_x[c] = 0;
      io_bad[c] = 0;
    }
    for (int c = tid; c < kCls * kPsCopies; c += kPsThreads) io_acc[c] = 0;
  }
  if (tid == 0) {
    s_io_slow = 0;
    s_near[0] = s_near[1] = 0;
  }
  __syncthreads();

  // a thread's four consecutive entries of a row in the chunk at f0 (`none`
  // past the row's reads)
  auto load4 = [&](const auto* row, int64_t f0, int32_t v[kPsPer], int32_t none) {
    const int64_t f = f0 + kPsPer * tid;
    if (f0 + kPsChunk <= Mi) {
      std::remove_cv_t<std::remove_reference_t<decltype(*row)>> w[kPsPer];
      __builtin_memcpy(w, row + f, sizeof(w));
#pragma unroll
      for (int j = 0; j < kPsPer; ++j) v[j] = w[j];
    } else {
#pragma unroll
      for (int j = 0; j < kPsPer; ++j) {
        const int32_t w = row[f + j < Mi ? f + j : 0];
        v[j] = f + j < Mi ? w : none;
      }
    }
  };
  auto gather = [&](const int32_t k[kPsPer], int64_t s[kPsPer]) {
#pragma unroll
    for (int j = 0; j < kPsPer; ++j) {
      const bool in = k[j] >= 0 && k[j] < r.F;
      const int64_t v = sizes[in ? k[j] : 0];
      s[j] = in ? v : 0;
    }
  };
  // position whose consumption read f waits for, from its window (-1: none)
  auto look = [&](int64_t f, int32_t fl) -> int64_t {
    int64_t g = int64_t(fl) - 1;
    if (g > f - 1) g = f - 1;
    return g < -1 ? -1 : g;
  };
  // t of the waits that have left the ring by the chunk at f0
  auto far_waits = [&](int64_t f0, const int32_t fl[kPsPer], double w[kPsPer]) {
#pragma unroll
    for (int j = 0; j < kPsPer; ++j) {
      const int64_t f = f0 + kPsPer * tid + j;
      const int64_t g = f < Mi ? look(f, fl[j]) : -1;
      w[j] = tr[g >= 0 && g < f0 - kRing ? g : 0];  // unconditional; used for such g only
    }
  };

  // marks the chunk at f0 when one of its reads waits for another (bit 0),
  // and when one of its first reads does (bit 1); of the row's first reads,
  // when one waits for a read of its own 64 (bit 2) or of the 64 before (bit 3)
  auto mark_near = [&](int64_t f0, const int32_t fl[kPsPer]) {
    uint32_t near = 0;
#pragma unroll
    for (int j = 0; j < kPsPer; ++j) {
      const int64_t f = f0 + kPsPer * tid + j;
      const int64_t g = f < Mi ? look(f, fl[j]) : -1, b = f & ~int64_t(63);
      if (g >= f0) near |= kPsPer * tid < kPsMinStep ? 3u : 1u;
      if (f0 == 0 && f < kPsHead && g >= 0) near |= g >= b ? 4u : (g >= b - 64 ? 8u : 0u);
    }
    if (near) atomicOr(&s_near[(f0 / kPsChunk) & 1], near);
  };
  // each class's sum after the chunk from the chunk's units, or a mark that
  // the chunk's reads have to be added up in order (one wave)
  auto io_check = [&]() -> bool {
    bool any = false;
    for (int c = lane; c < kCls; c += 64) {
      uint64_t sum = 0;
#pragma unroll
      for (int q = 0; q < kPsCopies; ++q) {
        sum += io_acc[c * kPsCopies + q];
        io_acc[c * kPsCopies + q] = 0;
      }
      const uint64_t x = io_x[c];
      const bool slow = io_bad[c] != 0u || (sum != 0u && x + sum >= binade_of(double_of(x)).top);
      if (slow) io_bad[c] = 1;
      else io_x[c] = x + sum;
      any = any || slow;
    }
    return __ballot(any) != 0u;
  };
  // the marked classes' fetch times of the chunk's reads from `from` on (st_f,
  // st_c), in stream order (one wave): 64 at a time where the sum stays inside
  // its binade
  auto io_ordered = [&](int from, int n) {
    for (int c = 0; c < kCls; ++c) {
      if (io_bad[c] == 0u) continue;
      double x = double_of(io_x[c]);
      for (int b = from; b < n; b += 64) {
        const int at = b + lane;
        const double v = st_f[at];
        const bool on = at < n && (kPolicy != kNoPFS || st_c[at] == c);
        const uint64_t m = __ballot(on);
        if (m == 0) continue;
        const Binade bx = binade_of(x);
        bool stop = false;
        const uint64_t d = units(v, bx, &stop);
        const uint64_t sum = read_lane64(wave_inclusive_scan64(on ? d : 0ull), 63);
        if (__ballot(on && stop) == 0 && bits_of(x) + sum < bx.top) {
          x = double_of(bits_of(x) + sum);
        } else {
          for (uint64_t mm = m; mm; mm &= mm - 1) x = x + rl_d(v, __builtin_ctzll(mm));
        }
      }
      if (lane == 0) {
        io_x[c] = bits_of(x);
        io_bad[c] = 0;
      }
    }
  };

  double Q = 0.0, Y = 0.0;  // Q and y = t + u after the last read
  // The row's first h reads, stepped 64 at a time from the staged terms: one
  // wave takes the Q chain, a second the t chain of the 64 before, the last
  // the sums by class. A batch that waits for the 64 before it (`prev`: there
  // is one) gets its Q chain after they are in; none waits inside itself.
  auto head = [&](int h, bool prev) {
    const int nb = (h + 63) / 64;
    // a batch's terms are requested from LDS before the barrier in front of it
    int32_t gn = -1;
    double wn = 0.0, rn = 0.0, un = 0.0, fn = 0.0;
    int cn = 0;
    auto request = [&](int b) {
      const int x = b < h ? b + lane : lane;
      if (kStaged && wave == 0) {
        gn = st_g[x];
        wn = st_w[x];
        rn = st_rd[x];
      }
      if (wave == 1) {
        un = st_u[x];
        if (kPolicy == kNaive) rn = st_rd[x];
      }
      if (kIo && wave == kPsWaves - 1) {
        fn = st_f[x];
        if (kPolicy == kNoPFS) cn = st_c[x];
      }
    };
    request(0);
    auto q_chain = [&](int b) {
      const double wl = gn >= 0 ? rt.p0 * ring[gn & (kRing - 1)] : wn;
      const double rl = rn;
      request(b + 64);
      double qb = 0.0;  // lane q: Q after read b + q
      auto step = [&](int q) {
        Q = __builtin_fmax(Q, rl_d(wl, q));
        Q = Q + rl_d(rl, q);
        qb = lane == q ? Q : qb;
      };
      if (h - b >= 64) {  // straight line: later operands are formed while earlier steps finish
#pragma unroll
        for (int q = 0; q < 64; ++q) step(q);
      } else {
        for (int q = 0; q < h - b; ++q) step(q);
      }
      st_w[b + lane] = qb;
    };
    auto t_chain = [&](int b) {
      const double ul = un, rl = rn;
      request(b + 64);
      const double al = kStaged ? st_w[b + lane] / rt.p0 : 0.0;
      double tb = 0.0;  // lane q: t of read b + q
      auto step = [&](int q) {
        double tf = Y;
        if (kPolicy == kNaive) tf = Y + rl_d(rl, q);
        if (kStaged) {
          tf = rl_d(al, q);
          if (b + q > 0) tf = __builtin_fmax(tf, Y);
        }
        tb = lane == q ? tf : tb;
        Y = tf + rl_d(ul, q);
      };
      if (h - b >= 64) {
#pragma unroll
        for (int q = 0; q < 64; ++q) step(q);
      } else {
        for (int q = 0; q < h - b; ++q) step(q);
      }
      if (b + lane < h) ring[b + lane] = tb;
    };
    double a0 = 0.0, a1 = 0.0;  // the sums of class `lane` and of class 64 + lane
    auto io_chain = [&](int b) {
      const double fl = fn;
      const int cl = cn;
      request(b + 64);
      // every step adds the read's fetch time in its class's lane and +0 in
      // the others (no sum is -0)
      auto step = [&](int q) {
        const int c = kPolicy == kNoPFS ? __builtin_amdgcn_readlane(cl, q) : 0;
        const double f = rl_d(fl, q);
        a0 = a0 + (c == lane ? f : 0.0);
        if (K > 64) a1 = a1 + (c == lane + 64 ? f : 0.0);
      };
      if (h - b >= 64) {
#pragma unroll
        for (int q = 0; q < 64; ++q) step(q);
      } else {
        for (int q = 0; q < h - b; ++q) step(q);
      }
    };
    if (kStaged) {
      for (int k = 0; k <= nb; ++k) {
        bool late = false;
        if (wave == 0 && k < nb) {
          late = prev && __ballot(64 * k + lane < h && gn >= 0 && gn >= 64 * k - 64) != 0u;
          if (!late) q_chain(64 * k);
        }
        if (wave == 1 && k > 0) t_chain(64 * k - 64);
        if (wave == kPsWaves - 1 && k < nb) io_chain(64 * k);
        __syncthreads();
        if (prev) {  // uniform
          if (late) q_chain(64 * k);
          __syncthreads();
        }
      }
    } else {
      for (int k = 0; k < nb; ++k) {
        if (wave == 1) t_chain(64 * k);
        if (kIo && wave == kPsWaves - 1) io_chain(64 * k);
      }
    }
    if (wave == 0 && lane == 0) s_Q = Q;
    if (wave == 1 && lane == 0) s_Y = Y;
    if (kIo && wave == kPsWaves - 1) {
      if (lane < kCls) io_x[lane] = bits_of(a0);
      if (lane + 64 < kCls) io_x[lane + 64] = bits_of(a1);
    }
    __syncthreads();
    Q = s_Q;
    Y = s_Y;
  };

  int32_t kA[kPsPer], cA[kPsPer] = {}, fA[kPsPer] = {}, cB[kPsPer] = {}, fB[kPsPer] = {};
  int64_t sB[kPsPer];
  double wB[kPsPer] = {};
  if (Mi > 0) {
    load4(Rr, 0, kA, -1);
    if (kPolicy == kNoPFS) load4(Sr, 0, cB, 0);
    if (kStaged) load4(Fr, 0, fB, 0);
    gather(kA, sB);
    load4(Rr, kPsChunk, kA, -1);
    if (kPolicy == kNoPFS) load4(Sr, kPsChunk, cA, 0);
    if (kStaged) load4(Fr, kPsChunk, fA, 0);
    if (kStaged) {
      mark_near(0, fB);
      __syncthreads();
    }
  }
  const int i0 = kPsPer * tid;
  for (int64_t f0 = 0; f0 < Mi; f0 += kPsChunk) {
    const int n = Mi - f0 < kPsChunk ? int(Mi - f0) : kPsChunk;
    // per-read terms, in the definition's expressions
    double u[kPsPer], fetch[kPsPer], rd[kPsPer], W[kPsPer];
    int cls[kPsPer];
    int32_t g[kPsPer];  // the position waited for, from the chunk's start (negative: before it)
#pragma unroll
    for (int j = 0; j < kPsPer; ++j) {
      const double s = double(sB[j]);
      cls[j] = ps_class(kPolicy, cB[j], rt.J);
      if (rt.rcp) {
        u[j] = div_rcp(s, rt.c, rt.rc);
        fetch[j] = kIo ? div_rcp(s, thr[cls[j]], rthr[cls[j]]) : 0.0;
        rd[j] = kIo ? fetch[j] + div_rcp(s, rt.wthr, rt.rwthr) : 0.0;
      } else {
        u[j] = s / rt.c;
        fetch[j] = kIo ? s / thr[cls[j]] : 0.0;
        rd[j] = kIo ? fetch[j] + s / rt.wthr : 0.0;
      }
      W[j] = 0.0;
      g[j] = -1;
      if (kStaged) {
        const int64_t gp = i0 + j < n ? look(f0 + i0 + j, fB[j]) : -1;
        g[j] = int32_t(gp - f0);
        const double near = ring[gp & (kRing - 1)];
        const double tg = gp >= f0 - kRing ? near : wB[j];
        W[j] = gp >= 0 && gp < f0 ? rt.p0 * tg : 0.0;
      }
    }
    // the next chunk's sizes and far waits, the one after's ids
    gather(kA, sB);
    if (kStaged) far_waits(f0 + kPsChunk, fA, wB);
#pragma unroll
    for (int j = 0; j < kPsPer; ++j) {
      cB[j] = cA[j];
      fB[j] = fA[j];
    }
    load4(Rr, f0 + 2 * kPsChunk, kA, -1);
    if (kPolicy == kNoPFS) load4(Sr, f0 + 2 * kPsChunk, cA, 0);
    if (kStaged) load4(Fr, f0 + 2 * kPsChunk, fA, 0);
    const uint32_t near = kStaged ? uint32_t(__builtin_amdgcn_readfirstlane(int(s_near[(f0 / kPsChunk) & 1]))) : 0u;
    if (kStaged) mark_near(f0 + kPsChunk, fB);

    // the chunk's terms to LDS, for a wave that takes reads of all threads
    auto stage = [&]() {
#pragma unroll
      for (int j = 0; j < kPsPer; ++j) {
        st_u[i0 + j] = u[j];
        if (kIo) st_rd[i0 + j] = rd[j];
        if (kStaged) {
          st_w[i0 + j] = W[j];
          st_g[i0 + j] = g[j];
        }
      }
    };
    auto stage_io = [&]() {
      if (!kIo) return;
#pragma unroll
      for (int j = 0; j < kPsPer; ++j) {
        st_f[i0 + j] = fetch[j];
        if (kPolicy == kNoPFS) st_c[i0 + j] = uint8_t(cls[j]);
      }
    };
    int pos = 0;
    constexpr int kHead = kPolicy == kPerfect ? kPsHeadPerfect : (kPolicy == kNaive ? kPsHeadNaive : kPsHead);
    // (said to be unlikely, the steps' uniform values spill, not the chunk loop's:
    // rows of 7.2M reads, 16 workers, Naive 20,059 -> 19,813 us)
    if (__builtin_expect(f0 == 0 && !(near & 4u), 0)) {
      stage();
      stage_io();
      __syncthreads();
      if (tid == 0) s_near[0] = 0;
      const int hmax = (near & 8u) ? kPsHeadPrev
                       : kPsThreads == kPsMany && (near & 2u) ? kPsHeadShort
                       : kPsThreads == kPsMany && kPolicy == kNaive && gridDim.x > 2 * kPsUnits
                           ? kPsHeadNaiveMany
                           : kHead;
      pos = n < hmax ? n : hmax;
      head(pos, (near & 8u) != 0u);
    }
    const int pos0 = pos;

    // fetch-time sums: this chunk's units by class
    if (kIo && pos0 < n) {
      uint64_t sum = 0;
      uint32_t bad = 0;
#pragma unroll
      for (int j = 0; j < kPsPer; ++j) {
        bool stop = false;
        uint64_t d = units(fetch[j], binade_of(double_of(io_x[cls[j]])), &stop);
        const bool on = i0 + j >= pos0 && i0 + j < n;
        if (!on) d = 0;
        bad |= stop && on ? 1u << j : 0u;
        if (kPolicy == kNoPFS)
          atomicAdd(reinterpret_cast<unsigned long long*>(&io_acc[cls[j] * kPsCopies + (lane & (kPsCopies - 1))]),
                    (unsigned long long)(d));
        else
          sum += d;
      }
      if (bad) {
#pragma unroll
        for (int j = 0; j < kPsPer; ++j)
          if ((bad >> j) & 1u) io_bad[cls[j]] = 1;
      }
      if (kPolicy != kNoPFS) {
        sum = wave_inclusive_scan64(sum);
        if (lane == 63) io_acc[wave] = sum;
      }
    }

    // the chunk's reads from pos on by one wave
    auto wave_chain = [&](int pos) {
      int p = pos;
      while (p < n) {
        auto load = [&](double* uu, double* rr, double* ww, int32_t* gg) {
          const int x = p + lane < n ? p + lane : n - 1;
          *uu = st_u[x];
          *rr = kIo ? st_rd[x] : 0.0;
          *ww = kStaged ? st_w[x] : 0.0;
          *gg = kStaged ? st_g[x] : -1;
          if (kStaged && *gg >= 0 && *gg < p) *ww = rt.p0 * ring[(f0 + *gg) & (kRing - 1)];
        };
        double ul, rl, wl;
        int32_t gl;
        load(&ul, &rl, &wl, &gl);
        const bool on = p + lane < n;
        const Binade wq = binade_of(Q), wy = binade_of(Y);
        bool stop = false, unknown = false;
        Link l{0, 0}, ex;
        uint64_t qx = 0, c = 0;
        if (kStaged) {
          unknown = gl >= p;
          stop = unknown || bits_of(wl) >= wq.top;
          const uint64_t d = units(rl, wq, &stop);
          if (on) l = Link{d, bits_of(wl) + d};
          l = wave_link_scan<true>(l);
          qx = apply<true>(bits_of(Q), l);
          stop = stop || qx >= wq.top;
          c = bits_of(rt.rcp ? div_rcp(double_of(qx), rt.p0, rt.rp0) : double_of(qx) / rt.p0);
          stop = stop || c >= wy.top;
        }
        uint64_t d = units(ul, wy, &stop);
        if (kPolicy == kNaive) {
          c = units(rl, wy, &stop);
          d += c;
        }
        l = on ? Link{d, kStaged ? c + d : 0ull} : Link{0, 0};
        l = wave_link_scan<kStaged>(l);
        ex = wave_link_shift<kStaged>(l);
        const uint64_t ye = apply<kStaged>(bits_of(Y), ex), yx = apply<kStaged>(bits_of(Y), l);
        const uint64_t tb = kPolicy == kNaive ? ye + c : max_u64(ye, c);
        stop = stop || yx >= wy.top;
        const uint64_t m = __ballot(on && stop);
        int step = m ? __builtin_ctzll(m) : (n - p < 64 ? n - p : 64);
        if (lane < step) ring[(f0 + p + lane) & (kRing - 1)] = double_of(tb);
        if (step > 0) {
          if (kStaged) Q = double_of(read_lane64(qx, step - 1));
          Y = double_of(read_lane64(yx, step - 1));
        }
        auto one = [&](double uk, double rk, double wk, int64_t f, bool rcp) -> double {
          double tf = Y;
          if (kPolicy == kNaive) tf = Y + rk;
          if (kStaged) {
            Q = __builtin_fmax(Q, wk);
            Q = Q + rk;
            tf = rcp ? div_rcp(Q, rt.p0, rt.rp0) : Q / rt.p0;
            if (f > 0) tf = __builtin_fmax(tf, Y);
          }
          Y = tf + uk;
          return tf;
        };
        if (m && ((__ballot(unknown) >> step) & 1u) == 0u) {
          const double tf = one(rl_d(ul, step), rl_d(rl, step), rl_d(wl, step), f0 + p + step, false);
          if (lane == 0) ring[(f0 + p + step) & (kRing - 1)] = tf;
          ++step;
        }
        p += step;
        if (step >= kPsMinWave || p >= n) continue;
        // read by read
        load(&ul, &rl, &wl, &gl);
        const int nb = n - p < 64 ? n - p : 64;
        double tl = 0.0;  // lane q: t of read p + q
        auto steps = [&](bool rcp) {
          for (int q = 0; q < nb; ++q) {
            const int gq = __builtin_amdgcn_readlane(gl, q) - p;
            const double wk = kStaged && gq >= 0 ? rt.p0 * rl_d(tl, gq & 63) : rl_d(wl, q);
            const double tf = one(rl_d(ul, q), rl_d(rl, q), wk, f0 + p + q, rcp);
            tl = lane == q ? tf : tl;
          }
        };
        // 64 reads of at most 2^363 seconds each (a 63-bit size over a rate
        // above 2^-300) keep Q and its quotients inside the range of div_rcp
        const bool plain = binade_of(Q).base != 0 && binade_of(Y).base != 0 && Q < 0x1p400 && Y < 0x1p400 &&
                           __ballot(lane < nb && !(ul >= 0.0 && rl >= 0.0 && wl >= 0.0 && wl < 0x1p700)) == 0;
        if (kStaged && rt.rcp && plain) steps(true);
        else steps(false);
        if (lane < nb) ring[(f0 + p + lane) & (kRing - 1)] = tl;
        p += nb;
      }
      if (lane == 0) {
        s_Q = Q;
        s_Y = Y;
      }
    };

    int shorts = 0;
    bool first = true, io_slow = false;
    if ((near & 2u) && pos < n) {
      // short windows: one wave from the start, another for the sums
      stage();
      stage_io();
      __syncthreads();
      if (tid == 0) s_near[(f0 / kPsChunk) & 1] = 0;
      if (wave == 0) wave_chain(pos);
      if (wave == kPsWaves - 1 && io_check()) io_ordered(pos0, n);
      __syncthreads();
      Q = s_Q;
      Y = s_Y;
      pos = n;
    }
    while (pos < n) {
      const Binade bq = binade_of(Q), by = binade_of(Y);
      uint32_t stops = 0;  // bit j: the scan does not hold at this thread's read j
      bool act[kPsPer];
      Link lq[kPsPer];     // of each read
      uint64_t qv[kPsPer]; // bits of Q after it
      uint64_t q_in = 0, q_end = 0;
#pragma unroll
      for (int j = 0; j < kPsPer; ++j) act[j] = i0 + j >= pos && i0 + j < n;
      if (kStaged) {
        Link l{0, 0};
#pragma unroll
        for (int j = 0; j < kPsPer; ++j) {
          bool stop = false;
          if (near) {  // uniform
            const double tg = ring[(f0 + g[j]) & (kRing - 1)];
            if (g[j] >= 0 && g[j] < pos) W[j] = rt.p0 * tg;
            stop = g[j] >= pos;
          }
          stop = stop || bits_of(W[j]) >= bq.top;
          const uint64_t d = units(rd[j], bq, &stop);
          lq[j] = act[j] ? Link{d, bits_of(W[j]) + d} : Link{0, 0};
          if (act[j] && stop) stops |= 1u << j;
          l = then<true>(l, lq[j]);
        }
        const Link inc = wave_link_scan<true>(l);
        const Link ex = wave_link_shift<true>(inc);
        if (lane == 63) s_q[wave] = inc;
        __syncthreads();
        uint64_t before;
        block_links<true, kPsWaves>(s_q, wave, lane, bits_of(Q), &before, &q_end);
        q_in = apply<true>(before, ex);
        uint64_t x = q_in;
#pragma unroll
        for (int j = 0; j < kPsPer; ++j) {
          x = apply<true>(x, lq[j]);
          if (act[j] && x >= bq.top) stops |= 1u << j;
          qv[j] = x;
        }
      } else if (kIo && first) {
        __syncthreads();  // the units by class are in
      }
      if (kIo && first && wave == kPsWaves - 1) {
        if (kStaged && lane == 0) s_near[(f0 / kPsChunk) & 1] = 0;  // read by every wave before the barrier
        const bool slow = io_check();
        if (slow && lane == 0) s_io_slow = 1;
      }
      // y: the same over u, with Q / p0 as the floor
      Link ly[kPsPer];
      uint64_t cb[kPsPer];   // bits of Q / p0 (Naive: the units of read(f))
      uint64_t y_in = 0, y_end = 0;
      {
        Link l{0, 0};
#pragma unroll
        for (int j = 0; j < kPsPer; ++j) {
          bool stop = false;
          cb[j] = 0;
          uint64_t d = units(u[j], by, &stop);
          if (kStaged) {
            cb[j] = bits_of(rt.rcp ? div_rcp(double_of(qv[j]), rt.p0, rt.rp0) : double_of(qv[j]) / rt.p0);
            stop = stop || cb[j] >= by.top;
          }
          if (kPolicy == kNaive) {
            cb[j] = units(rd[j], by, &stop);
            d += cb[j];
          }
          ly[j] = act[j] ? Link{d, kStaged ? cb[j] + d : 0ull} : Link{0, 0};
          if (act[j] && stop) stops |= 1u << j;
          l = then<kStaged>(l, ly[j]);
        }
        const Link inc = wave_link_scan<kStaged>(l);
        const Link ex = wave_link_shift<kStaged>(inc);
        if (lane == 63) s_y[wave] = inc;
        __syncthreads();
        uint64_t before;
        block_links<kStaged, kPsWaves>(s_y, wave, lane, bits_of(Y), &before, &y_end);
        y_in = apply<kStaged>(before, ex);
      }
      {
        uint64_t x = y_in;
#pragma unroll
        for (int j = 0; j < kPsPer; ++j) {
          const uint64_t tb = kPolicy == kNaive ? x + cb[j] : max_u64(x, cb[j]);
          x = apply<kStaged>(x, ly[j]);
          if (act[j]) {
            if (x >= by.top) stops |= 1u << j;
            // values past the first stop are rewritten before anything reads them
            ring[(f0 + i0 + j) & (kRing - 1)] = double_of(tb);
          }
        }
      }
      // the first read at which the scan does not hold
      const uint32_t mine = stops ? uint32_t(i0 + __builtin_ctz(stops)) : ~0u;
      const uint64_t has = __ballot(stops != 0u);
      if (lane == 0) s_stop[wave] = ~0u;
      if (has && lane == __builtin_ctzll(has)) s_stop[wave] = mine;
      __syncthreads();
      if (first) io_slow = s_io_slow != 0u;
      first = false;
      const uint32_t sv = s_stop[lane & (kPsWaves - 1)];
      const uint64_t sm = __ballot(sv != ~0u) & ((1u << kPsWaves) - 1u);
      if (sm == 0) {
        if (kStaged) Q = double_of(q_end);
        Y = double_of(y_end);
        break;
      }
      const int k = __builtin_amdgcn_readlane(int(sv), __builtin_ctzll(sm));
      if (k / kPsPer == tid) {
        // this thread's read k: the values before it hold; step it with
        // ordinary operations unless its wait is still unknown
        uint64_t qx = q_in, yx = y_in;
        double uk = 0, rk = 0, wk = 0;
        int32_t gk = -1;
#pragma unroll
        for (int j = 0; j < kPsPer; ++j) {
          if (j < (k % kPsPer)) {
            if (kStaged) qx = apply<true>(qx, lq[j]);
            yx = apply<kStaged>(yx, ly[j]);
          }
          if (j == (k % kPsPer)) {
            uk = u[j];
            rk = rd[j];
            wk = W[j];
            gk = g[j];
          }
        }
        double q = double_of(qx), y = double_of(yx);
        const bool known = gk < pos;
        if (known) {
          double tf = y;
          if (kPolicy == kNaive) tf = y + rk;
          if (kStaged) {
            q = __builtin_fmax(q, wk);
            q = q + rk;
            tf = q / rt.p0;
            if (f0 + k > 0) tf = __builtin_fmax(tf, y);
          }
          ring[(f0 + k) & (kRing - 1)] = tf;
          y = tf + uk;
        }
        s_Q = q;
        s_Y = y;
        s_pos = known ? k + 1 : k;
      }
      __syncthreads();
      Q = s_Q;
      Y = s_Y;
      const int np = s_pos;
      if (np - pos < kPsMinStep) ++shorts;
      pos = np;
      if (shorts < (f0 == 0 && kPolicy != kPerfect ? kPsShortsFirst : kPsShorts) || pos >= n) continue;

      // one wave goes on from here
      stage();
      __syncthreads();
      if (wave == 0) wave_chain(pos);
      __syncthreads();
      Q = s_Q;
      Y = s_Y;
      break;
    }

    if (kIo && io_slow) {
      stage_io();
      __syncthreads();
      if (wave == 0) io_ordered(pos0, n);
      if (tid == 0) s_io_slow = 0;
      __syncthreads();
    }

    // the chunk's t, from the ring
    double tv[kPsPer];
#pragma unroll
    for (int j = 0; j < kPsPer; ++j) tv[j] = ring[(f0 + i0 + j) & (kRing - 1)];
    if (i0 + kPsPer <= n) {
      __builtin_memcpy(tr + f0 + i0, tv, sizeof(tv));
    } else {
#pragma unroll
      for (int j = 0; j < kPsPer; ++j)
        if (i0 + j < n) tr[f0 + i0 + j] = tv[j];
    }
  }
  for (int64_t f = Mi + tid; f < M; f += kPsThreads) tr[f] = -1.0;
  for (int c = tid; c < K; c += kPsThreads)
    io[i * K + c] = kIo && c < kCls ? double_of(io_x[c]) : 0.0;
  if (tid == 0) finish[i] = Mi > 0 ? Y : 0.0;
}

int policy_impl(const nopfs_job* job, const int32_t* R, const int64_t* sizes, const int16_t* src,
                const int32_t* fill, const nopfs_model* model, int32_t policy, double* t,
                double* finish, double* io, hipStream_t st) {
  Shape s;
  int rc = make_shape(job, &s);
  if (rc) return rc;
  if ((rc = model_check(model))) return rc;
  if (policy < kPerfect || policy > kNoPFS) return fail(NOPFS_EINVAL, "policy must be 0..3");
  if (!sizes || !finish || !io) return fail(NOPFS_EINVAL, "sizes, finish and io must be non-NULL");
  if (s.M_max > 0) {
    if (!R || !t) return fail(NOPFS_EINVAL, "R and t must be non-NULL");
    if (policy >= kStaging && !fill) return fail(NOPFS_EINVAL, "fill must be non-NULL for the staging policies");
    if (policy == kNoPFS && !src) return fail(NOPFS_EINVAL, "src must be non-NULL for NoPFS");
  }
  if (s.N >= (int64_t(1) << 31)) return fail(NOPFS_ERANGE, "N too large for one launch");
  PsShape r{s.F, s.N, s.B, s.M_max, s.E, s.drop_last};
  PsRates rt{};
  rt.J = model->J;
  rt.thr[0] = model->pfs_t / model->pfs_gamma;
  for (int32_t j = 0; j < model->J; ++j) {
    const double own = model->r[j] / model->p[j];
    rt.thr[1 + j] = model->b_c < own ? model->b_c : own;
    rt.thr[1 + model->J + j] = own;
  }
  for (int c = 1 + 2 * model->J; c < kPsClasses; ++c) rt.thr[c] = rt.thr[0];
  const double wb = model->w0 / model->p0;
  rt.wthr = model->beta < wb ? model->beta : wb;
  rt.c = model->c;
  rt.p0 = model->p0;
  bool ok = true;
  auto reciprocal = [&](double b) {
    const double y = 1.0 / b;
    ok = ok && rcp_ok(b, y);
    return y;
  };
  for (int c = 0; c < kPsClasses; ++c) rt.rthr[c] = reciprocal(rt.thr[c]);
  rt.rwthr = reciprocal(rt.wthr);
  rt.rc = reciprocal(rt.c);
  rt.rp0 = reciprocal(rt.p0);
  rt.rcp = ok;
  auto run = [&](auto threads) {
    constexpr int kT = decltype(threads)::value;
    const dim3 grid(uint32_t(s.N)), block(kT);
    switch (policy) {
      case kPerfect:
        return launch("ps_sim_perfect", ps_sim<kPerfect, kT>, grid, block, 0, st, r, R, sizes, src,
                      fill, rt, t, finish, io);
      case kNaive:
        return launch("ps_sim_naive", ps_sim<kNaive, kT>, grid, block, 0, st, r, R, sizes, src,
                      fill, rt, t, finish, io);
      case kStaging:
        return launch("ps_sim_staging", ps_sim<kStaging, kT>, grid, block, 0, st, r, R, sizes, src,
                      fill, rt, t, finish, io);
      default:
        return launch("ps_sim_nopfs", ps_sim<kNoPFS, kT>, grid, block, 0, st, r, R, sizes, src,
                      fill, rt, t, finish, io);
    }
  };
  return s.N <= kPsUnits ? run(std::integral_constant<int, kPsFew>()) : run(std::integral_constant<int, kPsMany>());
}

}  // namespace
}  // namespace nopfs

extern "C" int nopfs_policy_sim(const nopfs_job* job, const int32_t* R, const int64_t* sizes,
                                const int16_t* src, const int32_t* fill, const nopfs_model* model,
                                int32_t policy, double* t, double* finish, double* io,
                                void* hip_stream) {
  try {
    return nopfs::policy_impl(job, R, sizes, src, fill, model, policy, t, finish, io,
                              static_cast<hipStream_t>(hip_stream));
  } catch (const std::bad_alloc&) {
    return nopfs::fail(NOPFS_ENOMEM, "host allocation failed");
  } catch (...) {
    return nopfs::fail(NOPFS_EDEVICE, "unexpected host exception");
  }
}
