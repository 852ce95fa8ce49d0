// Single-pulse search over dedispersed series: per-trial statistics and the
// boxcar matched filter with run extraction.
//
// The paper names a single-pulse search stage (Section 2.1) without giving its
// statistic.  The one computed here (documented in gsp.h): population mean and
// sigma of each trial's series from exact integer moments; for every box end
// e and width w, snr = (box sum - w mu) / (sigma sqrt(w)); best over widths;
// one candidate per maximal run of best >= threshold.
//
// The kernels work on a table of series jobs.  A job is the n_dm trials of
// one plan row: either a whole dedispersed row (batch search) or one
// streaming window whose boxes may reach back into retained samples of the
// previous window (a look-back region in front of the window).  Both kernels
// stride over their work items, so the same code serves the per-call batch
// launches (one item per workgroup or wave) and the fixed-grid launches of the
// streaming graph.
//
// Both are streaming passes over the int32 DM-time data, k_stats bound by HBM
// (5.9 TB/s), k_search by its vector instructions:
//  k_stats  one workgroup per trial, 8 loads in flight per lane, 128-bit
//           integer moment sums, mu and sigma finished in double;
//  k_search one wave per (trial, segment of box ends): segment plus look-back
//           read once, exact int64 prefix sums by wave scans into a per-wave
//           LDS ring, an integer prefilter per width, exact double SNRs only
//           where a box can pass, and run fragments appended with one atomic
//           each (joined on the host).
#include <algorithm>
#include <cstring>
#include <vector>

#include "gsp_internal.h"

namespace gsp {

__device__ __forceinline__ int find_job_by_trial(const SeriesTable *t, int g) {
  int lo = 0, hi = t->n_jobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (t->job[mid].trial0 <= g)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ int find_job_by_item(const SeriesTable *t, int64_t b) {
  int lo = 0, hi = t->n_jobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (t->job[mid].block0 <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// ---------------------------------------------------------------------------
// statistics
// ---------------------------------------------------------------------------
static constexpr int kStatsThreads = 256;

__global__ __launch_bounds__(kStatsThreads) void k_stats(const SeriesTable *__restrict__ tb,
                                                          double *__restrict__ musig,
                                                          const uint32_t *__restrict__ need) {
  __shared__ int64_t r1[kStatsThreads];
  __shared__ unsigned __int128 r2[kStatsThreads];
  const int n_trials = tb->n_trials;
  for (int g = blockIdx.x; g < n_trials; g += gridDim.x) {
    if (need && need[g] == 0) continue;  // a trial nobody reads: left as it was
    const SeriesJob &J = tb->job[find_job_by_trial(tb, g)];
    const int64_t n = J.n;
    const int32_t *x = as_global(J.x) + (int64_t)(g - J.trial0) * J.pitch + J.e_begin;
    const int64_t x0 = n > 0 ? x[0] : 0;
    int64_t s1 = 0;
    unsigned __int128 s2 = 0;
    auto add = [&](int32_t xv) {
      const int64_t v = (int64_t)xv - x0;
      s1 += v;
      const uint64_t a = (uint64_t)(v < 0 ? -v : v);
      s2 += (unsigned __int128)(a * a);
    };
    constexpr int kU = 8;  // loads in flight per thread
    int64_t k = threadIdx.x;
    for (; k + (kU - 1) * kStatsThreads < n; k += kU * kStatsThreads) {
      int32_t v[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) v[u] = x[k + u * kStatsThreads];
#pragma unroll
      for (int u = 0; u < kU; ++u) add(v[u]);
    }
    for (; k < n; k += kStatsThreads) add(x[k]);
    r1[threadIdx.x] = s1;
    r2[threadIdx.x] = s2;
    __syncthreads();
    for (int h = kStatsThreads / 2; h > 0; h >>= 1) {
      if (threadIdx.x < h) {
        r1[threadIdx.x] += r1[threadIdx.x + h];
        r2[threadIdx.x] += r2[threadIdx.x + h];
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      if (n > 0) {
        const double dn = (double)n;
        const double m1 = (double)r1[0] / dn;
        const double m2 = (double)r2[0] / dn;
        const double var = m2 - m1 * m1;
        musig[2 * g] = (double)x0 + m1;
        musig[2 * g + 1] = var > 0.0 ? sqrt(var) : 0.0;
      } else {
        musig[2 * g] = 0.0;
        musig[2 * g + 1] = 0.0;
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// boxcar search
// ---------------------------------------------------------------------------
// One wave owns one item: a trial and a segment [s0, s1) of its box ends.  It
// walks the samples from lo = max(first valid sample, s0 - (w_max - 1)) in
// blocks of 512: each lane holds two runs of 4 samples, added up in the lane
// and by two wave-wide scans (DPP) plus the running carry to the exact prefix
// sums C of the samples less the trial's integer mean c, and these go, four to
// an LDS access, into a per-wave ring that keeps the last RING of them.  A box
// (e, w) sums to C(e) - C(e - w) + w c.  Per width an integer prefilter finds
// whether any box of the block reaches the bound of its width (in 32 bits, on
// the ring's low halves, wherever no sample within a box's reach lies
// 2^31 / w_max or more from c, so that every box's C difference fits): 8
// differences and a maximum per lane.  Only blocks where one does, or that
// hold a large sample, are looked at box end by box end (64 a step, the widths
// that passed), and only
// ends that pass there get the exact double SNR.  Runs of flagged ends are
// followed across steps and blocks inside the wave and written as fragments
// (one atomic each).  Waves never wait for each other: there is no workgroup
// barrier after the widths are loaded.
//
// What bounds it: vector instructions, some 260 per block of a wave (10 widths;
// 80% busy).  4.57 GB of a survey beam, widths 1 to 512: 1.36 ms (3.79 when each
// step of 64 samples had its own scan and each box end its own LDS read and
// compare; 1.84 with flat loads, which LDS waits include; 3 workgroups per CU
// instead of 4, from 1 KB more LDS, 2.2).
static constexpr int kSearchThreads = 256;
static constexpr int kSearchBlock = 512;  // samples per block: 8 steps of 64

__global__ void k_zero_counter(unsigned long long *c) { *c = 0ull; }

struct SearchArgs {
  const SeriesTable *tb;
  const double *musig;
  const int32_t *widths;  // sorted, unique
  int32_t nw, wmax;
  int32_t tile;           // box ends per item
  float thr;
  Frag *frags;
  int64_t cap;
  unsigned long long *counter;
};

// One step of the wave scan: v plus v of the lane CTRL selects (DPP), 0 where
// the row mask or the row boundary gives no source.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int64_t add_dpp(int64_t v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROW_MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)v >> 32), CTRL, ROW_MASK, 0xf, false);
  return v + (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Inclusive scan of an int64 over the 64 lanes: shifts inside rows of 16,
// then the row totals broadcast to the following rows.
__device__ __forceinline__ int64_t wave_scan_i64(int64_t x) {
  x = add_dpp<0x111, 0xf>(x);  // row_shr:1
  x = add_dpp<0x112, 0xf>(x);  // row_shr:2
  x = add_dpp<0x114, 0xf>(x);  // row_shr:4
  x = add_dpp<0x118, 0xf>(x);  // row_shr:8
  x = add_dpp<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
  x = add_dpp<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
  return x;
}

// The same of an int32, for partial sums known to fit.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int32_t add_dpp_i32(int32_t v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ int32_t wave_scan_i32(int32_t x) {
  x = add_dpp_i32<0x111, 0xf>(x);
  x = add_dpp_i32<0x112, 0xf>(x);
  x = add_dpp_i32<0x114, 0xf>(x);
  x = add_dpp_i32<0x118, 0xf>(x);
  x = add_dpp_i32<0x142, 0xa>(x);
  x = add_dpp_i32<0x143, 0xc>(x);
  return x;
}

__device__ __forceinline__ int64_t readlane_i64(int64_t v, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int64_t lane63(int64_t v) { return readlane_i64(v, 63); }

// Four consecutive samples of a series (4-byte aligned).  A series is read as
// global memory: through a pointer read from the job table the compiler would
// take flat loads, which every wait for LDS also waits for.
typedef int32_t Quad __attribute__((ext_vector_type(4), aligned(4)));
typedef const __attribute__((address_space(1))) int32_t *SeriesPtr;
__device__ __forceinline__ Quad load_quad(SeriesPtr p) {
  return *(const __attribute__((address_space(1))) Quad *)p;
}

// max of m and the four differences p[i] - q (mod 2^32, as signed)
__device__ __forceinline__ int32_t max4(int32_t m, const uint32_t *p, int32_t a, int32_t b, int32_t c, int32_t d) {
  m = max(max(m, (int32_t)(p[0] - (uint32_t)a)), (int32_t)(p[1] - (uint32_t)b));
  return max(max(m, (int32_t)(p[2] - (uint32_t)c)), (int32_t)(p[3] - (uint32_t)d));
}

// Per-wave LDS: the prefix ring, the step's exact best SNR and width per
// lane, and the open run.
template <int RING>
struct SearchWaveLds {
  // the centred prefix sums, low and high halves: C after sample e at (e - lo) mod RING
  alignas(16) int32_t ring_lo[RING], ring_hi[RING];
  // of each 4 the smallest (low half; they differ by less than 2^24); the first 64 again behind the last
  int32_t qmin[RING / 4 + 64];
  __device__ int64_t get(int j) const {
    return (int64_t)(((uint64_t)(uint32_t)ring_hi[j] << 32) | (uint32_t)ring_lo[j]);
  }
  __device__ void put(int j, int64_t v) {
    ring_lo[j] = (int32_t)(uint32_t)v;
    ring_hi[j] = (int32_t)(uint32_t)((uint64_t)v >> 32);
  }
  double sb[64];
  uint8_t sk[64];
  int64_t o_first, o_peak;
  double o_snr;
  int32_t o_k, o_left;
};

// Four waves per SIMD (at most 128 VGPRs): occupancy hides the LDS and
// memory latency better than the registers a lower occupancy would free.
template <int RING>
__global__ __launch_bounds__(kSearchThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_search(SearchArgs a) {
  static_assert((RING & (RING - 1)) == 0, "ring length is a power of two");
  extern __shared__ __align__(16) int64_t lds64[];
  __shared__ __align__(16) int32_t wsh[64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwaves = blockDim.x >> 6;
  SearchWaveLds<RING> &W = reinterpret_cast<SearchWaveLds<RING> *>(lds64)[wave];
  const SeriesTable *tb = a.tb;
  const int64_t n_items = tb->n_items;
  const double thr = (double)a.thr;
  const int nw = a.nw;
  if ((int)threadIdx.x < nw) wsh[threadIdx.x] = a.widths[threadIdx.x];
  __syncthreads();  // the only workgroup barrier
  // widths that are no multiple of 4 (a mask), and lane i: the i-th of the others
  const uint64_t unaligned = __ballot(lane < nw && (wsh[min(lane, nw - 1)] & 3) != 0);
  const uint64_t every = nw < 64 ? (1ull << nw) - 1 : ~0ull;
  const uint64_t aligned = every & ~unaligned;
  const int n_al = __popcll(aligned), n4 = (n_al + 3) & ~3;
  int lane_qk = 0;
  for (uint64_t m = aligned, i = 0; m; m &= m - 1, ++i)
    if (lane == (int)i) lane_qk = __builtin_ctzll(m);
  const int lane_q4 = lane < n_al ? wsh[lane_qk] >> 2 : 1;

  for (int64_t b = (int64_t)blockIdx.x * nwaves + wave; b < n_items; b += (int64_t)gridDim.x * nwaves) {
    const SeriesJob &J = tb->job[find_job_by_item(tb, b)];
    const int64_t n = J.n;
    const int64_t local = b - J.block0;
    const int trial = (int)(local / J.tiles);
    const int64_t seg = local - (int64_t)trial * J.tiles;
    const int g = J.trial0 + trial;
    const double mu = a.musig[2 * g], sigma = a.musig[2 * g + 1];
    // an integer near the mean (any value is exact; near the mean keeps the
    // centred samples small)
    const int64_t cmean = (int64_t)fmin(fmax(rint(mu), -2147483648.0), 2147483647.0);
    if (!(sigma > 0.0)) continue;  // uniform over the wave
    SeriesPtr x = (SeriesPtr)(J.x + (int64_t)trial * J.pitch + J.e_begin);  // relative positions
    const int64_t look = J.look;
    const int64_t s0 = seg * a.tile;
    const int64_t s1 = min(s0 + (int64_t)a.tile, n);
    // whole blocks before s0 where there are samples, so that a segment's
    // blocks are whole but for the series' last
    const int64_t reach_blocks = (a.wmax - 1 + kSearchBlock - 1) / kSearchBlock;
    int64_t lo = s0 - reach_blocks * kSearchBlock;
    if (lo < -look) lo = max(-look, s0 - (int64_t)(a.wmax - 1));

    // prefilter bounds: a box can reach the threshold only if its sum is
    // >= w mu + thr sigma sqrt(w); lim sits 2 below that bound (far more than
    // its double rounding), so every box end the exact test flags passes
    // (lane k holds width k and its bound; the loops below read them with
    // readlane, so they cost no LDS round trip)
    // The bound is kept against the centred sums: C difference >= lim - w c,
    // in 64 bits and, clamped, in 32 (a clamp only lets more ends through).
    int lane_w = 0;
    int64_t lane_lim = INT64_MAX;
    int32_t lane_l32 = INT32_MAX;
    double lane_wmu = 0.0, lane_den = 1.0;  // w mu and sigma sqrt(w), as the exact SNR takes them
    if (lane < nw) {
      lane_w = wsh[lane];
      const double wd = (double)lane_w;
      lane_wmu = wd * mu;
      lane_den = sigma * sqrt(wd);
      const double bound = wd * mu + thr * sigma * sqrt(wd);
      lane_lim = bound < -4.0e18 ? INT64_MIN : (bound > 4.0e18 ? INT64_MAX : (int64_t)floor(bound) - 2);
      if (lane_lim != INT64_MIN && lane_lim != INT64_MAX) lane_lim -= cmean * (int64_t)lane_w;
      lane_l32 = (int32_t)max((int64_t)INT32_MIN, min((int64_t)INT32_MAX, lane_lim));
    }
    int32_t lane_ql = __shfl(lane_l32, lane_qk, 64);
    if (lane >= n_al) lane_ql = INT32_MAX;
    // samples this far from c or farther make the 32-bit prefilter unsafe for
    // the boxes that reach them (w_max of them sum to less than 2^31 in size)
    // (8 more for the bounds over groups of 4 ends and 4 starts)
    const int64_t big = (int64_t)(0x7FFFFFFF / (uint32_t)(a.wmax + 8));
    // samples nearer to c than this have block sums in 32 bits (and are not
    // big); 0: c so large that the differences themselves might wrap
    const int32_t near =
        cmean > -(int64_t(1) << 30) && cmean < (int64_t(1) << 30) ? (int32_t)min((int64_t)(1 << 21), big) : 0;
    int64_t last_big = -(reach_blocks + 1);   // the last block holding such a sample
    int64_t last_slow = -(reach_blocks + 1);  // the last block without group minima
    if (lane == 0) {  // C(lo - 1)
      W.put(RING - 1, 0);
      W.qmin[RING / 4 - 1] = 0;
    }
    __builtin_amdgcn_wave_barrier();

    bool open = false;
    int64_t o_first = 0, o_peak = 0, o_last = 0;
    double o_snr = 0.0;
    int o_k = 0, o_left = 0;
    auto emit = [&](int64_t t_first, int64_t t_last, int64_t e_peak, double snr, int k, int left, int right) {
      const unsigned long long idx = atomicAdd(a.counter, 1ull);
      if ((int64_t)idx < a.cap) {
        Frag f;
        f.trial = g;
        f.width = wsh[k - 1];
        f.t_first = J.abs0 + t_first;
        f.t_last = J.abs0 + t_last;
        f.e_peak = J.abs0 + e_peak;
        f.snr = snr;
        f.open_left = left;
        f.open_right = right;
        a.frags[idx] = f;
      }
    };

    const int64_t count = s1 - lo;
    const int64_t nblk = (count + kSearchBlock - 1) / kSearchBlock;
    const int64_t nfull = count / kSearchBlock;  // blocks with all their samples before s1
    // the quads of the next block in flight: samples eb + 4 lane .. + 3 and 256 further
    Quad q0 = {}, q1 = {};
    if (nfull > 0) {
      q0 = load_quad(x + lo + 4 * lane);
      q1 = load_quad(x + lo + 256 + 4 * lane);
    }
    int64_t carry = 0;
    for (int64_t blk = 0; blk < nblk; ++blk) {
      const int64_t eb = lo + blk * kSearchBlock;  // position of lane 0, step 0
      const int r0 = (int)(eb - lo);
      // ---- exact centred prefix sums into the ring ----
      uint32_t p32[8];  // low halves of C after samples eb + 256 j + 4 lane + i, at 4 j + i
      int32_t qmax[2] = {0, 0}, ymax = 0;  // of each 4 sums and of the lane's samples the largest
      bool quads = false;
      if (blk < nfull) {
        const Quad c0 = q0, c1 = q1;
        if (blk + 1 < nfull) {
          q0 = load_quad(x + eb + kSearchBlock + 4 * lane);
          q1 = load_quad(x + eb + kSearchBlock + 256 + 4 * lane);
        }
        int32_t y[8];
        uint32_t far = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          y[i] = (int32_t)((uint32_t)(i < 4 ? c0[i & 3] : c1[i & 3]) - (uint32_t)cmean);
          far = max(far, (uint32_t)y[i] + (uint32_t)(near - 1));
        }
        ymax = max(max(max(y[0], y[1]), max(y[2], y[3])), max(max(y[4], y[5]), max(y[6], y[7])));
        quads = near > 0 && __ballot(far > 2u * (uint32_t)near - 2u) == 0ull;
        if (quads) {  // |x - c| < near: sums of the block fit 32 bits
#pragma unroll
          for (int i = 1; i < 8; ++i)
            if (i != 4) y[i] += y[i - 1];
          const int32_t in0 = wave_scan_i32(y[3]), in1 = wave_scan_i32(y[7]);
          const int32_t t0 = __builtin_amdgcn_readlane(in0, 63), t1 = __builtin_amdgcn_readlane(in1, 63);
          const int32_t ex[2] = {in0 - y[3], in1 - y[7] + t0};
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int32_t *s = y + 4 * j;
            const uint32_t base = (uint32_t)carry + (uint32_t)ex[j];
            qmax[j] = (int32_t)(base + (uint32_t)max(max(s[0], s[1]), max(s[2], s[3])));
            const int32_t low = (int32_t)(base + (uint32_t)min(min(s[0], s[1]), min(s[2], s[3])));
            W.qmin[((r0 >> 2) & (RING / 4 - 1)) + 64 * j + lane] = low;
            if (j == 0 && (r0 & (RING - 1)) == 0) W.qmin[RING / 4 + lane] = low;
          }
          int4 h[2];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int64_t P = carry + (int64_t)(ex[i >> 2] + y[i]);
            p32[i] = (uint32_t)P;
            reinterpret_cast<int32_t *>(&h[i >> 2])[i & 3] = (int32_t)(uint32_t)((uint64_t)P >> 32);
          }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int at = (r0 + 256 * j + 4 * lane) & (RING - 1);
            *reinterpret_cast<int4 *>(&W.ring_lo[at]) =
                make_int4((int)p32[4 * j], (int)p32[4 * j + 1], (int)p32[4 * j + 2], (int)p32[4 * j + 3]);
            *reinterpret_cast<int4 *>(&W.ring_hi[at]) = h[j];
          }
          carry += (int64_t)(t0 + t1);
        }
      }
      if (!quads) {  // the last block of a segment, or samples far from c: 64 samples at a time
        bool blk_big = false;
#pragma unroll 1
        for (int it = 0; it < 8; ++it) {
          const int64_t e = eb + 64 * it + lane;
          // (positions past the segment count as c, i.e. add nothing)
          const int64_t y = e < s1 ? (int64_t)x[min(e, s1 - 1)] - cmean : 0;
          const int64_t P = carry + wave_scan_i64(y);
          blk_big |= __ballot(y <= -big || y >= big) != 0ull;
          carry = lane63(P);
          W.put((r0 + 64 * it + lane) & (RING - 1), P);
        }
        if (blk_big) last_big = blk;
        // box starts lie one position further back than box samples: in one
        // block more than reach_blocks where w_max is 1 above a multiple of 512
        last_slow = blk + ((a.wmax - 1) % kSearchBlock == 0 ? 1 : 0);
      }
      __builtin_amdgcn_wave_barrier();
      if (eb + kSearchBlock - 1 < s0) continue;  // look-back block: sums only

      // every box of every end starts at or after the first sample
      const bool full = max(eb, s0) - (int64_t)(a.wmax - 1) >= -look;
      // ---- integer prefilter.  32 bits wherever every box of the block sums
      // to less than 2^31 in size about w c: C differences of the ring's low
      // halves are exact then ----
      const bool bits32 = full && blk - last_big > reach_blocks;
      uint64_t pass = every;  // widths of which a box may reach its bound in this block
      if (quads && bits32) {
        // does any box of the block reach its width's bound?  First the
        // largest of 4 ends less the smallest of their starts' quad (two
        // quads where w is no multiple of 4), which is seldom above a bound
        // that no box reaches: the widths that are multiples of 4 four at a
        // time, without a branch, so that their LDS reads overlap.  Then
        // exactly, for the widths left: per lane the 8 prefix sums w before
        // its own, two aligned quads, or two pairs of neighbouring ones.
        const int at0 = (r0 >> 2) + lane;
        uint64_t need = every;
        pass = 0;
        if (blk - last_slow > reach_blocks) {
          need = 0;
          for (int k = 0; k < n4; k += 4) {
            uint64_t h[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int32_t *m = &W.qmin[(at0 - __builtin_amdgcn_readlane(lane_q4, k + u)) & (RING / 4 - 1)];
              const int32_t d = max((int32_t)((uint32_t)qmax[0] - (uint32_t)m[0]),
                                    (int32_t)((uint32_t)qmax[1] - (uint32_t)m[64]));
              h[u] = __ballot(d >= __builtin_amdgcn_readlane(lane_ql, k + u));
            }
            if (h[0] | h[1] | h[2] | h[3])
#pragma unroll
              for (int u = 0; u < 4; ++u)
                if (h[u] && k + u < n_al) need |= 1ull << __builtin_amdgcn_readlane(lane_qk, k + u);
          }
          for (uint64_t odd = unaligned; odd; odd &= odd - 1) {
            const int k = __builtin_ctzll(odd);
            const int w = __builtin_amdgcn_readlane(lane_w, k);
            int32_t d = ymax;  // w = 1
            if (w > 1) {
              const int32_t *m = &W.qmin[(at0 - (w >> 2)) & (RING / 4 - 1)];
              const int32_t *mm = &W.qmin[(at0 - (w >> 2) - 1) & (RING / 4 - 1)];
              d = max(max((int32_t)((uint32_t)qmax[0] - (uint32_t)m[0]), (int32_t)((uint32_t)qmax[1] - (uint32_t)m[64])),
                      max((int32_t)((uint32_t)qmax[0] - (uint32_t)mm[0]),
                          (int32_t)((uint32_t)qmax[1] - (uint32_t)mm[64])));
            }
            if (__ballot(d >= __builtin_amdgcn_readlane(lane_l32, k))) need |= 1ull << k;
          }
        }
        const int4 *ring4 = reinterpret_cast<const int4 *>(W.ring_lo);
        for (; need; need &= need - 1) {
          const int k = __builtin_ctzll(need);
          const int w = __builtin_amdgcn_readlane(lane_w, k);
          const int at = at0 - (w >> 2);
          int32_t best = INT32_MIN;
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int4 B = ring4[(at + 64 * j) & (RING / 4 - 1)];
            if ((w & 3) == 0) {
              best = max4(best, p32 + 4 * j, B.x, B.y, B.z, B.w);
              continue;
            }
            const int4 A = ring4[(at + 64 * j - 1) & (RING / 4 - 1)];
            if ((w & 3) == 1)
              best = max4(best, p32 + 4 * j, A.w, B.x, B.y, B.z);
            else if ((w & 3) == 2)
              best = max4(best, p32 + 4 * j, A.z, A.w, B.x, B.y);
            else
              best = max4(best, p32 + 4 * j, A.y, A.z, A.w, B.x);
          }
          if (__ballot(best >= __builtin_amdgcn_readlane(lane_l32, k))) pass |= 1ull << k;
        }
        if (pass == 0ull && !open) continue;
      }
      // ---- box ends that may reach it, 64 a step; widths outer: per width the
      // 8 ring reads are issued together, each compare leaves a wave mask ----
      uint64_t mk[8];
#pragma unroll
      for (int it = 0; it < 8; ++it) mk[it] = 0;
      if (pass && bits32) {
        uint32_t pv[8];
#pragma unroll
        for (int it = 0; it < 8; ++it) pv[it] = (uint32_t)W.ring_lo[(r0 + lane + 64 * it) & (RING - 1)];
        for (uint64_t ks = pass; ks; ks &= ks - 1) {
          const int k = __builtin_ctzll(ks);
          const int w = __builtin_amdgcn_readlane(lane_w, k);
          const int32_t L = __builtin_amdgcn_readlane(lane_l32, k);
          const int bw = r0 + lane - w;
          uint32_t qv[8];
#pragma unroll
          for (int it = 0; it < 8; ++it) qv[it] = (uint32_t)W.ring_lo[(bw + 64 * it) & (RING - 1)];
#pragma unroll
          for (int it = 0; it < 8; ++it) mk[it] |= __ballot((int32_t)(pv[it] - qv[it]) >= L);
        }
      } else if (pass) {
        int64_t pv[8];
#pragma unroll
        for (int it = 0; it < 8; ++it) pv[it] = W.get((r0 + lane + 64 * it) & (RING - 1));
        for (uint64_t ks = pass; ks; ks &= ks - 1) {
          const int k = __builtin_ctzll(ks);
          const int w = __builtin_amdgcn_readlane(lane_w, k);
          const int64_t L = readlane_i64(lane_lim, k);
          const int bw = r0 + lane - w;
          int64_t qv[8];
#pragma unroll
          for (int it = 0; it < 8; ++it) qv[it] = W.get((bw + 64 * it) & (RING - 1));
#pragma unroll
          for (int it = 0; it < 8; ++it)
            mk[it] |= __ballot((pv[it] - qv[it] >= L) & (full | ((int64_t)w <= eb + 64 * it + lane + look + 1)));
        }
      }
      uint32_t mbits = 0;
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int64_t e = eb + 64 * it + lane;
        mbits |= (uint32_t)(((mk[it] >> lane) & 1ull) & (e >= s0) & (e < s1)) << it;
      }

      // ---- exact SNR and runs, step by step ----
#pragma unroll 1
      for (int it = 0; it < 8; ++it) {
        const int64_t e0 = eb + 64 * it;
        const int64_t e = e0 + lane;
        const bool maybe = (mbits >> it) & 1u;
        if (__ballot(maybe) == 0ull && !open) continue;
        bool fl = false;
        double bs = 0.0;
        int kb = 0;
        if (maybe) {
          const int re = (int)(e - lo);
          const int64_t q1 = W.get(re & (RING - 1));
          // only widths whose integer sum passes the prefilter bound can
          // reach the threshold; when one does, the best width is among them
          // (a width below its bound has an SNR below the threshold), so the
          // others are skipped, for the whole wave when none of its lanes pass
          for (uint64_t ks = pass; ks; ks &= ks - 1) {
            const int k = __builtin_ctzll(ks);
            const int w = __builtin_amdgcn_readlane(lane_w, k);
            if ((int64_t)w > e + look + 1) break;  // box would start before the first sample
            const int64_t d = q1 - W.get((re - w) & (RING - 1));  // C difference
            const bool over = d >= readlane_i64(lane_lim, k);
            if (__ballot(over) == 0ull) continue;
            const double sum = (double)(d + cmean * (int64_t)w);
            const double wmu = __builtin_bit_cast(double, readlane_i64(__builtin_bit_cast(int64_t, lane_wmu), k));
            const double den = __builtin_bit_cast(double, readlane_i64(__builtin_bit_cast(int64_t, lane_den), k));
            const double snr = (sum - wmu) / den;
            if (over && (kb == 0 || snr > bs)) {
              bs = snr;
              kb = k + 1;
            }
          }
          fl = kb != 0 && bs >= thr;
        }
        const uint64_t m = __ballot(fl);
        if (open && !(m & 1ull)) {  // the open run ended on the previous step
          if (lane == 0) emit(o_first, o_last, o_peak, o_snr, o_k, o_left, 0);
          open = false;
        }
        if (m == 0ull) continue;
        W.sb[lane] = bs;
        W.sk[lane] = (uint8_t)kb;
        __builtin_amdgcn_wave_barrier();
        const bool last_step = e0 + 63 >= s1 - 1;  // the segment's last box end is on this step
        const bool start = fl && (lane == 0 || !((m >> (lane - 1)) & 1ull));
        // the run's last lane and, at its first lane, its peak (ties keep the
        // earlier box end): lane by lane where runs are short, else all lanes
        // together, each taking in twice as many of its run's lanes every time
        const uint64_t above = ~(m >> lane);
        const int l = lane + (above ? __builtin_ctzll(above) : 64) - 1;
        int pk = lane;
        double ps = bs;
        uint64_t runs8 = m & (m >> 1);
        runs8 &= runs8 >> 2;
        runs8 &= runs8 >> 4;
        if (runs8) {
#pragma unroll
          for (int d = 1; d < 64; d *= 2) {
            const double s = __shfl_down(ps, d, 64);
            const int p = __shfl_down(pk, d, 64);
            if (lane + d <= l && s > ps) {
              ps = s;
              pk = p;
            }
          }
        }
        if (start) {
          if (!runs8)
            for (int q = lane + 1; q <= l; ++q) {
              const double s = W.sb[q];
              if (s > ps) {
                ps = s;
                pk = q;
              }
            }
          int64_t f_first = e0 + lane, f_peak = e0 + pk;
          double f_snr = ps;
          int f_k = W.sk[pk];
          int f_left = (f_first == s0 && s0 > 0) ? 1 : 0;
          if (lane == 0 && open) {  // continues the open run
            f_first = o_first;
            f_left = o_left;
            if (!(ps > o_snr)) {
              f_peak = o_peak;
              f_snr = o_snr;
              f_k = o_k;
            }
          }
          if (l == 63 && !last_step) {  // still open: hand over to the next step
            W.o_first = f_first;
            W.o_peak = f_peak;
            W.o_snr = f_snr;
            W.o_k = f_k;
            W.o_left = f_left;
          } else {
            const int64_t f_last = e0 + l;
            emit(f_first, f_last, f_peak, f_snr, f_k, f_left, (f_last == s1 - 1 && s1 < n) ? 1 : 0);
          }
        }
        __builtin_amdgcn_wave_barrier();
        open = ((m >> 63) & 1ull) && !last_step;
        if (open) {
          o_first = W.o_first;
          o_peak = W.o_peak;
          o_snr = W.o_snr;
          o_k = W.o_k;
          o_left = W.o_left;
          o_last = e0 + 63;
        }
      }
    }
    if (open && lane == 0) emit(o_first, o_last, o_peak, o_snr, o_k, o_left, (o_last == s1 - 1 && s1 < n) ? 1 : 0);
    __builtin_amdgcn_wave_barrier();  // per-wave LDS reused by the next item
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static const void *search_kernel(int ring) {
  switch (ring) {
    case 1024: return (const void *)k_search<1024>;
    case 2048: return (const void *)k_search<2048>;
    case 4096: return (const void *)k_search<4096>;
    default: return (const void *)k_search<8192>;
  }
}

void set_search_attributes(const SearchTiling &tl) {
  check_hip(hipFuncSetAttribute(search_kernel(tl.ring), hipFuncAttributeMaxDynamicSharedMemorySize, (int)tl.lds),
            "set search LDS size");
}

SearchTiling search_tiling(int32_t max_width) {
  SearchTiling t;
  // the ring holds the sums of one block plus w_max before it
  t.ring = 1024;
  while (t.ring < max_width + kSearchBlock) t.ring *= 2;
  if (t.ring > 8192) fail(GSP_EINVAL, "widths too large for the search ring (at most 7680)");
  size_t per_wave = 0;
  switch (t.ring) {
    case 1024: per_wave = sizeof(SearchWaveLds<1024>); break;
    case 2048: per_wave = sizeof(SearchWaveLds<2048>); break;
    case 4096: per_wave = sizeof(SearchWaveLds<4096>); break;
    default: per_wave = sizeof(SearchWaveLds<8192>); break;
  }
  t.waves = (int)std::max<size_t>(1, std::min<size_t>(kSearchThreads / 64, (size_t)(128 * 1024) / per_wave));
  t.lds = per_wave * (size_t)t.waves;
  // long segments keep the look-back re-read small; at least 16 blocks
  t.tile = std::max(8192, ((max_width - 1) / kSearchBlock + 1) * kSearchBlock * 16);
  return t;
}

// Segments of a whole plan's search, whose fragment buffer grows with what is
// found: halved, down to twice the look-back, while the plan gives fewer waves
// than the chip holds (16 a CU).  A quick look's 200 trials of 16384 samples
// are 400 waves of 8192 box ends, 43 us, or 3200 of 1024, 22 us (16 since).
static SearchTiling batch_tiling(const gsp_dmt_desc *desc, int32_t max_width) {
  SearchTiling t = search_tiling(max_width);
  const int smallest = std::max(1, (max_width - 2 + kSearchBlock) / kSearchBlock) * kSearchBlock * 2;
  auto items = [&](int tile) {
    int64_t n = 0;
    for (int s = 0; s < desc->n_seg; ++s) n += (int64_t)desc->seg[s].n_dm * ((desc->n_out[s] + tile - 1) / tile);
    return n;
  };
  while (t.tile / 2 >= smallest && items(t.tile) < 16 * 256) t.tile /= 2;
  return t;
}

template <class Table>
static void finalize_jobs(Table &t, const SearchTiling &tl) {
  int64_t nb = 0;
  int32_t trials = 0;
  for (int j = 0; j < t.n_jobs; ++j) {
    SeriesJob &J = t.job[j];
    J.tiles = (J.n + tl.tile - 1) / tl.tile;
    J.block0 = nb;
    J.trial0 = trials;
    nb += (int64_t)J.n_dm * J.tiles;
    trials += J.n_dm;
  }
  t.n_items = nb;
  t.n_trials = trials;
}
void finalize_table(SeriesTable &t, const SearchTiling &tl) { finalize_jobs(t, tl); }

void launch_stats_table(gsp_ctx *ctx, const SeriesTable *tb_dev, int64_t grid, double *musig, double bytes,
                        hipStream_t st, const uint32_t *need) {
  if (grid <= 0) return;
  ProfScope prof(ctx, "stats", st, bytes);
  hipLaunchKernelGGL(k_stats, dim3((unsigned)grid), dim3(kStatsThreads), 0, st, tb_dev, musig, need);
  check_hip(hipGetLastError(), "launch statistics kernel");
}

void launch_search_table(gsp_ctx *ctx, const SeriesTable *tb_dev, int64_t grid, const SearchTiling &tl,
                         const double *musig, const int32_t *widths_dev, int32_t n_widths, int32_t max_width,
                         float thr, Frag *frags, int64_t cap, unsigned long long *counter, double bytes,
                         hipStream_t st, bool zeroed) {
  SearchArgs a;
  a.tb = tb_dev;
  a.musig = musig;
  a.widths = widths_dev;
  a.nw = n_widths;
  a.wmax = max_width;
  a.tile = tl.tile;
  a.thr = thr;
  a.frags = frags;
  a.cap = cap;
  a.counter = counter;
  if (!zeroed) hipLaunchKernelGGL(k_zero_counter, dim3(1), dim3(1), 0, st, counter);
  if (grid <= 0) return;
  if (grid >= (1LL << 31)) fail(GSP_EOVERFLOW, "too many search workgroups");
  ProfScope prof(ctx, "search", st, bytes);
  const dim3 blk((unsigned)(64 * tl.waves));
  switch (tl.ring) {
    case 1024: hipLaunchKernelGGL(k_search<1024>, dim3((unsigned)grid), blk, tl.lds, st, a); break;
    case 2048: hipLaunchKernelGGL(k_search<2048>, dim3((unsigned)grid), blk, tl.lds, st, a); break;
    case 4096: hipLaunchKernelGGL(k_search<4096>, dim3((unsigned)grid), blk, tl.lds, st, a); break;
    default: hipLaunchKernelGGL(k_search<8192>, dim3((unsigned)grid), blk, tl.lds, st, a); break;
  }
  check_hip(hipGetLastError(), "launch search kernel");
}

// Batch: one job per plan row over the whole dedispersed output.  The job table
// and the widths go to the device as arguments of the kernel that puts them in
// place (and clears the fragment counter): copies of the 80 KB table, twice, of
// the widths and of the counter took some 40 us of a quick look's 140.
struct BatchJobs {
  SeriesJob job[GSP_MAX_SEG];
  int32_t n_jobs, n_trials;
  int64_t n_items;
  int32_t widths[64];
  int32_t n_widths;
};
static_assert(sizeof(BatchJobs) < 4000, "kernel argument size");

__global__ __launch_bounds__(64) void k_put_batch(BatchJobs b, SeriesTable *t, int32_t *widths,
                                                  unsigned long long *counter) {
  const int j = threadIdx.x;
  if (j < b.n_jobs) t->job[j] = b.job[j];
  if (j < b.n_widths) widths[j] = b.widths[j];
  if (j == 0) {
    t->n_jobs = b.n_jobs;
    t->n_trials = b.n_trials;
    t->n_items = b.n_items;
    if (counter) *counter = 0ull;
  }
}

static SeriesTable *put_batch(gsp_ctx *ctx, const gsp_dmt_desc *desc, const int32_t *dmt, const SearchTiling &tl,
                              const std::vector<int32_t> &widths, unsigned long long *counter, BatchJobs &b,
                              hipStream_t st) {
  std::memset(&b, 0, sizeof(b));
  b.n_jobs = desc->n_seg;
  for (int s = 0; s < desc->n_seg; ++s) {
    SeriesJob &J = b.job[s];
    J.x = dmt + desc->offset[s];
    J.pitch = desc->n_out[s];
    J.n = desc->n_out[s];
    J.n_dm = desc->seg[s].n_dm;
  }
  finalize_jobs(b, tl);
  b.n_widths = (int32_t)widths.size();
  std::copy(widths.begin(), widths.end(), b.widths);
  ctx->jobs.device = ctx->device;
  ctx->jobs.reserve(sizeof(SeriesTable));
  if (b.n_widths) {
    ctx->widths.device = ctx->device;
    ctx->widths.reserve(sizeof(b.widths));
  }
  hipLaunchKernelGGL(k_put_batch, dim3(1), dim3(64), 0, st, b, ctx->jobs.as<SeriesTable>(), ctx->widths.as<int32_t>(),
                     counter);
  check_hip(hipGetLastError(), "launch table setup");
  ctx->stats.device = ctx->device;
  ctx->stats.reserve((size_t)desc->n_trials * 2 * sizeof(double));
  return ctx->jobs.as<SeriesTable>();
}

void launch_stats(gsp_ctx *ctx, const int32_t *dmt, const gsp_dmt_desc *desc, hipStream_t st,
                  const uint32_t *need) {
  BatchJobs b;
  SeriesTable *d = put_batch(ctx, desc, dmt, search_tiling(1), {}, nullptr, b, st);
  // bytes: the int32 DM-time array read once (the selected trials' rows only
  // when `need` is given; not known on the host then)
  launch_stats_table(ctx, d, b.n_trials, ctx->stats.as<double>(), need ? 0.0 : 4.0 * (double)desc->total, st,
                     need);
}

const double *stats_musig(gsp_ctx *ctx, const gsp_dmt_desc *) { return ctx->stats.as<double>(); }

void launch_search(gsp_ctx *ctx, const int32_t *dmt, const gsp_dmt_desc *desc, const std::vector<int32_t> &widths,
                   float thr, bool stats, Frag *frags, int64_t cap, unsigned long long *counter, hipStream_t st) {
  const SearchTiling tl = batch_tiling(desc, widths.back());
  BatchJobs b;
  SeriesTable *d = put_batch(ctx, desc, dmt, tl, widths, counter, b, st);
  // bytes: the int32 DM-time array read once (look-back overlap not counted)
  const double bytes = 4.0 * (double)desc->total;
  if (stats) launch_stats_table(ctx, d, b.n_trials, ctx->stats.as<double>(), bytes, st, nullptr);
  set_search_attributes(tl);
  launch_search_table(ctx, d, (b.n_items + tl.waves - 1) / tl.waves, tl, stats_musig(ctx, desc),
                      ctx->widths.as<int32_t>(), (int32_t)widths.size(), widths.back(), thr, frags, cap, counter, bytes,
                      st, true);
}

}  // namespace gsp
