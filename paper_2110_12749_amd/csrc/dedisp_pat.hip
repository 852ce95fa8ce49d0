// Brute-force dedispersion by shared partial sums: the pattern tile.
//
// What is computed is the same as k_dedisp (paper Section 2.3): for every DM
// trial i and output sample t, out[i][t] = sum_c Y[c][t + d(i, c)], exact
// integers.
//
// How.  Take 8 neighbouring channels (a group) and a tile of neighbouring
// trials.  The delays of the group's channels relative to its earliest one,
// (d(i, c) - d(i, c0)), its "pattern", take few distinct values over the
// tile: on the 1000-1500 MHz survey plan about 0.15 patterns per trial over 96
// trials at D = 1, 0.2 to 0.33 over 64 trials at D = 2 to 8.  So the sum of the 8
// channels is formed once per pattern, S[x] = sum_c Y[c][x + diff(c)], for the
// x its trials read, and every trial adds one value per group, S of its
// pattern at its own d(i, c0), instead of 8 samples.
//
//  * The partial sums are products with one-hot matrices and run on the
//    matrix cores (v_mfma_i32_16x16x64_i8): rows = 16 positions x, columns =
//    16 patterns, k = 8 channels x 8 shifts, B[(c, s)][p] = 1 where pattern p
//    reads channel c at shift s.  A lane's operand A is a window of 8
//    consecutive samples of a channel, so it is a plain load: the host lets
//    every channel's shifts start at a 4-byte boundary (loads from other
//    addresses take 4 times as long: 65 against 16 clocks per 64 lanes).  A
//    lane's 8 consecutive x take one 16-byte load (uint8; 4 to a 12-byte load
//    gave a wide band's D = 1 row 44.6 ms, now 40.3), 4 take two (16 bits); x +
//    1 multiplies the window of x with the one-hot matrix moved on by a sample.
//    uint8 samples enter as x - 128 (signed bytes; the accumulator starts at
//    128 per channel); the 11-bit sums of D <= 8 samples enter as two bytes
//    (x >> 4) and (x & 15) whose one-hot weights are 16 and 1.  Sums are exact
//    in int32.
//  * S is kept in LDS as dwords (S[x], S[x + 256]): the tile's outputs t and
//    t + 256 sit in one dword, so a trial's read at any delay is an aligned
//    dword, no shifted second copy is needed, and one three-operand add sums
//    2 outputs x 16 channels = 32 sample-adds.  The 16-bit halves are carried
//    into a second accumulator before they can overflow (PatArgs::flush).
//  * 8 building waves fill the next pass's LDS buffer while 8 summing waves
//    add the current one; one workgroup per CU (160 KB of LDS, 128 registers).
//
// What bounds it: the vector units of both kinds of waves and the LDS reads,
// each at 60 to 75 % of their time (a workgroup's summing alone takes 31 ms of
// the survey's D = 1 row, its building alone 37, both 49.7), with the loads of
// the building waves third.  Measured on the survey plan (4096 channels, 2^20
// samples, rows D = 1, 2, 4, 8): 49.7, 25.1, 12.8 and 7.0 ms (129, 84, 60 and
// 40 T sample-adds/s) against 111, 78, 29 and 11 ms on the byte-quad tile
// (D = 1) and the 16-bit tile; on 270-1620 MHz the D = 1 row takes 40.3 ms
// against 70.7.
#include <algorithm>
#include <array>
#include <cstring>
#include <thread>
#include <type_traits>

#include "dedisp_tile.h"

namespace gsp {

static constexpr int kPatG = 8;          // channels per group
static constexpr int kPatShifts = 7;     // shifts of a channel inside a subgroup of patterns (and one for odd positions)
static constexpr int kPatH = 256;        // a dword holds outputs t and t + kPatH
static constexpr int kPatK = kPatH / 64; // dwords per lane and trial
static constexpr int kPatSum = 8;        // summing waves
static constexpr int kPatBuild = 8;      // building waves
static constexpr int kPatRec = 4 * 16 * 3;  // dwords of a pattern block's records
static constexpr int kPatLdsDw = 20480;  // LDS dwords of one buffer (two buffers: 160 KB, one workgroup per CU)

typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_a __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x3_a __attribute__((ext_vector_type(3), aligned(4)));
typedef uint32_t u32x4_a __attribute__((ext_vector_type(4), aligned(4)));

// positions between a building lane's rows (and the 4 or 8 of each that it
// takes): with uint8 samples a 16-byte load holds the windows of 8 positions;
// 16-bit ones would need 32 registers more
constexpr int pat_rows(int NB) { return NB == 1 ? 8 : 4; }
// Samples of one channel from a lane's first position on: NB = 1: 16; NB = 2:
// 8, and 8 from the third on
template <int NB>
struct PatRaw {
  uint32_t w[4 * NB];
};

// TPW: trials per summing wave; NB: bytes per staged sample
template <int TPW, int NB>
__device__ __forceinline__ void pat_tile(const PatArgs &a, const int L, uint32_t *lds) {
  static_assert(TPW % 2 == 0, "trials are read in pairs");
  constexpr int NP = kPatBuild;
  const int dm_tile = L % a.n_dm_tiles, t_tile = L / a.n_dm_tiles;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int NC = kPatSum;  // summing waves
  const int t0 = t_tile * 2 * kPatH;
  const int p_first = a.tile_pass[dm_tile];
  const int n_pass = a.tile_pass[dm_tile + 1] - p_first - 1;

  // pass records, 64 at a time in registers (lane l: pass w0 + l), taken by readlane
  int w0 = 0;
  int win = 0;
  auto fetch_window = [&](int from) {
    w0 = from;
    win = a.passes[p_first + min(from + lane, n_pass)].x;
    asm volatile("" : "+v"(win));  // waits here, not at every use
  };
  auto g_begin = [&](int j) { return __builtin_amdgcn_readlane(win, j - w0); };
  if (wave >= NC) {
    // ---- building waves ----
    // Wave bw takes the tile's units bw, bw + NP, ... (a multiple of NP in each
    // pass).  What a unit needs is loaded while the units before it are
    // computed: its header (a scalar load), its channel offsets, then its
    // samples and patterns into one of NS register sets.  (Loads run up to 4
    // units past the tile's last one; the table has that many to spare.)
    __builtin_amdgcn_s_setprio(2);
    constexpr int RS = pat_rows(NB);
    const int bw = wave - NC;
    const int m = lane & 15, kg = lane >> 4;  // A: row m (positions x + RS m + j); B: column m; k: channels 2kg, 2kg + 1
    typedef const __attribute__((address_space(4))) int cint;
    typedef const __attribute__((address_space(4))) PatUnit cunit;
    cint *passes = (cint *)(a.passes + p_first);
    int u = passes[1] + bw;  // the next unit to compute
    cunit *up = (cunit *)a.units + u;
    struct Unit {
      int64_t base;
      int x, rel, chan, rec;
    };
    auto header = [&](int k) { return Unit{up[k * NP].base, up[k * NP].x, up[k * NP].rel, up[k * NP].chan, up[k * NP].rec}; };
    const uint32_t co_off = 8 * kg, rec_off = 12 * lane;
    auto load_co = [&](const Unit &h) {
      return *reinterpret_cast<const int2 *>(reinterpret_cast<const char *>(a.chan) + (int64_t)h.chan * (4 * kPatG) + co_off);
    };
    struct Set {             // a unit's inputs
      PatRaw<NB> raw[2][2];  // samples [half][channel of the lane's pair]
      u32x3_a r;             // the lane's pattern record
      int x, rel;            // first position, less the subgroup's first one
    };
    const uint32_t lane_x = (uint32_t)(t0 + RS * m) * NB;
    auto load = [&](Set &s, const Unit &h, const int2 co) {
      const uint8_t *base = a.Y + h.base + h.x * NB;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t vo = (uint32_t)(e ? co.y : co.x) + lane_x;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const uint8_t *p = base + vo + hf * kPatH * NB;
          uint32_t *w = s.raw[hf][e].w;
#pragma unroll
          for (int q = 0; q < NB; ++q) {
            const u32x4_a v = *reinterpret_cast<const u32x4_a *>(p + 4 * q);
            w[4 * q] = v.x, w[4 * q + 1] = v.y, w[4 * q + 2] = v.z, w[4 * q + 3] = v.w;
          }
        }
      }
      s.r = *reinterpret_cast<const u32x3_a *>(reinterpret_cast<const char *>(a.pats) + (int64_t)h.rec * 768 + rec_off);
      s.x = h.x;
      s.rel = h.rel;
    };
    // Operand A of half hf and k step ks, for position offsets 2 j2 and 2 j2 + 1
    // (the latter multiplies the one-hot columns moved on by one sample)
    auto make_a = [&](const Set &s, int hf, int ks, int j2) {
      v4i A;
      if constexpr (NB == 1) {  // the lane's two channels, 8 bytes each
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          uint32_t w[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) w[q] = s.raw[hf][e].w[q] ^ 0x80808080u;  // x - 128
          const int f = j2 >> 1;
          A[2 * e] = (int)((j2 & 1) ? __builtin_amdgcn_alignbyte(w[f + 1], w[f], 2) : w[f]);
          A[2 * e + 1] = (int)((j2 & 1) ? __builtin_amdgcn_alignbyte(w[f + 2], w[f + 1], 2) : w[f + 1]);
        }
      } else {  // channel ks of the two, 16 bytes
#pragma unroll
        for (int q = 0; q < 4; ++q) A[q] = (int)s.raw[hf][ks].w[4 * j2 + q];
      }
      return A;
    };
    const v4i bias = NB == 1 ? v4i{128 * kPatG, 128 * kPatG, 128 * kPatG, 128 * kPatG} : v4i{0, 0, 0, 0};
    // Pattern record of a lane: {LDS dword of the subgroup's first position,
    // the pattern's first position less that one | positions << 16 (both
    // multiples of 4 RS), one-hot bytes or words: for each of the lane's two
    // channels 8 bits per 64 bits of operand B, shift (6 bits) and validity}
    auto compute = [&](const Set &s, uint32_t *dst) {
      v4i B[2][NB];  // for position offsets 2 j2, and 2 j2 + 1: the same shifts plus one
      constexpr uint32_t one = NB == 1 ? 1u : 0x1001u;  // NB = 2: weight 16 on the high byte, 1 on the low one
#pragma unroll
      for (int q = 0; q < 2 * NB; ++q) {  // 64 bits of B at a time
        const uint32_t f = s.r.z >> (8 * q);
        const uint32_t w = NB == 1 ? (f >> 6) & 1u : ((f >> 6) & 1u) * one;
        const uint64_t v = (uint64_t)w << (f & 63u);
        B[0][q >> 1][2 * (q & 1)] = (int)(uint32_t)v;
        B[0][q >> 1][2 * (q & 1) + 1] = (int)(uint32_t)(v >> 32);
        if constexpr (NB == 1) {
          B[1][0][2 * q] = (int)(uint32_t)(v << 8);
          B[1][0][2 * q + 1] = (int)(uint32_t)((v << 8) >> 32);
        }
      }
      if constexpr (NB == 2)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            B[1][ks][q] = (int)(q ? __builtin_amdgcn_alignbyte((uint32_t)B[0][ks][q], (uint32_t)B[0][ks][q - 1], 2)
                                  : (uint32_t)B[0][ks][q] << 16);
      // D: products for x + kPatH, then, with these in the high half, for x.
      // NB = 1 has registers to keep both and join them on the way to the
      // LDS (a shift and or per dword, no moves); NB = 2 starts the second
      // from the first
      v4i D[2][4];
      const uint32_t p = (uint32_t)(s.rel + 4 * RS * kg);
      const bool valid = p - (s.r.y & 0xFFFFu) < (s.r.y >> 16);
      uint32_t *d = dst + (s.r.x + p);
#pragma unroll
      for (int j4 = 0; j4 < RS / 4; ++j4) {  // position offsets 4 j4 + jj
#pragma unroll
        for (int hf = 1; hf >= 0; --hf) {
#pragma unroll
          for (int ks = 0; ks < NB; ++ks) {
            const v4i A[2] = {make_a(s, hf, ks, 2 * j4), make_a(s, hf, ks, 2 * j4 + 1)};
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
              const v4i c = ks ? D[hf][jj] : NB == 1 || hf ? bias : D[1][jj] << 16;
              D[hf][jj] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[jj >> 1], B[jj & 1][ks], c, 0, 0, 0);
            }
          }
        }
        // lane (column m, row block kg): positions x = s.x + 4 RS kg + RS q + 4 j4 + jj
        if (valid) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            v4i w;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) w[jj] = NB == 1 ? D[0][jj][q] | D[1][jj][q] << 16 : D[0][jj][q];
            *reinterpret_cast<v4i *>(d + RS * q + 4 * j4) = w;
          }
        }
        if (j4 + 1 < RS / 4) __builtin_amdgcn_sched_barrier(0);  // registers for one half's products
      }
    };
    // NS sets in turn: unit k's inputs are in set k % NS, those of the NS - 1
    // units before it in flight; its offsets are loaded a unit before its samples
    constexpr int NS = 2;
    Set set[NS];
    int2 co[NS];      // offsets of the unit whose samples go to set k next
    Unit hd[NS];      // and its header
    // (the loads in the order of the steps, so that their waits count alike)
#pragma unroll
    for (int k = 0; k < NS; ++k) hd[k] = header(k);
#pragma unroll
    for (int k = 0; k < NS - 1; ++k) co[k] = load_co(hd[k]);
#pragma unroll
    for (int k = 0; k < NS - 1; ++k) {
      if (k == NS - 2) co[NS - 1] = load_co(hd[NS - 1]);
      __builtin_amdgcn_sched_barrier(0);
      load(set[k], hd[k], co[k]);
      __builtin_amdgcn_sched_barrier(0);
    }
    hd[0] = header(NS);
    int pass = 0, ue = passes[3];  // the pass being built and its end
    uint32_t *dst = lds;
    auto step = [&](auto kc) {     // returns whether the tile is done
      constexpr int k = decltype(kc)::value, l = (k + NS - 1) % NS;
      // offsets before samples: the wait for them leaves the samples in flight
      co[k] = load_co(hd[k]);
      __builtin_amdgcn_sched_barrier(0);
      load(set[l], hd[l], co[l]);
      up += NP;
      hd[(k + 1) % NS] = header(NS);
      __builtin_amdgcn_sched_barrier(0);
      compute(set[k], dst);
      __builtin_amdgcn_sched_barrier(0);
      u += NP;
      if (u < ue) return false;
      wg_barrier();  // the pass is built, the one before it summed
      if (++pass == n_pass) return true;
      dst = lds + (pass & 1) * kPatLdsDw;
      ue = passes[2 * pass + 3];
      return false;
    };
    while (true) {
      if (step(std::integral_constant<int, 0>())) break;
      if (step(std::integral_constant<int, 1>())) break;
      if constexpr (NS == 3)
        if (step(std::integral_constant<int, 2>())) break;
    }
    wg_barrier();  // the last pass is summed
    return;
  }

  // ---- summing waves ----
  constexpr int NPR = TPW / 2;      // offset dwords per group
  constexpr int GPR = 64 / NPR;     // groups whose offsets one register (a dword per lane) holds
  const int i_wave = dm_tile * TPW * NC + wave * TPW;
  uint32_t roff[2], noff[2];
  auto load_off = [&](int j) {
    const int gb = g_begin(j), ge = g_begin(j + 1);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int g = min(gb + r * GPR + lane / NPR, ge - 1);
      noff[r] = a.addr[(int64_t)g * (a.n_dm_pad >> 1) + (i_wave >> 1) + lane % NPR];
    }
  };
  // acc: sums of the two outputs of a dword in its 16-bit halves, below
  // 65536; car: multiples of 2048 carried out of them
  uint32_t acc[TPW][kPatK], car[TPW][kPatK];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int k = 0; k < kPatK; ++k) acc[t][k] = car[t][k] = 0;
  const uint32_t *cur = lds;
  auto ld = [&](uint32_t off, int q, int t, uint32_t *v) {  // trial t's dwords of the group with offsets at lane q of off
    const uint32_t pair = (uint32_t)__builtin_amdgcn_readlane((int)off, q + (t >> 1));
    const uint32_t o = (t & 1) ? pair >> 16 : pair & 0xFFFFu;
    const uint32_t *src = cur + o + lane;
#pragma unroll
    for (int k = 0; k < kPatK; ++k) v[k] = src[64 * k];
  };
  int left = a.flush;  // groups that may be added before the next carry
  auto carry = [&]() {
    left = a.flush;
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int k = 0; k < kPatK; ++k) {
        car[t][k] += (acc[t][k] >> 11) & 0x001F001Fu;
        acc[t][k] &= 0x07FF07FFu;
      }
  };
  fetch_window(0);
  load_off(0);
  wg_barrier();  // pass 0 built
  for (int kc = 0; kc < n_pass; ++kc) {
    if (kc + 3 > w0 + 63) fetch_window(kc);
    const int ng = g_begin(kc + 1) - g_begin(kc);
#pragma unroll
    for (int r = 0; r < 2; ++r) roff[r] = noff[r];
    if (kc + 1 < n_pass) load_off(kc + 1);
    cur = lds + (kc & 1) * kPatLdsDw;
    // two groups at a time: one three-operand add sums both into a trial's
    // dword; two trials' dwords of both in flight
    auto lane_of = [&](int g) { return (g < GPR ? g : g - GPR) * NPR; };
    auto off_of = [&](int g) { return g < GPR ? roff[0] : roff[1]; };
    int g = 0;
    for (; g + 1 < ng; g += 2) {
      const uint32_t oa = off_of(g), ob = off_of(g + 1);
      const int qa = lane_of(g), qb = lane_of(g + 1);
      uint32_t va[2][kPatK], vb[2][kPatK];
      ld(oa, qa, 0, va[0]);
      ld(ob, qb, 0, vb[0]);
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        if (t + 1 < TPW) {
          ld(oa, qa, t + 1, va[(t + 1) & 1]);
          ld(ob, qb, t + 1, vb[(t + 1) & 1]);
        }
#pragma unroll
        for (int k = 0; k < kPatK; ++k) acc[t][k] = acc[t][k] + va[t & 1][k] + vb[t & 1][k];
      }
      left -= 2;
      if (left < 2) carry();
    }
    if (g < ng) {
      const uint32_t oa = off_of(g);
      const int qa = lane_of(g);
      uint32_t va[2][kPatK];
      ld(oa, qa, 0, va[0]);
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        if (t + 1 < TPW) ld(oa, qa, t + 1, va[(t + 1) & 1]);
#pragma unroll
        for (int k = 0; k < kPatK; ++k) acc[t][k] += va[t & 1][k];
      }
      left -= 1;
      if (left < 2) carry();
    }
    wg_barrier();  // pass kc summed, pass kc + 1 built
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int i = i_wave + t;
    if (i >= a.n_dm) break;
    int32_t *orow = a.out + (int64_t)i * a.out_pitch;
#pragma unroll
    for (int k = 0; k < kPatK; ++k) {
      const uint32_t s[2] = {(acc[t][k] & 0xFFFFu) + ((car[t][k] & 0xFFFFu) << 11) - a.excess,
                             (acc[t][k] >> 16) + ((car[t][k] >> 16) << 11) - a.excess};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t tt = (int64_t)t0 + h * kPatH + lane + 64 * k;
        if (tt < a.n_out && tt >= a.t_lo) orow[tt] = (int32_t)s[h];
      }
    }
  }
}

template <int TPW, int NB>
__global__ __launch_bounds__(64 * (kPatSum + kPatBuild)) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_dedisp_pat(PatArgs a) {
  extern __shared__ __align__(16) uint32_t lds[];
  pat_tile<TPW, NB>(a, xcd_remap(blockIdx.x, a.n_dm_tiles * a.n_t_tiles), lds);
}

// The tiles of a job table, one per workgroup; the grid, fixed when a graph is
// captured, may hold more.
template <int TPW, int NB>
__global__ __launch_bounds__(64 * (kPatSum + kPatBuild)) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_dedisp_pat_jobs(const PatJobTable *tb) {
  extern __shared__ __align__(16) uint32_t lds[];
  typedef const __attribute__((address_space(4))) PatJobTable ctable;  // scalar loads
  ctable *t = (ctable *)tb;
  const int n_items = (int)t->n_items;
  if ((int)blockIdx.x >= n_items) return;
  const int L = xcd_remap(blockIdx.x, n_items);
  int lo = 0, hi = t->n_jobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((int)t->job[mid].item0 <= L)
      lo = mid;
    else
      hi = mid - 1;
  }
  static_assert(sizeof(PatArgs) % 8 == 0, "copied by 8 bytes");
  typedef const __attribute__((address_space(4))) uint64_t cu64;
  cu64 *src = (cu64 *)&t->job[lo].a;
  uint64_t w[sizeof(PatArgs) / 8];
#pragma unroll
  for (int k = 0; k < (int)(sizeof(PatArgs) / 8); ++k) w[k] = src[k];
  PatArgs a;
  __builtin_memcpy(&a, w, sizeof(a));
  a.Y = as_global(a.Y);
  a.addr = as_global(a.addr);
  a.tile_pass = as_global(a.tile_pass);
  a.passes = as_global(a.passes);
  a.units = as_global(a.units);
  a.chan = as_global(a.chan);
  a.pats = as_global(a.pats);
  a.out = as_global(a.out);
  pat_tile<TPW, NB>(a, L - (int)t->job[lo].item0, lds);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
bool pat_shape_supported(const DedispShape &s) {
  return s.kind == 4 && s.groups == kPatK && (s.tpw == 12 || s.tpw == 8) && s.waves == kPatSum &&
         s.chunk >= 1;
}

// groups of a pass: the summing waves hold their offsets in two registers
static int pat_max_groups(const DedispShape &s) { return std::min(s.chunk, 2 * (64 / (s.tpw / 2))); }

namespace {

// One DM tile's tables, indices relative to the tile's own first entry
struct PatTile {
  std::vector<int32_t> passes;  // {first group, first unit}
  std::vector<PatUnit> units;   // base: not yet known
  std::vector<int32_t> chan;
  std::vector<uint32_t> pats;
  std::vector<uint32_t> addr;   // [n_groups][MT / 2]
  int64_t far = 0;              // samples read past a tile's first output
  double built = 0;             // LDS dwords built
  const char *err = nullptr;
};

struct Pattern {
  int32_t diff[kPatG];  // delays relative to the group's earliest channel
  int32_t lo, hi;       // range of that channel's delay over the pattern's trials
};

void build_pat_tile(const RowTables &rt, int i0, int MT, const std::vector<int32_t> &first, PatTile &T) {
  const int nchan = rt.nchan, n_dm = rt.n_dm, ng = (int)first.size();
  const int NB = rt.D == 1 ? 1 : 2, RS = pat_rows(NB), run = 4 * RS - 1;
  const int32_t *d = rt.delays_host.data();
  T.addr.assign((size_t)ng * (MT / 2), 0);
  std::vector<Pattern> P;
  std::vector<int32_t> pat_of(MT), dst, xs;
  int64_t used = 0;
  int in_pass = 0;
  // a pass's work goes to the building waves in turn, 16 RS positions of a
  // subgroup (all their pattern blocks) to the one with the least so far;
  // their unit lists are interleaved, all filled up to the same length
  // with units of block 0, which has no patterns
  struct Work {
    int32_t sub, x, rel, blk, nblk, g;
  };
  std::vector<Work> todo;
  T.pats.assign(kPatRec, 0);
  std::vector<std::vector<PatUnit>> list(kPatBuild);
  auto end_pass = [&]() {
    for (auto &l : list) l.clear();
    for (const Work &w : todo) {
      auto &l = *std::min_element(list.begin(), list.end(), [](auto &p, auto &q) { return p.size() < q.size(); });
      for (int b = 0; b < w.nblk; ++b) l.push_back({0, w.x, w.rel, w.sub, w.blk + b, w.g, 0});
    }
    size_t n = 0;
    for (auto &l : list) n = std::max(n, l.size());
    const Work &w = todo.back();
    for (size_t k = 0; k < n; ++k)
      for (auto &l : list) T.units.push_back(k < l.size() ? l[k] : PatUnit{0, w.x, 0, w.sub, 0, w.g, 0});
    todo.clear();
  };
  const int max_g = pat_max_groups(rt.shape);
  for (int g = 0; g < ng; ++g) {
    const int c_lo = g * kPatG, nc = std::min(kPatG, nchan - c_lo);
    const int c0 = first[g];
    P.clear();
    for (int j = 0; j < MT; ++j) {
      const int32_t *row = d + (int64_t)std::min(i0 + j, n_dm - 1) * nchan + c_lo;
      const int32_t o = row[c0 - c_lo];
      Pattern n;
      for (int c = 0; c < kPatG; ++c) n.diff[c] = c < nc ? row[c] - o : 0;
      int k = (int)P.size() - 1;
      while (k >= 0 && std::memcmp(P[k].diff, n.diff, sizeof(n.diff)) != 0) --k;
      if (k < 0) {
        k = (int)P.size();
        n.lo = n.hi = o;
        P.push_back(n);
      } else {
        P[k].lo = std::min(P[k].lo, o);
        P[k].hi = std::max(P[k].hi, o);
      }
      pat_of[j] = k;
    }
    // LDS windows of whole runs of 4 RS positions (what a lane writes); the 16-byte
    // chunk of a position differs by 1 mod RS between neighbouring patterns,
    // which spreads the writes of 16 patterns over the banks (73 B/clk/CU
    // against 16 where they agree)
    const int np = (int)P.size();
    dst.resize(np);
    xs.resize(np);
    auto place = [&](int64_t at) {
      for (int k = 0; k < np; ++k) {
        const int32_t s = P[k].lo & ~run, e = (P[k].hi + kPatH + run) & ~run;
        xs[k] = s;
        while ((((at - s) >> 2) & (RS - 1)) != (k & (RS - 1))) at += 4;
        dst[k] = (int32_t)at;
        at += e - s;
      }
      return at;
    };
    int64_t end = place(used);
    if (in_pass == 0 || end > kPatLdsDw || in_pass >= max_g) {
      if (in_pass) end_pass();
      T.passes.push_back(g);
      T.passes.push_back((int32_t)(T.units.size()));
      end = place(0);
      in_pass = 0;
      if (end > kPatLdsDw) {
        T.err = "a channel group's partial sums do not fit the LDS";
        return;
      }
    }
    T.built += (double)(end - (in_pass ? used : 0));
    used = end;
    ++in_pass;
    for (int j = 0; j < MT; ++j) {
      const int32_t o = d[(int64_t)std::min(i0 + j, n_dm - 1) * nchan + c0];
      const int k = pat_of[j];
      T.addr[(size_t)g * (MT / 2) + j / 2] |= (uint32_t)(dst[k] + o - xs[k]) << (16 * (j & 1));
    }
    // subgroups: consecutive patterns whose shifts span at most 7 per channel,
    // counted from a 4-byte boundary of the staged row
    const int32_t al = 4 / NB - 1;
    for (int s = 0; s < np;) {
      int32_t lo[kPatG], hi[kPatG];
      std::copy(P[s].diff, P[s].diff + kPatG, lo);
      std::copy(P[s].diff, P[s].diff + kPatG, hi);
      int e = s + 1;
      for (; e < np; ++e) {
        bool ok = true;
        for (int c = 0; c < nc && ok; ++c)
          ok = std::max(hi[c], P[e].diff[c]) - (std::min(lo[c], P[e].diff[c]) & ~al) < kPatShifts;
        if (!ok) break;
        for (int c = 0; c < nc; ++c) {
          lo[c] = std::min(lo[c], P[e].diff[c]);
          hi[c] = std::max(hi[c], P[e].diff[c]);
        }
      }
      for (int c = 0; c < nc; ++c) lo[c] &= ~al;
      const int32_t sub = (int32_t)(T.chan.size() / (2 * kPatG));  // two entries per channel
      int32_t max_lo = 0;
      for (int c = 0; c < kPatG; ++c) {
        const int cc = c < nc ? c : 0;  // absent channels read the first one, weight 0
        T.chan.push_back(cc);           // channel of the group ...
        T.chan.push_back(lo[cc]);       // ... and its first shift (byte offsets once the pitch is known)
        max_lo = std::max(max_lo, lo[cc]);
      }
      const int32_t blk0 = (int32_t)(T.pats.size() / kPatRec);
      const int nblk = (e - s + 15) / 16;
      std::vector<int32_t> bs(nblk, INT32_MAX), be(nblk, 0);  // positions each block covers
      for (int k = s; k < e; ++k) {
        bs[(k - s) / 16] = std::min(bs[(k - s) / 16], xs[k]);
        be[(k - s) / 16] = std::max(be[(k - s) / 16], (P[k].hi + kPatH + run) & ~run);
      }
      const int32_t x0 = *std::min_element(bs.begin(), bs.end()), x1 = *std::max_element(be.begin(), be.end());
      if (x1 - x0 >= 65536 - 16 * RS) {
        T.err = "a channel group's delays spread too wide";
        return;
      }
      T.pats.resize(T.pats.size() + (size_t)nblk * kPatRec, 0);
      for (int k = s; k < e; ++k) {
        uint32_t *blk = T.pats.data() + (size_t)(blk0 + (k - s) / 16) * kPatRec;
        const uint32_t len = (uint32_t)(((P[k].hi + kPatH + run) & ~run) - xs[k]);
        for (int kg = 0; kg < 4; ++kg) {
          uint32_t *r = blk + 3 * (16 * kg + (k - s) % 16);
          r[0] = (uint32_t)(dst[k] - (xs[k] - x0));
          r[1] = (uint32_t)(xs[k] - x0) | len << 16;
          for (int q = 0; q < 2; ++q) {
            const int c = 2 * kg + q;
            if (c >= nc) continue;
            const uint32_t sh = (uint32_t)(P[k].diff[c] - lo[c]);
            if (NB == 1)
              r[2] |= (64 | 8 * sh) << (8 * q);  // byte sh of 8
            else
              r[2] |= (64 | 16 * (sh & 3)) << (16 * q + 8 * (sh >> 2));  // word sh of 8, 4 to each 64 bits
          }
        }
      }
      for (int32_t x = x0; x < x1; x += 16 * RS) {
        int b0 = nblk, b1 = -1;
        for (int b = 0; b < nblk; ++b)
          if (bs[b] < x + 16 * RS && be[b] > x) {
            b0 = std::min(b0, b);
            b1 = b;
          }
        if (b1 < 0) continue;
        todo.push_back({sub, x, x - x0, blk0 + b0, b1 - b0 + 1, g});
        T.far = std::max<int64_t>(T.far, x + 15 * RS + kPatH + max_lo + 16);
      }
      s = e;
    }
  }
  end_pass();
  T.passes.push_back(ng);  // sentinel
  T.passes.push_back((int32_t)(T.units.size()));
}

}  // namespace

void pat_tables_host(const RowTables &rt, PatHost &H) {
  const DedispShape &sh = rt.shape;
  if (rt.D > 8) fail(GSP_EINVAL, "the pattern tile sums at most 8 samples (11 bits)");
  if (!pat_shape_supported(sh)) fail(GSP_EINVAL, "unsupported dedispersion shape");
  const int nchan = rt.nchan, n_dm = rt.n_dm;
  const int ng = (nchan + kPatG - 1) / kPatG;
  if (ng >= (1 << 22)) fail(GSP_EINVAL, "too many channels for the pattern tile");
  // carried multiples of 2048 stay below 65536
  if ((int64_t)255 * rt.D * nchan / 2048 >= 65000) fail(GSP_EINVAL, "sums too large for the pattern tile");
  const int NB = rt.D == 1 ? 1 : 2;
  const int MT = sh.trials_per_block();
  const int n_tiles = (n_dm + MT - 1) / MT;
  // earliest channel of each group: the same for every trial (delays of all
  // trials fall with frequency), taken at the last one
  std::vector<int32_t> first(ng);
  const int32_t *dl = rt.delays_host.data() + (int64_t)(n_dm - 1) * nchan;
  for (int g = 0; g < ng; ++g) {
    const int c1 = std::min(nchan, (g + 1) * kPatG);
    first[g] = (int32_t)(std::min_element(dl + g * kPatG, dl + c1) - dl);
  }
  std::vector<PatTile> tiles(n_tiles);
  const int n_thr = (int)std::max(1u, std::min({16u, std::thread::hardware_concurrency(), (unsigned)n_tiles}));
  std::vector<std::exception_ptr> errs(n_thr);
  auto work = [&](int k) {
    try {
      for (int tl = k; tl < n_tiles; tl += n_thr) build_pat_tile(rt, tl * MT, MT, first, tiles[tl]);
    } catch (...) {
      errs[k] = std::current_exception();
    }
  };
  {
    std::vector<std::thread> thr;
    try {
      for (int k = 1; k < n_thr; ++k) thr.emplace_back(work, k);
    } catch (...) {  // no more threads: the remaining shares run here
      for (int k = (int)thr.size() + 1; k < n_thr; ++k) work(k);
    }
    work(0);
    for (auto &t : thr) t.join();
  }
  for (auto &e : errs)
    if (e) std::rethrow_exception(e);
  int64_t far = 0;
  double built = 0;
  size_t n_units = 0, n_chan = 0, n_pats = 0, n_passes = 0;
  for (const PatTile &T : tiles) {
    if (T.err) fail(GSP_EINVAL, T.err);
    far = std::max(far, T.far);
    built += T.built;
    n_units += T.units.size();
    n_chan += T.chan.size() / (2 * kPatG);
    n_pats += T.pats.size();
    n_passes += T.passes.size() / 2;
  }
  if (std::max({n_units, n_chan * kPatG, n_pats, n_passes}) >= (size_t)INT32_MAX / 16)
    fail(GSP_EINVAL, "pattern tables too large");
  const int64_t T2 = 2 * kPatH;
  const int64_t n_t = (rt.n_out + T2 - 1) / T2;
  const int64_t pitch = (std::max({rt.N, (n_t - 1) * T2 + far, rt.pitch_override}) + 255) / 256 * 256;
  // byte offsets inside a group's rows are 32 bits
  if (pitch * NB * (kPatG + 1) >= (1LL << 31)) fail(GSP_EINVAL, "row too long for the pattern tile's 32-bit offsets");

  H.addr.assign((size_t)ng * n_tiles * (MT / 2), 0);
  H.passes.reserve(2 * n_passes);
  H.units.reserve(n_units + 4 * kPatBuild);
  H.chan.reserve(kPatG * n_chan);
  H.pats.reserve(n_pats);
  for (int tl = 0; tl < n_tiles; ++tl) {
    PatTile &T = tiles[tl];
    const int32_t i_off = (int32_t)H.units.size(), c_off = (int32_t)(H.chan.size() / kPatG),
                  b_off = (int32_t)(H.pats.size() / kPatRec);
    H.tile_pass.push_back((int32_t)(H.passes.size() / 2));
    for (size_t k = 0; k < T.passes.size(); k += 2) {
      H.passes.push_back(T.passes[k]);
      H.passes.push_back(T.passes[k + 1] + i_off);
    }
    for (PatUnit v : T.units) {
      v.base = (int64_t)v.group * kPatG * pitch * NB;
      v.chan += c_off;
      v.rec += b_off;
      H.units.push_back(v);
    }
    for (size_t k = 0; k < T.chan.size(); k += 2)
      H.chan.push_back((int32_t)((T.chan[k] * pitch + T.chan[k + 1]) * NB));
    H.pats.insert(H.pats.end(), T.pats.begin(), T.pats.end());
    for (int g = 0; g < ng; ++g)
      std::copy(T.addr.begin() + (size_t)g * (MT / 2), T.addr.begin() + (size_t)(g + 1) * (MT / 2),
                H.addr.begin() + ((size_t)g * n_tiles + tl) * (MT / 2));
    T = PatTile();
  }
  for (int k = 0; k < 4 * kPatBuild; ++k) H.units.push_back(H.units.back());  // read ahead of the last tile's end
  H.tile_pass.push_back((int32_t)(H.passes.size() / 2));
  H.pitch = pitch;
  H.built = built;
}

// Clocks of a row on the pattern tile, from the work that its tables list:
// rounds of 256 workgroups (one to a CU), each some 10000 or 22000 clocks
// (filling and draining), 208 per building unit of 128 positions (183 for
// 16-bit samples' 64) and 8.5 per trial and group of 8 channels.  Fitted to the
// same 126 rows as the other tiles, to 7 %; D > 1 then 17 % up, so that no row
// came out slower than on the other tile.
double pat_clocks(const RowTables &rt, const PatHost &H) {
  const int ng = (rt.nchan + kPatG - 1) / kPatG, MT = rt.shape.trials_per_block();
  const int64_t n_dm_tiles = (rt.n_dm + MT - 1) / MT;
  const int64_t tiles = n_dm_tiles * ((rt.n_out + 2 * kPatH - 1) / (2 * kPatH));
  const double units = (double)(H.units.size() - 4 * kPatBuild) / (double)n_dm_tiles;
  const double rounds = (double)((tiles + 255) / 256);
  return rt.D == 1 ? 8.4e3 + rounds * (9.9e3 + 208.0 * units + 8.54 * MT * ng)
                   : 1.17 * (0.5e3 + rounds * (21.9e3 + 183.0 * units + 8.67 * MT * ng));
}

// Whether the pattern tile beats the row's other default (the byte-quad tile's
// estimate, which does not see how wide its copies are, 25 % up).  It does
// not where the channels are so wide, or the trials so far apart, that most
// trials have patterns of their own (64 channels over 500 MHz, 688 trials at
// D = 2: 0.229 against 0.184 ms), nor for few trials of a tile.  Over the 126
// rows the defaults so chosen take 1.78 times less time in the mean than
// without the pattern tile, the fastest choice for each row 1.79 times.
bool pat_tables_pay(const RowTables &rt, const PatHost &H) {
  double other = plain_clocks(rt.n_dm, rt.n_out, rt.nchan);
  if (rt.D == 1 && rt.nchan % 4 == 0) other = std::min(other, 1.25 * quad_clocks(rt.n_dm, rt.n_out, rt.nchan));
  return pat_clocks(rt, H) < other;
}

// Whether 64 trials per tile are faster than the 96 of rt.  With many tiles it
// is the trials' padding that decides: a tile's building costs about 24 trials'
// sums (the survey's D = 1 row: 49.7 ms for 16 tiles of 96, 54.9 for 24 of
// 64), so that the second set of tables is built only where rounds are few
// (1024 channels, 782 trials, 17900 outputs: 0.336 ms in 2 rounds of 96, 0.257
// in 2 of 64).
static bool fewer_trials_faster(const RowTables &rt, const PatHost &H) {
  auto padded = [&](int t) { return (int64_t)(rt.n_dm + 8 * t - 1) / (8 * t) * (8 * t + 24); };
  const int64_t tiles = (int64_t)((rt.n_dm + 95) / 96) * ((rt.n_out + 2 * kPatH - 1) / (2 * kPatH));
  if (tiles > 8 * 256) return padded(8) < padded(12);
  RowTables small;
  small.n_dm = rt.n_dm;
  small.D = rt.D;
  small.nchan = rt.nchan;
  small.N = rt.N;
  small.n_out = rt.n_out;
  small.max_delay = rt.max_delay;
  small.shape = rt.shape;
  small.shape.tpw = 8;
  small.delays_host = rt.delays_host;
  PatHost S;
  try {
    pat_tables_host(small, S);
  } catch (const Error &) {
    return false;
  }
  return pat_clocks(small, S) < pat_clocks(rt, H);
}

void build_pat_tables(gsp_ctx *ctx, RowTables &rt, bool must) {
  // small rows keep the other tile, whose tables are smaller: up to 2048 times
  // 64 trials, 512 outputs and a group at D = 1, where that is the byte-quad
  // tile, 1024 at others
  const int64_t t_tiles = (rt.n_out + 2 * kPatH - 1) / (2 * kPatH);
  if (!must && rt.n_dm * t_tiles * ((rt.nchan + kPatG - 1) / kPatG) <= 64 * (rt.D == 1 ? 2048 : 1024))
    fail(GSP_EINVAL, "too small a row for the pattern tile");
  PatHost H;
  pat_tables_host(rt, H);
  if (!must && rt.shape.tpw == 12 && fewer_trials_faster(rt, H))
    fail(GSP_EINVAL, "fewer trials per pattern tile are faster on this row");
  if (!must && !pat_tables_pay(rt, H)) fail(GSP_EINVAL, "the pattern tile does not pay on this row");
  upload_pat_tables(ctx, rt, H);
}

int64_t pat_table_bytes(const PatHost &H) {
  return (int64_t)((H.tile_pass.size() + H.passes.size() + H.chan.size() + H.pats.size() + H.addr.size()) * 4 +
                   H.units.size() * sizeof(PatUnit));
}

void upload_pat_tables(gsp_ctx *ctx, RowTables &rt, const PatHost &H) {
  rt.q_pitch = H.pitch;
  rt.lds_bytes = 2 * kPatLdsDw * 4;
  rt.q_staged_dw = H.built;
  rt.n_passes = (int32_t)(H.passes.size() / 2);
  rt.max_chunk = pat_max_groups(rt.shape);
  rt.shape.chunk = rt.max_chunk;
  auto upload = [&](DevBuf &b, const void *src, size_t bytes, const char *what) {
    b.device = ctx->device;
    b.reserve(std::max<size_t>(bytes, 16));
    check_hip(hipMemcpy(b.ptr, src, bytes, hipMemcpyHostToDevice), what);
  };
  upload(rt.q_tile_pass, H.tile_pass.data(), H.tile_pass.size() * 4, "copy pattern pass index");
  upload(rt.q_passes, H.passes.data(), H.passes.size() * 4, "copy pattern passes");
  upload(rt.q_items, H.units.data(), H.units.size() * sizeof(PatUnit), "copy pattern units");
  upload(rt.q_chan, H.chan.data(), H.chan.size() * 4, "copy pattern channel offsets");
  upload(rt.q_copies, H.pats.data(), H.pats.size() * 4, "copy patterns");
  upload(rt.addr, H.addr.data(), H.addr.size() * 4, "copy pattern LDS offsets");
}

template <int TPW, int NB>
static void launch_p(const PatArgs &a, int64_t lds, hipStream_t st) {
  auto kern = k_dedisp_pat<TPW, NB>;
  check_hip(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds),
            "set LDS size");
  hipLaunchKernelGGL(kern, dim3(a.n_dm_tiles * a.n_t_tiles), dim3(64 * (kPatSum + kPatBuild)), (size_t)lds, st, a);
}

PatArgs pat_args(const RowTables &rt, const uint8_t *Y, int32_t *out, int64_t out_pitch, int32_t t_lo, int64_t n_out) {
  PatArgs a;
  std::memset(&a, 0, sizeof(a));
  a.excess = rt.D == 1 ? 128 * (-rt.nchan & (kPatG - 1)) : 0;
  a.Y = Y;
  a.addr = rt.addr.as<uint32_t>();
  a.tile_pass = rt.q_tile_pass.as<int32_t>();
  a.passes = rt.q_passes.as<int2>();
  a.units = rt.q_items.as<PatUnit>();
  a.chan = rt.q_chan.as<int32_t>();
  a.pats = rt.q_copies.as<uint32_t>();
  a.out = out;
  a.out_pitch = out_pitch;
  a.n_out = n_out;
  a.t_lo = t_lo;
  a.n_dm = rt.n_dm;
  const int MT = rt.shape.trials_per_block();
  a.n_dm_tiles = (rt.n_dm + MT - 1) / MT;
  a.n_dm_pad = a.n_dm_tiles * MT;
  const int64_t n_t = (n_out + 2 * kPatH - 1) / (2 * kPatH);
  if ((int64_t)a.n_dm_tiles * n_t >= (1LL << 31)) fail(GSP_EOVERFLOW, "too many dedispersion tiles");
  a.n_t_tiles = (int32_t)n_t;
  // a half holds at most 2047 after a carry; each group adds at most 255 D kPatG
  a.flush = (65535 - 2047) / (255 * rt.D * kPatG);  // >= 3 for D <= 8; at least 2 are added between carries
  return a;
}

void launch_dedisp_pat(gsp_ctx *ctx, const RowTables &rt, int32_t *out_row, hipStream_t st) {
  const PatArgs a = pat_args(rt, ctx->staged.as<uint8_t>(), out_row, rt.n_out, 0, rt.n_out);
  ProfScope prof(ctx, "dedisperse_pattern", st, (double)rt.n_dm * (double)rt.n_out * (double)rt.nchan);
  switch (rt.shape.tpw * 4 + (rt.D == 1 ? 1 : 2)) {
    case 12 * 4 + 1: launch_p<12, 1>(a, rt.lds_bytes, st); break;
    case 12 * 4 + 2: launch_p<12, 2>(a, rt.lds_bytes, st); break;
    case 8 * 4 + 1: launch_p<8, 1>(a, rt.lds_bytes, st); break;
    case 8 * 4 + 2: launch_p<8, 2>(a, rt.lds_bytes, st); break;
    default: fail(GSP_EINVAL, "unsupported dedispersion shape");
  }
  check_hip(hipGetLastError(), "launch dedispersion kernel");
}

int pat_form(const RowTables &rt) { return rt.D > 1 ? 2 : rt.shape.tpw == 8 ? 1 : 0; }

static const void *pat_jobs_kernel(int form) {
  return form == 0   ? (const void *)k_dedisp_pat_jobs<12, 1>
         : form == 1 ? (const void *)k_dedisp_pat_jobs<8, 1>
                     : (const void *)k_dedisp_pat_jobs<8, 2>;
}

void set_pat_jobs_attributes(int form) {
  check_hip(hipFuncSetAttribute(pat_jobs_kernel(form), hipFuncAttributeMaxDynamicSharedMemorySize, 2 * kPatLdsDw * 4),
            "set LDS size");
}

void launch_pat_jobs(int form, const PatJobTable *tb_dev, int64_t grid, hipStream_t st) {
  const dim3 g((unsigned)grid), blk(64 * (kPatSum + kPatBuild));
  const size_t lds = 2 * kPatLdsDw * 4;
  switch (form) {
    case 0: hipLaunchKernelGGL((k_dedisp_pat_jobs<12, 1>), g, blk, lds, st, tb_dev); break;
    case 1: hipLaunchKernelGGL((k_dedisp_pat_jobs<8, 1>), g, blk, lds, st, tb_dev); break;
    default: hipLaunchKernelGGL((k_dedisp_pat_jobs<8, 2>), g, blk, lds, st, tb_dev); break;
  }
  check_hip(hipGetLastError(), "launch pattern jobs");
}

}  // namespace gsp
