// rbq_topp_select: adaptive Top-p selection (Algorithm 2 step 3; Section 4.1).
//
// The selected set is { i : S_i >= s* } where s* is the largest score value
// whose "mass at or above" reaches p of the softmax total. Instead of a sort
// (O(n log n)) or Algorithm 3's ternary search over values, s* is found as the
// boundary key K* (the order-preserving 32-bit key of its fp32 score): a
// histogram of softmax masses over bins of the score finds the bin that holds
// it, and the few keys inside that bin are ranked by their masses.
//
// Masses. A key's mass relative to a reference r (a part's maximum, or the
// row maximum M) is exp2((S - r) * sm_scale * log2(e)) in fp32, as a 2^-40
// fixed-point integer (2^-48 for rows of 16385 to 32768 keys); histogram sums are
// 64-bit integer sums, so they are exact and do not depend on the order of the
// additions. Parts are combined with the factors
// exp2((m_j - M) * sm_scale * log2(e)) in fp64 in a fixed order, so the selection
// is bitwise deterministic. The per-key rounding (less than one unit) and the fp32
// exponential keep the cumulative mass within about 2e-6 of the exact one (fp32
// rounding of the exponent's argument dominates for keys far below the maximum).
//
// First level. A key's bin is the step of its mass on a logarithmic grid:
// floor(S * sm_scale * log2(e) * 64), 4096 bins of 1/64 octave below the maximum
// (monotone in S, so every key of a higher bin ranks above every key of a lower
// one; 63 octaves, past which a key has no mass in these units). A bin then holds
// under 2 % of the keys of an octave: of the 131072 keys of a row about 500 are
// left to be ranked inside the crossing bin (a bin of the key's top 12 bits held
// up to 10,000), and the LDS additions spread over hundreds of bins.
//
// Rows longer than kSelRowMax: three kernels, one block per (row, part), a part
// being spb consecutive sub-chunks of 16384 keys:
//   1 hist   per part: its maximum m_j and the histogram of masses relative to
//            m_j, bins aligned on the absolute grid so that parts can be merged:
//            64 sums of 64 bins and the 64-bin sections that hold mass (plain
//            stores: no atomics outside LDS).
//   2 cand   every block of a row merges the row's records in fp64: the total
//            Z, the target T = p Z and the bin where the mass from the top
//            reaches T, with the mass still needed inside it. Then it marks its
//            part's keys above that bin in a bitmap and hands its keys inside
//            the bin (the candidates, with their positions) to the last kernel.
//            An irregular row (scores that the grid cannot hold, or more
//            candidates in a part than its buffer takes, which the part's mass
//            inside the bin bounds) gets K* here instead, by an exact three-level
//            select over all of its keys in every block: ten times the time.
//   3 final  ranks the row's candidates (masses relative to M) and so finds K*,
//            adds the part's candidates >= K* to its bitmap and expands the bitmap
//            into ascending indices at the offset given by the selected counts of
//            the parts before it. It reads no scores.
// Shorter rows: one kernel, one block per row, the scores in registers from the
// first load to the last store (sel_row_kernel).
//
// What bounds them: at 32 rows the launch, the dependent loads and the barriers;
// at hundreds of rows the instructions per key and, in passes 1 and 2, reading
// the scores (from the memory side: a kernel boundary does not leave them in the
// L2). A section that all 16 waves of a block repeat costs about 16 cycles an
// instruction, one that a single wave does about 6, so the merges and crossings
// are wave 0's. Kernel times in us, three passes or one block per row, with bins
// of 12 key bits and three passes over the scores before:
//   32 rows of 130816 keys, p = 0.95 / 0.8   7.4 + 6.7 + 7.8 / 7.8 + 7.0 + 5.8
//                          before            7.6 + 8.0 + 10.6 / 7.9 + 7.8 + 8.5
//   256 rows of 131072 keys, p = 0.95        32 + 31 + 18, before 32 + 33 + 61
//   512 rows of 2032 .. 32512 keys           27 (one block per row), before 18 + 19 + 32
// The parts of a row run on one XCD (tile_place, one row per tile group).
//
// Ragged batches (seq_n / seq_p != NULL): row r of sequence b = r / Hq has
// seq_n[b] keys (clamped to [0, n]; n stays the row stride and sizes the grid)
// and its own p = seq_p[b]. Blocks past a row's keys leave at once; rows whose
// p is >= 1 skip the first two passes, and the last pass selects every key. Where
// n calls for three passes, the rows of up to kSelRowMax keys are still selected by
// one block each, in a launch before them: a row's form, and so the rounding of its
// sums, depends on its own length only. (us a call, before / with that launch: 16
// sequences of 4K to 64K keys 71 / 65, of 33K to 63K 74 / 76; 4 of 10K to 48K 23 / 31.)
#include <algorithm>
#include <climits>
#include <cmath>
#include <type_traits>

#include "rbq_device.h"
#include "rbq_internal.h"

namespace rbq {
namespace {

typedef unsigned long long u64;
constexpr int kT = kSelThreads;
constexpr int kPT = kSelPerThread;
constexpr int kSub = kSelSub;
constexpr int kTW = kT / kWave;            // waves per block
constexpr float kFix = 1099511627776.0f;   // 2^40

// fp32 to integers as the hardware converts: towards zero and towards minus
// infinity, saturating, a NaN to 0
__device__ __forceinline__ uint32_t cvt_u32(float x) {
  uint32_t r;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}
__device__ __forceinline__ int cvt_floor(float x) {
  int r;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// softmax mass of one score in units of 2^-32 / whole relative to m (s <= m),
// truncated; every pass evaluates it with the same instructions, so the same score
// always gets the same mass. (Whole and fractional part of `whole` times the mass:
// every step but the exponential is exact. A NaN gives no mass.)
constexpr float kWhole = 256.f;         // units of 2^-40: sums of up to 2^24 keys
constexpr float kWholeFine = 65536.f;   // units of 2^-48: sums of up to 2^16
__device__ __forceinline__ u64 fixed_mass(float s, float m, float scale_log2e, float whole = kWhole) {
  const float a = __builtin_amdgcn_exp2f(__fmul_rn(__fsub_rn(s, m), scale_log2e)) * whole;
  const uint32_t lo = cvt_u32(__builtin_amdgcn_fractf(a) * 4294967296.f);
  return (u64(cvt_u32(a)) << 32) | lo;
}

// inverse of score_key (-0 comes back as +0, which has the same mass)
__device__ __forceinline__ float key_score(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// ---------------------------------------------------------------- wave and block scans
// 64-bit DPP move with a row mask (rows left out of the mask read 0)
#define RBQ_DPP_U64_M(v, ctrl, rmask)                                                                     \
  ((uint64_t(uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t((v) >> 32)), (ctrl), (rmask), 0xF, false))) \
    << 32) |                                                                                              \
   uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(v)), (ctrl), (rmask), 0xF, false)))
#define RBQ_DPP_F64_M(v, ctrl, rmask) \
  __builtin_bit_cast(double, RBQ_DPP_U64_M(__builtin_bit_cast(uint64_t, (v)), ctrl, rmask))

// inclusive prefix sums over the lanes of a wave: row shifts within rows of 16,
// then row broadcasts across them
__device__ __forceinline__ u64 wave_incl_scan_u64(u64 x) {
  x += RBQ_DPP_U64_M(x, 0x111, 0xF);   // row_shr:1
  x += RBQ_DPP_U64_M(x, 0x112, 0xF);   // row_shr:2
  x += RBQ_DPP_U64_M(x, 0x114, 0xF);   // row_shr:4
  x += RBQ_DPP_U64_M(x, 0x118, 0xF);   // row_shr:8
  x += RBQ_DPP_U64_M(x, 0x142, 0xA);   // row_bcast:15 into rows 1, 3
  x += RBQ_DPP_U64_M(x, 0x143, 0xC);   // row_bcast:31 into rows 2, 3
  return x;
}
__device__ __forceinline__ double wave_incl_scan_f64(double x) {
  x += RBQ_DPP_F64_M(x, 0x111, 0xF);
  x += RBQ_DPP_F64_M(x, 0x112, 0xF);
  x += RBQ_DPP_F64_M(x, 0x114, 0xF);
  x += RBQ_DPP_F64_M(x, 0x118, 0xF);
  x += RBQ_DPP_F64_M(x, 0x142, 0xA);
  x += RBQ_DPP_F64_M(x, 0x143, 0xC);
  return x;
}
__device__ __forceinline__ double readlane_f64(double v, int l) {
  return __builtin_bit_cast(double, readlane_u64(__builtin_bit_cast(uint64_t, v), l));
}

// Exclusive prefix of one u32 per lane over the wave, and the wave's total.
__device__ __forceinline__ uint32_t wave_excl_scan_u32(uint32_t v, uint32_t* total) {
  uint32_t x = v;
  x += RBQ_DPP_U32(x, 0x111);   // row_shr:1
  x += RBQ_DPP_U32(x, 0x112);   // row_shr:2
  x += RBQ_DPP_U32(x, 0x114);   // row_shr:4
  x += RBQ_DPP_U32(x, 0x118);   // row_shr:8: inclusive within each row of 16
  x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x142, 0xA, 0xF, false));   // row_bcast:15 into rows 1, 3
  x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x143, 0xC, 0xF, false));   // row_bcast:31 into rows 2, 3
  *total = uint32_t(__builtin_amdgcn_readlane(int(x), 63));
  return x - v;
}

struct Crossing {
  uint32_t bin;
  uint32_t ok;   // 0: the histogram holds no mass
  u64 need;
};

// Given the mass strictly above a thread's four consecutive bins (b3 the
// highest) and need within (above, above + their sum], the bin where the suffix
// sum reaches need and what is still needed inside it.
__device__ __forceinline__ void crossing_in4(int first, u64 above, u64 need, u64 b0, u64 b1, u64 b2, u64 b3,
                                             Crossing* out) {
  u64 cum = above;
  int bin = first;
  if (cum + b3 >= need) {
    bin = first + 3;
  } else {
    cum += b3;
    if (cum + b2 >= need) {
      bin = first + 2;
    } else {
      cum += b2;
      if (cum + b1 >= need) {
        bin = first + 1;
      } else {
        cum += b1;
      }
    }
  }
  out->bin = uint32_t(bin);
  out->need = need - cum;
  out->ok = 1u;
}

// a non-negative fp64 mass as u64 (rounded up), saturating
__device__ __forceinline__ u64 mass_ceil(double x) {
  return x <= 0.0 ? 0ull : x >= 1.8446744073709550e19 ? ~0ull : u64(ceil(x));
}

// Crossing search over the kSelBins u64 masses of one row in LDS (bins ordered
// by key): the highest bin b whose suffix sum (bins >= b) reaches `need` (p > 0:
// the share p of the histogram's total), and the mass still needed inside it. need is clamped into [1, total]; a
// histogram without mass gives ok = 0. All threads call it (4 bins each); the
// result is valid in *out after the trailing barrier. wsum: kTW words of LDS.
__device__ __forceinline__ void block_crossing_4096(const u64* h, u64 need, float p, u64* wsum, Crossing* out) {
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  const u64 b0 = h[4 * t], b1 = h[4 * t + 1], b2 = h[4 * t + 2], b3 = h[4 * t + 3];
  const u64 s = (b0 + b1) + (b2 + b3);
  const u64 inc = wave_incl_scan_u64(s);
  if (lane == kWave - 1) wsum[w] = inc;
  __syncthreads();
  u64 before = 0, total = 0;
#pragma unroll
  for (int v = 0; v < kTW; ++v) {
    const u64 x = wsum[v];
    before += v < w ? x : 0ull;
    total += x;
  }
  const u64 above = total - (before + inc);   // mass of the bins above this thread's four
  if (p > 0.f) need = mass_ceil(double(p) * double(total));
  need = need < 1ull ? 1ull : need > total ? total : need;
  if (total == 0) {
    if (t == 0) {
      out->bin = 0;
      out->ok = 0;
      out->need = 0;
    }
  } else if (above < need && above + s >= need) {   // exactly one thread
    crossing_in4(4 * t, above, need, b0, b1, b2, b3, out);
  }
  __syncthreads();
}

// A row's key count and p: the call's, or its sequence's in a ragged batch. A
// p outside (0, 1] is clamped into it (<= 0 or NaN: the smallest positive p,
// which keeps the top key and its ties).
struct RowSel {
  int n;
  float p;
};
__device__ __forceinline__ RowSel row_sel(const int32_t* __restrict__ seq_n, const float* __restrict__ seq_p, int hq,
                                          int row, int n, float p) {
  RowSel r{n, p};
  const int b = row / hq;
  if (seq_n) r.n = min(max(seq_n[b], 0), n);
  if (seq_p) {
    const float v = seq_p[b];
    r.p = v > 0.f ? fminf(v, 1.f) : 1e-30f;
  }
  return r;
}

// The (row, part) of this block: tile (KV group, part), the group's rows in
// the tile's consecutive slots (group = rows per KV group, 1 when unknown).
struct SelWork {
  int row, part;
  bool ok;
};
__device__ __forceinline__ SelWork sel_work(const TilePlace& tp, int group) {
  int g, j, s;
  SelWork w;
  w.ok = tile_of(tp, group, int(blockIdx.x), g, j, s);
  w.row = g * group + s;
  w.part = j;
  return w;
}

// The keys of a sub-chunk at `base`: wave w holds the 64 kPT keys from
// base + 64 kPT w on, step k of it 64 consecutive ones (one ballot is one word
// of the row's selection bitmap, and a wave's words are consecutive).
template <int PT>
__device__ __forceinline__ int key_at(int base, int k) {
  return base + int(threadIdx.x / kWave) * (kWave * PT) + k * kWave + lane_id();
}
// the thread's PT scores, all loads in flight; past `end` the last key again (the values are masked)
template <int PT>
__device__ __forceinline__ void load_keys(const float* __restrict__ s, int base, int end, float* v) {
  if (base + kT * PT <= end) {   // block-uniform: one address for all of them
    const float* p = s + key_at<PT>(base, 0);
#pragma unroll
    for (int k = 0; k < PT; ++k) v[k] = p[k * kWave];
  } else {
#pragma unroll
    for (int k = 0; k < PT; ++k) v[k] = s[min(key_at<PT>(base, k), end - 1)];
  }
}

// ballot straight from a comparison
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Lanes K .. K + 3 of (lo, hi) become the wave-uniform words w[0 .. 3]. The
// wait states come first because the words are usually ballots: gfx950 needs
// two between a vector instruction that writes a scalar register and one that
// reads it, and the compiler does not look into the asm to place them.
template <int K>
__device__ __forceinline__ void words_to_lanes(const uint64_t* w, uint32_t& lo, uint32_t& hi) {
  asm volatile(
      "s_nop 1\n\t"
      "v_writelane_b32 %0, %2, %10\n\tv_writelane_b32 %1, %3, %10\n\t"
      "v_writelane_b32 %0, %4, %11\n\tv_writelane_b32 %1, %5, %11\n\t"
      "v_writelane_b32 %0, %6, %12\n\tv_writelane_b32 %1, %7, %12\n\t"
      "v_writelane_b32 %0, %8, %13\n\tv_writelane_b32 %1, %9, %13"
      : "+v"(lo), "+v"(hi)
      : "s"(uint32_t(w[0])), "s"(uint32_t(w[0] >> 32)), "s"(uint32_t(w[1])), "s"(uint32_t(w[1] >> 32)),
        "s"(uint32_t(w[2])), "s"(uint32_t(w[2] >> 32)), "s"(uint32_t(w[3])), "s"(uint32_t(w[3] >> 32)), "n"(K),
        "n"(K + 1), "n"(K + 2), "n"(K + 3));
}
// body(K) for the compile-time steps K = 0, 4, 8, .. below `steps` (a multiple of four, <= PT)
template <int PT, int K = 0, class F>
__device__ __forceinline__ void for_groups(int steps, F& body) {
  if constexpr (K < PT) {
    if (K < steps) {   // block-uniform
      body(std::integral_constant<int, K>{});
      for_groups<PT, K + 4>(steps, body);
    }
  }
}
// set bits of a wave-uniform word below this lane
__device__ __forceinline__ int bits_below(uint64_t w) {
  return int(__builtin_amdgcn_mbcnt_hi(uint32_t(w >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(w), 0u)));
}

// The words that lanes 0 .. 31 of a wave hold in (lo, hi), one 32-bit half per
// lane: lane 2 k + s gets half s of lane k's word.
__device__ __forceinline__ uint32_t half_words(uint32_t lo, uint32_t hi) {
  const int src = lane_id() >> 1;
  const uint32_t a = uint32_t(__shfl(int(lo), src, kWave)), b = uint32_t(__shfl(int(hi), src, kWave));
  return (lane_id() & 1) ? b : a;
}
// the low `left` bits of a 32-bit word (none for left <= 0)
__device__ __forceinline__ uint32_t low_bits(int left) { return left >= 32 ? ~0u : left > 0 ? (1u << left) - 1u : 0u; }

// The smallest score whose key is K, for comparing scores instead of keys:
// exact (S >= value <=> key(S) >= K) unless it is a NaN pattern.
__device__ __forceinline__ float key_floor(uint32_t K) { return key_score(K); }

// ---------------------------------------------------------------- the logarithmic grid
// The bin of a score: floor(S * c), c = sm_scale * log2(e) * 64. Bins are
// integers below 2^30, in fp32 (where every value from 2^23 on is one) or int.
__device__ __forceinline__ int grid_bin(float s, float c) { return cvt_floor(__fmul_rn(s, c)); }
// The window of kSelBins bins below a maximum: `top` is the absolute index of
// the group of 64 bins that holds it, the window the 64 groups up to it. It
// reaches 63 octaves down, where a key has no mass left in these units (and so
// has every key that the window leaves out).
struct GridWindow {
  int top, base;   // group of the maximum; first bin of the window
  bool ok;         // the grid can hold this maximum (false for a NaN or an infinity)
};
__device__ __forceinline__ GridWindow grid_window(float m, float c) {
  GridWindow g;
  g.ok = fabsf(__fmul_rn(m, c)) < 1073741824.f;
  g.top = g.ok ? grid_bin(m, c) >> 6 : 0;
  g.base = g.ok ? (g.top - (kSelCoarse - 1)) * kSelFine : INT_MAX;   // (not ok: the histogram is not used)
  return g;
}
// One key's mass into the histogram.
__device__ __forceinline__ void grid_add(u64* h, float s, float m, float scale_log2e, float c, int base,
                                         float whole = kWhole) {
  // (64-bit integer LDS atomics: under the contention of a few popular bins
  // they run several times faster than fp32 ones)
  const u64 e = fixed_mass(s, m, scale_log2e, whole);
  const uint32_t d = uint32_t(grid_bin(s, c)) - uint32_t(base);
  if (d < uint32_t(kSelBins)) atomicAdd(&h[d], e);
}

// per-row state written by pass 2 (part 0) for pass 3
struct RowState {
  float M;          // row maximum
  int bin;          // the crossing bin
  double need;      // mass still needed inside it (2^-40 units relative to M)
  uint32_t exact;   // an irregular row: the marked keys are final and K* is
  uint32_t kstar;   // this
  double pad;
};
static_assert(sizeof(RowState) == kSelStateWords * 4, "state words per row");

// ---------------------------------------------------------------- pass 1: part histograms
// per-part record of pass 1 (at the start of its kSelPart1Bytes slot)
struct P1Head {
  float m;          // the part's maximum
  int top;          // its GridWindow::top
  uint32_t ok;      // its GridWindow::ok
};

template <bool RAGGED, bool MULTI>
__global__ __launch_bounds__(kT, 8) void sel_hist_kernel(const float* __restrict__ scores, int n, int spb, TilePlace tp,
                                                      int group, float scale_log2e,
                                                      unsigned char* __restrict__ part1,
                                                      const int32_t* __restrict__ seq_n,
                                                      const float* __restrict__ seq_p, int hq) {
  __shared__ u64 h[kSelBins];
  __shared__ float red[kTW];
  const SelWork wk = sel_work(tp, group);
  if (!wk.ok) return;
  const int parts = tp.parts;
  const RowSel rs = RAGGED ? row_sel(seq_n, seq_p, hq, wk.row, n, 0.5f) : RowSel{n, 0.5f};
  const int k0 = wk.part * spb * kSub;
  if (k0 >= rs.n || (RAGGED && (rs.n <= kSelRowMax || rs.p >= 1.f))) return;   // block-uniform: no histogram needed
  const int k1 = min(rs.n, k0 + spb * kSub);
  const float* srow = scores + int64_t(wk.row) * n;
  const int t = threadIdx.x;
  const float c = scale_log2e * kSelPerOctave;
  float v[kPT];
  load_keys<kPT>(srow, k0, k1, v);
#pragma unroll
  for (int k = 0; k < kSelBins / kT; ++k) h[k * kT + t] = 0ull;
  // the part's maximum
  float m = -INFINITY;
  for (int base = k0; base < k1; base += kSub) {
    if (MULTI && base > k0) load_keys<kPT>(srow, base, k1, v);
#pragma unroll
    for (int k = 0; k < kPT; ++k) m = fmaxf(m, v[k]);   // (lanes past k1 hold the last key again)
    if (!MULTI) break;
  }
  m = wave_max_dpp(m);
  if (lane_id() == 0) red[t / kWave] = m;
  __syncthreads();   // (also orders the clearing of h before the adds)
#pragma unroll
  for (int w = 0; w < kTW; ++w) m = fmaxf(m, red[w]);
  const GridWindow g = grid_window(m, c);
  for (int base = k0; base < k1; base += kSub) {
    if (MULTI) load_keys<kPT>(srow, base, k1, v);   // (read again: from L2)
    if (base + kSub <= k1) {
#pragma unroll
      for (int k = 0; k < kPT; ++k) grid_add(h, v[k], m, scale_log2e, c, g.base);
    } else {
#pragma unroll
      for (int k = 0; k < kPT; ++k)
        if (key_at<kPT>(base, k) < k1) grid_add(h, v[k], m, scale_log2e, c, g.base);
    }
    if (!MULTI) break;
  }
  __syncthreads();
  // the sums of 64 bins: 4 bins per thread, a 16-lane row per sum
  const u64 b0 = h[4 * t], b1 = h[4 * t + 1], b2 = h[4 * t + 2], b3 = h[4 * t + 3];
  u64 s4 = (b0 + b1) + (b2 + b3);
  s4 += RBQ_DPP_U64(s4, 0xB1);    // quad_perm [1,0,3,2]
  s4 += RBQ_DPP_U64(s4, 0x4E);    // quad_perm [2,3,0,1]
  s4 += RBQ_DPP_U64(s4, 0x141);   // row_half_mirror
  s4 += RBQ_DPP_U64(s4, 0x140);   // row_mirror
  unsigned char* P1 = part1 + (int64_t(wk.row) * parts + wk.part) * kSelPart1Bytes;
  if ((t & 15) == 0) reinterpret_cast<u64*>(P1 + kSelP1Coarse)[t >> 4] = s4;
  if (s4) {   // (sections without mass are not written and never read)
    u32x4* dst = reinterpret_cast<u32x4*>(P1 + kSelP1Sec + size_t(8) * (4 * t));
    dst[0] = u32x4{uint32_t(b0), uint32_t(b0 >> 32), uint32_t(b1), uint32_t(b1 >> 32)};
    dst[1] = u32x4{uint32_t(b2), uint32_t(b2 >> 32), uint32_t(b3), uint32_t(b3 >> 32)};
  }
  if (t == 0) *reinterpret_cast<P1Head*>(P1) = P1Head{m, g.top, g.ok};
}

// ---------------------------------------------------------------- pass 2: candidates
// per-part record of pass 2 (at the start of its kSelPart2Bytes slot), followed
// at kSelP2Cand by the candidates {key, index in the row}
struct P2Head {
  uint32_t above_cnt;   // keys above the crossing bin
  uint32_t cand_cnt;    // keys inside it (only the first cand_cap are stored)
};
// Where pass 2 leaves the bitmap of a part's keys above the crossing bin: the
// caller's selection bitmap, which pass 3 completes; without one, the end of the
// part's candidate room, as long as that leaves half of it (kOwnMapMax
// sub-chunks); otherwise nowhere, and pass 3 compares the scores with K*. The room
// for candidates is the same with and without the caller's bitmap, so that the
// fused step and the separate call settle the same rows by the exact select.
constexpr int kMapWords = kSub / kWave;   // words of a sub-chunk
constexpr int kOwnMapMax = 4;
struct MapPlan {
  u64* masks;        // the caller's [rows][words], or NULL
  int words;
  int cand_cap;      // candidates a part stores
  bool own;          // the part's own bitmap follows its candidates
};
inline MapPlan map_plan(u64* masks, int words, int spb) {
  const bool room = spb <= kOwnMapMax;
  return MapPlan{masks, words, room ? kSelCandCap - kMapWords * spb : kSelCandCap, room && masks == nullptr};
}
__device__ __forceinline__ u64* part_map(const MapPlan& mp, unsigned char* P2, int row, int k0) {
  if (mp.masks) return mp.masks + int64_t(row) * mp.words + k0 / kWave;
  return mp.own ? reinterpret_cast<u64*>(P2 + kSelP2Cand) + mp.cand_cap : nullptr;
}

// The products S * c of the keys inside the crossing bin are those in [lo, hi):
// fp32 holds halves up to 2^23 in magnitude (the bin of -2^23 has -2^23 + 1/2, too)
// and integers only, or less, from there on.
struct BinEdges {
  float lo, hi;
};
__device__ __forceinline__ BinEdges bin_edges(int bin) {
  BinEdges e;
  e.lo = float(bin);
  e.hi = bin >= -8388608 && bin < 8388608 ? e.lo + 1.f : __uint_as_float(__float_as_uint(e.lo) + (bin > 0 ? 1 : -1));
  return e;
}
// Four steps' keys against the crossing bin: lanes K .. K + 3 of `above` and
// `mid` get the words of the keys above it and inside it (NaN: neither).
struct LaneWords {
  uint32_t lo, hi;
};
template <int K>
__device__ __forceinline__ void classify4(const float* v, const BinEdges& e, float c, LaneWords& above, LaneWords& mid) {
  uint64_t a[4], m[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const float x = __fmul_rn(v[u], c);
    a[u] = ballot(x >= e.hi);
    m[u] = ballot(x >= e.lo) & ~a[u];
  }
  words_to_lanes<K>(a, above.lo, above.hi);
  words_to_lanes<K>(m, mid.lo, mid.hi);
}

// Exact three-level select over every key of an irregular row, masses relative to M: K*.
__device__ __forceinline__ uint32_t exact_select_row(const float* __restrict__ srow, int nr, float M,
                                                     float scale_log2e, float p, u64* h, u64* wsum, Crossing* cr) {
  const int t = threadIdx.x;
  uint32_t prefix = 0;
  u64 need = 0;
  // levels: bits 31..20 (all keys), 19..8 (keys in the first bin), 7..0 (keys in both)
#pragma unroll 1
  for (int level = 0; level < 3; ++level) {
    const int shift = level == 0 ? 20 : level == 1 ? 8 : 0;
    const uint32_t mask = level == 2 ? 0xffu : 0xfffu;
    const int hshift = level == 0 ? 32 : level == 1 ? 20 : 8;   // bits that must match the prefix
    for (int b = t; b < kSelBins; b += kT) h[b] = 0;
    __syncthreads();
#pragma unroll 1
    for (int base = 0; base < nr; base += kSub) {
      float v[kPT];
      load_keys<kPT>(srow, base, nr, v);
#pragma unroll
      for (int k = 0; k < kPT; ++k) {
        const uint32_t key = score_key(v[k]);
        const bool match = hshift == 32 || (key >> hshift) == prefix;
        if (key_at<kPT>(base, k) < nr && match) {
          const u64 e = fixed_mass(v[k], M, scale_log2e);
          if (e) atomicAdd(&h[(key >> shift) & mask], e);
        }
      }
    }
    __syncthreads();
    block_crossing_4096(h, need, level == 0 ? p : 0.f, wsum, cr);
    const uint32_t bin = cr->ok ? cr->bin : 0u;   // (no mass left: the lowest bin, every key of the prefix)
    prefix = (prefix << (level == 2 ? 8 : 12)) | bin;
    need = cr->need;
    __syncthreads();   // every thread has read *cr
  }
  return prefix;
}

// ballots of a sub-chunk's keys >= K* (by value: scores >= the smallest score of key K*)
template <int PT>
__device__ __forceinline__ void select_ballots(const float* v, int base, int end, uint32_t kstar, uint64_t* bal) {
  const float fstar = key_floor(kstar);   // (NaN for K* = 0: every key, by keys)
  if (!__builtin_isnan(fstar)) {          // (block-uniform)
#pragma unroll
    for (int k = 0; k < PT; ++k) bal[k] = ballot(v[k] >= fstar) & ballot(key_at<PT>(base, k) < end);
  } else {
#pragma unroll
    for (int k = 0; k < PT; ++k) bal[k] = ballot(score_key(v[k]) >= kstar) & ballot(key_at<PT>(base, k) < end);
  }
}

// (Two blocks per CU need 8 waves per SIMD, for which four scalar registers, and in the
// ragged form one vector register, are kept in scratch; with those in registers one
// block fits, and 256 rows of 131072 keys take 97 us for 84.)
template <bool RAGGED, bool MULTI>
__global__ __launch_bounds__(kT, 8) void sel_cand_kernel(const float* __restrict__ scores, int n, int spb, TilePlace tp,
                                                      int group, float p, float scale_log2e,
                                                      const unsigned char* __restrict__ part1,
                                                      unsigned char* __restrict__ part2, uint32_t* __restrict__ state,
                                                      MapPlan mp, const int32_t* __restrict__ seq_n,
                                                      const float* __restrict__ seq_p, int hq) {
  // the parts' group sums, then their bins of the crossing group (or an exact select's histogram)
  __shared__ double val_s[kSelMaxParts][kSelCoarse];
  __shared__ int shift_s[kSelMaxParts];   // groups from the part's maximum up to the row's
  __shared__ uint32_t cnt_s[kTW];
  __shared__ uint32_t cand_n;
  __shared__ u64 wsum[kTW];
  __shared__ Crossing cr;
  __shared__ int i1_s, bin_s;             // the crossing group's place in the row's window, the crossing bin
  __shared__ bool exact_s;
  const SelWork wk = sel_work(tp, group);
  if (!wk.ok) return;
  const int parts = tp.parts;
  const RowSel rs = RAGGED ? row_sel(seq_n, seq_p, hq, wk.row, n, p) : RowSel{n, p};
  const int k0 = wk.part * spb * kSub;
  if (k0 >= rs.n || (RAGGED && (rs.n <= kSelRowMax || rs.p >= 1.f))) return;   // block-uniform
  const int k1 = min(rs.n, k0 + spb * kSub);
  const int parts_r = (rs.n + spb * kSub - 1) / (spb * kSub);   // parts holding keys of this row
  const float* srow = scores + int64_t(wk.row) * n;
  const int t = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const float c = scale_log2e * kSelPerOctave;
  const unsigned char* P1row = part1 + int64_t(wk.row) * parts * kSelPart1Bytes;
  auto P1 = [&](int j) { return P1row + int64_t(j) * kSelPart1Bytes; };
  // The merge: a wave loads parts wave, wave + kTW, ..; wave 0 adds them up (a
  // step that all 16 waves repeat costs 16 cycles, one that wave 0 does about 6).
  P1Head hl{};
  if (wave == 0) hl = *reinterpret_cast<const P1Head*>(P1(min(lane, parts_r - 1)));   // lane j: part j
  u64 g0 = 0ull;   // this wave's first part's group sum `lane`
  if (wave < parts_r) g0 = reinterpret_cast<const u64*>(P1(wave) + kSelP1Coarse)[lane];
  float v[kPT];
  load_keys<kPT>(srow, k0, k1, v);   // lands during the merge
  if (t == 0) cand_n = 0;
  for (int j = wave; j < parts_r; j += kTW)
    val_s[j][lane] = double(j == wave ? g0 : reinterpret_cast<const u64*>(P1(j) + kSelP1Coarse)[lane]);
  // (wave 0) the row maximum, the parts' factors and shifts against it
  float M = -INFINITY;
  double fac = 0.0, need1 = 0.0, need = 0.0;
  int top = 0, l1 = 0, shift = kSelCoarse;
  bool bad = false;
  if (wave == 0) {
    const bool in = lane < parts_r;
    M = wave_max_dpp(in ? hl.m : -INFINITY);
    fac = in ? exp2((double(hl.m) - double(M)) * double(scale_log2e)) : 0.0;
    const bool ok = in && hl.ok;
    top = wave_max_i32(ok ? hl.top : INT_MIN / 2);   // the row's window: the 64 groups up to here
    shift = ok ? min(top - hl.top, kSelCoarse) : kSelCoarse;
    shift_s[lane] = shift;
    // (the grid misses a part that counts: its maximum is out of the grid's
    // range, or infinite, which makes the factor a NaN)
    bad = ballot(in && !ok && !(fac == 0.0)) != 0ull;
  }
  __syncthreads();
  if (wave == 0) {
    // Level 1: group i of the row's window (i = 63 on top) is group i + shift of
    // a part's. Lane l holds group 63 - l, so the prefix sums over the lanes are
    // the masses from the top down to each group.
    double C = 0.0;
    for (int j = 0; j < parts_r; ++j) {   // in part order
      const int i = kSelCoarse - 1 - lane + __builtin_amdgcn_readlane(shift, j);
      const double x = val_s[j][min(i, kSelCoarse - 1)];
      C += (i < kSelCoarse ? x : 0.0) * readlane_f64(fac, j);
    }
    const double x1 = wave_incl_scan_f64(C);
    const double T = double(rs.p) * readlane_f64(x1, kWave - 1);
    const u64 hit = ballot(x1 >= T);   // (lane 63 holds the total, >= T)
    const bool found = hit != 0ull && !bad && T > 0.0;   // (otherwise an irregular row)
    l1 = found ? __builtin_ctzll(hit) : 0;
    need1 = T - (l1 > 0 ? readlane_f64(x1, l1 - 1) : 0.0);
    if (lane == 0) {
      i1_s = kSelCoarse - 1 - l1;
      exact_s = !found;
    }
  }
  __syncthreads();
  bool exact = exact_s;
  if (!exact) {   // block-uniform
    // Level 2: the crossing group's 64 bins
    const int i1 = i1_s;
    for (int j = wave; j < parts_r; j += kTW) {
      const int ij = i1 + shift_s[j];
      u64 x = 0ull;
      // (a section without mass was not written: its group sum tells)
      if (ij < kSelCoarse && val_s[j][ij] > 0.0)
        x = reinterpret_cast<const u64*>(P1(j) + kSelP1Sec)[ij * kSelFine + lane];
      val_s[j][lane] = double(x);
    }
    __syncthreads();
    if (wave == 0) {
      double F = 0.0;
      for (int j = 0; j < parts_r; ++j) F += val_s[j][kSelFine - 1 - lane] * readlane_f64(fac, j);
      const double x2 = wave_incl_scan_f64(F);
      const u64 hit = ballot(x2 >= need1);
      int l2;
      if (hit) {
        l2 = __builtin_ctzll(hit);
      } else {   // (the sums fell short of need1 by rounding: the lowest bin with mass)
        const u64 nzb = ballot(F > 0.0);
        l2 = nzb ? 63 - __builtin_clzll(nzb) : kWave - 1;
      }
      need = need1 - (l2 > 0 ? readlane_f64(x2, l2 - 1) : 0.0);
      const int bin = (top - l1) * kSelFine + kSelFine - 1 - l2;
      // At most how many keys a part has inside the bin: its mass there over the
      // least mass of one key there (the product S * c is off by up to 2^-24 of
      // itself, the mass by far less than 1e-3 octaves, its truncation by one unit
      // of the part that shrinks a unit most). Every block of the row comes to the
      // same answer for all parts (lane j: part j), so all of them know that the
      // candidates fit. (The row's mass against one part's room sent ordinary rows
      // of a million keys to the exact select: 8 rows of 1048576 normal scores,
      // sigma 1.5 nats, p = 0.95, 604 us; now 42.)
      const float slack = float(abs(bin)) * 0x1p-22f + 0.1f;
      const float x0 = float(double(bin) - double(M) * double(c)) - slack;
      const float least = __builtin_amdgcn_exp2f(x0 * (1.f / kSelPerOctave)) * kFix - 1.f;
      const double mass = lane < parts_r ? val_s[lane][kSelFine - 1 - l2] * fac : 0.0;
      const bool fits = ballot(lane < parts_r && !(mass < double(least) * double(mp.cand_cap))) == 0ull;
      if (lane == 0) {
        bin_s = bin;
        exact_s = !fits;
      }
    }
    __syncthreads();
    exact = exact_s;
  }
  unsigned char* P2 = part2 + (int64_t(wk.row) * parts + wk.part) * kSelPart2Bytes;
  u64* map = part_map(mp, P2, wk.row, k0);
  if (exact) {   // block-uniform: an irregular row, K* from all of its keys
    if (t == 0) wsum[0] = __float_as_uint(M);
    __syncthreads();   // (every wave is done with val_s, too)
    M = __uint_as_float(uint32_t(wsum[0]));
    const uint32_t kstar =
        exact_select_row(srow, rs.n, M, scale_log2e, rs.p, reinterpret_cast<u64*>(&val_s[0][0]), wsum, &cr);
    uint32_t ac = 0;
    for (int base = k0; base < k1; base += kSub) {
      uint64_t bal[kPT];
      load_keys<kPT>(srow, base, k1, v);
      select_ballots<kPT>(v, base, k1, kstar, bal);
      uint32_t lo = 0u, hi = 0u;
      auto put = [&](auto k) { words_to_lanes<k>(bal + k, lo, hi); };
      for_groups<kPT>(kPT, put);
      const u64 w = lane < kPT ? (u64(hi) << 32) | lo : 0ull;
      if (map && lane < kPT) map[(base - k0) / kWave + wave * kPT + lane] = w;
      ac += uint32_t(__popcll(w));
    }
    ac = uint32_t(wave_sum_i32(int(ac)));
    if (lane == 0) cnt_s[wave] = ac;
    __syncthreads();
    if (t == 0) {
      uint32_t a = 0;
#pragma unroll
      for (int w = 0; w < kTW; ++w) a += cnt_s[w];
      *reinterpret_cast<P2Head*>(P2) = P2Head{a, 0u};
      if (wk.part == 0)
        *reinterpret_cast<RowState*>(state + int64_t(wk.row) * kSelStateWords) =
            RowState{M, 0, 0.0, 1u, kstar, 0.0};
    }
    return;
  }
  // The keys above the bin into the bitmap, those inside it into the candidate
  // list: lane l holds the 32-bit word of keys 32 l .. of its wave's 1024, and
  // goes through the few candidates in it (whose scores are in the cache).
  const BinEdges be = bin_edges(bin_s);
  u32x2* cand = reinterpret_cast<u32x2*>(P2 + kSelP2Cand);
  uint32_t ac = 0;   // this lane's words' keys above the bin
  for (int base = k0; base < k1; base += kSub) {
    if (MULTI && base > k0) load_keys<kPT>(srow, base, k1, v);
    LaneWords lw{0u, 0u}, lm{0u, 0u};
    auto step4 = [&](auto k) { classify4<k>(v + k, be, c, lw, lm); };
    for_groups<kPT>(kPT, step4);
    const int first = base + wave * (kPT * kWave) + 32 * lane;   // of this lane's word (lanes 0 .. 31)
    const uint32_t in = lane < 2 * kPT ? low_bits(k1 - first) : 0u;
    const uint32_t above = half_words(lw.lo, lw.hi) & in;
    uint32_t mid = half_words(lm.lo, lm.hi) & in;
    ac += uint32_t(__popc(above));
    uint32_t wcnt;
    uint32_t pos = wave_excl_scan_u32(uint32_t(__popc(mid)), &wcnt);
    if (wcnt) {   // wave-uniform: one reservation per wave
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(&cand_n, wcnt);
      pos += uint32_t(__builtin_amdgcn_readfirstlane(int(at)));
      for (; mid; mid &= mid - 1u, ++pos) {
        const int i = first + __builtin_ctz(mid);
        if (pos < uint32_t(mp.cand_cap)) cand[pos] = u32x2{score_key(srow[i]), uint32_t(i)};
      }
    }
    if (map && lane < 2 * kPT) reinterpret_cast<uint32_t*>(map)[(first - k0) / 32] = above;
    if (!MULTI) break;
  }
  ac = uint32_t(wave_sum_i32(int(ac)));
  if (lane == 0) cnt_s[wave] = ac;
  __syncthreads();   // (also completes the candidate count)
  if (wave == 0) {
    const uint32_t a = uint32_t(wave_sum_i32(lane < kTW ? int(cnt_s[lane]) : 0));
    if (t == 0) {
      *reinterpret_cast<P2Head*>(P2) = P2Head{a, min(cand_n, uint32_t(mp.cand_cap))};
      if (wk.part == 0)
        *reinterpret_cast<RowState*>(state + int64_t(wk.row) * kSelStateWords) =
            RowState{M, bin_s, need, 0u, 0u, 0.0};
    }
  }
}

// ---------------------------------------------------------------- ranking the candidates
// K* among the candidate keys (at least one): the largest key whose mass at or
// above (masses relative to M, need in the same units) reaches need; 0 when none
// does (every candidate is selected). All kThr threads call it; keys(body) calls
// body(key) for this thread's share of the candidates. The candidates fall
// into 256 sub-bins of the crossing bin, wave 0 finds the sub-bin where the mass
// reaches need, and the few keys inside that one are compared in pairs; where it
// holds more than 64 (ties, or a bin that is one fp32 value) the step repeats on
// 256 steps of the range of their keys.
// rank_clear comes before the barrier that publishes the keys.
constexpr int kSubBins = 256, kPairMax = kWave;
struct RankLds {
  u64 h[kSubBins];
  uint32_t rest[kPairMax];
  Crossing cr;
  uint32_t cnt, kmin, kmax, kstar;
};
template <int kThr>
__device__ __forceinline__ void rank_clear(RankLds& L) {
  for (int b = threadIdx.x; b < kSubBins; b += kThr) L.h[b] = 0ull;
  if (threadIdx.x == 0) {
    L.cnt = 0u;
    L.kmin = 0xffffffffu;
    L.kmax = 0u;
  }
}
template <int kThr, class Keys>
__device__ __forceinline__ uint32_t rank_candidates(const Keys& keys, u64 need, float M, float scale_log2e, float c,
                                                    int bin, RankLds& L, float whole = kWhole) {
  const int t = threadIdx.x, lane = lane_id();
  need = need < 1ull ? 1ull : need;
  uint32_t lo = 0u, hi = 0xffffffffu;   // the open keys
  int shift = -1;                       // -1: sub-bins of the bin; otherwise 2^shift keys per step
#pragma unroll 1
  for (;;) {   // at most five rounds
    auto slot = [&](uint32_t key) {
      if (shift >= 0) return int((key - lo) >> shift);
      return min(max(int((__fmul_rn(key_score(key), c) - float(bin)) * float(kSubBins)), 0), kSubBins - 1);
    };
    keys([&](uint32_t key) {
      if (key >= lo && key <= hi) {
        const u64 e = fixed_mass(key_score(key), M, scale_log2e, whole);
        if (e) atomicAdd(&L.h[slot(key)], e);
      }
    });
    __syncthreads();
    if (t < kWave) {
      const u64 b0 = L.h[4 * t], b1 = L.h[4 * t + 1], b2 = L.h[4 * t + 2], b3 = L.h[4 * t + 3];
      const u64 s = (b0 + b1) + (b2 + b3);
      const u64 inc = wave_incl_scan_u64(s);
      const u64 total = readlane_u64(inc, kWave - 1);
      const u64 nd = need > total ? total : need;
      const u64 above = total - inc;
      if (total == 0) {
        if (t == 0) L.cr.ok = 0u;
      } else if (above < nd && above + s >= nd) {   // one lane
        crossing_in4(4 * t, above, nd, b0, b1, b2, b3, &L.cr);
      }
    }
    __syncthreads();
    if (!L.cr.ok) return 0u;   // block-uniform: no candidate has mass
    const int cs = int(L.cr.bin);
    need = L.cr.need;
    // (counted up to one more than fit, or ties would queue for the counter)
    uint32_t mn = 0xffffffffu, mx = 0u;
    keys([&](uint32_t key) {
      if (key >= lo && key <= hi && slot(key) == cs) {
        mn = min(mn, key);
        mx = max(mx, key);
        if (__hip_atomic_load(&L.cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <= uint32_t(kPairMax)) {
          const uint32_t pos = atomicAdd(&L.cnt, 1u);
          if (pos < uint32_t(kPairMax)) L.rest[pos] = key;
        }
      }
    });
    __syncthreads();
    const int r = int(L.cnt);
    if (r <= kPairMax) {   // block-uniform
      if (t < kWave) {
        const uint32_t key = lane < r ? L.rest[lane] : 0u;
        const u64 e = lane < r ? fixed_mass(key_score(key), M, scale_log2e, whole) : 0ull;
        u64 sum = 0;
        for (int i = 0; i < r; ++i)
          sum += uint32_t(__builtin_amdgcn_readlane(int(key), i)) >= key ? readlane_u64(e, i) : 0ull;
        const uint32_t best = wave_max_u32(lane < r && sum >= need ? key : 0u);
        if (t == 0) L.kstar = best;
      }
      __syncthreads();
      return L.kstar;
    }
    mn = ~wave_max_u32(~mn);
    mx = wave_max_u32(mx);
    if (lane == 0 && mn <= mx) {   // (a wave with a key there)
      atomicMin(&L.kmin, mn);
      atomicMax(&L.kmax, mx);
    }
    __syncthreads();
    lo = L.kmin;
    hi = L.kmax;
    if (lo == hi) return lo;   // block-uniform: all of them tie
    const int bits = 32 - __clz(hi - lo);
    shift = bits > 8 ? bits - 8 : 0;
    __syncthreads();   // every thread has read L
    rank_clear<kThr>(L);
    __syncthreads();
  }
}

// This lane's set bits, lowest first, as positions first + bit into dst[0 ..]: the
// lanes of a wave go through their 32-bit words side by side.
__device__ __forceinline__ void stage_bits(uint32_t bits, int first, uint16_t* dst) {
  while (bits) {
    *dst++ = uint16_t(first + __builtin_ctz(bits));
    bits &= bits - 1u;
  }
}

// ---------------------------------------------------------------- pass 3: resolve K* and write
// Half the threads of the other passes: a block has only the row's candidates
// and its part's 256 bitmap words per sub-chunk to go through, and the row's
// blocks wait mostly on the one round of loads at the start.
constexpr int kFT = 512, kFW = kFT / kWave;
constexpr int kFPT = kSub / kFT;   // 64-key steps per wave and sub-chunk
static_assert(kFPT * 2 == kWave, "a lane per 32-bit word of a wave's keys");

template <bool RAGGED, bool MULTI>
__global__ __launch_bounds__(kFT) void sel_final_kernel(const float* __restrict__ scores, int n, int spb, TilePlace tp,
                                                        int group, float p, float scale_log2e, unsigned char* part2,
                                                        const uint32_t* __restrict__ state,
                                                        int32_t* __restrict__ sel_idx,
                                                        int32_t* __restrict__ sel_count, MapPlan mp,
                                                        const int32_t* __restrict__ seq_n,
                                                        const float* __restrict__ seq_p, int hq) {
  // the row's candidate keys, part by part; then the selected positions of a sub-chunk
  __shared__ uint32_t ck[kSelCandLds];
  __shared__ int32_t ci[kSelCandCap];        // this part's candidates' indices
  __shared__ uint32_t word_s[2 * kMapWords]; // the sub-chunk's bitmap
  __shared__ RankLds rank;
  __shared__ uint32_t before_s, sel_s;
  __shared__ int wave_cnt[kFW];
  const SelWork wk = sel_work(tp, group);
  if (!wk.ok) return;
  const int parts = tp.parts;
  const RowSel rs = RAGGED ? row_sel(seq_n, seq_p, hq, wk.row, n, p) : RowSel{n, p};
  const int k0 = wk.part * spb * kSub;
  if (k0 >= rs.n || (RAGGED && rs.n <= kSelRowMax)) return;   // block-uniform: no key of this row here
  const int k1 = min(rs.n, k0 + spb * kSub);
  const int span = spb * kSub;
  const int parts_r = (rs.n + span - 1) / span;
  const int t = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const float* srow = scores + int64_t(wk.row) * n;
  unsigned char* P2row = part2 + int64_t(wk.row) * parts * kSelPart2Bytes;
  // the bitmap as 32-bit words: thread t owns word t of a sub-chunk, positions 32 t .. 32 t + 31
  uint32_t* map =
      reinterpret_cast<uint32_t*>(part_map(mp, P2row + int64_t(wk.part) * kSelPart2Bytes, wk.row, k0));
  const bool all = RAGGED && rs.p >= 1.f;   // every key of the row (the first two passes skipped it)
  uint32_t kstar = 0u;                      // keys >= kstar are selected (every key is >= 0)
  int offset = k0, total_sel = rs.n, own_n = 0;
  uint32_t next = 0u;                       // this thread's word of the coming sub-chunk
  if (!all) {
    // one round of loads: the bitmap word, the row's state and heads in every
    // wave, the first 64 candidates of the wave's first part (whatever their number)
    if (map) next = map[t];
    const RowState rst = *reinterpret_cast<const RowState*>(state + int64_t(wk.row) * kSelStateWords);
    const P2Head hl = *reinterpret_cast<const P2Head*>(P2row + int64_t(min(lane, parts_r - 1)) * kSelPart2Bytes);
    const u32x2 pre = reinterpret_cast<const u32x2*>(P2row + int64_t(min(wave, parts_r - 1)) * kSelPart2Bytes +
                                                     kSelP2Cand)[lane];
    rank_clear<kFT>(rank);
    if (t == 0) before_s = sel_s = 0u;
    const P2Head hd = lane < parts_r ? hl : P2Head{0u, 0u};
    uint32_t ncand, nabove;
    const uint32_t cb = wave_excl_scan_u32(hd.cand_cnt, &ncand);
    const uint32_t ab = wave_excl_scan_u32(hd.above_cnt, &nabove);
    const int C = int(ncand);
    // More candidates than the LDS holds (a million keys, or scores within a few
    // hundredths of a nat): gone through where pass 2 left them, in the L2.
    const bool held = C <= kSelCandLds;
    const int own0 = __builtin_amdgcn_readlane(int(cb), wk.part);
    own_n = __builtin_amdgcn_readlane(int(hd.cand_cnt), wk.part);
    auto list = [&](int j) {
      return reinterpret_cast<const u32x2*>(P2row + int64_t(j) * kSelPart2Bytes + kSelP2Cand);
    };
    for (int j = wave; j < parts_r; j += kFW) {
      const int c0 = __builtin_amdgcn_readlane(int(cb), j), cn = __builtin_amdgcn_readlane(int(hd.cand_cnt), j);
      if (!held && j != wk.part) continue;   // (wave-uniform)
      const u32x2* cand = list(j);
      auto put = [&](int i, u32x2 e) {
        if (i >= cn) return;
        if (held) ck[c0 + i] = e.x;
        if (j == wk.part) ci[i] = int32_t(e.y);
      };
      int i = lane;
      if (j == wave) {
        put(i, pre);
        i += kWave;
      }
      for (; i < cn; i += 4 * kWave) {   // (four loads in flight)
        if (cn - (i - lane) <= kWave) {  // (wave-uniform)
          put(i, cand[i]);
          break;
        }
        u32x2 e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = cand[min(i + u * kWave, cn - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) put(i + u * kWave, e[u]);
      }
    }
    __syncthreads();
    auto before = [&](auto body) {   // body(key, whether it is of a part before this one)
      if (held) {                    // (block-uniform)
        for (int i = t; i < C; i += kFT) body(ck[i], i < own0);
      } else {
        for (int j = wave; j < parts_r; j += kFW) {
          const int cn = __builtin_amdgcn_readlane(int(hd.cand_cnt), j);
          const u32x2* cand = list(j);
          for (int i = lane; i < cn; i += 4 * kWave) {
            uint32_t key[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) key[u] = cand[min(i + u * kWave, cn - 1)].x;
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (i + u * kWave < cn) body(key[u], j < wk.part);
          }
        }
      }
    };
    auto keys = [&](auto body) { before([&](uint32_t key, bool) { body(key); }); };
    kstar = rst.exact ? rst.kstar : 0u;
    if (C > 0) {   // block-uniform
      const float c = scale_log2e * kSelPerOctave;
      kstar = rank_candidates<kFT>(keys, mass_ceil(rst.need), rst.M, scale_log2e, c, rst.bin, rank);
      if (kstar == 0u) {   // (block-uniform) their masses fall short by rounding: all of them are selected
        keys([&](uint32_t key) { atomicMin(&rank.kmin, key); });
        __syncthreads();
        kstar = rank.kmin;
      }
      // selected candidates of the parts before this one, and of the row
      int nb = 0, ns = 0;
      before([&](uint32_t key, bool b) {
        ns += key >= kstar ? 1 : 0;
        nb += key >= kstar && b ? 1 : 0;
      });
      ns = wave_sum_i32(ns);
      nb = wave_sum_i32(nb);
      if (lane == 0 && ns) atomicAdd(&sel_s, uint32_t(ns));
      if (lane == 0 && nb) atomicAdd(&before_s, uint32_t(nb));
      for (int i = t; i < own_n; i += kFT)
        if ((held ? ck[own0 + i] : list(wk.part)[i].x) < kstar) ci[i] = -1;
      __syncthreads();
    }
    offset = __builtin_amdgcn_readlane(int(ab), wk.part) + int(before_s);
    total_sel = int(nabove) + int(sel_s);
  }

  // Ascending expansion, sub-chunk by sub-chunk. The positions are gathered in
  // LDS and leave as whole lines (stores of the few selected keys of each 64
  // took four times as many).
  int32_t* out = sel_idx + int64_t(wk.row) * n;
  uint16_t* stage = reinterpret_cast<uint16_t*>(ck);
  static_assert(sizeof(ck) >= kSub * sizeof(uint16_t), "every position of a sub-chunk");
  for (int base = k0; base < k1; base += kSub) {
    uint32_t w = 0u;
    if (all) {
      const int left = k1 - (base + 32 * t);
      w = left >= 32 ? ~0u : left > 0 ? (1u << left) - 1u : 0u;
    } else if (map) {   // (block-uniform branches)
      w = next;
      if (MULTI && base + kSub < k1) next = map[(base + kSub - k0) / 32 + t];
      if (own_n > 0) {
        word_s[t] = w;
        __syncthreads();
        for (int i = t; i < own_n; i += kFT) {
          const int d = ci[i] - base;
          if (ci[i] >= 0 && d >= 0 && d < kSub) atomicOr(&word_s[d >> 5], 1u << (d & 31));
        }
        __syncthreads();
        w = word_s[t];
      }
    } else {
      const float fstar = key_floor(kstar);   // (NaN for K* = 0: every key, by keys)
      const bool byval = !__builtin_isnan(fstar);
      const int i0 = base + wave * (kFPT * kWave) + lane;
#pragma unroll 4
      for (int k = 0; k < kFPT; ++k) {
        const int i = i0 + k * kWave;
        const float x = srow[min(i, k1 - 1)];
        const uint64_t b = ballot(byval ? x >= fstar : score_key(x) >= kstar) & ballot(i < k1);
        if (lane == 2 * k) w = uint32_t(b);
        if (lane == 2 * k + 1) w = uint32_t(b >> 32);
      }
    }
    if (mp.masks) map[(base - k0) / 32 + t] = w;
    uint32_t wtot;
    const uint32_t excl = wave_excl_scan_u32(uint32_t(__popc(w)), &wtot);
    if (lane == 0) wave_cnt[wave] = int(wtot);
    __syncthreads();
    int o = 0, sub_tot = 0;
#pragma unroll
    for (int x = 0; x < kFW; ++x) {
      const int y = wave_cnt[x];
      o += x < wave ? y : 0;
      sub_tot += y;
    }
    stage_bits(w, 32 * t, stage + o + int(excl));
    __syncthreads();
    int32_t* dst = out + offset;
    for (int i = t; i < sub_tot; i += kFT) dst[i] = base + int(stage[i]);
    if (!MULTI) break;
    offset += sub_tot;
    __syncthreads();   // word_s, wave_cnt and stage are rewritten for the next sub-chunk
  }
  // the part holding the row's last key writes the count
  if (wk.part == parts_r - 1 && t == 0) sel_count[wk.row] = total_sel;
}

// ---------------------------------------------------------------- short rows: one block per row
// The whole selection of a row of at most 1024 PT keys: maximum, grid histogram,
// crossing bin, candidates, K*, bitmap and indices, with the scores in registers
// throughout and one launch instead of three. The row is spread evenly over the
// waves: each takes `steps` times 64 consecutive keys (a multiple of four, so a
// short row of a ragged batch costs what its own length does). An irregular row
// (see above) takes the three key levels instead of the grid and the candidates.
template <bool RAGGED, int PT>
__global__ __launch_bounds__(kT) void sel_row_kernel(const float* __restrict__ scores, int n, float p,
                                                     float scale_log2e, int32_t* __restrict__ sel_idx,
                                                     int32_t* __restrict__ sel_count, u64* __restrict__ masks,
                                                     int mask_words, const int32_t* __restrict__ seq_n,
                                                     const float* __restrict__ seq_p, int hq) {
  // the histogram, then the candidate keys, then the selected positions
  constexpr int kPool = std::max(int(sizeof(u64)) * kSelBins, PT * kT * int(sizeof(uint16_t)));
  constexpr int kRowCand = kPool / int(sizeof(uint32_t));   // (all keys of a row of 8192)
  __shared__ __attribute__((aligned(16))) unsigned char pool[kPool];
  u64* h = reinterpret_cast<u64*>(pool);
  uint32_t* ck = reinterpret_cast<uint32_t*>(pool);
  __shared__ RankLds rank;
  __shared__ u64 wsum[kTW];
  __shared__ Crossing cr;
  __shared__ float red[kTW];
  __shared__ uint32_t cand_n;
  __shared__ int wave_cnt[kTW];
  const int row = blockIdx.x;
  const RowSel rs = RAGGED ? row_sel(seq_n, seq_p, hq, row, n, p) : RowSel{n, p};
  const int t = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int nr = rs.n;
  if (RAGGED && nr > PT * kT) return;   // block-uniform: a row of the three passes
  if (nr == 0) {   // block-uniform: a row without keys selects none
    if (t == 0) sel_count[row] = 0;
    return;
  }
  const float* srow = scores + int64_t(row) * n;
  const float c = scale_log2e * kSelPerOctave;
  const int steps = (nr + 4 * kT - 1) / (4 * kT) * 4;   // 64-key steps per wave (<= PT)
  const int first = wave * steps * kWave + lane;        // this lane's key of step 0
  float v[PT];
  auto groups = [&](auto body) { for_groups<PT>(steps, body); };
  auto each = [&](auto body) {   // body(k) for every step
    groups([&](auto k4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) body(k4 + u);
    });
  };
  // the phases below form what they need of a score again: keeping bins, keys
  // or masses of PT scores from one phase to the next would not fit the registers
  auto forget = [&]() {
    each([&](int k) {
      float x = v[k];
      asm volatile("" : "+v"(x));
      v[k] = x;
    });
  };
  each([&](int k) { v[k] = srow[min(first + k * kWave, nr - 1)]; });
  const bool all = RAGGED && rs.p >= 1.f;   // every key of the row
  uint32_t kstar = 0u;                      // keys >= kstar are selected (every key is >= 0)
  // lane 2 k + s holds half s of the bitmap word of the wave's step k: positions pos0 .. pos0 + 31
  static_assert(PT <= kWave / 2, "a lane per half word");
  const int pos0 = wave * steps * kWave + 32 * lane;
  const uint32_t in = lane < 2 * steps ? low_bits(nr - pos0) : 0u;   // its positions inside the row
  uint32_t word = in;                                                // the selected ones
  if (!all) {
#pragma unroll
    for (int k = 0; k < kSelBins / kT; ++k) h[k * kT + t] = 0ull;
    if (t == 0) cand_n = 0u;
    rank_clear<kT>(rank);
    float m = -INFINITY;
    each([&](int k) {   // (lanes past the row: no mass, no bin)
      v[k] = first + k * kWave < nr ? v[k] : -INFINITY;
      m = fmaxf(m, v[k]);
    });
    m = wave_max_dpp(m);
    if (lane == 0) red[wave] = m;
    __syncthreads();   // (also orders the clearing of h before the adds)
    m = row_max(red[lane & (kTW - 1)]);
    const GridWindow g = grid_window(m, c);
    // A row of more than one sub-chunk has finer units: its masses are not relative
    // to the maximum of their own sub-chunk, as those of a longer row are.
    const float whole = nr > kSub ? kWholeFine : kWhole;
    each([&](int k) { grid_add(h, v[k], m, scale_log2e, c, g.base, whole); });
    forget();
    __syncthreads();
    // the total, the target and the crossing bin: wave w holds bins 256 w ..,
    // and the wave with the crossing looks for it alone
    const u64 b0 = h[4 * t], b1 = h[4 * t + 1], b2 = h[4 * t + 2], b3 = h[4 * t + 3];
    const u64 s = (b0 + b1) + (b2 + b3);
    const u64 ws = wave_sum_u64(s);
    if (lane == 0) wsum[wave] = ws;
    __syncthreads();
    u64 upto = wsum[lane & (kTW - 1)];   // lane l (of 16): mass of the bins of waves 0 .. l
    upto += RBQ_DPP_U64_M(upto, 0x111, 0xF);
    upto += RBQ_DPP_U64_M(upto, 0x112, 0xF);
    upto += RBQ_DPP_U64_M(upto, 0x114, 0xF);
    upto += RBQ_DPP_U64_M(upto, 0x118, 0xF);
    const u64 total = readlane_u64(upto, kTW - 1);
    u64 need = mass_ceil(double(rs.p) * double(total));
    need = need > total ? total : need;
    const bool fast = g.ok && total > 0ull;   // block-uniform
    bool byscore = !fast;                     // K* compared with all scores in the end
    if (fast) {
      const u64 wabove = total - readlane_u64(upto, wave);   // mass of the bins of the waves above
      if (wabove < need && wabove + ws >= need) {            // one wave
        const u64 above = wabove + (ws - wave_incl_scan_u64(s));
        if (above < need && above + s >= need) crossing_in4(4 * t, above, need, b0, b1, b2, b3, &cr);   // one lane
      }
      __syncthreads();
      const int bin = g.base + int(cr.bin);
      const u64 need_bin = cr.need;
      // the keys above the bin, and those inside it as candidates (as pass 2)
      const BinEdges be = bin_edges(bin);
      LaneWords lw{0u, 0u}, lm{0u, 0u};
      groups([&](auto k) { classify4<k>(v + k, be, c, lw, lm); });
      word = half_words(lw.lo, lw.hi) & in;
      uint32_t mid = half_words(lm.lo, lm.hi) & in;
      uint32_t wcnt;
      uint32_t pos = wave_excl_scan_u32(uint32_t(__popc(mid)), &wcnt);
      if (wcnt) {   // wave-uniform: one reservation per wave
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&cand_n, wcnt);
        pos += uint32_t(__builtin_amdgcn_readfirstlane(int(at)));
        uint32_t q = pos;
        for (uint32_t m2 = mid; m2; m2 &= m2 - 1u, ++q)
          if (q < uint32_t(kRowCand)) ck[q] = score_key(srow[pos0 + __builtin_ctz(m2)]);
      }
      __syncthreads();
      const int C = int(cand_n);
      // (the candidates' masses are those the histogram summed, so one of them
      // reaches need_bin; more than the LDS holds are gone through in the registers)
      byscore = C > kRowCand;
      if (!byscore) {
        auto held = [&](auto body) {
          for (int i = t; i < C; i += kT) body(ck[i]);
        };
        kstar = rank_candidates<kT>(held, need_bin, m, scale_log2e, c, bin, rank, whole);
        for (; mid; mid &= mid - 1u, ++pos)
          if (ck[pos] >= kstar) word |= mid & (0u - mid);
      } else if constexpr (PT * kT > kRowCand) {
        auto own = [&](auto body) {
          each([&](int k) {   // (lanes past the row: below every bin)
            float s1 = v[k];
            asm volatile("" : "+v"(s1));   // (as forget(), for each of the ranking's passes)
            const float x = __fmul_rn(s1, c);
            if (x >= be.lo && x < be.hi) body(score_key(s1));
          });
        };
        kstar = rank_candidates<kT>(own, need_bin, m, scale_log2e, c, bin, rank, whole);
      }
    }
    if (!fast) {   // three levels over the row's keys
      u64 rest = 0;
      uint32_t prefix = 0;
#pragma unroll 1
      for (int level = 0; level < 3; ++level) {
        const int shift = level == 0 ? 20 : level == 1 ? 8 : 0;
        const uint32_t mask = level == 2 ? 0xffu : 0xfffu;
        const int hshift = level == 0 ? 32 : level == 1 ? 20 : 8;   // bits that must match the prefix
        forget();
        __syncthreads();   // every thread is done with h and cr
        for (int b = t; b < kSelBins; b += kT) h[b] = 0ull;
        __syncthreads();
        each([&](int k) {
          const uint32_t key = score_key(v[k]);
          const bool match = hshift == 32 || (key >> hshift) == prefix;
          if (match) {   // (lanes past the row add no mass)
            const u64 e = fixed_mass(v[k], m, scale_log2e, whole);
            if (e) atomicAdd(&h[(key >> shift) & mask], e);
          }
        });
        __syncthreads();
        block_crossing_4096(h, rest, level == 0 ? rs.p : 0.f, wsum, &cr);
        const uint32_t bin = cr.ok ? cr.bin : 0u;   // (no mass left: the lowest bin, every key of the prefix)
        prefix = (prefix << (level == 2 ? 8 : 12)) | bin;
        rest = cr.need;
      }
      kstar = prefix;
    }
    if (byscore) {   // block-uniform
      forget();
      const float fstar = key_floor(kstar);   // (NaN for K* = 0: every key, by keys)
      const bool byval = !__builtin_isnan(fstar);
      LaneWords lw{0u, 0u};
      groups([&](auto k4) {
        uint64_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = ballot(byval ? v[k4 + u] >= fstar : score_key(v[k4 + u]) >= kstar);
        words_to_lanes<k4>(w, lw.lo, lw.hi);
      });
      word = half_words(lw.lo, lw.hi) & in;
    }
  }
  // ascending indices: wave-major, then lane
  uint32_t wsel;
  const uint32_t excl = wave_excl_scan_u32(uint32_t(__popc(word)), &wsel);
  if (lane == 0) wave_cnt[wave] = int(wsel);
  // (the other half of the last word too: it may hold no key)
  if (masks && lane < 2 * steps && (pos0 & ~63) < nr)
    reinterpret_cast<uint32_t*>(masks + int64_t(row) * mask_words)[pos0 / 32] = word;
  __syncthreads();
  uint32_t upto = uint32_t(wave_cnt[lane & (kTW - 1)]);   // lane l (of 16): waves 0 .. l
  upto += RBQ_DPP_U32(upto, 0x111);
  upto += RBQ_DPP_U32(upto, 0x112);
  upto += RBQ_DPP_U32(upto, 0x114);
  upto += RBQ_DPP_U32(upto, 0x118);
  const int tot = __builtin_amdgcn_readlane(int(upto), kTW - 1);
  const int o = __builtin_amdgcn_readlane(int(upto), wave) - int(wsel);
  // the positions through LDS, as in the final pass above
  uint16_t* stage = reinterpret_cast<uint16_t*>(pool);
  stage_bits(word, pos0, stage + o + int(excl));
  __syncthreads();
  int32_t* out = sel_idx + int64_t(row) * n;
  for (int i = t; i < tot; i += kT) out[i] = int(stage[i]);
  if (t == 0) sel_count[row] = tot;
}

constexpr int kAllThreads = 256;
__global__ __launch_bounds__(kAllThreads) void topp_all_kernel(int n, int32_t* __restrict__ sel_idx,
                                                               int32_t* __restrict__ sel_count,
                                                               u64* __restrict__ masks, int mask_words) {
  const int row = blockIdx.y;
  const int i = blockIdx.x * kAllThreads + threadIdx.x;
  if (i < n) sel_idx[int64_t(row) * n + i] = i;
  if (blockIdx.x == 0 && threadIdx.x == 0) sel_count[row] = n;
  if (masks && (i & 63) == 0 && i / 64 < mask_words) {
    const int left = n - i;   // keys [i, i + 64) that exist
    masks[int64_t(row) * mask_words + i / 64] = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1 : 0ull;
  }
}

// rows of up to `most` keys (n: their stride)
template <bool RAGGED>
void sel_rows(int rows, hipStream_t stream, int most, int n, const float* scores, float p, float scale_log2e,
              int32_t* sel_idx, int32_t* sel_count, u64* masks, int mask_words, const int32_t* seq_n,
              const float* seq_p, int heads_q) {
#define RBQ_SEL_ROW(PT)                                                                                            \
  sel_row_kernel<RAGGED, PT><<<rows, kT, 0, stream>>>(scores, n, p, scale_log2e, sel_idx, sel_count, masks, mask_words, \
                                                      seq_n, seq_p, heads_q)
  if (most <= 4 * kT) RBQ_SEL_ROW(4);
  else if (most <= 8 * kT) RBQ_SEL_ROW(8);
  else if (most <= 16 * kT) RBQ_SEL_ROW(16);
  else RBQ_SEL_ROW(32);
#undef RBQ_SEL_ROW
}

template <bool RAGGED, bool MULTI>
void sel_passes(int rows, hipStream_t stream, int n, const ToppPlan& pl, const float* scores, float p,
                float scale_log2e, const ToppWorkspace& w, int32_t* sel_idx, int32_t* sel_count, u64* masks,
                int mask_words, const int32_t* seq_n, const float* seq_p, int heads_q) {
  const TilePlace tp = tile_place(rows, pl.parts, kPlaceGroup);
  const dim3 grid(unsigned(tile_grid(tp, 1)));
  const MapPlan mp = map_plan(masks, mask_words, pl.spb);
  sel_hist_kernel<RAGGED, MULTI><<<grid, kT, 0, stream>>>(scores, n, pl.spb, tp, 1, scale_log2e, w.part1, seq_n,
                                                          seq_p, heads_q);
  sel_cand_kernel<RAGGED, MULTI><<<grid, kT, 0, stream>>>(scores, n, pl.spb, tp, 1, p, scale_log2e, w.part1, w.part2,
                                                          w.state, mp, seq_n, seq_p, heads_q);
  sel_final_kernel<RAGGED, MULTI><<<grid, kFT, 0, stream>>>(scores, n, pl.spb, tp, 1, p, scale_log2e, w.part2, w.state,
                                                           sel_idx, sel_count, mp, seq_n, seq_p, heads_q);
}

}  // namespace

rbq_status launch_topp(int32_t rows, int32_t n, const float* scores, float p, float sm_scale, int32_t* sel_idx,
                       int32_t* sel_count, void* ws, hipStream_t stream, unsigned long long* masks,
                       const int32_t* seq_n, const float* seq_p, int32_t heads_q) {
  const int mask_words = topp_mask_words(n);
  const bool ragged = seq_n != nullptr || seq_p != nullptr;   // per-row counts / p: decided on the device
  if (n == 0 || (p >= 1.0f && !ragged)) {
    // every key (or none) is selected
    const int cover = masks ? mask_words * 64 : n;
    const dim3 grid(cover > 0 ? (cover + kAllThreads - 1) / kAllThreads : 1, rows);
    topp_all_kernel<<<grid, kAllThreads, 0, stream>>>(n, sel_idx, sel_count, masks, mask_words);
    return hipGetLastError() == hipSuccess ? RBQ_OK : RBQ_EDEVICE;
  }
  const float scale_log2e = float(double(sm_scale) * 1.4426950408889634);
  if (n <= kSelRowMax) {
    if (ragged)
      sel_rows<true>(rows, stream, n, n, scores, p, scale_log2e, sel_idx, sel_count, masks, mask_words, seq_n, seq_p,
                     heads_q);
    else
      sel_rows<false>(rows, stream, n, n, scores, p, scale_log2e, sel_idx, sel_count, masks, mask_words, nullptr,
                      nullptr, heads_q);
    return hipGetLastError() == hipSuccess ? RBQ_OK : RBQ_EDEVICE;
  }
  if (seq_n)
    sel_rows<true>(rows, stream, kSelRowMax, n, scores, p, scale_log2e, sel_idx, sel_count, masks, mask_words, seq_n,
                   seq_p, heads_q);
  const ToppPlan pl = topp_plan(n);
  const ToppWorkspace w = topp_workspace(ws, rows, n);
#define RBQ_SEL_PASSES(RG, MU)                                                                               \
  sel_passes<RG, MU>(rows, stream, n, pl, scores, p, scale_log2e, w, sel_idx, sel_count, masks, mask_words, \
                     RG ? seq_n : nullptr, RG ? seq_p : nullptr, heads_q)
  if (ragged) {
    if (pl.spb > 1) RBQ_SEL_PASSES(true, true); else RBQ_SEL_PASSES(true, false);
  } else {
    if (pl.spb > 1) RBQ_SEL_PASSES(false, true); else RBQ_SEL_PASSES(false, false);
  }
#undef RBQ_SEL_PASSES
  return hipGetLastError() == hipSuccess ? RBQ_OK : RBQ_EDEVICE;
}

}  // namespace rbq
