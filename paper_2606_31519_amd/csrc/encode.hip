// rbq_encode_keys: index construction (Algorithm 1; Section 3.2; Appendix A.2).
//
//   x = k - c_k,  r = P^T x  (the row x * P),  bits = [r > 0],
//   alpha' = sum_j |r_j| / ||x||,  f = ||x|| / alpha',  g = <c_q, x>
//
// The rotation is the only dense contraction on the path, so it runs on the
// matrix cores: long runs of keys as described at encode_long_kernel, up to 4096
// keys per head (every window of the lazy update) with v_mfma_f32_32x32x2_f32
// (fp32 in, fp32 accumulate: the sign decisions need fp32 accuracy, bf16 products
// of P would flip signs of small components). Each wave keeps its 32 output columns of P in registers as the
// MFMA B operands (64 floats per lane, all requested at once), and a tile of
// 32 centred keys is staged in LDS. In the 32x32 accumulator layout lane l
// holds output column l % 32, so one wave ballot of (r > 0) over a register
// yields two packed 32-bit code words directly.
//
// With RBQ_ENCODE_SET_CENTROID a two-pass deterministic column mean over the
// new keys first sets c_k (fixed-order partial sums, no atomics).
#include <algorithm>

#include "encode_dev.h"
#include "rbq_device.h"
#include "rbq_internal.h"

namespace rbq {
namespace {

// ---------------------------------------------------------------- centroid
// D / 8 threads per key row (8 dimensions each), 2048 / D row groups
template <int DT, int D = kHeadDim>
__global__ __launch_bounds__(256) void centroid_partial_kernel(const void* __restrict__ keys, int64_t keys_ld,
                                                               int n_new, float* __restrict__ partial,
                                                               int chunks) {
  constexpr int TPR = D / 8, RG = 256 / TPR;
  __shared__ float red[RG][D + 4];
  const int bh = blockIdx.y;
  const int c = blockIdx.x;
  const int rg = threadIdx.x / TPR;     // row group
  const int t = threadIdx.x % TPR;      // dims [8t, 8t + 8)
  const int r0 = c * kCentroidChunk;
  const int r1 = min(n_new, r0 + kCentroidChunk);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr int kPieces = DT == RBQ_BF16 ? 1 : 2;   // 16-byte pieces of a thread's dimensions
  const u32x4* base = reinterpret_cast<const u32x4*>(static_cast<const char*>(keys) +
                                                     (int64_t(bh) * keys_ld * D + 8 * t) * (2 * kPieces));
  auto load = [&](int r, u32x4* v) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) v[i] = base[int64_t(r) * (D / 8 * kPieces) + i];
  };
  auto add = [&](const u32x4* v) {
    if constexpr (DT == RBQ_BF16) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[2 * i] += bf16_lo(v[0][i]);
        acc[2 * i + 1] += bf16_hi(v[0][i]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += __uint_as_float(v[(i / 4) % kPieces][i % 4]);
    }
  };
  constexpr int kBatch = 8;   // rows in flight per thread, added in order (8 x 130816 bf16 keys: 51 -> 46 us)
  int r = r0 + rg;
  for (; r + (kBatch - 1) * RG < r1; r += kBatch * RG) {
    u32x4 v[kBatch][kPieces];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) load(r + i * RG, v[i]);
#pragma unroll
    for (int i = 0; i < kBatch; ++i) add(v[i]);
  }
  for (; r < r1; r += RG) {
    u32x4 v[kPieces];
    load(r, v);
    add(v);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) red[rg][8 * t + k] = acc[k];
  __syncthreads();
  if (threadIdx.x < D) {
    float s = 0.f;
#pragma unroll
    for (int g = 0; g < RG; ++g) s += red[g][threadIdx.x];
    partial[(int64_t(bh) * chunks + c) * D + threadIdx.x] = s;
  }
}

// The chunks' sums in order, 32 of them loaded at a time: 6 us for the 128 chunks of
// 128K keys, one load after the other 31.
template <int D = kHeadDim>
__global__ __launch_bounds__(D) void centroid_final_kernel(const float* __restrict__ partial, int chunks,
                                                           int n_new, float* __restrict__ c_k) {
  constexpr int kBatch = 32;
  const int bh = blockIdx.x;
  const float* p = partial + int64_t(bh) * chunks * D + threadIdx.x;
  float s = 0.f;
  for (int c0 = 0; c0 < chunks; c0 += kBatch) {
    float v[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) v[i] = p[int64_t(min(c0 + i, chunks - 1)) * D];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) s += c0 + i < chunks ? v[i] : 0.f;
  }
  c_k[int64_t(bh) * D + threadIdx.x] = s / float(n_new);
}

// ---------------------------------------------------------------- encode
template <int DT, bool ROT, int D>
__global__ __launch_bounds__(kEncThreads) void encode_kernel(EncodeArgs ea) {
  encode_tiles<DT, ROT, false, D>(ea, blockIdx.y, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------- encode, long runs of keys
// The rotation on the fp16 matrix cores at fp32 accuracy. A key is scaled by the
// power of two that puts its largest component into [2^14, 2^15), P by one that
// does the same for its largest entry, and both are split into two fp16 parts,
// hi + mid (22 bits of each value); then
//   r = (hm + mh) + hh,
// three products that are exact in fp32, the small ones summed first. What is left
// out (the mid x mid products and the bits past the 22nd) is about 7e-8 of a
// component's rms, and there are 8 roundings of the large sum where the fp32 form
// has 65: against 64 bits the components are off by 1.1e-7 of their rms instead of
// 1.45e-7, the factors by 7.3e-8 instead of 9.3e-8, and no sign is (kNearZero).
// (Three bf16 parts and six products were off by 0.7e-7, in 200 us where this
// form took 123 before the signs' second look, which costs 2.)
//
// The product is taken transposed, r^T = P^T x^T: a lane then holds 16 output
// dimensions of ONE key (key l % 32 of its tile in lane l), so a key's sign word,
// sum |r|, ||x||^2 and <c_q, x> need one exchange between the wave's halves and
// nothing else: no barrier and no LDS after P's parts are laid out in it (64 KB at
// D = 128, in operand order, for a block of 12 waves per CU). Waves go through
// tiles of 32 keys on their own, straight from global memory: a lane's operand of
// a step is 8 consecutive dimensions of its key.
//
// Bound: the matrix cores and the vector ALUs that centre and split, at the clock
// the card holds under them (1.5 to 1.6 GHz measured). 8 heads x 130816 bf16 keys,
// D = 128: 125 us, the fp32 form 336; with the centroid 158 us a call, before 390.
// (fp32 keys, whose coming tile takes twice the registers: 8 waves)
constexpr int long_waves(int dt) { return dt == RBQ_BF16 ? 12 : 8; }
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

// x as hi + mid fp16 parts
struct Parts8 {
  f16x8 h, m;
};
__device__ __forceinline__ Parts8 split8(f32x8 x) {
  Parts8 p;
  p.h = __builtin_convertvector(x, f16x8);
  p.m = __builtin_convertvector(x - __builtin_convertvector(p.h, f32x8), f16x8);
  return p;
}
// the exponent e of the power of two that takes a largest magnitude a into
// [2^14, 2^15) (at most 2^127 for the smallest, 2^-114 for an infinity)
__device__ __forceinline__ int scale_exp(float a) {
  return min(141 - int((__float_as_uint(a) >> 23) & 0xffu), 127);
}
__device__ __forceinline__ float exp2_int(int e) { return __uint_as_float(uint32_t(e + 127) << 23); }   // |e| <= 127

__device__ __forceinline__ float dot4(f32x4 a, f32x4 b) {
  return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x)));
}
__device__ __forceinline__ float max_abs8(f32x8 x, float m) {   // (pairs: one three-way maximum each)
#pragma unroll
  for (int i = 0; i < 8; i += 2) m = fmaxf(fmaxf(m, fabsf(x[i])), fabsf(x[i + 1]));
  return m;
}
// Components this close to zero are formed again in 64 bits for their sign: in the
// scaled units about 2e-6 of a component's rms (1e-6 for keys with all components
// alike), ten times the rounding error, met in one of 150 tiles of 32 keys. More than
// two exact zeros among 16 components are no chance (a key at the centroid, sparse
// keys under a sparse P) and stay zeros.
// Of 2.8e9 bits against 64 bits 68 were off without this, 80 in the fp32 form, and
// none are with it.
constexpr float kNearZero = 1024.f;
template <int DT, int D>
__device__ __forceinline__ double component_f64(const char* key, const float* ck, const float* p) {
  double r = 0.0;
#pragma unroll 16
  for (int d = 0; d < D; ++d) {
    const float x = DT == RBQ_BF16 ? __uint_as_float(uint32_t(reinterpret_cast<const uint16_t*>(key)[d]) << 16)
                                   : reinterpret_cast<const float*>(key)[d];
    r = fma(double(x) - double(ck[d]), double(p[d * D]), r);
  }
  return r;
}
// x of this lane + x of the lane 32 away
__device__ __forceinline__ float sum_halves(float x) { return x + __shfl_xor(x, 32, kWave); }

template <int DT, bool ROT, int D>
__global__ __launch_bounds__(long_waves(DT) * kWave) void encode_long_kernel(EncodeArgs ea, int blocks_per_head) {
  constexpr int kLongWaves = long_waves(DT);
  constexpr int W = D / 32;         // code words per key, 32-row blocks of P^T
  constexpr int S = D / 16;         // steps of 16 dimensions
  constexpr int kElem = DT == RBQ_BF16 ? 2 : 4;
  constexpr int kPieces = kElem / 2;   // 16-byte pieces of 8 dimensions
  __shared__ f16x8 pt_s[W][S][2][kWave];   // P^T's parts, lane-major
  __shared__ float ck_s[D], cq_s[D];
  __shared__ float red[kLongWaves];
  __shared__ int next_s;
  __shared__ uint16_t near_s[W][kLongWaves][kWave];   // (a lane's own: no wait between its write and its read)
  const int bh = blockIdx.x / blocks_per_head, bx = blockIdx.x % blocks_per_head;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
  const int key_l = lane & 31, half = lane >> 5;
  const int n_new = ea.n_new;
  const int tiles = (n_new + 31) / 32;
  const char* keys = static_cast<const char*>(ea.keys) + int64_t(bh) * ea.keys_ld * D * kElem + 16 * kPieces * half;

  u32x4 raw[S][kPieces];   // the coming tile's key: dimensions 16 s + 8 half .. + 8
  auto load_tile = [&](int tile) {
    const int key = min(tile * 32 + key_l, n_new - 1);   // (keys past n_new are never stored)
    const u32x4* kp = reinterpret_cast<const u32x4*>(keys + int64_t(key) * D * kElem);
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int i = 0; i < kPieces; ++i) raw[s][i] = kp[s * 2 * kPieces + i];
  };
  // The block's tiles, every blocks_per_head-th from the last one down (a centroid
  // pass before has just read those), go to its waves one by one: dealt out in
  // advance, the waves that a SIMD favours end early and leave the others alone.
  auto tile_at = [&](int q) { return tiles - 1 - bx - q * blocks_per_head; };
  int tile = tile_at(wave);
  if (threadIdx.x == 0) next_s = kLongWaves;
  // P's fragment (jb, s): rows 32 jb + lane % 32 of P^T, dimensions as above (all requested at once)
  constexpr int kFrags = (W * S + kLongWaves - 1) / kLongWaves;
  f32x8 pf[kFrags];
  float pmax = 0.f;
#pragma unroll
  for (int u = 0; u < kFrags; ++u) {
    const int f = min(wave + u * kLongWaves, W * S - 1);
    const float* p = ea.P + (16 * (f % S) + 8 * half) * D + 32 * (f / S) + key_l;
#pragma unroll
    for (int i = 0; i < 8; ++i) pf[u][i] = p[i * D];
  }
  if (tile >= 0) load_tile(tile);   // (after P: loads are waited for in order)
  float cq_own = 0.f;
  if (threadIdx.x < D) {
    ck_s[threadIdx.x] = ea.c_k[int64_t(bh) * D + threadIdx.x];
    if (ea.c_q) cq_own = ea.c_q[int64_t(bh) * D + threadIdx.x];
    cq_s[threadIdx.x] = cq_own;
  }
#pragma unroll
  for (int u = 0; u < kFrags; ++u) pmax = max_abs8(pf[u], pmax);
  pmax = wave_max_dpp(pmax);
  if (lane == 0) red[wave] = pmax;
  const bool has_cq = __syncthreads_or(cq_own != 0.f);   // (no query centroid: g = 0 for every key)
#pragma unroll
  for (int w = 0; w < kLongWaves; ++w) pmax = fmaxf(pmax, red[w]);
  const int pexp = scale_exp(pmax);
#pragma unroll
  for (int u = 0; u < kFrags; ++u) {
    const int f = min(wave + u * kLongWaves, W * S - 1);   // (past the last: the same values again)
    const Parts8 q = split8(pf[u] * -exp2_int(pexp));
    pt_s[f / S][f % S][0][lane] = q.h;
    pt_s[f / S][f % S][1][lane] = q.m;
  }
  __syncthreads();

  while (tile >= 0) {
    // centre this tile's keys; their norms, their products with c_q and their largest components
    f32x8 v[S];
    float nn[4] = {0.f, 0.f, 0.f, 0.f}, gg[4] = {0.f, 0.f, 0.f, 0.f};   // (short chains: fewer roundings in a row)
    float top = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if constexpr (DT == RBQ_BF16) {
        v[s] = __builtin_convertvector(__builtin_bit_cast(bf16x8, raw[s][0]), f32x8);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[s][i] = __uint_as_float(raw[s][(i / 4) % kPieces][i % 4]);
      }
      const int d = 16 * s + 8 * half;
      v[s] -= *reinterpret_cast<const f32x8*>(&ck_s[d]);
      nn[s % 4] += dot4(v[s].lo, v[s].lo) + dot4(v[s].hi, v[s].hi);
      top = max_abs8(v[s], top);
      __builtin_amdgcn_sched_barrier(0);   // (a step at a time, for the registers' sake)
    }
    if (has_cq) {   // block-uniform
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const f32x8 cq = *reinterpret_cast<const f32x8*>(&cq_s[16 * s + 8 * half]);
        gg[s % 4] += dot4(cq.lo, v[s].lo) + dot4(cq.hi, v[s].hi);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    float norm2 = sum_halves((nn[0] + nn[1]) + (nn[2] + nn[3])), g = sum_halves((gg[0] + gg[1]) + (gg[2] + gg[3]));
    // (left to the compiler, the sums are formed after the products from values kept in scratch memory)
    asm volatile("" : "+v"(norm2), "+v"(g));
    const int xexp = scale_exp(fmaxf(top, __shfl_xor(top, 32, kWave)));
    const float scale = exp2_int(xexp);
    Parts8 x[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      x[s] = split8(v[s] * scale);
      __builtin_amdgcn_sched_barrier(0);
    }
    int q = 0;
    if (lane == 0) q = atomicAdd(&next_s, 1);
    const int coming = tile_at(__builtin_amdgcn_readfirstlane(q));
    if (coming >= 0) load_tile(coming);   // lands during the products

    const int key = tile * 32 + key_l;
    uint32_t word[W];
    uint32_t open = 0u;   // words (of any lane's key) with a component whose sign is still open
    float absum = 0.f;
#pragma unroll 1
    for (int jp = 0; jp < W; jp += 2) {   // two words at a time: two chains of products
      f32x16 a[2] = {f32x16{0.f}, f32x16{0.f}};
      auto frag = [&](int j, int s, int part) { return pt_s[jp + j][s][part][lane]; };
      // the small products first (h m + m h), then the large ones on their sum
      f16x8 ph[2][2], pm[2][2];   // [step % 2][word]: this step's parts of P^T and the next one's
#pragma unroll
      for (int j = 0; j < 2; ++j) ph[0][j] = frag(j, 0, 0), pm[0][j] = frag(j, 0, 1);
#pragma unroll
      for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          ph[(s + 1) % 2][j] = frag(j, (s + 1) % S, 0);   // (after the last step: the second pass's first)
          if (s + 1 < S) pm[(s + 1) % 2][j] = frag(j, s + 1, 1);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) a[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(pm[s % 2][j], x[s].h, a[j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 2; ++j) a[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ph[s % 2][j], x[s].m, a[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (s + 1 < S) {
#pragma unroll
          for (int j = 0; j < 2; ++j) ph[(s + 1) % 2][j] = frag(j, s + 1, 0);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) a[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ph[s % 2][j], x[s].h, a[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      // register i of a[j]: -r of dimension 32 (jp + j) + 8 (i / 4) + 4 half + i % 4 of this lane's key
      float low = kNearZero;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint32_t bits = 0u;
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16; i += 2) low = fminf(fminf(low, fabsf(a[j][i])), fabsf(a[j][i + 1]));
#pragma unroll
        for (int i = 15; i >= 0; --i) {
          const float r = a[j][i];
          sum[i % 4] += fabsf(r);
          bits = (bits << 1) | (__float_as_uint(r) >> 31);   // 1 iff r > 0 (a zero sum is +0)
          if (ROT) {
            if (key < n_new)
              ea.rot_out[(int64_t(bh) * n_new + key) * D + 32 * (jp + j) + 8 * (i / 4) + 4 * half + i % 4] =
                  0.f - ldexpf(r, -xexp - pexp);
          }
        }
        absum += (sum[0] + sum[1]) + (sum[2] + sum[3]);
        bits = ((bits & 0xf000u) << 12) | ((bits & 0xf00u) << 8) | ((bits & 0xf0u) << 4) | (bits & 0xfu);
        bits <<= 4 * half;
        bits |= uint32_t(__shfl_xor(int(bits), 32, kWave));
#pragma unroll
        for (int w = 0; w < W; ++w) word[w] = w == jp + j ? bits : word[w];
      }
      if (__any(low < kNearZero)) {
        open |= 1u << jp;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          uint32_t m = 0u, z = 0u;
#pragma unroll
          for (int i = 15; i >= 0; --i) m = (m << 1) | uint32_t(fabsf(a[j][i]) < kNearZero);
#pragma unroll
          for (int i = 15; i >= 0; --i) z = (z << 1) | uint32_t(a[j][i] == 0.f);
          near_s[jp + j][wave][lane] = uint16_t(__popc(z) > 2 ? m & ~z : m);
        }
      }
    }
    if (open != 0u) {   // wave-uniform
      int row = min(key, n_new - 1), half4 = 4 * half;
      asm volatile("" : "+v"(row), "+v"(half4));   // (formed here, not kept in registers through the products)
      const char* kp = static_cast<const char*>(ea.keys) + int64_t(bh) * ea.keys_ld * D * kElem + int64_t(row) * D * kElem;
      const uint32_t own = 0x0f0f0f0fu << half4;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        if (!((open >> (w & ~1)) & 1u)) continue;
        for (uint32_t near = near_s[w][wave][lane]; near; near &= near - 1) {
          const int i = __builtin_ctz(near), d = 8 * (i / 4) + half4 + i % 4;
          const uint32_t one = component_f64<DT, D>(kp, ck_s, ea.P + 32 * w + d) > 0.0 ? 1u : 0u;
          word[w] = (word[w] & ~(1u << d)) | (one << d);
        }
        word[w] = (word[w] & own) | uint32_t(__shfl_xor(int(word[w] & own), 32, kWave));
      }
    }
    absum = ldexpf(sum_halves(absum), -xexp - pexp);
    if (half == 0 && key < n_new) {
      const float nrm = sqrtf(norm2);
      const float alpha_p = nrm > 0.f ? absum / nrm : 0.f;
      const float f = alpha_p > 0.f ? norm2 / absum : 0.f;   // (= ||x|| / alpha', with two roundings fewer)
      const int64_t o = int64_t(bh) * ea.cap + ea.offset + key;
      if constexpr (W == 4)
        *reinterpret_cast<u32x4*>(ea.codes + o * W) = u32x4{word[0], word[1], word[2], word[3]};
      else
        *reinterpret_cast<u32x2*>(ea.codes + o * W) = u32x2{word[0], word[1]};
      if (ea.kfac16 != nullptr)
        ea.kfac16[o] = compact_factor(f);
      else
        *reinterpret_cast<f32x2*>(ea.kfac + o * 2) = f32x2{f, g};
      if (ea.alpha_out)
        ea.alpha_out[int64_t(bh) * n_new + key] = alpha_p * (D == 128 ? 0.08838834764831845f : 0.125f);   // 1/sqrt(D)
    }
    tile = coming;
  }
}

template <int DT, int D>
rbq_status launch_dt(int32_t batch, int32_t heads_kv, const void* keys, int64_t keys_ld, int32_t n_new,
                     int32_t offset, int32_t cap, const float* P, const float* c_q, float* c_k, uint32_t* codes,
                     float* kfac, uint32_t flags, float* alpha_out, void* ws, float* rot_out, hipStream_t stream,
                     uint16_t* kfac16) {
  constexpr int kLongBlocks = 256;   // one block per CU: P's parts fill most of its LDS
  const int bhs = batch * heads_kv;
  if (flags & RBQ_ENCODE_SET_CENTROID) {
    const int chunks = (n_new + kCentroidChunk - 1) / kCentroidChunk;
    float* partial = static_cast<float*>(ws);
    centroid_partial_kernel<DT, D><<<dim3(chunks, bhs), 256, 0, stream>>>(keys, keys_ld, n_new, partial, chunks);
    centroid_final_kernel<D><<<bhs, D, 0, stream>>>(partial, chunks, n_new, c_k);
  }
  EncodeArgs ea{keys, keys_ld, n_new, offset, cap, P, c_q, c_k, codes, kfac, alpha_out, rot_out};
  ea.kfac16 = kfac16;
  if (n_new > kEncodeLongMin) {
    const int tiles = (n_new + 31) / 32;
    constexpr int kWaves = long_waves(DT);
    const int bph = std::max(1, std::min(kLongBlocks / bhs, (tiles + kWaves - 1) / kWaves));
    if (rot_out)
      encode_long_kernel<DT, true, D><<<bph * bhs, kWaves * kWave, 0, stream>>>(ea, bph);
    else
      encode_long_kernel<DT, false, D><<<bph * bhs, kWaves * kWave, 0, stream>>>(ea, bph);
    return hipGetLastError() == hipSuccess ? RBQ_OK : RBQ_EDEVICE;
  }
  const dim3 grid(encode_blocks_per_head(n_new, bhs), bhs);
  if (rot_out)
    encode_kernel<DT, true, D><<<grid, kEncThreads, 0, stream>>>(ea);
  else
    encode_kernel<DT, false, D><<<grid, kEncThreads, 0, stream>>>(ea);
  return hipGetLastError() == hipSuccess ? RBQ_OK : RBQ_EDEVICE;
}

}  // namespace

rbq_status launch_encode(int32_t batch, int32_t heads_kv, const void* keys, int32_t keys_dtype, int64_t keys_ld,
                         int32_t n_new, int32_t offset, int32_t cap, const float* P, const float* c_q, float* c_k,
                         uint32_t* codes, float* kfac, uint32_t flags, float* alpha_out, void* ws,
                         float* rot_out, hipStream_t stream, uint16_t* kfac16, int32_t head_dim) {
  if (n_new == 0) return RBQ_OK;
#define RBQ_ENCODE_LAUNCH(DT, D)                                                                                   \
  launch_dt<DT, D>(batch, heads_kv, keys, keys_ld, n_new, offset, cap, P, c_q, c_k, codes, kfac, flags, alpha_out, \
                   ws, rot_out, stream, kfac16)
  if (head_dim == 64)
    return keys_dtype == RBQ_BF16 ? RBQ_ENCODE_LAUNCH(RBQ_BF16, 64) : RBQ_ENCODE_LAUNCH(RBQ_F32, 64);
  return keys_dtype == RBQ_BF16 ? RBQ_ENCODE_LAUNCH(RBQ_BF16, kHeadDim) : RBQ_ENCODE_LAUNCH(RBQ_F32, kHeadDim);
#undef RBQ_ENCODE_LAUNCH
}

}  // namespace rbq
