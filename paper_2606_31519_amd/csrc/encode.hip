// rbq_encode_keys: index construction (Algorithm 1; Section 3.2; Appendix A.2).
//
//   x = k - c_k,  r = P^T x  (the row x * P),  bits = [r > 0],
//   alpha' = sum_j |r_j| / ||x||,  f = ||x|| / alpha',  g = <c_q, x>
//
// The rotation is the only dense contraction on the path, so it runs on the
// matrix cores with v_mfma_f32_32x32x2_f32 (fp32 in, fp32 accumulate: the sign
// decisions need fp32 accuracy, bf16 products of P would flip signs of small
// components). Runs of any length take the same kernel, so an index has the same
// rows, bit for bit, whether its keys were encoded at once or as they came. (Two
// fp16 parts per value, 22 bits, took 125 us for 8 heads x 130816 keys instead of
// 336, but gave other factors than the windows' and other signs near zero.)
// Each wave keeps its 32 output columns of P in registers as the MFMA B operands
// (64 floats per lane, all requested at once), and a tile of
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

template <int DT, int D>
rbq_status launch_dt(int32_t batch, int32_t heads_kv, const void* keys, int64_t keys_ld, int32_t n_new,
                     int32_t offset, int32_t cap, const float* P, const float* c_q, float* c_k, uint32_t* codes,
                     float* kfac, uint32_t flags, float* alpha_out, void* ws, float* rot_out, hipStream_t stream,
                     uint16_t* kfac16) {
  const int bhs = batch * heads_kv;
  if (flags & RBQ_ENCODE_SET_CENTROID) {
    const int chunks = (n_new + kCentroidChunk - 1) / kCentroidChunk;
    float* partial = static_cast<float*>(ws);
    centroid_partial_kernel<DT, D><<<dim3(chunks, bhs), 256, 0, stream>>>(keys, keys_ld, n_new, partial, chunks);
    centroid_final_kernel<D><<<bhs, D, 0, stream>>>(partial, chunks, n_new, c_k);
  }
  const dim3 grid(encode_blocks_per_head(n_new, bhs), bhs);
  EncodeArgs ea{keys, keys_ld, n_new, offset, cap, P, c_q, c_k, codes, kfac, alpha_out, rot_out};
  ea.kfac16 = kfac16;
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
