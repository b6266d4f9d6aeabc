// rbq_quantize_query: query pre-processing and INT4 quantisation
// (Algorithm 2 step 1; Section 3.3 "Query Quantization"; Appendix A.3.2).
//
// One block per query head; 2 x 128 threads share the 128 x 128 product (all
// loads of a thread in flight at once), then one wave, two dimensions per lane:
//   y = q - c_q, A = ||y||, u = y / A, q'[j] = sum_d P[d][j] u[d]   (q' = P^T u)
//   q_l = min q', q_r = max q', Delta = (q_r - q_l) / L,
//   q_u = clamp(floor((q' - q_l) / Delta + 1/2), 0, L)
// with L = 2^B_q - 1 levels above the lowest (B_q = 4, L = 15, unless the
// caller asks for fewer bits).
// The code of each dimension is decided in fp32 with every operation rounded
// separately (no contraction; IEEE division), so the oracle can repeat the
// decision exactly from the same q'. Bit-plane j of the codes is one wave
// ballot per 64 dimensions. The cost is one 128 x 128 matrix-vector product
// per head, amortised over all keys (Section 3.1). A launch of few blocks is bound
// by its chain of steps: three barriers, wave reductions on the DPP paths and an
// epilogue within one wave (32 heads: 4.5 us; with twelve barriers and
// reductions through LDS permutes 5.1).
#include "encode_dev.h"
#include "quantize_dev.h"
#include "rbq_device.h"
#include "rbq_internal.h"

namespace rbq {
namespace {

// query head `row` (= b * Hq + h), by the kQAll threads of the calling block
template <int D>
__device__ __forceinline__ void quantize_row(const QuantArgs& qa, int row) {
  constexpr int kQParts = QShape<D>::kQParts;
  const float* __restrict__ q = qa.q;
  const float* __restrict__ P = qa.P;
  const float* __restrict__ c_q = qa.c_q;
  const float* __restrict__ c_k = qa.c_k;
  const int Hq = qa.Hq, Hkv = qa.Hkv;
  __shared__ float u_s[D];
  __shared__ float part_s[kQParts][D];
  __shared__ f32x2 red[kQAll / kWave];
  const int b = row / Hq;
  const int h = row - b * Hq;
  const int grp = b * Hkv + h / (Hq / Hkv);    // (b, kv head)
  const int j = threadIdx.x % D;               // output dimension
  const int part = threadIdx.x / D;            // which share of the input dimensions

  // this group's D / kQParts rows of P, requested before anything else (they do not depend on q)
  constexpr int kRows = D / kQParts;
  float pv[kRows];
#pragma unroll
  for (int k = 0; k < kRows; ++k) pv[k] = P[(part * kRows + k) * D + j];

  float qj = 0.f, y = 0.f, ck = 0.f;
  if (part == 0) {
    qj = q[int64_t(row) * D + j];
    const float cq = c_q ? c_q[int64_t(grp) * D + j] : 0.f;
    ck = c_k[int64_t(grp) * D + j];
    y = qj - cq;
  }
  // the first D threads hold the vector; the block's sums include zeros from the others
  const float yy = wave_dot(y, y), qc = wave_dot(qj, ck);
  if (lane_id() == 0) red[threadIdx.x / kWave] = f32x2{yy, qc};
  __syncthreads();
  float A = 0.f, B0 = 0.f;
#pragma unroll
  for (int i = 0; i < kQAll / kWave; ++i) {
    A += red[i].x;
    B0 += red[i].y;
  }
  A = sqrtf(A);
  if (part == 0) u_s[j] = A > 0.f ? y / A : 0.f;
  __syncthreads();

  // q'[j] = sum_d P[d][j] u[d]: each group takes kRows rows of P (loaded above)
  float acc = 0.f;
#pragma unroll
  for (int k = 0; k < kRows; ++k) acc = fmaf(pv[k], u_s[part * kRows + k], acc);
  part_s[part][j] = acc;
  __syncthreads();
  if (threadIdx.x >= kWave) return;

  quantize_finish<D>(qa, row, part_s, A, B0, true);   // one wave's: no more barriers
}

template <int D>
__global__ __launch_bounds__(kQAll) void quantize_kernel(QuantArgs qa) { quantize_row<D>(qa, blockIdx.x); }

// One launch for the query quantisation and the lazy index update of the
// decode step (they are independent): blocks [0, rows) quantise one query
// head each, the others encode the window keys as encode_kernel would.
static_assert(kQAll == kEncThreads, "both roles run on blocks of the same size");
template <int DT, bool RAGGED, int D = kHeadDim>
__global__ __launch_bounds__(kQAll) void quantize_flush_kernel(QuantArgs qa, EncodeArgs ea, int rows, int per_head) {
  const int blk = blockIdx.x;
  if (blk < rows) {
    quantize_row<D>(qa, blk);
  } else {
    const int e = blk - rows;
    encode_tiles<DT, false, RAGGED, D>(ea, e / per_head, e % per_head, per_head);
  }
}

}  // namespace

rbq_status launch_quantize(int32_t batch, int32_t heads_q, int32_t heads_kv, const float* q, const float* P,
                           const float* c_q, const float* c_k, uint32_t* qplanes, float* qscal, float* qrot_out,
                           hipStream_t stream, int32_t bits, int32_t head_dim) {
  const QuantArgs qa{q, P, c_q, c_k, qplanes, qscal, qrot_out, heads_q, heads_kv, (1 << bits) - 1, bits > 4 ? 8 : 4};
  if (head_dim == 64)
    quantize_kernel<64><<<batch * heads_q, kQAll, 0, stream>>>(qa);
  else
    quantize_kernel<kHeadDim><<<batch * heads_q, kQAll, 0, stream>>>(qa);
  return hipGetLastError() == hipSuccess ? RBQ_OK : RBQ_EDEVICE;
}

rbq_status launch_quantize_flush(int32_t batch, int32_t heads_q, int32_t heads_kv, const float* q, const float* P,
                                 const float* c_q, const float* c_k, uint32_t* qplanes, float* qscal,
                                 const void* keys, int32_t keys_dtype, int64_t keys_ld, int32_t n_new, int32_t offset,
                                 int32_t cap, uint32_t* codes, float* kfac, hipStream_t stream, const int32_t* seq_off,
                                 const int32_t* seq_cnt, int32_t off_max, uint16_t* kfac16, int32_t head_dim) {
  if (n_new == 0)
    return launch_quantize(batch, heads_q, heads_kv, q, P, c_q, c_k, qplanes, qscal, nullptr, stream, 4, head_dim);
  const QuantArgs qa{q, P, c_q, c_k, qplanes, qscal, nullptr, heads_q, heads_kv, 15, 4};
  const EncodeArgs ea{keys,  keys_ld, n_new,   offset,  cap,     P,       c_q,     c_k,     codes,
                      kfac,  nullptr, nullptr, seq_off, seq_cnt, off_max, heads_kv, kfac16};
  const int rows = batch * heads_q, bhs = batch * heads_kv;
  const int per_head = encode_blocks_per_head(n_new, bhs);
  const int blocks = rows + per_head * bhs;
  const bool rg = seq_off != nullptr;
  if (head_dim == 64) {
    if (keys_dtype == RBQ_BF16) {
      if (rg)
        quantize_flush_kernel<RBQ_BF16, true, 64><<<blocks, kQAll, 0, stream>>>(qa, ea, rows, per_head);
      else
        quantize_flush_kernel<RBQ_BF16, false, 64><<<blocks, kQAll, 0, stream>>>(qa, ea, rows, per_head);
    } else {
      if (rg)
        quantize_flush_kernel<RBQ_F32, true, 64><<<blocks, kQAll, 0, stream>>>(qa, ea, rows, per_head);
      else
        quantize_flush_kernel<RBQ_F32, false, 64><<<blocks, kQAll, 0, stream>>>(qa, ea, rows, per_head);
    }
    return hipGetLastError() == hipSuccess ? RBQ_OK : RBQ_EDEVICE;
  }
  if (keys_dtype == RBQ_BF16) {
    if (rg)
      quantize_flush_kernel<RBQ_BF16, true><<<blocks, kQAll, 0, stream>>>(qa, ea, rows, per_head);
    else
      quantize_flush_kernel<RBQ_BF16, false><<<blocks, kQAll, 0, stream>>>(qa, ea, rows, per_head);
  } else {
    if (rg)
      quantize_flush_kernel<RBQ_F32, true><<<blocks, kQAll, 0, stream>>>(qa, ea, rows, per_head);
    else
      quantize_flush_kernel<RBQ_F32, false><<<blocks, kQAll, 0, stream>>>(qa, ea, rows, per_head);
  }
  return hipGetLastError() == hipSuccess ? RBQ_OK : RBQ_EDEVICE;
}

}  // namespace rbq
