// The query quantisation's device code (see quantize.hip), shared with the fused
// quantisation and scan of small launches (score.hip).
#pragma once

#include "rbq_device.h"

namespace rbq {

constexpr int kQAll = 256;            // threads per block
// The matrix-vector product is split over kQAll / D thread groups (2 at D = 128, 4 at D = 64).
template <int D>
struct QShape {
  static constexpr int kQParts = kQAll / D;
};

// The code of one rotated component, every operation rounded on its own.
__device__ __forceinline__ int quant_code(float x, float ql, float delta, float top) {
#pragma clang fp contract(off)
  if (!(delta > 0.f)) return 0;
  const float t = __fdiv_rn(__fsub_rn(x, ql), delta);
  float r = floorf(__fadd_rn(t, 0.5f));
  r = fminf(fmaxf(r, 0.f), top);
  return int(r);
}

struct QuantArgs {
  const float* q;
  const float* P;
  const float* c_q;      // or NULL
  const float* c_k;
  uint32_t* qplanes;
  float* qscal;
  float* qrot_out;       // or NULL
  int Hq, Hkv;
  int levels;            // 2^B_q - 1
  int planes;            // bit-planes written per head: 4 (B_q <= 4) or 8
};

// The last stage of head `row`, one wave: the rotated components from the thread
// groups' shares, the codes, their bit-planes and the scalars (A and B0 given).
template <int D>
struct QuantRow {
  uint64_t bal[8][D / kWave];   // bit-plane m of dimensions 64 t .. + 64
  float ql, qr, delta;
  int su;
  // lane l < RBQ_QSCAL_STRIDE: scalar l
  __device__ __forceinline__ float scalar(int l, float A, float B0) const {
    return l == 0 ? ql : l == 1 ? delta : l == 2 ? float(su) : l == 3 ? A : l == 4 ? B0 : l == 5 ? qr : 0.f;
  }
};
template <int D>
__device__ __forceinline__ QuantRow<D> quantize_finish(const QuantArgs& qa, int row, const float (*part_s)[D],
                                                       float A, float B0, bool store) {
  constexpr int T = D / kWave, W = D / 32, kQParts = QShape<D>::kQParts;   // (W words per bit-plane)
  const int lane = lane_id();
  QuantRow<D> o;
  float r[T], ql, qr;
#pragma unroll
  for (int t = 0; t < T; ++t) {   // (the groups' shares in a fixed order)
    r[t] = part_s[0][t * kWave + lane];
#pragma unroll
    for (int p = 1; p < kQParts; ++p) r[t] += part_s[p][t * kWave + lane];
    if (qa.qrot_out) qa.qrot_out[int64_t(row) * D + t * kWave + lane] = r[t];
    ql = t ? fminf(ql, r[t]) : r[t];
    qr = t ? fmaxf(qr, r[t]) : r[t];
  }
  o.ql = wave_min(ql);
  o.qr = wave_max(qr);
  {
#pragma clang fp contract(off)
    o.delta = __fdiv_rn(__fsub_rn(o.qr, o.ql), float(qa.levels));
  }
  int code[T];
#pragma unroll
  for (int t = 0; t < T; ++t) code[t] = quant_code(r[t], o.ql, o.delta, float(qa.levels));

  // the ballot's low half is word 2 t of the plane, its high half word 2 t + 1
  uint32_t* planes = qa.qplanes + int64_t(row) * qa.planes * W;
  o.su = 0;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    if (m >= qa.planes) break;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const uint64_t bal = __ballot((code[t] >> m) & 1);
      o.bal[m][t] = bal;
      o.su += int(__popcll(bal)) << m;
      if (store && lane == 0)
        *reinterpret_cast<u32x2*>(planes + m * W + 2 * t) = u32x2{uint32_t(bal), uint32_t(bal >> 32)};
    }
  }
  if (store && lane < RBQ_QSCAL_STRIDE)
    qa.qscal[int64_t(row) * RBQ_QSCAL_STRIDE + lane] = o.scalar(lane, A, B0);
  return o;
}

}  // namespace rbq
