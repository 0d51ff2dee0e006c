// Absorbed query in fp32: the body of one workgroup, shared by the stand-alone absorb kernel and the front kernel of
// an fp32 decode step.
#pragma once
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

// Workgroup = (64 latent columns or the RoPE part, head, 8 rows); four lanes share an output column and take 16-byte
// pieces of its row of W_K^(h) in turn, all requested before the queries are staged (one thread per column walking
// its own row was 5.0 us at 4 heads x 64, r = 64).
constexpr int kFrontRows = 8;
template <int DH4>  // d_head / 16: pieces per lane; 0: any d_head
__device__ __forceinline__ void absorb_f32_block(const AbsorbArgs& a, int bx, int h, int bz, float* sq) {
  const int tid = threadIdx.x, dh = a.d_head, r = a.r, dR = a.d_rope, E = r + dR;
  const int row0 = bz * kFrontRows, rows = a.rows - row0 < kFrontRows ? a.rows - row0 : kFrontRows;
  float* qcat = reinterpret_cast<float*>(a.qcat) + ((size_t)row0 * a.n_heads + h) * E;
  const size_t pitch = (size_t)a.n_heads * E;
  if (bx == r / 64) {  // RoPE part
    const float* qr = reinterpret_cast<const float*>(a.q_rope) + ((size_t)row0 * a.n_heads + h) * dR;
    for (int i = tid; i < rows * dR; i += kBlock)
      qcat[(size_t)(i / dR) * pitch + r + i % dR] = qr[(size_t)(i / dR) * a.n_heads * dR + i % dR] * a.scale_log2;
    return;
  }
  const int n = 64 * bx + (tid >> 2), q4 = tid & 3;
  const float* w = reinterpret_cast<const float*>(a.w_uk) + ((size_t)h * r + n) * dh + 4 * q4;
  float4 wv[DH4 > 0 ? DH4 : 1];
  if constexpr (DH4 > 0) {
#pragma unroll
    for (int i = 0; i < DH4; ++i) wv[i] = *reinterpret_cast<const float4*>(w + 16 * i);
  }
  const float* q = reinterpret_cast<const float*>(a.q) + ((size_t)row0 * a.n_heads + h) * dh;
  for (int i = tid; i < rows * dh / 4; i += kBlock)
    *reinterpret_cast<float4*>(sq + 4 * i) =
        *reinterpret_cast<const float4*>(q + (size_t)(4 * i / dh) * a.n_heads * dh + 4 * i % dh);
  __syncthreads();
  for (int row = 0; row < rows; ++row) {
    float dot = 0.f;
    auto piece = [&](const float4& x, int i) {
      const float4 y = *reinterpret_cast<const float4*>(sq + row * dh + 16 * i + 4 * q4);
      dot += x.x * y.x + x.y * y.y + x.z * y.z + x.w * y.w;
    };
    if constexpr (DH4 > 0) {
#pragma unroll
      for (int i = 0; i < DH4; ++i) piece(wv[i], i);
    } else {
      for (int i = 0; i < dh / 16; ++i) piece(*reinterpret_cast<const float4*>(w + 16 * i), i);
    }
    dot = group_reduce<4>(dot, LaneSum());
    if (q4 == 0) qcat[(size_t)row * pitch + n] = dot * a.scale_log2;
  }
}

}  // namespace mtla
