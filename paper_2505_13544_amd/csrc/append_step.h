// The append of a decode step: exactly one candidate token of one sequence, by the 256 threads of a workgroup.
#pragma once
#include "bounds.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

constexpr int kMaxRPerThread = 4;  // r <= 1024 with 256 threads
// d_hyper <= 256 (mtla_create): a thread of a workgroup holds at most one element of a row of the hyper-network's width

constexpr int kTPR = 4;                 // lanes sharing one hyper-network row
constexpr int kRowsPerPass = kBlock / kTPR;

// 8 consecutive elements of storage type T, kept raw until they are needed.
template <typename T>
struct Chunk8;
template <>
struct Chunk8<bf16> {
  uint4 raw;
  __device__ __forceinline__ void load(const bf16* p) { raw = *reinterpret_cast<const uint4*>(p); }
  __device__ __forceinline__ void store(bf16* p) const { *reinterpret_cast<uint4*>(p) = raw; }
  __device__ __forceinline__ void unpack(float (&o)[8]) const {
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};
template <>
struct Chunk8<float> {
  typedef float vec4 __attribute__((ext_vector_type(4)));  // (a float4 kept across the kernel's barriers ends up in scratch)
  vec4 lo, hi;
  __device__ __forceinline__ void load(const float* p) {
    lo = *reinterpret_cast<const vec4*>(p);
    hi = *reinterpret_cast<const vec4*>(p + 4);
  }
  __device__ __forceinline__ void store(float* p) const {
    *reinterpret_cast<vec4*>(p) = lo;
    *reinterpret_cast<vec4*>(p + 4) = hi;
  }
  __device__ __forceinline__ void unpack(float (&o)[8]) const {
    o[0] = lo.x; o[1] = lo.y; o[2] = lo.z; o[3] = lo.w;
    o[4] = hi.x; o[5] = hi.y; o[6] = hi.z; o[7] = hi.w;
  }
};

// Nothing but the positional branch G[slot] depends on the sequence position, so the
// length, the latent, the old tail, the key and the thread's pieces of hyp_A are all
// requested at once (NCH = pieces per thread of one hyp_A row, r / 32), and the G row as soon as the
// length, the first to arrive, is there: it travels while Linear(c) is formed (asked for behind it, it was a
// second trip to memory: 0.8 us of a step's 2.5 at r = 256, 1.0 of 4.9 at r = 512).
// TC = element type of c_new: the storage type, or float when the caller's projection hands the
// latent over unrounded (the merge and the hyper-network then see it in full precision and the cache
// row is rounded once).
template <typename T, int NCH, typename TC = T>
struct AppendStep {
  float told[kMaxRPerThread], cel[kMaxRPerThread];  // elements tid, tid + 256, .. of the tail shadow and of the latent
  Chunk8<T> krv, ach[NCH];
  float bias, g_pre;

  static __host__ __device__ size_t floats(const AppendArgs& a) { return (size_t)a.d_hyper + 4 + 8 + a.r; }  // of `smem`

  // What does not depend on the length.
  __device__ __forceinline__ void request(const AppendArgs& a, int b, int tid) {
    const int r = a.r, dR = a.d_rope, dy = a.d_hyper, q = tid & (kTPR - 1), y = tid / kTPR;
    const TC* crow = reinterpret_cast<const TC*>(a.c_new) + (size_t)b * r;
    const float* tail = a.tail_c ? a.tail_c + (size_t)b * r : nullptr;
#pragma unroll
    for (int i = 0; i < kMaxRPerThread; ++i) {
      const int e = tid + i * kBlock;
      told[i] = (tail && e < r) ? tail[e] : 0.f;
      cel[i] = e < r ? to_f32(crow[e]) : 0.f;
    }
    krv.load(reinterpret_cast<const T*>(a.kr_new) + (size_t)b * dR + 8 * (tid < dR / 8 ? tid : 0));  // stored by the first dR / 8 threads
    bias = 0.f;
    if (!a.w_override && y < dy) {
      const T* A = reinterpret_cast<const T*>(a.hyp_A);
      const T* ha = reinterpret_cast<const T*>(a.hyp_a);
#pragma unroll
      for (int i = 0; i < NCH; ++i) ach[i].load(A + (size_t)y * r + 8 * (q + i * kTPR));
      if (ha) bias = to_f32(ha[y]);
    }
  }
  // This thread's element of the slot's row of G.
  __device__ __forceinline__ void request_slot(const AppendArgs& a, int tid, int p0) {
    g_pre = 0.f;
    if (!a.w_override && tid < a.d_hyper) {
      const int slot_c = slots_inside(p0, a.stride, a.max_slots - 1);  // a full sequence, or a length below zero, is refused
      g_pre = to_f32(reinterpret_cast<const T*>(a.hyp_G)[(size_t)slot_c * a.d_hyper + tid]);
    }
  }
  // The merge weight; barriers inside.  smem: floats(a) floats.
  __device__ __forceinline__ float weight(const AppendArgs& a, int b, int tid, float* smem) {
    float* sg = smem;               // [dy] Linear(c)
    float* red = smem + a.d_hyper;  // [4]
    // [r] the latent as fp32 (normalised in the whole-layer call): the hyper-network's rows read it from
    // here instead of every thread holding its own copy of the pieces it needs (at r = 512 that copy was 64
    // registers, and with them the fused front kernel of a decode step fitted two workgroups per unit)
    float* sc_row = smem + a.d_hyper + 4 + 8;
    const int r = a.r, dy = a.d_hyper, q = tid & (kTPR - 1), y = tid / kTPR;
    const bool hyper = !a.w_override;
    const bool ln = sizeof(TC) == 4 && a.ln_eps > 0.f;  // whole-layer call: normalise the unrounded latent first
    // y = (v - mean) / sqrt(var + eps), two passes over the row in fp32; every thread ends up with the same mean and 1/sigma.
    if (ln) {
      const T* ln_g = reinterpret_cast<const T*>(a.ln_gamma);
      const T* ln_b = reinterpret_cast<const T*>(a.ln_beta);
      float* lred = smem + a.d_hyper + 4;  // [8]
      float part = 0.f;
#pragma unroll
      for (int i = 0; i < kMaxRPerThread; ++i) part += cel[i];
      part = wave_sum(part);
      if ((tid & (kWave - 1)) == 0) lred[tid / kWave] = part;
      __syncthreads();
      const float ln_mean = (lred[0] + lred[1] + lred[2] + lred[3]) / r;
      part = 0.f;
#pragma unroll
      for (int i = 0; i < kMaxRPerThread; ++i) {
        const int e = tid + i * kBlock;
        if (e < r) part += (cel[i] - ln_mean) * (cel[i] - ln_mean);
      }
      part = wave_sum(part);
      if ((tid & (kWave - 1)) == 0) lred[4 + tid / kWave] = part;
      __syncthreads();
      const float ln_inv = 1.0f / sqrtf((lred[4] + lred[5] + lred[6] + lred[7]) / r + a.ln_eps);
#pragma unroll
      for (int i = 0; i < kMaxRPerThread; ++i) {
        const int e = tid + i * kBlock;
        if (e < r) {
          cel[i] = (cel[i] - ln_mean) * ln_inv;
          if (ln_g) cel[i] *= to_f32(ln_g[e]);
          if (ln_b) cel[i] += to_f32(ln_b[e]);
        }
      }
    }
    if (hyper) {
#pragma unroll
      for (int i = 0; i < kMaxRPerThread; ++i) {
        const int e = tid + i * kBlock;
        if (e < r) sc_row[e] = cel[i];
      }
      __syncthreads();
      // ---- Linear(c), rows y < 64 from the registers, further rows (dy > 64) straight from memory
      const T* A = reinterpret_cast<const T*>(a.hyp_A);
      const T* ha = reinterpret_cast<const T*>(a.hyp_a);
      auto reduce = [&](float dot, int yy, float bia) {
        dot = group_reduce<4>(dot, LaneSum());
        if (yy < dy && q == 0) sg[yy] = dot + bia;
      };
      float dot = 0.f;
      if (y < dy) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
          float av[8], cv[8];
          ach[i].unpack(av);
          load8(sc_row + 8 * (q + i * kTPR), cv);
#pragma unroll
          for (int j = 0; j < 8; ++j) dot += av[j] * cv[j];
        }
      }
      reduce(dot, y, bias);
      for (int yy = y + kRowsPerPass; yy - y < dy; yy += kRowsPerPass) {
        dot = 0.f;
        if (yy < dy) {
          for (int i = 0; i < NCH; ++i) {
            float av[8], cv[8];
            load8(A + (size_t)yy * r + 8 * (q + i * kTPR), av);
            load8(sc_row + 8 * (q + i * kTPR), cv);
#pragma unroll
            for (int j = 0; j < 8; ++j) dot += av[j] * cv[j];
          }
        }
        reduce(dot, yy, yy < dy && ha ? to_f32(ha[yy]) : 0.f);
      }
    }
    __syncthreads();
    if (!hyper) return a.w_override[b];
    // the sum of hyper_logit, with the row already in registers
    float zp = tid < dy ? sg[tid] * g_pre : 0.f;
    zp = wave_sum(zp);
    if ((tid & (kWave - 1)) == 0) red[tid >> 6] = zp;
    __syncthreads();
    const float z = (red[0] + red[1]) + (red[2] + red[3]);
    return 1.f / (1.f + expf(-z));
  }
};

}  // namespace

}  // namespace mtla
