// mtla_cache_append kernels: hyper-network merge weight, then the temporal
// merge of the new latent into the strided cache (Section "Inference using
// MTLA": Eq. (infer-linear) and the update rule; RoPE-key rule of Section
// "Decoupled Rotary Position Embedding").
//
// Every cache row has exactly one writer.  A decode step (one token per sequence) is a single
// launch of `batch` workgroups that also advances seq_len (append_step_kernel).  A bulk append
// (prefix) runs one workgroup per (sequence, group of touched slots) with the hyper-network on
// the matrix cores (append_bulk_kernel, append_bulk_f32_kernel in prefill_front.hip) or one workgroup per touched slot
// (append_kernel, other hyper-network widths and strides), and a second tiny kernel advances seq_len once every workgroup has
// read the old value.
#include "absorb_f32.h"
#include "absorb_mfma.h"
#include "append_step.h"
#include "bounds.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

// Linear(c): sg[y] = a[y] + sum_n A[y][n] sc[n] for every row y < dy.  Four adjacent lanes
// share a row and take 8-element pieces round-robin (contiguous 64-byte reads of A,
// conflict-free reads of sc); all loads of a pass are issued before the first use.
template <typename T>
__device__ __forceinline__ void hyper_linear(const T* A, const T* ha, const float* sc, float* sg,
                                             int r, int dy, int tid) {
  const int q = tid & (kTPR - 1);
  for (int y0 = 0; y0 < dy; y0 += kRowsPerPass) {
    const int y = y0 + tid / kTPR;
    float dot = 0.f;
    if (y < dy) {
      const T* Arow = A + (size_t)y * r;
      for (int c8 = q; c8 < r / 8; c8 += kTPR) {
        float wv[8];
        load8(Arow + 8 * c8, wv);
#pragma unroll
        for (int j = 0; j < 8; ++j) dot += wv[j] * sc[8 * c8 + j];
      }
    }
    dot = group_reduce<4>(dot, LaneSum());
    if (y < dy && q == 0) sg[y] = dot + (ha ? to_f32(ha[y]) : 0.f);
  }
}

// <Linear(c), Linear(pe_j)> = sum_y sg[y] G[slot][y], reduced over the workgroup; red: [4] floats.
template <typename T>
__device__ __forceinline__ float hyper_logit(const float* sg, const T* Grow, float* red, int dy, int tid) {
  float zp = tid < dy ? sg[tid] * to_f32(Grow[tid]) : 0.f;
  zp = wave_sum(zp);
  if ((tid & (kWave - 1)) == 0) red[tid >> 6] = zp;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// One workgroup per sequence.
template <typename T, int NCH, typename TC = T>
__device__ __forceinline__ void append_step_block(const AppendArgs& a, int b, float* smem) {
  const int tid = threadIdx.x, s = a.stride, r = a.r, dR = a.d_rope;
  AppendStep<T, NCH, TC> st;
  const int p0 = a.seq_len[b];
  const int n = a.n_new ? a.n_new[b] : 1;
  st.request(a, b, tid);
  st.request_slot(a, tid, p0);
  const float w = st.weight(a, b, tid, smem);
  if (n < 1) return;
  if (const int refused = append_status(p0, 1, s, a.max_slots)) {
    if (tid == 0) *a.status = refused;
    return;
  }
  const int slot = p0 / s;
  const bool continuing = (p0 - slot * s) != 0;
  float* tail = a.tail_c ? a.tail_c + (size_t)b * r : nullptr;
  T* crow_out = reinterpret_cast<T*>(a.cache_c) + cache_row(a.pages, b, slot, a.max_slots) * r;
#pragma unroll
  for (int i = 0; i < kMaxRPerThread; ++i) {
    const int e = tid + i * kBlock;
    if (e < r) {
      const float old = continuing ? (tail ? st.told[i] : to_f32(crow_out[e])) : 0.f;
      const float v = old + w * st.cel[i];
      crow_out[e] = from_f32<T>(v);
      if (tail) tail[e] = v;
    }
  }
  if (tid < dR / 8) st.krv.store(reinterpret_cast<T*>(a.cache_kr) + cache_row(a.pages, b, slot, a.max_slots) * dR + 8 * tid);
  if (tid == 0) {
    if (a.w_out) a.w_out[b] = w;
    if (a.slot_out) a.slot_out[b] = slot;
    a.seq_len[b] = p0 + 1;  // every thread took p0 before the barrier
  }
}

template <typename T, int NCH>
__global__ __launch_bounds__(kBlock) void append_step_kernel(AppendArgs a) {
  extern __shared__ float smem[];
  append_step_block<T, NCH>(a, blockIdx.x, smem);
}

// Front of a fused decode step (bf16 storage): the two things the pass over the cache waits
// for, neither of which needs the other -- the append of the step's token (workgroups below
// `batch`) and the absorbed queries (the rest, numbered like the absorb kernel's grid) -- in one
// launch, so a step pays one kernel start and one round trip to memory for both.
// Four workgroups per unit (128 registers, and with heads of 128 exactly a quarter of its LDS): what a step of 256 sequences launches is then resident at
// once.  The whole-layer call's queries are fp32 and take twice the room: heads of 128 come to 48 KB a workgroup, three of them.
template <int NCH, int KK, typename TC>
__global__ __launch_bounds__(kBlock, 4) void decode_front_kernel(AppendArgs ap, AbsorbArgs ab, int gx, int gy) {
  extern __shared__ float smem[];
  const int blk = blockIdx.x;
  if (blk < ap.batch) {
    append_step_block<bf16, NCH, TC>(ap, blk, smem);
    return;
  }
  const int i = blk - ap.batch;
  const int bx = i % gx, rest = i / gx;
  absorb_mfma_block<KK, sizeof(TC) == 4>(ab, bx, rest % gy, rest / gy, reinterpret_cast<unsigned char*>(smem));  // the whole-layer call hands q, q^R and c over unrounded
}

// Front of an fp32 decode step, split the same way (the append as a launch of its own took 3.1 us and the absorption
// behind it 5.0 us at 4 heads x 64, r = 64).
template <int NCH, int DH4>
__global__ __launch_bounds__(kBlock) void decode_front_f32_kernel(AppendArgs ap, AbsorbArgs ab, int gx, int gy) {
  extern __shared__ float smem[];
  const int blk = blockIdx.x;
  if (blk < ap.batch) {
    append_step_block<float, NCH>(ap, blk, smem);
    return;
  }
  const int i = blk - ap.batch, rest = i / gx;
  absorb_f32_block<DH4>(ab, i % gx, rest % gy, rest / gy, smem);
}

// One slot of a bulk append: tokens [t_lo, t_hi) of the call fold into `slot` of sequence b.
// Called by every thread of the workgroup (barriers inside).
template <typename T>
__device__ __forceinline__ void append_slot(const AppendArgs& a, int b, int p0, int n, int slot, float* smem) {
  float* sc = smem;              // [r] current token's latent in fp32
  float* sg = smem + a.r;        // [dy] Linear(c)
  float* red = sg + a.d_hyper;   // [4] per-wave partial of the hyper-network logit
  const int tid = threadIdx.x;
  const int s = a.stride, r = a.r, dR = a.d_rope, dy = a.d_hyper;
  const long long slot_first = (long long)slot * s;
  const int t_lo = int((slot_first > p0 ? slot_first : (long long)p0) - p0);
  const long long slot_end = slot_first + s;
  const int t_hi = int((slot_end < (long long)p0 + n ? slot_end : (long long)p0 + n) - p0);

  T* crow_out = reinterpret_cast<T*>(a.cache_c) + cache_row(a.pages, b, slot, a.max_slots) * r;
  float* tail = a.tail_c ? a.tail_c + (size_t)b * r : nullptr;
  const T* A = reinterpret_cast<const T*>(a.hyp_A);
  const T* ha = reinterpret_cast<const T*>(a.hyp_a);
  const T* G = reinterpret_cast<const T*>(a.hyp_G);

  float acc[kMaxRPerThread];
  const bool continuing = slot_first < p0;  // the slot already holds earlier tokens
#pragma unroll
  for (int i = 0; i < kMaxRPerThread; ++i) {
    const int e = tid + i * kBlock;
    acc[i] = 0.f;
    if (continuing && e < r) acc[i] = tail ? tail[e] : to_f32(crow_out[e]);
  }

  for (int t = t_lo; t < t_hi; ++t) {
    const size_t tok = (size_t)b * a.n_new_max + t;
    const T* crow = reinterpret_cast<const T*>(a.c_new) + tok * r;
#pragma unroll
    for (int i = 0; i < kMaxRPerThread; ++i) {
      const int e = tid + i * kBlock;
      if (e < r) sc[e] = to_f32(crow[e]);
    }
    __syncthreads();
    float w;
    if (a.w_override) {
      w = a.w_override[tok];
    } else {
      hyper_linear(A, ha, sc, sg, r, dy, tid);
      __syncthreads();
      const float z = hyper_logit(sg, G + (size_t)slot * dy, red, dy, tid);
      w = 1.f / (1.f + expf(-z));
    }
#pragma unroll
    for (int i = 0; i < kMaxRPerThread; ++i) {
      const int e = tid + i * kBlock;
      if (e < r) acc[i] += w * sc[e];
    }
    if (tid == 0) {
      if (a.w_out) a.w_out[tok] = w;
      if (a.slot_out) a.slot_out[tok] = slot;
    }
    __syncthreads();  // sc / red are rewritten by the next token
  }

  const bool is_open_slot = (t_hi == n);  // last slot touched: remains the sequence's tail
#pragma unroll
  for (int i = 0; i < kMaxRPerThread; ++i) {
    const int e = tid + i * kBlock;
    if (e < r) {
      crow_out[e] = from_f32<T>(acc[i]);
      if (tail && is_open_slot) tail[e] = acc[i];
    }
  }
  // RoPE key: the slot keeps the key of the newest token folded into it.
  const T* kr_src = reinterpret_cast<const T*>(a.kr_new) + ((size_t)b * a.n_new_max + (t_hi - 1)) * dR;
  T* kr_dst = reinterpret_cast<T*>(a.cache_kr) + cache_row(a.pages, b, slot, a.max_slots) * dR;
  for (int e = tid; e < dR; e += kBlock) kr_dst[e] = kr_src[e];
}

// Bulk append, any storage type: one workgroup per (sequence, slot touched), tokens of the slot in
// order.  The tail shadow is read by the first slot of a call and written by the last: workgroup 0
// of the sequence takes both, one after the other, so the read precedes the write.
template <typename T>
__global__ __launch_bounds__(kBlock) void append_kernel(AppendArgs a) {
  extern __shared__ float smem[];
  const int b = blockIdx.y, kslot = blockIdx.x, s = a.stride;
  const int p0 = a.seq_len[b];
  int n = a.n_new ? a.n_new[b] : a.n_new_max;
  n = n < 0 ? 0 : (n > a.n_new_max ? a.n_new_max : n);
  if (n == 0) return;
  if (const int refused = append_status(p0, n, s, a.max_slots)) {
    if (kslot == 0 && threadIdx.x == 0) *a.status = refused;
    return;
  }
  const int first_slot = p0 / s, last_slot = int(((long long)p0 + n - 1) / s);
  const int slot = first_slot + kslot;
  if (slot < last_slot || (slot == last_slot && kslot == 0)) append_slot<T>(a, b, p0, n, slot, smem);
  if (kslot == 0 && last_slot > first_slot) append_slot<T>(a, b, p0, n, last_slot, smem);
}

__global__ void advance_len_kernel(AppendArgs a) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= a.batch) return;
  const int p0 = a.seq_len[b];
  int n = a.n_new ? a.n_new[b] : a.n_new_max;
  n = n < 0 ? 0 : (n > a.n_new_max ? a.n_new_max : n);
  if (append_status(p0, n, a.stride, a.max_slots) == 0) a.seq_len[b] = p0 + n;
}

__global__ void fill_zero_kernel(int32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Plain streaming read for benchmarks: every workgroup walks its own contiguous share of the buffer
// with 16-byte loads, two 16 KB pieces per wavefront in flight, and folds what it reads into one word.
__global__ __launch_bounds__(kBlock) void stream_read_kernel(const uint4* __restrict__ p, size_t n_vec, uint32_t* out) {
  const size_t per = (n_vec + gridDim.x - 1) / gridDim.x;
  const size_t lo = blockIdx.x * per, hi = lo + per < n_vec ? lo + per : n_vec;
  uint32_t acc = 0;
  for (size_t i = lo + threadIdx.x; i < hi; i += 8 * kBlock) {
    uint4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const size_t j = i + (size_t)u * kBlock;
      v[u] = p[j < hi ? j : hi - 1];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  if (acc == 0x9e3779b9u) *out = acc;  // keeps the loads alive; practically never taken
}

}  // namespace

// 16 bytes in registers.  (An array of HIP's uint4 kept across a loop body's branches goes to scratch or LDS.)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Beam reordering of the sequence state: a gather of whole sequences.  Workgroup (x, b) copies every
// gridDim.x-th run of 256 16-byte pieces of the live rows of source sequence src_index[b] (four
// loads in flight per thread); workgroup (0, b) also copies the tail shadow and the length.
__global__ __launch_bounds__(kBlock) void reorder_kernel(ReorderArgs a) {
  const int b = blockIdx.y, tid = threadIdx.x;
  const int src = a.src_index[b];
  if (src < 0 || src >= a.max_batch) {  // refuse: destination sequence untouched
    if (blockIdx.x == 0 && tid == 0) *a.status = 1;  // MTLA_ERR_INVALID_ARG
    return;
  }
  const int len = a.src_len[src];
  const int live = live_slots(len, a.stride, a.max_slots);
  const size_t row_c = (size_t)a.max_slots * a.r * a.elem, row_kr = (size_t)a.max_slots * a.d_rope * a.elem;
  const u32x4* sc = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(a.src_c) + src * row_c);
  const u32x4* sk = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(a.src_kr) + src * row_kr);
  u32x4* dc = reinterpret_cast<u32x4*>(reinterpret_cast<char*>(a.dst_c) + b * row_c);
  u32x4* dk = reinterpret_cast<u32x4*>(reinterpret_cast<char*>(a.dst_kr) + b * row_kr);
  // slots first_slot .. live-1 (rows are multiples of 16 bytes)
  const int first = a.first_slot < live ? a.first_slot : live;
  const size_t o_c = (size_t)first * a.r * a.elem / 16, o_k = (size_t)first * a.d_rope * a.elem / 16;
  sc += o_c;
  dc += o_c;
  sk += o_k;
  dk += o_k;
  const size_t n_c = (size_t)(live - first) * a.r * a.elem / 16, n_k = (size_t)(live - first) * a.d_rope * a.elem / 16;
  const size_t step = (size_t)gridDim.x * kBlock;
  for (size_t i = (size_t)blockIdx.x * kBlock + tid; i < n_c + n_k; i += 4 * step) {
    u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t j = i + u * step;
      const size_t jj = j < n_c + n_k ? j : n_c + n_k - 1;  // past the end: read and dropped (a guarded read sends v to scratch)
      v[u] = jj < n_c ? sc[jj] : sk[jj - n_c];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t j = i + u * step;
      if (j < n_c + n_k) {
        if (j < n_c) dc[j] = v[u];
        else dk[j - n_c] = v[u];
      }
    }
  }
  if (blockIdx.x == 0) {
    if (a.src_tail && a.dst_tail)
      for (int e = tid; e < a.r; e += kBlock) a.dst_tail[(size_t)b * a.r + e] = a.src_tail[(size_t)src * a.r + e];
    if (tid == 0) a.dst_len[b] = len;
  }
}

// Beam reordering over paged storage: one workgroup per destination sequence.  Pages below the one the
// next token will be written to are complete and never change again: the destination's table row takes the
// source's entries for them.  That page becomes the destination's fresh page; the source's live rows of it
// (at most one page, none when the next token opens a page) are copied over, unless the destination takes the
// source's own page over (fresh page = the source's page: nothing to copy, for the one destination that does).
__global__ __launch_bounds__(kBlock) void fork_paged_kernel(ForkArgs a) {
  const int b = blockIdx.y, part = blockIdx.x, n_parts = gridDim.x, tid = threadIdx.x;  // the copy is dealt over n_parts workgroups
  const int src = a.src_index[b];
  int fresh = a.fresh[b];
  if (src < 0 || src >= a.max_batch) {  // refuse: destination untouched
    if (part == 0 && tid == 0) *a.status = 1;  // MTLA_ERR_INVALID_ARG
    return;
  }
  const int len = a.src_len[src];
  const int live = live_slots(len, a.stride, a.max_slots);
  const int P = 1 << a.src.shift;
  const int next_slot = len > 0 ? len / a.stride : 0;           // the slot the next token goes into
  const int pw = (next_slot < a.max_slots ? next_slot : a.max_slots - 1) >> a.src.shift;
  const int32_t* srow = a.src.table + (size_t)src * a.src.max_pages;
  int sp = srow[pw];  // requested before it is known whether the page holds live rows (any entry is readable)
  if (fresh < 0 || fresh >= a.src.n_pages) {
    if (part == 0 && tid == 0) *a.status = 1;
    fresh = fresh < 0 ? 0 : a.src.n_pages - 1;
  }
  if (part == 0) {
    int32_t* drow = a.dst_table + (size_t)b * a.src.max_pages;
    for (int k = tid; k < pw; k += kBlock) drow[k] = srow[k];
    if (tid == 0) {
      drow[pw] = fresh;
      a.dst_len[b] = len;
    }
    for (int e = tid; e < a.r; e += kBlock) a.dst_tail[(size_t)b * a.r + e] = a.src_tail[(size_t)src * a.r + e];
  }
  const int n_rows = live - pw * P;  // live rows of the page being written to (<= P)
  if (n_rows <= 0) return;
  sp = sp < 0 ? 0 : (sp < a.src.n_pages ? sp : a.src.n_pages - 1);
  if (sp == fresh) return;           // the destination takes the source's page over
  const size_t n_c = (size_t)n_rows * a.r / 8, n_k = (size_t)n_rows * a.d_rope / 8;  // 16-byte pieces (bf16)
  const u32x4* sc = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(a.cache_c) + (size_t)sp * P * a.r);
  const u32x4* sk = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(a.cache_kr) + (size_t)sp * P * a.d_rope);
  u32x4* dc = reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(a.cache_c) + (size_t)fresh * P * a.r);
  u32x4* dk = reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(a.cache_kr) + (size_t)fresh * P * a.d_rope);
  constexpr int U = 8;  // pieces in flight per thread
  const size_t step = (size_t)n_parts * kBlock;
  for (size_t i = (size_t)part * kBlock + tid; i < n_c + n_k; i += U * step) {
    u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t j = i + (size_t)u * step;
      const size_t jj = j < n_c + n_k ? j : n_c + n_k - 1;  // past the end: read and dropped (a guarded read sends v to scratch)
      v[u] = jj < n_c ? sc[jj] : sk[jj - n_c];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t j = i + (size_t)u * step;
      if (j < n_c + n_k) {
        if (j < n_c) dc[j] = v[u];
        else dk[j - n_c] = v[u];
      }
    }
  }
}

hipError_t launch_fork_paged(const ForkArgs& a, hipStream_t st) {
  const size_t page_bytes = ((size_t)a.r + a.d_rope) * 2 << a.src.shift;
  size_t parts = (page_bytes + (16u << 10) - 1) / (16u << 10);  // about 16 KB of a page per workgroup
  parts = parts < 1 ? 1 : (parts > 16 ? 16 : parts);
  hipLaunchKernelGGL(fork_paged_kernel, dim3((unsigned)parts, a.batch), dim3(kBlock), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_reorder(const ReorderArgs& a, hipStream_t st) {
  const size_t seq_bytes = (size_t)a.max_slots * (a.r + a.d_rope) * a.elem;
  size_t nx = (seq_bytes + (64u << 10) - 1) / (64u << 10);  // about 64 KB per workgroup and pass
  nx = nx < 1 ? 1 : (nx > 64 ? 64 : nx);
  hipLaunchKernelGGL(reorder_kernel, dim3((unsigned)nx, a.batch), dim3(kBlock), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_stream_read(const void* p, size_t bytes, int32_t* out, int workgroups, hipStream_t st) {
  hipLaunchKernelGGL(stream_read_kernel, dim3(workgroups), dim3(kBlock), 0, st, reinterpret_cast<const uint4*>(p),
                     bytes / 16, reinterpret_cast<uint32_t*>(out));
  return hipGetLastError();
}

hipError_t launch_fill_zero(int32_t* p, int n, hipStream_t st) {
  hipLaunchKernelGGL(fill_zero_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

bool decode_front_supported(const AppendArgs& ap, const AbsorbArgs& ab) {
  const bool nch = ap.r == 64 || ap.r == 128 || ap.r == 256 || ap.r == 512;
  const bool kk = ab.d_head == 32 || ab.d_head == 64 || ab.d_head == 128;
  return nch && kk && ab.out_bf16 && ap.n_new_max == 1 && ab.rows == ap.batch;
}

hipError_t launch_decode_front(const AppendArgs& ap, const AbsorbArgs& ab, hipStream_t st) {
  const int gx = absorb_col_blocks(ab.r) + 1, gy = ab.n_heads;
  const int gz = (ab.rows + absorb_rows_per_block(ab.rows) - 1) / absorb_rows_per_block(ab.rows);
  const dim3 grid(ap.batch + gx * gy * gz), block(kBlock);
  const size_t append = AppendStep<bf16, 1>::floats(ap) * sizeof(float);
#define MTLA_FRONT(N, K)                                                                                \
  if (ap.r == 32 * N && ab.d_head == 32 * K) {                                                          \
    const size_t absorb = ap.c_new_f32 ? AbsorbLds<K, true>::bytes : AbsorbLds<K, false>::bytes, smem = append > absorb ? append : absorb; \
    if (ap.c_new_f32)                                                                                   \
      hipLaunchKernelGGL((decode_front_kernel<N, K, float>), grid, block, smem, st, ap, ab, gx, gy);    \
    else                                                                                                \
      hipLaunchKernelGGL((decode_front_kernel<N, K, bf16>), grid, block, smem, st, ap, ab, gx, gy);     \
    return hipGetLastError();                                                                           \
  }
  MTLA_FRONT(2, 1) MTLA_FRONT(2, 2) MTLA_FRONT(2, 4)
  MTLA_FRONT(4, 1) MTLA_FRONT(4, 2) MTLA_FRONT(4, 4)
  MTLA_FRONT(8, 1) MTLA_FRONT(8, 2) MTLA_FRONT(8, 4)
  MTLA_FRONT(16, 1) MTLA_FRONT(16, 2) MTLA_FRONT(16, 4)
#undef MTLA_FRONT
  return hipErrorInvalidValue;
}

hipError_t launch_decode_front_f32(const AppendArgs& ap, const AbsorbArgs& ab, hipStream_t st) {
  const int gx = ab.r / 64 + 1, gy = ab.n_heads, gz = (ab.rows + kFrontRows - 1) / kFrontRows;
  const dim3 grid(ap.batch + gx * gy * gz), block(kBlock);
  const size_t append_f = AppendStep<float, 1>::floats(ap), absorb_f = (size_t)kFrontRows * ab.d_head;
  const size_t smem = (append_f > absorb_f ? append_f : absorb_f) * sizeof(float);
#define MTLA_FRONT(N)                                                                                           \
  if (ap.r == 32 * N) {                                                                                         \
    switch (ab.d_head / 32) {                                                                                   \
      case 1: hipLaunchKernelGGL((decode_front_f32_kernel<N, 2>), grid, block, smem, st, ap, ab, gx, gy); break;   \
      case 2: hipLaunchKernelGGL((decode_front_f32_kernel<N, 4>), grid, block, smem, st, ap, ab, gx, gy); break;   \
      case 4: hipLaunchKernelGGL((decode_front_f32_kernel<N, 8>), grid, block, smem, st, ap, ab, gx, gy); break;   \
      default: hipLaunchKernelGGL((decode_front_f32_kernel<N, 0>), grid, block, smem, st, ap, ab, gx, gy); break;  \
    }                                                                                                           \
    return hipGetLastError();                                                                                   \
  }
  MTLA_FRONT(2) MTLA_FRONT(4) MTLA_FRONT(8) MTLA_FRONT(16)
#undef MTLA_FRONT
  return hipErrorInvalidValue;
}

hipError_t launch_append(const AppendArgs& a, int dtype, hipStream_t st) {
  const size_t smem = (size_t)(a.r + a.d_hyper + 4) * sizeof(float);
  if (a.n_new_max == 1) {  // decode step: one workgroup per sequence, advances seq_len itself
    const size_t smem1 = AppendStep<float, 1>::floats(a) * sizeof(float);
    const dim3 grid(a.batch), block(kBlock);
#define MTLA_STEP(TT, N)                                                            \
  if (a.r == 32 * N) {                                                               \
    hipLaunchKernelGGL((append_step_kernel<TT, N>), grid, block, smem1, st, a);      \
    return hipGetLastError();                                                        \
  }
    if (dtype == 0) {
      MTLA_STEP(float, 2) MTLA_STEP(float, 4) MTLA_STEP(float, 8) MTLA_STEP(float, 16)
    } else {
      MTLA_STEP(bf16, 2) MTLA_STEP(bf16, 4) MTLA_STEP(bf16, 8) MTLA_STEP(bf16, 16)
    }
#undef MTLA_STEP
    return hipErrorInvalidValue;
  }
  // slots a call can touch per sequence: a partly filled first slot plus the rest
  const int n_slots = (a.n_new_max + a.stride - 2) / a.stride + 1;
  const dim3 grid(n_slots, a.batch), block(kBlock);
  if (append_bulk_supported(a, dtype)) {
    const hipError_t e = launch_append_bulk(a, dtype, st);
    if (e != hipSuccess) return e;
  } else if (dtype == 0)
    hipLaunchKernelGGL(append_kernel<float>, grid, block, smem, st, a);
  else
    hipLaunchKernelGGL(append_kernel<bf16>, grid, block, smem, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(advance_len_kernel, dim3((a.batch + 255) / 256), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace mtla
