// 16-bit path, what is neither a contraction nor a GEMM epilogue: weight re-layout, embedding gather,
// cache compaction and the plain <-> fragment layout conversions.  Number formats: see bf16_layout.h.
#include <algorithm>

#include "bf16_layout.h"
#include "ded_kernels.h"
#include "step_ends.h"

namespace ded {

namespace {

__device__ inline float wave_sum(float v) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
__device__ inline float block_sum_256(float v, float* sh) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}

struct F8 {
  float v[8];
};
__device__ inline F8 load8(const float* p) {
  F8 r;
  float4 a = *reinterpret_cast<const float4*>(p);
  float4 b = *reinterpret_cast<const float4*>(p + 4);
  r.v[0] = a.x; r.v[1] = a.y; r.v[2] = a.z; r.v[3] = a.w;
  r.v[4] = b.x; r.v[5] = b.y; r.v[6] = b.z; r.v[7] = b.w;
  return r;
}
__device__ inline void store8(float* p, const F8& r) {
  *reinterpret_cast<float4*>(p) = make_float4(r.v[0], r.v[1], r.v[2], r.v[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(r.v[4], r.v[5], r.v[6], r.v[7]);
}
__device__ inline uint32_t pk(uint16_t lo, uint16_t hi) { return (uint32_t)lo | ((uint32_t)hi << 16); }
// eight floats -> hi and lo planes
__device__ inline void to_f16x8_split(const F8& r, uint4& hi, uint4& lo) {
  uint16_t h[8], l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) split_f16(r.v[i], h[i], l[i]);
  hi = make_uint4(pk(h[0], h[1]), pk(h[2], h[3]), pk(h[4], h[5]), pk(h[6], h[7]));
  lo = make_uint4(pk(l[0], l[1]), pk(l[2], l[3]), pk(l[4], l[5]), pk(l[6], l[7]));
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Source feature of packed feature n (see PERM_* in ded_kernels.h).  F = half the row count for PERM_GATE_UP.
__device__ inline int packw_source_row(int n, int perm, int F) {
  if (perm == PERM_NONE) return n;
  const int t = (n >> 4) & 3, e = n & 15;
  if (perm == PERM_ROPE) {  // per 128-dim head: group j holds dims [32j, 32j+32) and their partners + 64
    const int head = n >> 7, j = (n >> 6) & 1;
    const int dim = 32 * j + 16 * (t & 1) + e + (t >= 2 ? 64 : 0);
    return head * 128 + dim;
  }
  const int f = 32 * (n >> 6) + 16 * (t & 1) + e;  // PERM_GATE_UP: gate f in tiles 0,1, up f in tiles 2,3
  return t >= 2 ? F + f : f;
}

// dst: PackW (f16) with the feature count padded to a multiple of 64 (padding features are zero)
__global__ void pack_weight_kernel(uint4* __restrict__ dst, const bf16_t* __restrict__ src, int N, int K, int perm) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // destination 16-byte unit
  int64_t total = (int64_t)((N + 63) / 64 * 64) * K / 8;
  if (u >= total) return;
  int lane = (int)(u & 63);
  int64_t frag = u >> 6;
  int KT = K >> 5;
  int t = (int)(frag % PACKW_TILES);
  int64_t gk = frag / PACKW_TILES;
  int kt = (int)(gk % KT), ng = (int)(gk / KT);
  int n = ng * 64 + t * 16 + (lane & 15);
  int k = kt * 32 + (lane >> 4) * 8;
  uint4 out = make_uint4(0, 0, 0, 0);
  if (n < N) {
    int row = packw_source_row(n, perm, N / 2);
    uint4 in = *reinterpret_cast<const uint4*>(src + (int64_t)row * K + k);
    uint32_t w[4] = {in.x, in.y, in.z, in.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = pk(bf16_to_f16((uint16_t)(w[i] & 0xffffu)), bf16_to_f16((uint16_t)(w[i] >> 16)));
    out = make_uint4(w[0], w[1], w[2], w[3]);
  }
  dst[u] = out;
}
void bf16_pack_weight(bf16_t* dst, const bf16_t* src, int N, int K, int perm, hipStream_t s) {
  int64_t units = (int64_t)((N + 63) / 64 * 64) * K / 8;
  hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<uint4*>(dst), src, N, K, perm);
}

// ------------------------------------------------------------------------------------------
// Embedding gather: x = emb[token] (fp32 residual stream), y = (x * gain) as hi/lo f16 in PackX for the first
// GEMM, ssq[r][g] = sum of x^2 over the 64 features of group g (the consumer turns that into 1/rms).  The workgroups behind
// those of the rows do the step's front work.
__global__ __launch_bounds__(256) void bf16_embed_kernel(float* __restrict__ x, uint4* __restrict__ y,
                                                         float* __restrict__ ssq, const bf16_t* __restrict__ emb,
                                                         const float* __restrict__ gain, StepFront f, int RB, int d) {
  int r = blockIdx.x;
  if (r >= RB * 16) {
    step_front(f, r - RB * 16);
    return;
  }
  const bool real = r < f.rows;  // padding rows (up to the 64-row granule of the GEMMs) are cleared
  const bf16_t* src = emb + (int64_t)(real ? f.token[r] : 0) * d;
  for (int u = threadIdx.x; u < d / 8; u += 256) {  // d % 64 == 0: whole wavefront iterations only
    uint4 in = real ? *reinterpret_cast<const uint4*>(src + u * 8) : make_uint4(0, 0, 0, 0);
    uint32_t w[4] = {in.x, in.y, in.z, in.w};
    F8 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v.v[2 * i] = bf16_to_f32((uint16_t)(w[i] & 0xffffu));
      v.v[2 * i + 1] = bf16_to_f32((uint16_t)(w[i] >> 16));
    }
    store8(x + (int64_t)r * d + u * 8, v);
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) ss += v.v[i] * v.v[i];
    ss += __shfl_xor(ss, 1);  // 8 consecutive lanes = one 64-feature group
    ss += __shfl_xor(ss, 2);
    ss += __shfl_xor(ss, 4);
    if ((threadIdx.x & 7) == 0) ssq[(int64_t)r * (d / 64) + (u >> 3)] = ss;
    F8 g = load8(gain + u * 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) v.v[i] *= g.v[i];
    uint4 hi, lo;
    to_f16x8_split(v, hi, lo);
    y[packx_index(r, u * 8, RB, 0) >> 3] = hi;
    y[packx_index(r, u * 8, RB, 1) >> 3] = lo;
  }
}
void bf16_embed(float* x, bf16_t* y_packed, float* ssq, const bf16_t* emb, const float* gain, const StepFront& f,
                int rows_pad, int d, hipStream_t s) {
  hipLaunchKernelGGL(bf16_embed_kernel, dim3(rows_pad + step_front_blocks(f)), dim3(256), 0, s, x,
                     reinterpret_cast<uint4*>(y_packed), ssq, emb, gain, f, rows_pad / 16, d);
}

// ------------------------------------------------------------------------------------------
// Compaction in the fragment layouts.  Threads 0..15 move the sixteen 16-byte key units of a slot,
// threads 16..143 one value element each; every thread walks the path upwards (see the fp32 kernel).  Every workgroup does
// the approval walk of its sequence itself; the first of the sequence reports it.
__global__ __launch_bounds__(256) void bf16_kv_compact_kernel(bf16_t* const* __restrict__ kc, bf16_t* const* __restrict__ vc,
                                                              ApprovalWalk w, const int32_t* __restrict__ seq_p, int Hkv,
                                                              int cap) {
  __shared__ WalkShared sh;
  const int hd = 128;
  int layer = blockIdx.x, bh = blockIdx.y;
  int b = bh / Hkv;
  int P = seq_p[b];
  const int len = approval_walk(w, b, sh);
  if (layer == 0 && bh == b * Hkv) report_walk(w, b, sh, len);
  const int32_t* pth = sh.path;
  int t = threadIdx.x;
  if (t < 16) {
    bf16_t* K = kc[layer] + (int64_t)bh * cap * hd;
    for (int j = 0; j < len; ++j) {
      int src = pth[j];
      if (src != j)
        *reinterpret_cast<uint4*>(K + packk_index(P + j, t * 8)) =
            *reinterpret_cast<const uint4*>(K + packk_index(P + src, t * 8));
    }
  } else if (t < 16 + hd) {
    bf16_t* V = vc[layer] + (int64_t)bh * cap * hd;
    int hdim = t - 16;
    for (int j = 0; j < len; ++j) {
      int src = pth[j];
      if (src != j) V[packvt_index(P + j, hdim)] = V[packvt_index(P + src, hdim)];
    }
  }
}
void bf16_kv_compact(bf16_t* const* kc, bf16_t* const* vc, const ApprovalWalk& w, const StepMeta& m, const ModelDims& md, hipStream_t s) {
  hipLaunchKernelGGL(bf16_kv_compact_kernel, dim3(md.n_layers, m.batch * md.Hkv), dim3(256), 0, s, kc, vc, w, m.seq_p, md.Hkv,
                     md.cap);
}

// ------------------------------------------------------------------------------------------
// plain bf16 rows [n][hd] of one (sequence, kv head)  <->  slots [first, first + n) of its f16 cache fragments (to the
// cache: exact widening; back: round to bf16).  A workgroup takes the keys or the values of one 32-slot group of the cache, 8 KiB
// of fragments (both, one after the other, are two round trips to memory), in 16-byte units: a key unit is eight dims of one slot (a 16-byte piece of a
// plain row), a value unit eight slots of one dim, so values go through LDS.  Slots outside the range keep their
// contents (a group's first and last slots may belong to other tokens).
// Bound by memory traffic (plain + cache bytes once each).  One thread per element, with two-byte scattered accesses to
// the value fragments, took 13.4 us for 2001 slots of 8 heads; now 6.7 us to
// the cache, 6.3 us back (16.4 MB: 2.5 TB/s, a launch this small is half start-up).
constexpr int KV_LDS_ROW = 128 + 2;  // elements; the padding spreads a column over the banks

__device__ inline uint4 bf16_to_f16x8(uint4 v) {
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = pk(bf16_to_f16((uint16_t)(w[i] & 0xffffu)), bf16_to_f16((uint16_t)(w[i] >> 16)));
  return make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ inline uint4 f16_to_bf16x8(uint4 v) {
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    w[i] = pk(f32_to_bf16(f16_to_f32((uint16_t)(w[i] & 0xffffu))), f32_to_bf16(f16_to_f32((uint16_t)(w[i] >> 16))));
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// kb: 32-slot group; kc / vc: cache of the (sequence, kv head); kp / vp: its plain rows (row 0 = slot `first`), either may
// be null.  Called by 256 threads.
template <bool TO_CACHE>
__device__ inline void kv_group_copy(bf16_t* kc, bf16_t* vc, bf16_t* kp, bf16_t* vp, int first, int n, int kb,
                                     uint16_t* lds) {
  const int tid = threadIdx.x, slot0 = kb * 32;
  auto inside = [&](int slot) { return slot >= first && slot < first + n; };
  if (kp) {
    uint4* units = reinterpret_cast<uint4*>(kc) + (int64_t)kb * 512;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int u = tid + i * 256, lane = u & 63, m = lane & 15;
      const int slot = slot0 + (m >> 2) * 8 + ((u >> 8) & 1) * 4 + (m & 3), dim = ((u >> 6) & 3) * 32 + (lane >> 4) * 8;
      if (!inside(slot)) continue;
      bf16_t* plain = kp + (int64_t)(slot - first) * 128 + dim;
      if (TO_CACHE) units[u] = bf16_to_f16x8(load_row16(plain));
      else store_row16(plain, f16_to_bf16x8(units[u]));
    }
  }
  if (!vp) return;
  uint4* units = reinterpret_cast<uint4*>(vc) + (int64_t)kb * 512;
  uint32_t* l32 = reinterpret_cast<uint32_t*>(lds);
  if (TO_CACHE) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int u = tid + i * 256, row = u >> 4, dim = (u & 15) * 8;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (inside(slot0 + row)) v = bf16_to_f16x8(load_row16(vp + (int64_t)(slot0 + row - first) * 128 + dim));
      uint32_t* d = l32 + (row * KV_LDS_ROW + dim) / 2;
      d[0] = v.x, d[1] = v.y, d[2] = v.z, d[3] = v.w;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int u = tid + i * 256, lane = u & 63, dim = (u >> 6) * 16 + (lane & 15), k8 = (lane >> 4) * 8;
      uint16_t e[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) e[j] = lds[(k8 + j) * KV_LDS_ROW + dim];
      if (inside(slot0 + k8) && inside(slot0 + k8 + 7)) {
        units[u] = make_uint4(pk(e[0], e[1]), pk(e[2], e[3]), pk(e[4], e[5]), pk(e[6], e[7]));
      } else {
        uint16_t* d = reinterpret_cast<uint16_t*>(units + u);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (inside(slot0 + k8 + j)) d[j] = e[j];
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int u = tid + i * 256, lane = u & 63, dim = (u >> 6) * 16 + (lane & 15), k8 = (lane >> 4) * 8;
      const uint4 v = f16_to_bf16x8(units[u]);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) lds[(k8 + j) * KV_LDS_ROW + dim] = (uint16_t)(w[j >> 1] >> ((j & 1) * 16));
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int u = tid + i * 256, row = u >> 4, dim = (u & 15) * 8;
      if (!inside(slot0 + row)) continue;
      const uint32_t* d = l32 + (row * KV_LDS_ROW + dim) / 2;
      store_row16(vp + (int64_t)(slot0 + row - first) * 128 + dim, make_uint4(d[0], d[1], d[2], d[3]));
    }
  }
}

template <bool TO_CACHE>
__global__ __launch_bounds__(256) void bf16_kv_copy_kernel(bf16_t* __restrict__ kcache, bf16_t* __restrict__ vcache,
                                                           bf16_t* __restrict__ kp, bf16_t* __restrict__ vp, int seq,
                                                           int first, int n, int Hkv, int cap) {
  __shared__ __align__(16) uint16_t lds[32 * KV_LDS_ROW];
  const int g = blockIdx.y;
  const int64_t base = ((int64_t)seq * Hkv + g) * cap * 128, plain = (int64_t)g * n * 128;
  const bool keys = blockIdx.z == 0;  // or values
  kv_group_copy<TO_CACHE>(kcache + base, vcache + base, keys && kp ? kp + plain : nullptr, !keys && vp ? vp + plain : nullptr,
                          first, n, first / 32 + blockIdx.x, lds);
}
void bf16_kv_copy(bf16_t* kcache, bf16_t* vcache, bf16_t* k_plain, bf16_t* v_plain, bool to_cache, int seq,
                  int first, int n, const ModelDims& md, hipStream_t s) {
  if (n <= 0) return;
  const dim3 grid((first + n - 1) / 32 - first / 32 + 1, md.Hkv, 2);
  if (to_cache)
    hipLaunchKernelGGL((bf16_kv_copy_kernel<true>), grid, dim3(256), 0, s, kcache, vcache, k_plain, v_plain, seq, first, n,
                       md.Hkv, md.cap);
  else
    hipLaunchKernelGGL((bf16_kv_copy_kernel<false>), grid, dim3(256), 0, s, kcache, vcache, k_plain, v_plain, seq, first,
                       n, md.Hkv, md.cap);
}

// zero the slots [first, first + n) of one sequence (keys and values) in the fragment layouts
__global__ void bf16_kv_clear_kernel(bf16_t* __restrict__ kcache, bf16_t* __restrict__ vcache, int seq, int first,
                                     int Hkv, int cap) {
  const int hd = 128;
  int j = blockIdx.x, g = blockIdx.y, i = threadIdx.x;
  int64_t cbase = ((int64_t)seq * Hkv + g) * cap * hd;
  kcache[cbase + packk_index(first + j, i)] = 0;
  vcache[cbase + packvt_index(first + j, i)] = 0;
}
void bf16_kv_clear(bf16_t* kcache, bf16_t* vcache, int seq, int first, int n, const ModelDims& md, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(bf16_kv_clear_kernel, dim3(n, md.Hkv), dim3(128), 0, s, kcache, vcache, seq, first, md.Hkv, md.cap);
}

// tree K / V [B][Hkv][max_nodes][hd] -> cache slots P + node.  The step's description is still in host memory (seq_p, seq_n); the
// last workgroups of each row of the grid copy it to the device for the kernels that follow.  What the scatter itself needs of
// it travels with the launch for up to eight sequences: a round trip to the host at its head is 1.5 us of 5.
struct FewSequences {
  int32_t count, p[8], n[8];  // count 0: more of them, read the arrays
};
__global__ __launch_bounds__(256) void bf16_scatter_tree_kv_kernel(bf16_t* __restrict__ kc, bf16_t* __restrict__ vc,
                                                                   const bf16_t* __restrict__ kt,
                                                                   const bf16_t* __restrict__ vt,
                                                                   const int32_t* __restrict__ seq_p,
                                                                   const int32_t* __restrict__ seq_n, FewSequences few,
                                                                   const uint4* __restrict__ meta_src,
                                                                   uint4* __restrict__ meta_dst, int units, int Hkv, int cap,
                                                                   int max_nodes) {
  __shared__ __align__(16) uint16_t lds[32 * KV_LDS_ROW];
  if (blockIdx.x == gridDim.x - 1) {
    if (blockIdx.z) return;
    for (int u = blockIdx.y * 256 + threadIdx.x; u < units; u += gridDim.y * 256) meta_dst[u] = meta_src[u];
    return;
  }
  const int bh = blockIdx.y, b = bh / Hkv;
  int P = few.p[0], n = few.n[0];
#pragma unroll
  for (int i = 1; i < 8; ++i)
    if (b == i) P = few.p[i], n = few.n[i];
  if (!few.count) P = seq_p[b], n = seq_n[b];
  const int kb = P / 32 + blockIdx.x;
  if (kb * 32 >= P + n) return;
  const int64_t plain = (int64_t)bh * max_nodes * 128, base = (int64_t)bh * cap * 128;
  const bool keys = blockIdx.z == 0;  // or values
  kv_group_copy<true>(kc + base, vc + base, keys ? const_cast<bf16_t*>(kt) + plain : nullptr,
                      keys ? nullptr : const_cast<bf16_t*>(vt) + plain, P, n, kb, lds);
}
void bf16_scatter_tree_kv(bf16_t* kc, bf16_t* vc, const bf16_t* k_tree, const bf16_t* v_tree, const StepMeta& m,
                          const void* meta_src, void* meta_dst, int units, const int32_t* host_p, const int32_t* host_n,
                          const ModelDims& md, int max_nodes, hipStream_t s) {
  FewSequences few = {};
  if (m.batch <= 8) {
    few.count = m.batch;
    for (int b = 0; b < m.batch; ++b) few.p[b] = host_p[b], few.n[b] = host_n[b];
  }
  // a tree of n nodes touches at most (n + 30) / 32 + 1 groups
  hipLaunchKernelGGL(bf16_scatter_tree_kv_kernel, dim3((m.n_step + 30) / 32 + 2, m.batch * md.Hkv, 2), dim3(256), 0, s, kc,
                     vc, k_tree, v_tree, m.seq_p, m.seq_n, few, reinterpret_cast<const uint4*>(meta_src),
                     reinterpret_cast<uint4*>(meta_dst), units, md.Hkv, md.cap, max_nodes);
}

}  // namespace ded
