// Skinny 16-bit GEMM on the CDNA matrix cores with fused epilogues:
//   Y[r][n] = sum_k X[r][k] W[n][k] for a few tens of rows, followed in the same kernel by what the
//   decoder does with Y (rotary embedding + cache append, SiLU*up, residual add + next input, logits).
//
// At tree sizes (R <= 64 rows) the projection is bound by streaming the weights from HBM once.  What
// was measured on MI355X and shaped these kernels:
//   * plain 16-byte-per-lane streaming tops out near 6.2 TB/s for the chip and near 52 GB/s per CU,
//     so every CU has to stream its equal share (~24 GB/s) for the whole kernel, and whatever else a
//     CU loads (the activations) comes out of the same per-CU budget, even when it hits in L2;
//   * a wavefront that reads one contiguous stream is ~15 % faster than one that interleaves four;
//   * every launch costs ~3.5 us even back-to-back, and a small dependent kernel 6-10 us, which is
//     why the split-K reduction and the element-wise stages live in the GEMM's epilogue.
// Hence:
//   * weights are pre-laid-out (PackW, f16) as MFMA A-operand fragments in the order a wavefront
//     consumes them: 64-feature group -> k step -> 4 feature tiles -> lane; one k step of a group is
//     4 KiB of contiguous memory fetched by four coalesced 1 KiB loads straight into registers;
//   * activations (PackX, B operand, hi/lo f16 planes) are shared: in the "wide" kernel the NWN
//     wavefronts of a half-workgroup own NWN neighbouring feature groups over the same k range and
//     the activation chunks go through LDS once (double buffered, one barrier per chunk);
//   * narrow outputs use the "stream" kernel: one feature group per workgroup, the NW wavefronts
//     split the k range and combine through LDS in a fixed tree order;
//   * blockIdx.y is a global split-K.  Every slice is written to its own buffer; the workgroup that
//     finishes LAST for an output tile (atomic ticket, device-coherent slice accesses, no waiting) re-reads all
//     slices IN SLICE ORDER and runs the epilogue, so the result does not depend on arrival order.
// v_mfma_f32_16x16x32_f16: A = weights (M = 16 features), B = activations (N = 16 rows),
// C[m][n] lands in lane (n + 16*(m/4)), element m%4: four consecutive features of one row.
// X = hi + lo (two planes): both products accumulate into the same fp32 registers.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "bf16_layout.h"
#include "ded_kernels.h"

namespace ded {

namespace {

constexpr int TN = PACKW_TILES;  // feature tiles per group (fixed by the weight layout)
constexpr int PD = 4;            // k steps (of 32) per group of the k-range split
constexpr int RING = 2;          // k steps in flight per wavefront (stream kernel); divides PD

#ifdef DED_GEMM_TRACE
__device__ unsigned long long* g_trace = nullptr;  // [workgroup][wave][8] wall-clock stamps (debug builds only)
#define DED_STAMP(i)                                                                                       \
  if (g_trace && (threadIdx.x & 63) == 0)                                                                  \
    g_trace[((((size_t)blockIdx.y * gridDim.x + blockIdx.x) * (blockDim.x >> 6)) + (threadIdx.x >> 6)) * 8 + (i)] = \
        wall_clock64();
#else
#define DED_STAMP(i)
#endif

typedef float caller_f32x4_t __attribute__((ext_vector_type(4), aligned(4)));  // a caller's floats: aligned to themselves
typedef f32x4_t Acc[TN][4];  // 4 feature tiles x 4 row blocks

// With a single 64-row group the weights of a skinny GEMM are read exactly once per launch (ONCE): loaded with the
// non-temporal hint they stream through the caches without displacing anything, which measured ~12 % more read
// bandwidth on a plain streaming kernel (6.8 against 6.0 TB/s).  With two or three row groups the later rounds of
// the launch find the weights in the last-level cache, and the hint would cost that.
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
template <bool ONCE>
__device__ inline uint4 load_weights(const uint4* q) {
  if constexpr (ONCE) {
    const u32x4_t r = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(q));
    return make_uint4(r.x, r.y, r.z, r.w);
  } else {
    return *q;
  }
}
// A load that the compiler may move as it likes (nothing in the launch writes what it reads).
template <bool ONCE>
__device__ inline uint4 load_free(const uint4* q) {
  typedef const __attribute__((address_space(4))) u32x4_t invariant_t;
  const u32x4_t r = ONCE ? __builtin_nontemporal_load((invariant_t*)q) : *(invariant_t*)q;
  return make_uint4(r.x, r.y, r.z, r.w);
}
// Loads stay on their side of this: the compiler may not move them across a memory clobber (the pointers are not __restrict__)
// nor the scheduler across its own barrier.  Otherwise it sinks a prefetch to where its value is used.
__device__ __forceinline__ void pin_loads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Split-K slices travel between workgroups of one launch, which may sit on different XCDs with separate
// L2 caches.  Instead of device-scope fences (a whole-L2 write-back and invalidate per workgroup, measured
// at 3-4x the kernel time; even an acquire fence in the last workgroup alone, followed by plain 16-byte
// loads, was 10-20 % slower) the slices are written and read with device-scope relaxed atomic accesses, which
// go through to the memory side on their own; ordering comes from waiting for the stores to complete
// before the ticket is taken, and from the ticket's return value before the loads are issued.
// A slice is private to the kernel, so it is kept in accumulator order: tile (row group, feature group) ->
// (t, rb) -> half -> lane, 8 bytes each: every store / load instruction covers 512 contiguous bytes.
// -DDED_SPLITK_FENCES builds the memory-model-only variant instead (plain slice accesses, a release fence before
// the ticket and an acquire fence after it): the fallback should a future part or driver not give the
// write-through / read-through behaviour of device-scope atomics that the default relies on.
#ifdef DED_SPLITK_FENCES
__device__ inline void slice_store(unsigned long long* p, unsigned long long v) { *p = v; }
__device__ inline unsigned long long slice_load(const unsigned long long* p) { return *p; }
#else
__device__ inline void slice_store(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned long long slice_load(unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
#endif

__device__ inline unsigned long long pack2(float a, float b) {
  return ((unsigned long long)__float_as_uint(b) << 32) | __float_as_uint(a);
}
__device__ inline int64_t slice_tile_offset(int NG, int ng) { return ((int64_t)blockIdx.z * NG + ng) * (TN * 4 * 256); }

// Row blocks rb_lo .. rb_lo + RBN - 1 of the tile, which the wavefront holds in acc[t][0 .. RBN-1].
template <int RBN, typename A>
__device__ inline void store_slice(float* slice, int NG, int ng, int rb_lo, int lane, const A& acc) {
  unsigned long long* q = reinterpret_cast<unsigned long long*>(slice + slice_tile_offset(NG, ng) + rb_lo * 256) + lane;
#pragma unroll
  for (int t = 0; t < TN; ++t)
#pragma unroll
    for (int j = 0; j < RBN; ++j) {
      const f32x4_t v = acc[t][j];
      slice_store(q + (t * 4 + j) * 128, pack2(v[0], v[1]));
      slice_store(q + (t * 4 + j) * 128 + 64, pack2(v[2], v[3]));
    }
}

// acc[t][j] = sum over slices 0..splits-1 (in slice order) of row block rb_lo + j of the tile, j < RBN
template <int RBN, typename A>
__device__ inline void load_slices(const float* part, int64_t part_stride, int splits, int NG, int ng, int rb_lo, int lane,
                                   A& acc) {
#pragma unroll
  for (int t = 0; t < TN; ++t)
#pragma unroll
    for (int j = 0; j < RBN; ++j) acc[t][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const float* base = part + slice_tile_offset(NG, ng) + rb_lo * 256;
#pragma unroll 4
  for (int s = 0; s < splits; ++s) {
    unsigned long long* q =
        reinterpret_cast<unsigned long long*>(const_cast<float*>(base) + (int64_t)s * part_stride) + lane;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int j = 0; j < RBN; ++j) {
        unsigned long long a = slice_load(q + (t * 4 + j) * 128);
        unsigned long long b = slice_load(q + (t * 4 + j) * 128 + 64);
        acc[t][j] += f32x4_t{__uint_as_float((unsigned)a), __uint_as_float((unsigned)(a >> 32)),
                             __uint_as_float((unsigned)b), __uint_as_float((unsigned)(b >> 32))};
      }
  }
}

// acc[t][j] (in: this workgroup's own slice values, which it still holds) = sum over slices 0..S-1 in slice order,
// the own values standing in for slice `split`: only the S - 1 other slices are fetched, all loads in flight
// together.  The result does not depend on which workgroup arrived last.
template <int RBN, int S, typename A>
__device__ inline void sum_other_slices(const float* part, int64_t part_stride, int split, int NG, int ng, int rb_lo, int lane,
                                        A& acc) {
  const float* base = part + slice_tile_offset(NG, ng) + rb_lo * 256;
  unsigned long long a[S - 1][TN][RBN], b[S - 1][TN][RBN];
#pragma unroll
  for (int k = 0; k < S - 1; ++k) {
    const int sl = k + (k >= split ? 1 : 0);
    unsigned long long* q =
        reinterpret_cast<unsigned long long*>(const_cast<float*>(base) + (int64_t)sl * part_stride) + lane;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int j = 0; j < RBN; ++j) {
        a[k][t][j] = slice_load(q + (t * 4 + j) * 128);
        b[k][t][j] = slice_load(q + (t * 4 + j) * 128 + 64);
      }
  }
  f32x4_t own[TN][RBN];
#pragma unroll
  for (int t = 0; t < TN; ++t)
#pragma unroll
    for (int j = 0; j < RBN; ++j) own[t][j] = acc[t][j];
  // position p of the sum takes slice p: the own values at p == split, else the fetched slice k = p - (p > split)
#pragma unroll
  for (int p = 0; p < S; ++p) {
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int j = 0; j < RBN; ++j) {
        const int lo = p > 0 ? p - 1 : 0, hi = p < S - 1 ? p : S - 2;  // the fetched slice is one of a[lo], a[hi]
        const bool use_lo = p > split;
        const unsigned long long ua = use_lo ? a[lo][t][j] : a[hi][t][j];
        const unsigned long long ub = use_lo ? b[lo][t][j] : b[hi][t][j];
        const f32x4_t other = f32x4_t{__uint_as_float((unsigned)ua), __uint_as_float((unsigned)(ua >> 32)),
                                      __uint_as_float((unsigned)ub), __uint_as_float((unsigned)(ub >> 32))};
        const f32x4_t v = p == split ? own[t][j] : other;
        acc[t][j] = p == 0 ? v : acc[t][j] + v;
      }
  }
}

template <int RBN, typename A>
__device__ inline void sum_slices_keep_own(const float* part, int64_t part_stride, int split, int splits, int NG, int ng,
                                           int rb_lo, int lane, A& acc) {
  if (splits == 2) {
    sum_other_slices<RBN, 2>(part, part_stride, split, NG, ng, rb_lo, lane, acc);
  } else if (splits == 4) {
    sum_other_slices<RBN, 4>(part, part_stride, split, NG, ng, rb_lo, lane, acc);
  } else if (splits == 3) {
    sum_other_slices<RBN, 3>(part, part_stride, split, NG, ng, rb_lo, lane, acc);
  } else {
    load_slices<RBN>(part, part_stride, splits, NG, ng, rb_lo, lane, acc);  // all slices, the own one included
  }
}

__device__ inline uint2 pack4_f16(float a, float b, float c, float d) {
  return make_uint2((uint32_t)f32_to_f16(a) | ((uint32_t)f32_to_f16(b) << 16),
                    (uint32_t)f32_to_f16(c) | ((uint32_t)f32_to_f16(d) << 16));
}
__device__ inline void split4_f16(const float (&v)[4], uint2& hi, uint2& lo) {
  uint16_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) split_f16(v[i], h[i], l[i]);
  hi = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
  lo = make_uint2((uint32_t)l[0] | ((uint32_t)l[1] << 16), (uint32_t)l[2] | ((uint32_t)l[3] << 16));
}

// ------------------------------------------------------------------------------------------
// Epilogues.  Run by one wavefront on RBN row blocks (first one: rbase) of a 64-feature group; acc[t][j]
// holds row block rbase + j.  A lane holds, for row (rbase + j) * 16 + (lane & 15), the 4 features
// t * 16 + (lane >> 4) * 4 + i.  Feature groups of the QKV and gate/up matrices are interleaved at pack
// time (packw_source_row) so that tiles t and t + 2 of a group hold partner features: rotary pairs
// (i, i + 64), or gate / up.
// ------------------------------------------------------------------------------------------
// RMSNorm scale of the GEMM input rows: 1 / sqrt(sum(x^2) / d + eps), from the per-(row, 64-feature group)
// sums that the producer stored.  The sums were written by another kernel, usually from another XCD, and a
// load issued when they are needed costs ~3 us; at kernel start it would delay the first weight chunk (loads
// return in order).  So the wavefronts of a workgroup share the job: each fetches a slice of the groups for
// row rb0 * 16 + lane a few iterations before its k loop ends (ssq_issue; <= 8 float2 registers), adds them
// up after the loop, and the partial sums meet in LDS at the barrier the kernel has there anyway.
constexpr int SSQ_REGS = 8;
struct SsqPart {
  float2 v[SSQ_REGS];
};
__device__ inline void ssq_clear(SsqPart& p) {
#pragma unroll
  for (int i = 0; i < SSQ_REGS; ++i) p.v[i] = make_float2(0.f, 0.f);
}
// wavefront `wv` of `nwv` takes float2 units [wv * per, wv * per + per) of the row's ssq_groups / 2
__device__ inline void ssq_issue(const GemmEpilogue& e, int rb0, int lane, int wv, int nwv, SsqPart& p) {
  if (!e.ssq_in) return;
  const int n2 = e.ssq_groups >> 1, per = (n2 + nwv - 1) / nwv, g0 = wv * per;
  const float2* src = reinterpret_cast<const float2*>(e.ssq_in + (int64_t)(rb0 * 16 + lane) * e.ssq_groups);
#pragma unroll
  for (int i = 0; i < SSQ_REGS; ++i)
    if (i < per && g0 + i < n2) p.v[i] = src[g0 + i];
}
// partial sum of this wavefront's slice -> LDS (call before a workgroup barrier)
__device__ inline void ssq_publish(const GemmEpilogue& e, int rb0, int lane, int wv, int nwv, const SsqPart& p,
                                   float* s_ssq) {
  if (!e.ssq_in) return;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < SSQ_REGS; ++i) s += p.v[i].x + p.v[i].y;
  const int n2 = e.ssq_groups >> 1, per = (n2 + nwv - 1) / nwv, g0 = wv * per;
  const float2* src = reinterpret_cast<const float2*>(e.ssq_in + (int64_t)(rb0 * 16 + lane) * e.ssq_groups);
  for (int i = SSQ_REGS; i < per && g0 + i < n2; ++i) s += src[g0 + i].x + src[g0 + i].y;  // very wide rows only
  s_ssq[wv * 64 + lane] = s;
}
// after that barrier: scale of row rb0 * 16 + lane (partials added in wavefront order)
__device__ inline float ssq_scale(const GemmEpilogue& e, int lane, int nwv, const float* s_ssq) {
  if (!e.ssq_in) return 1.f;
  float s = 0.f;
  for (int w = 0; w < nwv; ++w) s += s_ssq[w * 64 + lane];
  return 1.0f / sqrtf(s * e.inv_k + e.eps);
}

// A wavefront may hold only T of the group's four feature tiles, from tile t0 on (paired epilogues: tiles t0 and t0 + 2).
template <int EPI, int RBN, int T = TN, bool RAGGED = false, typename A>
__device__ inline void run_epilogue(const GemmEpilogue& e, int ng, int N, int rb0, int rbase, float row_scale, int lane,
                                    A& acc, int t0 = 0) {
  // (RAGGED: rows from e.rows on are surplus ones of a last row tile, nothing is written for them)
  const int row_in = lane & 15, quad = lane >> 4;
  float scale[RBN];
#pragma unroll
  for (int j = 0; j < RBN; ++j) scale[j] = __shfl(row_scale, (rbase - rb0 + j) * 16 + row_in);

  if (EPI == EPI_LOGITS || EPI == EPI_TOP2) {
    // what the approval walk needs of a logits row, without the row: the best value of this 64-feature group, its
    // feature index (lowest on ties), the second best value, and whether any value is NaN or infinite
    uint4* dst = reinterpret_cast<uint4*>(e.top2_part);
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb) {
      if (RAGGED && (rbase + rb) * 16 >= e.rows) continue;
      const int64_t r = (int64_t)(rbase + rb) * 16 + row_in;
      float v1 = -INFINITY, v2 = -INFINITY;
      int i1 = 0x7fffffff, bad = 0;
      // the row itself too, where it is asked for: into the workspace and, for a real node, into the caller's [batch][max_nodes][V]
      float *own = nullptr, *out = nullptr;
      if constexpr (EPI == EPI_LOGITS) {
        own = e.out + r * e.out_stride;
        if (e.logits_out && r < e.rows) {
          const int b = e.blk_seq[r >> 4], node = (int)r - e.row0[b];
          if (node < e.seq_n[b]) out = e.logits_out + ((int64_t)b * e.max_nodes + node) * N;
        }
      }
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        const int n = (ng * TN + t) * 16 + quad * 4;
        if (n >= N) continue;
        const f32x4_t v = acc[t][rb] * scale[rb];
        if constexpr (EPI == EPI_LOGITS) {
          *reinterpret_cast<f32x4_t*>(own + n) = v;
          if (out) *reinterpret_cast<caller_f32x4_t*>(out + n) = v;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // ascending feature index: a later equal value never replaces the first
          const float x = v[i];
          bad |= !(fabsf(x) <= 3.402823466e38f);
          if (x > v1) {
            v2 = v1;
            v1 = x;
            i1 = n + i;
          } else if (x > v2) {
            v2 = x;
          }
        }
      }
#pragma unroll
      for (int off = 16; off <= 32; off <<= 1) {  // the four lanes that share the row
        const float ov1 = __shfl_xor(v1, off), ov2 = __shfl_xor(v2, off);
        const int oi1 = __shfl_xor(i1, off);
        bad |= __shfl_xor(bad, off);
        if (ov1 > v1 || (ov1 == v1 && oi1 < i1)) {
          v2 = fmaxf(v1, ov2);
          v1 = ov1;
          i1 = oi1;
        } else {
          v2 = fmaxf(v2, ov1);
        }
      }
      if (quad == 0)
        dst[r * e.top2_groups + ng] = make_uint4(__float_as_uint(v1), (uint32_t)i1, __float_as_uint(v2), (uint32_t)bad);
    }
  } else if (EPI == EPI_RESIDUAL) {
    // x += Y;  next GEMM input = (x * gain) as hi/lo f16 (its 1/rms is applied by the consumer);  sum(x^2) per group
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb) {
      if (RAGGED && (rbase + rb) * 16 >= e.rows) continue;
      const int r = (rbase + rb) * 16 + row_in;
      float ss = 0.f;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int n = (ng * TN + t0 + t) * 16 + quad * 4;
        float* xp = e.x + (int64_t)r * N + n;
        float4 xv = *reinterpret_cast<const float4*>(xp);
        float4 g = *reinterpret_cast<const float4*>(e.gain + n);
        float xn[4] = {xv.x + acc[t][rb][0], xv.y + acc[t][rb][1], xv.z + acc[t][rb][2], xv.w + acc[t][rb][3]};
        *reinterpret_cast<float4*>(xp) = make_float4(xn[0], xn[1], xn[2], xn[3]);
        ss += xn[0] * xn[0] + xn[1] * xn[1] + xn[2] * xn[2] + xn[3] * xn[3];
        if (T == 1) e.ssq_out[(int64_t)r * (N / 4) + n / 4] = ss;
        float y[4] = {xn[0] * g.x, xn[1] * g.y, xn[2] * g.z, xn[3] * g.w};
        uint2 hi, lo;
        split4_f16(y, hi, lo);
        *reinterpret_cast<uint2*>(e.y_packed + packx_index(r, n, e.rb_total, 0)) = hi;
        *reinterpret_cast<uint2*>(e.y_packed + packx_index(r, n, e.rb_total, 1)) = lo;
      }
      if (T == 1) continue;
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      if (quad == 0) e.ssq_out[(int64_t)r * (N / 64) + ng] = ss;
    }
  } else if (EPI == EPI_SILU) {
    // group ng = gate features [32 ng, 32 ng + 32) in tiles 0, 1 and the matching up features in tiles 2, 3
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb) {
      if (RAGGED && (rbase + rb) * 16 >= e.rows) continue;
      const int r = (rbase + rb) * 16 + row_in;
#pragma unroll
      for (int t = 0; t < T / 2; ++t) {
        const int f = ng * 32 + (t0 + t) * 16 + quad * 4;
        if (2 * f >= N) continue;
        float h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float gv = acc[t][rb][i] * scale[rb], uv = acc[t + T / 2][rb][i] * scale[rb];
          h[i] = gv / (1.0f + __expf(-gv)) * uv;
        }
        *reinterpret_cast<uint2*>(e.y_packed + packx_index(r, f, e.rb_total, 0)) = pack4_f16(h[0], h[1], h[2], h[3]);
      }
    }
  } else if (EPI == EPI_QKV) {
    // group ng = head slot ng / 2, dims [32 j, 32 j + 32) in tiles 0, 1 and their rotary partners (+64) in tiles 2, 3
    const int hs = ng >> 1, j = ng & 1;
    const int G = e.H / e.Hkv;
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb) {
      if (RAGGED && (rbase + rb) * 16 >= e.rows) continue;
      const int r = (rbase + rb) * 16 + row_in;
      if (r >= e.rows) continue;
      const int b = e.blk_seq[r >> 4], node = r - e.row0[b];
      const int n_b = e.seq_n[b];
      const bool real = node < n_b;
      const int slot = e.seq_p[b] + node;
#pragma unroll
      for (int t = 0; t < T / 2; ++t) {
        const int d0 = 32 * j + 16 * (t0 + t) + quad * 4;
        float a[4], c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a[i] = acc[t][rb][i] * scale[rb];
          c[i] = acc[t + T / 2][rb][i] * scale[rb];
        }
        if (hs < e.H + e.Hkv) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float2 cs = e.rope_tab[(int64_t)r * 64 + d0 + i];
            float ra = a[i] * cs.x - c[i] * cs.y;
            float rc = c[i] * cs.x + a[i] * cs.y;
            a[i] = ra;
            c[i] = rc;
          }
        }
        if (hs < e.H) {
          const int kvh = hs / G, g = hs - kvh * G;
          const int vr = g * ((n_b + 15) & ~15) + node;
          uint16_t* base = e.q_packed + ((int64_t)b * e.Hkv + kvh) * ((int64_t)G * e.n_step * 128 * 2);
          uint2 hi, lo;
          split4_f16(a, hi, lo);
          *reinterpret_cast<uint2*>(base + packq_index(vr, d0, 0)) = hi;
          *reinterpret_cast<uint2*>(base + packq_index(vr, d0, 1)) = lo;
          split4_f16(c, hi, lo);
          *reinterpret_cast<uint2*>(base + packq_index(vr, d0 + 64, 0)) = hi;
          *reinterpret_cast<uint2*>(base + packq_index(vr, d0 + 64, 1)) = lo;
        } else if (real && hs < e.H + e.Hkv) {
          uint16_t* base = e.k_cache + ((int64_t)b * e.Hkv + (hs - e.H)) * ((int64_t)e.cap * 128);
          *reinterpret_cast<uint2*>(base + packk_index(slot, d0)) = pack4_f16(a[0], a[1], a[2], a[3]);
          *reinterpret_cast<uint2*>(base + packk_index(slot, d0 + 64)) = pack4_f16(c[0], c[1], c[2], c[3]);
        } else if (real) {
          uint16_t* base = e.v_cache + ((int64_t)b * e.Hkv + (hs - e.H - e.Hkv)) * ((int64_t)e.cap * 128);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            base[packvt_index(slot, d0 + i)] = f32_to_f16(a[i]);
            base[packvt_index(slot, d0 + 64 + i)] = f32_to_f16(c[i]);
          }
        }
      }
    }
  }
}

// Split-K hand-over (splits > 1), second part: called by the whole workgroup after its wavefronts have issued their
// slice stores.  Returns true in the workgroup that arrived last for its output tile.
__device__ inline bool take_ticket(int splits, int* counters, int* s_flag) {
#ifdef DED_SPLITK_FENCES
  __atomic_thread_fence(__ATOMIC_RELEASE);  // agent scope is the default of a thread fence in HIP device code
#else
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): this wavefront's slice stores have completed
#endif
  DED_STAMP(4)
  __syncthreads();
  if (threadIdx.x == 0) {
    int* ticket = counters + (blockIdx.z * gridDim.x + blockIdx.x);
    int prev = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int last = prev == splits - 1;
    if (last) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
    *s_flag = last;
  }
  __syncthreads();
#ifdef DED_SPLITK_FENCES
  if (*s_flag) __atomic_thread_fence(__ATOMIC_ACQUIRE);
#endif
  DED_STAMP(5)
  return *s_flag != 0;
}

// The row blocks of a launch are dealt to its groups (blockIdx.z) as evenly as they go: at most four each, sizes that differ by
// one at most, and a kernel instance for the larger groups of 4 or of 3 (smaller ones take the branch with one block less).
// Groups that always ran as four fetched and multiplied blocks nobody reads, out of what bounds these kernels, ~50 GB/s into
// each CU.  In steps, us, always four / as dealt: 48 rows (7B shape) gate/up 43.0 / 38.3, QKV 31.6 / 29.8, O and down together
// 38.4 / 36.1; 97 rows 66.0 / 61.0, 41.3 / 38.9, 54.1 / 52.2; 144 rows of the 8B shape, QKV 34.4 / 30.1, O and down 92.5 / 84.5.
// The first `larger` groups have RBG blocks, the others RBG - 1 (a division in the kernel would cost it 0.2 us).
template <int RBG>
__device__ inline int group_first(int larger) { return (int)blockIdx.z * (RBG - 1) + min((int)blockIdx.z, larger); }

// How a launch reads its weights, and with that the order of its loads: once (a single group); by several groups; by several
// groups in more workgroups than CUs.
enum { READ_ONCE, READ_SHARED, READ_ROUNDS };

// ------------------------------------------------------------------------------------------
// Stream kernel: one feature group per workgroup, NW wavefronts split the k range.
// ------------------------------------------------------------------------------------------
template <int NW, int RBG>
struct StreamShared {
  float4 red[(NW > 1 ? NW / 2 : 1) * TN * RBG * 64];
  float ssq[NW * 64];
  int flag;
};
template <int NW, int PLANES, int EPI, int READS, int RBG, typename SH>
__device__ __forceinline__ void stream_group(SH& sh, float* __restrict__ part, int64_t part_stride, const uint4* xp,
                                             const uint4* wp, int RB, int rb0, int N, int KT, int splits,
                                             int* __restrict__ counters, const GemmEpilogue& epi) {
  constexpr bool ONCE = READS == READ_ONCE;
  float4* const red = sh.red;
  float* const s_ssq = sh.ssq;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ng = blockIdx.x;
  const int split = blockIdx.y;
  // this wavefront's k range, in units of RING steps (the finest grain the loop allows: K = 11008 over 16
  // wavefronts is 21 or 22 steps each, where whole groups of PD steps would give 20 or 24)
  const int units = KT / RING;
  const int parts = splits * NW;
  const int gi = split * NW + wave;
  // (32 bits: a 64-bit division takes 0.2 us.  At least 4 steps: the host launches no more wavefronts than K has groups of PD)
  const int k0 = gi * units / parts * RING, k1 = (gi + 1) * units / parts * RING;

  f32x4_t acc[TN][RBG];
#pragma unroll
  for (int t = 0; t < TN; ++t)
#pragma unroll
    for (int rb = 0; rb < RBG; ++rb) acc[t][rb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  DED_STAMP(0)
  SsqPart ssq;
  ssq_clear(ssq);
  // The ring: D steps' fragments in fixed registers, a step's refilled as soon as it is used up (the loads held there).  Straight
  // code from the first load to the last: a load under a condition makes the compiler's waits assume that it did not happen.
  // D = 4 where the registers of one plane allow it and no second workgroup wants them (one group: at most one workgroup per CU in
  // the measured shapes; 232 registers, two wavefronts per SIMD, against 152 and three).  us, D = 2 / 4: O and down together, 64 rows,
  // 7B shape 38.4 / 38.4, 13B 52.4 / 52.7; with two wavefronts (O of d = 2048, 64 rows) 25.0 / 11.9, since with fewer registers the
  // compiler fetches the slices two at a time.  Several groups, 2 / 4: 7B, 128 rows 54.3 / 53.7, 192 rows 79.8 / 84.9 (three
  // workgroups per CU).  Two planes: four steps of both do not fit.
  constexpr int D = PLANES == 1 && ONCE ? 4 : 2;
  static_assert((D == RING || D == 2 * RING) && D <= PD, "a range is whole units of RING steps, and at least PD steps");
  const int n = k1 - k0;
  const char* wsrc = reinterpret_cast<const char*>(wp) + (((int64_t)ng * KT + k0) * TN << 10);  // (uniform; the lane's offset apart)
  // per k step the activations of the group's row blocks x 2 planes (hi, lo) are one run of memory
  const char* xsrc = reinterpret_cast<const char*>(xp) + (int64_t)k0 * ((int64_t)RB << 11) + ((int64_t)rb0 << 11);
  const int64_t xstep = (int64_t)RB << 11;
  const uint32_t lane16 = lane << 4;
  uint4 wr[D][TN], xr[D][RBG * PLANES];
  auto issue = [&](int slot) {
    pin_loads();
#pragma unroll
    for (int t = 0; t < TN; ++t) wr[slot][t] = load_weights<ONCE>(reinterpret_cast<const uint4*>(wsrc + (t << 10) + lane16));
#pragma unroll
    for (int rb = 0; rb < RBG; ++rb)
#pragma unroll
      for (int p = 0; p < PLANES; ++p) xr[slot][rb * PLANES + p] = *reinterpret_cast<const uint4*>(xsrc + ((rb * 2 + p) << 10) + lane16);
    wsrc += TN << 10;
    xsrc += xstep;
    pin_loads();
  };
  auto compute = [&](int slot) {
#pragma unroll
    for (int p = 0; p < PLANES; ++p)  // 4 RBG independent accumulators between dependent products
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        f16x8_t a = __builtin_bit_cast(f16x8_t, wr[slot][t]);
#pragma unroll
        for (int rb = 0; rb < RBG; ++rb)
          acc[t][rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
              a, __builtin_bit_cast(f16x8_t, xr[slot][rb * PLANES + p]), acc[t][rb], 0, 0, 0);
      }
  };
  constexpr bool SSQ = EPI != EPI_RESIDUAL;
  int left = n - D;  // steps not requested yet
  if (D > RING && left % D) {  // what is beyond whole turns goes first; either way the places are in order after it
    constexpr int R = D - RING;
#pragma unroll
    for (int j = 0; j < D; ++j) issue((j + R) % D);
#pragma unroll
    for (int j = R; j < D; ++j) {
      compute(j);
      issue(j);
    }
    left -= RING;
  } else {
#pragma unroll
    for (int j = 0; j < D; ++j) issue(j);
  }
  // A step's place is refilled at once, or all of a turn's together where other workgroups on the CU have their loads in flight
  // meanwhile.  O and down together, us, at once / together: 7B shape, 128 rows 53.9 / 55.2, 13B, 192 rows 97.5 / 100.6 (at most one
  // workgroup per CU); down alone, more of them: 7B, 192 rows 57.9 / 54.3, 13B, 97 rows 55.2 / 53.7.
  auto turns_to = [&](int rest) {
    for (; left > rest; left -= D) {
      if (READS == READ_ROUNDS) {
#pragma unroll
        for (int j = 0; j < D; ++j) compute(j);
#pragma unroll
        for (int j = 0; j < D; ++j) issue(j);
      } else {
#pragma unroll
        for (int j = 0; j < D; ++j) {
          compute(j);
          issue(j);
        }
      }
    }
  };
  if constexpr (SSQ) {
    turns_to(12);
    ssq_issue(epi, rb0, lane, wave, NW, ssq);  // the row sums, a dozen steps before the end
  }
  turns_to(0);
#pragma unroll
  for (int j = 0; j < D; ++j) compute(j);
  ssq_publish(epi, rb0, lane, wave, NW, ssq, s_ssq);
  if (NW == 1) __syncthreads();

  DED_STAMP(2)
  // combine the NW k ranges: wave w += wave w + stride, stride = NW/2 .. 1
  if (NW > 1) {
#pragma unroll
    for (int stride = NW / 2; stride >= 1; stride >>= 1) {
      if (wave >= stride && wave < 2 * stride) {
        float4* dst = red + (int64_t)(wave - stride) * TN * RBG * 64 + lane;
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
          for (int rb = 0; rb < RBG; ++rb) {
            f32x4_t v = acc[t][rb];
            dst[(t * RBG + rb) * 64] = make_float4(v[0], v[1], v[2], v[3]);
          }
      }
      __syncthreads();
      if (wave < stride) {
        const float4* src = red + (int64_t)wave * TN * RBG * 64 + lane;
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
          for (int rb = 0; rb < RBG; ++rb) {
            float4 v = src[(t * RBG + rb) * 64];
            acc[t][rb] += f32x4_t{v.x, v.y, v.z, v.w};
          }
      }
      __syncthreads();
    }
  }
  DED_STAMP(3)
  const float row_scale = ssq_scale(epi, lane, NW, s_ssq);  // the reduction above had at least one barrier
  if (splits == 1) {
    if (wave == 0) run_epilogue<EPI, RBG>(epi, ng, N, rb0, rb0, row_scale, lane, acc);
  } else {
    if (wave == 0) store_slice<RBG>(part + (int64_t)split * part_stride, gridDim.x, ng, 0, lane, acc);
    // the wavefronts of the last workgroup share the tile's row blocks
    constexpr int RBN = (RBG + NW - 1) / NW;
    const int rb_lo = wave * RBN;
    if (take_ticket(splits, counters, &sh.flag) && rb_lo < RBG) {
      if (RBG % RBN == 0 || rb_lo + RBN <= RBG) {
        load_slices<RBN>(part, part_stride, splits, gridDim.x, ng, rb_lo, lane, acc);
        DED_STAMP(6)
        run_epilogue<EPI, RBN>(epi, ng, N, rb0, rb0 + rb_lo, row_scale, lane, acc);
      } else if constexpr (RBG % RBN) {
        load_slices<RBG % RBN>(part, part_stride, splits, gridDim.x, ng, rb_lo, lane, acc);
        run_epilogue<EPI, RBG % RBN>(epi, ng, N, rb0, rb0 + rb_lo, row_scale, lane, acc);
      }
    }
  }
  DED_STAMP(7)
}
// RBG: row blocks of the larger groups; others have one less.  (Two to three wavefronts per SIMD: for a fourth, which three blocks
// would fit, the compiler fetched the slices two at a time.  us, so / now: d = 2048, 80 rows O 13.1 / 10.1, down 20.0 / 17.1; d = 1024,
// K = 2816, 144 rows 12.9 / 9.9)
template <int NW, int PLANES, int EPI, int READS, int RBG>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 3)))
void gemm_stream_kernel(float* __restrict__ part, int64_t part_stride, const uint4* xp, const uint4* wp, int RB, int larger,
                        int N, int KT, int splits, int* __restrict__ counters, GemmEpilogue epi) {
  __shared__ StreamShared<NW, RBG> sh;
  const int rb0 = READS == READ_ONCE ? 0 : group_first<RBG>(larger);
  if (READS == READ_ONCE || (int)blockIdx.z < larger)
    stream_group<NW, PLANES, EPI, READS, RBG>(sh, part, part_stride, xp, wp, RB, rb0, N, KT, splits, counters, epi);
  else
    stream_group<NW, PLANES, EPI, READS, RBG - 1>(sh, part, part_stride, xp, wp, RB, rb0, N, KT, splits, counters, epi);
}

// ------------------------------------------------------------------------------------------
// Wide kernel: a workgroup owns NWN neighbouring feature groups over one k range.  Its 2 x NWN
// wavefronts form two halves: half h walks the h-th half of the k range, wavefront wn of a half owns
// feature group wn.  The activation chunks (CH k steps x 4 row blocks x PLANES) of each half are
// staged through LDS once per half (double buffered, one barrier per chunk), so the activations cost
// 1/NWN of what they would if every wavefront fetched its own.  Two wavefronts per SIMD overlap each
// other's LDS waits and barriers; the halves are added through LDS at the end (fixed order).
// ------------------------------------------------------------------------------------------
template <int NWN, int PLANES, int RBG>
struct WideShape {
  static constexpr int CH = (NWN == 4 || PLANES == 1) ? 2 : 1;  // k steps per activation chunk (<= 4 staged units / thread)
  static constexpr int STEP_U4 = RBG * PLANES * 64;             // uint4 units of activations per k step
  static constexpr int CHUNK_U4 = CH * STEP_U4;
  static constexpr int RED_U4 = 2 * NWN * TN * ((RBG + 1) / 2) * 64;  // what the halves exchange
  static constexpr int LDS_U4 = 2 * 2 * CHUNK_U4 > RED_U4 ? 2 * 2 * CHUNK_U4 : RED_U4;
};
template <int NWN, int PLANES, int RBG>
struct WideShared {
  uint4 lds[WideShape<NWN, PLANES, RBG>::LDS_U4];  // [half][buffer][chunk]; reused for the final reduction
  float ssq[2 * NWN * 64];
  int flag;
};
template <int NWN, int PLANES, int EPI, bool ONCE, int RBG, typename SH>
__device__ __forceinline__ void wide_group(SH& sh, float* __restrict__ part, int64_t part_stride, const uint4* xp, const uint4* wp,
                                           int RB, int rb0, int N, int KT, int splits,
                                           int* __restrict__ counters, const GemmEpilogue& epi) {
  using W = WideShape<NWN, PLANES, RBG>;
  constexpr int TH = NWN * 64;  // threads per half
  constexpr int CH = W::CH, STEP_U4 = W::STEP_U4, CHUNK_U4 = W::CHUNK_U4;
  constexpr int PER_THREAD = (CHUNK_U4 + TH - 1) / TH;
  uint4* const lds = sh.lds;
  float* const s_ssq = sh.ssq;
  const int half = threadIdx.x / TH;
  const int tid = threadIdx.x - half * TH, lane = tid & 63, wn = tid >> 6;
  uint4* xs = lds + half * 2 * CHUNK_U4;
  const int NG = (N + 16 * TN - 1) / (16 * TN);
  const int ng_raw = blockIdx.x * NWN + wn;
  const int ng = ng_raw < NG ? ng_raw : NG - 1;  // surplus wavefront of the last tile: valid reads, no store
  const int split = blockIdx.y;
  const int groups = KT / PD;
  const int g_begin = split * groups / splits, g_end = (split + 1) * groups / splits;
  const int n_chunks = (g_end - g_begin) * (PD / CH) / 2;  // per half; the range holds an even number of chunks
  const int kt0 = g_begin * PD + half * n_chunks * CH;

  f32x4_t acc[TN][RBG];
#pragma unroll
  for (int t = 0; t < TN; ++t)
#pragma unroll
    for (int rb = 0; rb < RBG; ++rb) acc[t][rb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const uint4* wsrc = wp + (((int64_t)ng * KT * TN) << 6) + lane;
  const uint4* xsrc = xp + ((int64_t)rb0 << 7);
  const int64_t xstep = (int64_t)RB << 7;

  struct WChunk {
    uint4 f[CH][TN];
  };
  struct XStage {
    uint4 u[PER_THREAD];
  };
  auto load_w = [&](int c) {
    WChunk w;
#pragma unroll
    for (int s = 0; s < CH; ++s)
#pragma unroll
      for (int t = 0; t < TN; ++t) w.f[s][t] = load_free<ONCE>(wsrc + (((int64_t)(kt0 + c * CH + s) * TN + t) << 6));
    return w;
  };
  // unit u of a chunk: step s = u / STEP_U4, inside the step (rb, plane, lane) in memory order
  auto load_x = [&](int c) {
    XStage x;
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      int u = tid + i * TH;
      if (CHUNK_U4 % TH == 0 || u < CHUNK_U4) {
        int s = u / STEP_U4, v = u - s * STEP_U4;
        int src = PLANES == 2 ? v : ((v >> 6) * 128 + (v & 63));  // one plane: skip the lo fragments
        x.u[i] = load_free<false>(xsrc + (int64_t)(kt0 + c * CH + s) * xstep + src);
      }
    }
    return x;
  };
  auto store_x = [&](int buf, const XStage& x) {
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      int u = tid + i * TH;
      if (CHUNK_U4 % TH == 0 || u < CHUNK_U4) xs[buf * CHUNK_U4 + u] = x.u[i];
    }
  };
  auto compute = [&](const WChunk& w, int buf) {
#pragma unroll
    for (int s = 0; s < CH; ++s) {
      f16x8_t b[RBG * PLANES];
#pragma unroll
      for (int i = 0; i < RBG * PLANES; ++i)
        b[i] = __builtin_bit_cast(f16x8_t, xs[buf * CHUNK_U4 + s * STEP_U4 + (i << 6) + lane]);
#pragma unroll
      for (int p = 0; p < PLANES; ++p)
#pragma unroll
        for (int t = 0; t < TN; ++t) {
          f16x8_t a = __builtin_bit_cast(f16x8_t, w.f[s][t]);
#pragma unroll
          for (int rb = 0; rb < RBG; ++rb)
            acc[t][rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b[rb * PLANES + p], acc[t][rb], 0, 0, 0);
        }
    }
  };

  DED_STAMP(0)
  // Software pipeline.  Loads return in order, so waiting for an activation chunk also waits for every
  // weight chunk issued before it: with activations one chunk ahead an iteration could not be shorter than
  // one HBM round trip (measured: 16 iterations of 1.4 us).  Hence activations are fetched TWO chunks ahead
  // (registers; the LDS copy stays double buffered) and weights THREE: the wait for activation chunk c + 1
  // then only needs loads that are two iterations old.  In every iteration the activation loads are issued
  // before the weight loads.  Both halves run the same number of iterations and barriers (n_chunks >= 2).
  // Kernel shapes whose chunks hold two k steps keep the shallower pipeline (activations one chunk ahead,
  // weights two): their iterations are twice as long, and the deeper one does not fit the register file.
  constexpr bool DEEP = CH == 1;
  SsqPart ssq;
  ssq_clear(ssq);
  const int wv = threadIdx.x >> 6;
  const int c_ssq = n_chunks - 14;  // fetch the row sums ~10 iterations before the loop ends
  if constexpr (DEEP) {
    // Weights three chunks ahead, activations two.  The ring slots are fixed registers (the loop is unrolled by the
    // ring length and leaves from the middle): a copy between slots would have to wait for the load that still
    // writes its source.  Of a single row group, whose weights all come from memory, the loads are pinned, activations in front of
    // weights, and the LDS stores behind the products: the compiler otherwise sinks a prefetch to the block of its first use, or
    // waits for activations of one iteration back before the products (48 rows, gate/up of a 7B shape: 49.0 us so, 38.4 pinned).
    // Several groups find the weights in the caches and take the compiler's order, loads between the products (gate/up of the 7B
    // shape, us, pinned / not: 128 rows 65.4 / 64.2, 176 rows 109.8 / 105.0, 192 rows 113.2 / 108.9; up to 97 rows within the noise
    // of a card).  Fetches past the range re-read its last chunk (in bounds, never used).
    const int c_max = n_chunks - 1;
    auto cl = [&](int c) { return c < c_max ? c : c_max; };
    auto load_w_pinned = [&](int c) {
      WChunk w;
#pragma unroll
      for (int t = 0; t < TN; ++t) w.f[0][t] = load_weights<ONCE>(wsrc + (((int64_t)(kt0 + c) * TN + t) << 6));
      return w;
    };
    auto load_x_pinned = [&](int c) {
      XStage x;
#pragma unroll
      for (int i = 0; i < PER_THREAD; ++i) {
        int u = tid + i * TH;
        if (CHUNK_U4 % TH != 0 && u >= CHUNK_U4) u = CHUNK_U4 - 1;  // surplus threads fetch the last unit again
        x.u[i] = xsrc[(int64_t)(kt0 + c) * xstep + u];              // CH == 1, two planes: unit u of the step
      }
      return x;
    };
    static_assert(!DEEP || (CH == 1 && PLANES == 2), "the pinned loads assume one two-plane k step per chunk");
    const int c_ssq4 = c_ssq > 0 ? c_ssq / 4 * 4 : 0;
    XStage xa = load_x_pinned(0), xb;  // xa: even chunks, xb: odd chunks
    WChunk w0 = load_w_pinned(0);
    xb = load_x_pinned(cl(1));
    WChunk w1 = load_w_pinned(cl(1));
    WChunk w2 = load_w_pinned(cl(2));
    WChunk w3;
    store_x(0, xa);
    __syncthreads();
    DED_STAMP(1)
    int c = 0;
    auto stage = [&](XStage& xl, WChunk& wl, const WChunk& w, int buf, const XStage& xs_) {
      xl = load_x_pinned(cl(c + 2));
      if (ONCE) pin_loads();
      wl = load_w_pinned(cl(c + 3));
      if (ONCE) pin_loads();
      compute(w, buf);
      if (ONCE) __builtin_amdgcn_sched_barrier(0);
      store_x(buf ^ 1, xs_);
      __syncthreads();
      ++c;
    };
    // (whole turns, the row sums, the rest: with the row sums' loads under a condition inside the loop the compiler waited for
    // every load in flight once per turn)
    while (c < c_ssq4) {
      stage(xa, w3, w0, 0, xb);
      stage(xb, w0, w1, 1, xa);
      stage(xa, w1, w2, 0, xb);
      stage(xb, w2, w3, 1, xa);
    }
    ssq_issue(epi, rb0, lane, wv, 2 * NWN, ssq);
    for (;;) {
      stage(xa, w3, w0, 0, xb);
      if (c >= n_chunks) break;
      stage(xb, w0, w1, 1, xa);
      if (c >= n_chunks) break;
      stage(xa, w1, w2, 0, xb);
      if (c >= n_chunks) break;
      stage(xb, w2, w3, 1, xa);
      if (c >= n_chunks) break;
    }
  } else {
    WChunk w0 = load_w(0);
    XStage x0 = load_x(0);
    WChunk w1 = load_w(1);
    int buf = 0;
    store_x(0, x0);
    __syncthreads();
    DED_STAMP(1)
    if (c_ssq < 0) ssq_issue(epi, rb0, lane, wv, 2 * NWN, ssq);
    for (int c = 0; c + 2 < n_chunks; ++c) {
      XStage xn = load_x(c + 1);
      WChunk w2 = load_w(c + 2);
      if (c == c_ssq) ssq_issue(epi, rb0, lane, wv, 2 * NWN, ssq);
      compute(w0, buf);
      store_x(buf ^ 1, xn);
      __syncthreads();
      // (held behind the barrier: in the instance of three row blocks the copies, which wait for every weight load in flight, were
      // moved in front of it, with the LDS stores behind them.  48 rows, us, moved / held: 8B shape gate/up 50.4 / 46.6, LM head
      // 175.9 / 171.1; 13B shape gate/up 58.9 / 54.7, QKV 37.6 / 36.6)
      __builtin_amdgcn_sched_barrier(0);
      w0 = w1;
      w1 = w2;
      buf ^= 1;
    }
    XStage xn = load_x(n_chunks - 1);  // last two chunks: nothing left to prefetch
    compute(w0, buf);
    store_x(buf ^ 1, xn);
    __syncthreads();
    compute(w1, buf ^ 1);
  }
  DED_STAMP(2)
  ssq_publish(epi, rb0, lane, threadIdx.x >> 6, 2 * NWN, ssq, s_ssq);
  // the halves are added through LDS: half 0 ends up with the first H0 row blocks of its feature group, half 1 with the others,
  // in acc[t][0..]; each half hands the other what it does not finish
  constexpr int H0 = (RBG + 1) / 2, H1 = RBG - H0;
  __syncthreads();
  {
    constexpr int HALF_U4 = TN * H0 * 64;
    float4* out = reinterpret_cast<float4*>(lds) + (half * NWN + wn) * HALF_U4 + lane;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int j = 0; j < H0; ++j) {
        const f32x4_t v = half == 0 ? acc[t][H0 + j < RBG ? H0 + j : RBG - 1] : acc[t][j];
        if (j < H1 || half == 1) out[(t * H0 + j) * 64] = make_float4(v[0], v[1], v[2], v[3]);
      }
    __syncthreads();
    const float4* in = reinterpret_cast<const float4*>(lds) + ((1 - half) * NWN + wn) * HALF_U4 + lane;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int j = 0; j < H0; ++j) {
        if (j < H1 || half == 0) {
          const float4 v = in[(t * H0 + j) * 64];
          const f32x4_t mine = half == 0 ? acc[t][j] : acc[t][H0 + j < RBG ? H0 + j : RBG - 1];
          acc[t][j] = mine + f32x4_t{v.x, v.y, v.z, v.w};
        }
      }
  }
  DED_STAMP(3)
  const float row_scale = ssq_scale(epi, lane, 2 * NWN, s_ssq);
  const bool store_ok = ng_raw < NG;
  // every wavefront finishes the row blocks it holds, or writes them as this workgroup's slice; in the last workgroup it then
  // fetches the same row blocks of the other slices and finishes those
  float* slice = part + (int64_t)split * part_stride;
  if (splits > 1) {
    if (store_ok) {
      if (H0 == H1) store_slice<H0>(slice, NG, ng, half * H0, lane, acc);
      else if (half == 0) store_slice<H0>(slice, NG, ng, 0, lane, acc);
      else store_slice<H1>(slice, NG, ng, H0, lane, acc);
    }
    if (!take_ticket(splits, counters, &sh.flag)) return;
  }
  if (!store_ok) return;
  auto finish = [&](auto held, int rb_lo) {
    constexpr int RBN = decltype(held)::value;
    if (splits > 1) sum_slices_keep_own<RBN>(part, part_stride, split, splits, NG, ng, rb_lo, lane, acc);
    DED_STAMP(6)
    run_epilogue<EPI, RBN>(epi, ng, N, rb0, rb0 + rb_lo, row_scale, lane, acc);
  };
  if (H0 == H1) finish(std::integral_constant<int, H0>(), half * H0);
  else if (half == 0) finish(std::integral_constant<int, H0>(), 0);
  else finish(std::integral_constant<int, H1>(), H0);
  DED_STAMP(7)
}
// RBG: row blocks of the larger groups; others have one less
template <int NWN, int PLANES, int EPI, bool ONCE, int RBG>
__global__ __launch_bounds__(NWN * 128, 2) void gemm_wide_kernel(float* __restrict__ part, int64_t part_stride,
                                                                 const uint4* xp,
                                                                 const uint4* wp, int RB, int larger, int N, int KT,
                                                                 int splits, int* __restrict__ counters,
                                                                 GemmEpilogue epi) {
  __shared__ WideShared<NWN, PLANES, RBG> sh;
  const int rb0 = ONCE ? 0 : group_first<RBG>(larger);
  if (ONCE || (int)blockIdx.z < larger)
    wide_group<NWN, PLANES, EPI, ONCE, RBG>(sh, part, part_stride, xp, wp, RB, rb0, N, KT, splits, counters, epi);
  else
    wide_group<NWN, PLANES, EPI, ONCE, RBG - 1>(sh, part, part_stride, xp, wp, RB, rb0, N, KT, splits, counters, epi);
}

// ------------------------------------------------------------------------------------------
// Slim kernel (one or two row blocks: plain decoding, small trees).  With 16 rows the activations of a projection are a
// fraction of its weights, so nothing is gained by sharing them between wavefronts, and a workgroup can take few
// features and the whole k range: one wavefront per k range, fragments straight into registers D steps ahead, no barrier
// in the loop; the wavefronts' sums meet in LDS and one wavefront per row block runs the epilogue.  No slices, no
// tickets.  The ranges are those of the skinny kernels' plan (`splits` slices of PER ranges each, SUB) and they are added
// in the order of those kernels, so that a row's result has the same bits in a small tree as in a larger one.
// T = 4: a whole 64-feature group; T = 2: tiles t0 and t0 + 2, the partners of the paired epilogues; T = 1: one tile, for
// the narrow residual projections (N = d gives one workgroup per CU); their sums of squares are kept per 4 features.
// Bound by the weight stream at 16 rows, by the activations out of the L2s (~13 TB/s) beyond.  7B widths, 16 rows, in a
// step: QKV 24.8 us, O 8.8, gate/up 37.6, down 18.2, LM head 47.8; plain decoding step 4.13 -> 3.43 ms.  The loops alone
// would allow 21.8 / 36 / 41 (QKV, gate/up, LM head): the rest is the rows' sums of squares, 64 KB per workgroup.
// 32 rows: 104 us per layer against 120 with the kernels above, 48 rows 124.
// ------------------------------------------------------------------------------------------
struct SlimRanges {
  int splits, per;  // slices, ranges per slice: 2 = halves of a wide kernel's slice, 4 / 1 = a stream kernel's wavefronts
  int units;        // k range of slice s: [s * units / splits, (s + 1) * units / splits) groups (wide: then halved), or
  int step;         // of range i: [i * units / (splits * per), ...) in units of `step` k steps (stream)
  int wide;
  int ssq_waves;    // wavefronts that share a row's sums of squares in the kernel of that plan
};

// ((v0 + v1) + v2) + v3 over the four lanes of a quad, in all of them
__device__ __forceinline__ float quad_sum(float v) {
  const int i = __float_as_int(v);
  const float a = __int_as_float(__builtin_amdgcn_mov_dpp(i, 0x00, 0xf, 0xf, true));
  const float b = __int_as_float(__builtin_amdgcn_mov_dpp(i, 0x55, 0xf, 0xf, true));
  const float c = __int_as_float(__builtin_amdgcn_mov_dpp(i, 0xaa, 0xf, 0xf, true));
  const float d = __int_as_float(__builtin_amdgcn_mov_dpp(i, 0xff, 0xf, 0xf, true));
  return ((a + b) + c) + d;
}

template <int T, int RBN, int PLANES, int EPI, int NWMAX>
__global__ __launch_bounds__(NWMAX * 64) void gemm_slim_kernel(const uint4* __restrict__ xp, const uint4* __restrict__ wp,
                                                               int RB, int N, int KT, SlimRanges rg, GemmEpilogue epi) {
  constexpr int STEP_REGS = (T + RBN * PLANES) * 4;
  constexpr int BUDGET = NWMAX > 8 ? 64 : 100;
  constexpr int D = STEP_REGS * 6 <= BUDGET ? 6 : STEP_REGS * 4 <= BUDGET ? 4 : STEP_REGS * 3 <= BUDGET ? 3 : 2;
  extern __shared__ float4 slim_lds[];  // [ranges][RBN][T][64], then the row's sums of squares [16 * RBN][d / 64]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ranges = blockDim.x >> 6;
  const int ng = blockIdx.x / (TN / T), t0 = blockIdx.x % (TN / T);
  int k0, k1;
  if (rg.wide) {
    const int sl = wave >> 1, b = sl * rg.units / rg.splits, e = (sl + 1) * rg.units / rg.splits, half = (e - b) * (PD / 2);
    k0 = b * PD + (wave & 1) * half, k1 = k0 + half;
  } else {
    k0 = wave * rg.units / ranges * rg.step, k1 = (wave + 1) * rg.units / ranges * rg.step;
  }
  // whole turns of the ring, the first `skip` places of them empty
  const int n = k1 - k0, turns = (n + D - 1) / D, skip = turns * D - n;
  const uint4* wsrc = wp + ((((int64_t)ng * KT + k0) * TN + t0) << 6) + lane;
  const uint4* xsrc = xp + (int64_t)k0 * ((int64_t)RB << 7) + lane;
  const int64_t xstep = (int64_t)RB << 7;

  uint4 wr[D][T], xr[D][RBN * PLANES];
  auto issue = [&](int j) {
#pragma unroll
    for (int t = 0; t < T; ++t) wr[j][t] = load_weights<true>(wsrc + ((T == 2 ? 2 * t : t) << 6));
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
      for (int p = 0; p < PLANES; ++p) xr[j][rb * PLANES + p] = xsrc[(rb * 2 + p) << 6];
    wsrc += TN * 64;
    xsrc += xstep;
  };
  f32x4_t acc[T][RBN];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb) acc[t][rb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int j) {
#pragma unroll
    for (int p = 0; p < PLANES; ++p)
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int rb = 0; rb < RBN; ++rb)
          acc[t][rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, wr[j][t]),
                                                              __builtin_bit_cast(f16x8_t, xr[j][rb * PLANES + p]),
                                                              acc[t][rb], 0, 0, 0);
  };

#pragma unroll
  for (int j = 0; j < D; ++j)
    if (j >= skip && turns > 0) issue(j);
  // the rows' sums of squares per 64 features, behind the first weights on their way; four features each or summed already
  float* s_ssq = reinterpret_cast<float*>(slim_lds + ranges * RBN * T * 64);
  const int d64 = KT / 2, row_len = d64 + 1;  // (odd: the rows start in different banks)
  float* s_part = s_ssq + 16 * RBN * row_len;  // [row][ssq_waves]
  if (epi.ssq_in) {
    const int total = 16 * RBN * d64;
    if (epi.ssq_groups == d64) {
      for (int i = threadIdx.x; i < total; i += blockDim.x) s_ssq[i + i / d64] = epi.ssq_in[i];
    } else {
      // in the order of the residual epilogue: tiles one after the other, then the four lanes of a row.  Coalesced: four
      // neighbouring lanes hold the four tiles of a group (a lane that reads all four touches four times the lines: gate/up
      // 42.9 us)
      const float4* src = reinterpret_cast<const float4*>(epi.ssq_in);
      const int total4 = total * 4, stride = blockDim.x;
      for (int i0 = threadIdx.x; i0 < total4; i0 += 8 * stride) {
        float4 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = src[min(i0 + q * stride, total4 - 4 + (lane & 3))];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float x = quad_sum(v[q].x), y = quad_sum(v[q].y), z = quad_sum(v[q].z), w = quad_sum(v[q].w);
          const int i = i0 + q * stride;
          if ((lane & 3) == 0 && i < total4) s_ssq[(i >> 2) + (i >> 2) / d64] = (x + y) + (z + w);
        }
      }
    }
    __syncthreads();
  }
  if (turns > 1) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      if (j >= skip) compute(j);
      issue(j);
    }
    for (int c = 2; c < turns; ++c) {
#pragma unroll
      for (int j = 0; j < D; ++j) {
        compute(j);
        issue(j);
      }
    }
#pragma unroll
    for (int j = 0; j < D; ++j) compute(j);
  } else if (turns == 1) {
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (j >= skip) compute(j);
  }

  if (epi.ssq_in) {  // pairs of groups in the shares that the plan's kernel gives its wavefronts
    const int n2 = d64 >> 1, per = (n2 + rg.ssq_waves - 1) / rg.ssq_waves;
    for (int i = threadIdx.x; i < 16 * RBN * rg.ssq_waves; i += blockDim.x) {
      const int r = i / rg.ssq_waves, w = i - r * rg.ssq_waves;
      const float* row = s_ssq + r * row_len;
      float p = 0.f;
#pragma unroll 4
      for (int g = w * per; g < min(n2, (w + 1) * per); ++g) p += row[2 * g] + row[2 * g + 1];
      s_part[i] = p;
    }
  }
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb) {
      const f32x4_t v = acc[t][rb];
      slim_lds[((wave * RBN + rb) * T + t) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
    }
  __syncthreads();
  // one wavefront per row block; with fewer ranges than row blocks the first takes the rest too
  for (int rb = wave; rb < RBN; rb += ranges) {
    auto at = [&](int w, int t) {
      const float4 v = slim_lds[((w * RBN + rb) * T + t) * 64 + lane];
      return f32x4_t{v.x, v.y, v.z, v.w};
    };
    f32x4_t sum[T][1];
#pragma unroll
    for (int t = 0; t < T; ++t) sum[t][0] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int sl = 0; sl < rg.splits; ++sl) {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int w = sl * rg.per;
        f32x4_t v = at(w, t);
        if (rg.per == 2) v += at(w + 1, t);
        if (rg.per == 4) v = (v + at(w + 2, t)) + (at(w + 1, t) + at(w + 3, t));
        sum[t][0] = sl == 0 ? v : sum[t][0] + v;
      }
    }
    float row_scale = 1.f;
    if (epi.ssq_in) {
      float s = 0.f;
      for (int w = 0; w < rg.ssq_waves; ++w) s += s_part[(rb * 16 + (lane & 15)) * rg.ssq_waves + w];
      row_scale = 1.0f / sqrtf(s * epi.inv_k + epi.eps);
    }
    run_epilogue<EPI, 1, T>(epi, ng, N, rb, rb, row_scale, lane, sum, t0);
  }
}

// ------------------------------------------------------------------------------------------
// Tile kernel (a few hundred rows and more: wide trees, prompt chunks, batches).  With that many rows per weight a projection
// needs the matrix cores and the operand stream at the same time, so operands have to be far ahead of the products
// without holding registers: every operand lies in memory as whole fragments, and the fragments go from memory straight
// into LDS (16 bytes per lane, 1 KiB per instruction): a ring of ST slots of one k step each, 96 - 144 KB, all but one or
// two of them in flight.  The slots are separate arrays and the loop is unrolled over them, so that the compiler sees
// that a slot's reads do not touch the slots still being filled and leaves the waits to the explicit counts; one barrier
// per slot.
// 8 wavefronts = 2 x 4: two groups of GPW x 64 features, four of RBW x 16 rows.  Where the registers allow it (AHEAD) the
// next slot's fragments are read while the present one's are multiplied.
// A workgroup (one per CU) walks a list of items: whole tiles, or one k range of a tile that is split so that a partly
// empty round fills up.  The partial sums of a split tile travel as slices as in the kernels above, ticketed per
// wavefront tile: every wavefront position has a last arriver of its own and no barrier is needed.  The first slots of
// the next item are requested before a tile's epilogue runs.
// What bounds it: at 512 rows and more the matrix cores at the chip's power limit (LM head of a 7B shape, 512 rows:
// 225 us with two planes = 1.19 PFLOP/s executed, and no more than 1.26 with operands that never leave the caches; gate/up
// of the 13B shape, 216 tiles of 256 x 256 in one round: 225 us between launches that draw less power, 250 in a step); at
// 256 rows the operand stream, ~55 GB/s into each CU (gate/up of a 7B shape 119 -> 101 us, QKV 73 -> 61, O 48 -> 27, down 78 -> 44).
// ------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void glb_void_t;
// lane i: 16 bytes at base + its offset -> dst[i].  (The offset is kept from view, as 32 bits: the compiler otherwise holds a
// 64-bit one per load across the loop, or spills it.)
// BUFFER: nothing where the offset is NO_LOAD, past the buffer's end, which the hardware checks.  With global loads to LDS in
// flight the compiler waits for every LDS read before it uses the first, which is what costs the tiles that read and multiply
// in one step (gate/up of the 8B shape, 2048 rows, us, global / buffer: 776 / 759).  The tiles that read a step ahead wait for
// all reads anyway, and setting up the buffer costs them (gate/up of the 7B shape, 256 rows: 100 / 103).
constexpr uint32_t NO_LOAD = 0xf0000000u;
template <bool BUFFER>
__device__ __forceinline__ void load_to_lds(const char* base, uint32_t offset, uint4* dst) {
  asm volatile("" : "+v"(offset));
  if constexpr (BUFFER) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, NO_LOAD, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)dst, 16, offset, 0, 0, 0);
  } else {
    __builtin_amdgcn_global_load_lds((glb_void_t*)(base + offset), (lds_void_t*)dst, 16, 0, 0);
  }
}
template <int N>
__device__ __forceinline__ void wait_loads() {  // all but the last N vector-memory operations, and every LDS read, are done
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x70);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void barrier_only() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Slices of the tile kernel: the same device-scope accesses (sc1: performed at the device's point of coherence) as
// slice_store / slice_load, 16 bytes per lane.
struct SliceRef {
  __amdgpu_buffer_rsrc_t r;
};
constexpr int AUX_DEVICE_SCOPE = 16;  // sc1
__device__ __forceinline__ SliceRef slice_ref(float* p, int bytes) {
  return SliceRef{__builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, 0x00020000)};
}
__device__ __forceinline__ void slice_store16(const SliceRef& s, int byte, f32x4_t v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), s.r, byte, 0, AUX_DEVICE_SCOPE);
}
__device__ __forceinline__ f32x4_t slice_load16(const SliceRef& s, int byte) {
  return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(s.r, byte, 0, AUX_DEVICE_SCOPE));
}

constexpr int TILE_WAVES = 8;
constexpr int SUM_PARTS = 8;  // most k ranges of a product that gemm_sum_slices_kernel adds
constexpr int TILE_LDS = 158 * 1024;  // of the CU's 160 KB, for the ring
template <int PLANES, int GPW, int RBW>
struct TileShape {
  static constexpr int FGS = 2, RGS = TILE_WAVES / FGS;
  static constexpr int FG = FGS * GPW;             // feature groups per workgroup
  static constexpr int RBT = RGS * RBW;            // row blocks per workgroup
  static constexpr int WF = FG * TN, XF = RBT * PLANES;  // fragments per k step
  static constexpr int SLOT_U4 = (WF + XF) * 64;
  static constexpr int ST_MAX = TILE_LDS / (SLOT_U4 * 16);
  static constexpr int ST = ST_MAX >= 6 ? 6 : ST_MAX >= 4 ? 4 : ST_MAX;
  static constexpr int TILE_ELEMS = FG * 64 * RBT * 16;
  static constexpr int ACC_REGS = GPW * TN * RBW * 4, FRAG_REGS = (GPW * TN + RBW * PLANES) * 4;
  static constexpr bool AHEAD = ACC_REGS + 2 * FRAG_REGS <= 168;  // room for two slots' fragments in registers
  static_assert(ST >= 3, "two slots in flight");
};

template <int PLANES, int EPI, int GPW, int RBW>
__global__ __launch_bounds__(512, 2) void gemm_tile_kernel(float* __restrict__ part, const uint4* __restrict__ xp,
                                                           const uint4* __restrict__ wp, int RB, int N, int KT, int tiles,
                                                           int row_tiles, int n_whole, int parts, int ssq_waves,
                                                           int* __restrict__ counters, GemmEpilogue epi) {
  using S = TileShape<PLANES, GPW, RBW>;
  constexpr int FGS = S::FGS, FG = S::FG, RBT = S::RBT, WF = S::WF, XF = S::XF, ST = S::ST;
  constexpr bool AHEAD = S::AHEAD;
  constexpr int WJ = WF / TILE_WAVES, XJ = (XF + TILE_WAVES - 1) / TILE_WAVES;
  constexpr int IN_FLIGHT = (ST - 2) * (WJ + XJ);  // this wavefront's loads issued after the slot it waits for
  static_assert(WF % TILE_WAVES == 0, "every wavefront fetches the same number of weight fragments");
  static_assert(IN_FLIGHT < 64, "the wait counter has 6 bits");
  __shared__ uint4 ring0[S::SLOT_U4], ring1[S::SLOT_U4], ring2[S::SLOT_U4];
  __shared__ uint4 ring3[ST > 3 ? S::SLOT_U4 : 1], ring4[ST > 4 ? S::SLOT_U4 : 1], ring5[ST > 5 ? S::SLOT_U4 : 1];
  __shared__ float s_scale[2][RBT * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fg = wave % FGS, rg = wave / FGS;
  const int NG = (N + 16 * TN - 1) / (16 * TN);
  // Work items: the first n_whole tiles whole, then the others in `parts` k ranges each, range by range.  At any time the
  // workgroups walk the same k range, so that activations (and the weights, between row tiles) meet in the L2s; items
  // next to each other run on one XCD (workgroup ids go to the 8 XCDs in turn).
  const int rest = tiles - n_whole, items = n_whole + rest * parts;
  // Tiles that are all whole are dealt to the XCDs in eight shares, so that a partly filled last round is spread over all of
  // them (gate/up of the 13B shape, 1024 rows, 432 tiles: 506 us with two XCDs idle in it, 473 so; of the 8B shape, 768
  // rows: 310 and 289).  Split ones are dealt round by round: in shares the XCDs walk different k ranges (O of the 7B shape,
  // 512 rows: 46 us round by round, 55 in shares).
  int item = blockIdx.x, step = gridDim.x, end = items;
  if ((gridDim.x & 7) == 0) {
    const int xcd = item & 7, slot = item >> 3;
    if (rest == 0) step >>= 3, item = (xcd * items >> 3) + slot, end = (xcd + 1) * items >> 3;
    else item = xcd * (step >> 3) + slot;
  }
  if (item >= end) return;
  const int64_t xstep = (int64_t)RB << 11;  // bytes of activations per k step
  const int real_rb = epi.rows >> 4;        // row blocks that exist: the operands are padded to 64 rows, and the last row tile may reach past them

  // The segment whose slots are being requested: tile, k range in slots, slots left to request; operand addresses as a
  // wavefront-uniform base that moves with k and a lane offset per load that is fixed inside a tile.
  int tile, part_id, kp, kp_end, req_left;
  const char *wbase, *xbase;
  uint32_t woff[WJ], xoff[XJ];
  auto open_segment = [&]() {
    if (item < n_whole) {
      tile = item, part_id = -1;
      kp = 0, kp_end = KT;
    } else {
      part_id = (item - n_whole) / rest;
      tile = item - part_id * rest;
      kp = part_id * (KT / PD) / parts * PD, kp_end = (part_id + 1) * (KT / PD) / parts * PD;
    }
    req_left = kp_end - kp;
    const int tf = tile / row_tiles, rb_tile = (tile - tf * row_tiles) * RBT;
    wbase = reinterpret_cast<const char*>(wp) + (((int64_t)tf * FG * KT + kp) << 12);
    xbase = reinterpret_cast<const char*>(xp) + kp * xstep + ((int64_t)rb_tile << 11);
#pragma unroll
    for (int j = 0; j < WJ; ++j) {
      const int f = j * TILE_WAVES + wave;
      const int g = min(f >> 2, NG - 1 - tf * FG);  // surplus feature groups re-read a valid one
      woff[j] = (((uint32_t)g * KT) << 12) + ((f & 3) << 10) + (lane << 4);
    }
#pragma unroll
    for (int j = 0; j < XJ; ++j) {
      const int f = min(j * TILE_WAVES + wave, XF - 1);
      // (surplus row blocks are not fetched, or, by global loads, a valid one again; what becomes of them is not stored)
      const int rb = f / PLANES, p = f % PLANES, valid = min(rb, real_rb - 1 - rb_tile);
      xoff[j] = AHEAD || rb == valid ? ((uint32_t)valid << 11) + (p << 10) + (lane << 4) : NO_LOAD;
    }
  };
  auto request = [&](uint4* slot) {
#pragma unroll
    for (int j = 0; j < WJ; ++j) load_to_lds<!AHEAD>(wbase, woff[j], slot + (j * TILE_WAVES + wave) * 64);
#pragma unroll
    for (int j = 0; j < XJ; ++j)
      load_to_lds<!AHEAD>(xbase, xoff[j], slot + (WF + min(j * TILE_WAVES + wave, XF - 1)) * 64);
    // (past the segment's end its last slot is read again, so that the loads in flight stay countable)
    --req_left;
    wbase += req_left > 0 ? 1 << 12 : 0;
    xbase += req_left > 0 ? xstep : 0;
  };
  auto request_first = [&]() {
    request(ring0);
    request(ring1);
    if constexpr (AHEAD || ST > 3) request(ring2);
    if constexpr (AHEAD ? ST > 3 : ST > 4) request(ring3);
    if constexpr (AHEAD ? ST > 4 : ST > 5) request(ring4);
    if constexpr (AHEAD && ST > 5) request(ring5);
  };

  Acc acc[GPW];
  // a slot's fragments in registers: the next slot's are read while the present one's are multiplied
  struct Frags {
    f16x8_t w[GPW * TN], x[RBW * PLANES];
  };
  Frags fa, fb;
  auto read = [&](const uint4* slot, Frags& f) {
    const uint4* lw = slot + fg * (GPW * TN) * 64 + lane;
    const uint4* lx = slot + (WF + rg * (RBW * PLANES)) * 64 + lane;
#pragma unroll
    for (int i = 0; i < RBW * PLANES; ++i) f.x[i] = __builtin_bit_cast(f16x8_t, lx[i << 6]);
#pragma unroll
    for (int i = 0; i < GPW * TN; ++i) f.w[i] = __builtin_bit_cast(f16x8_t, lw[i << 6]);
  };
  auto compute = [&](const Frags& f) {
#pragma unroll
    for (int gw = 0; gw < GPW; ++gw)
#pragma unroll
      for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int p = 0; p < PLANES; ++p)
#pragma unroll
          for (int rb = 0; rb < RBW; ++rb)
            acc[gw][t][rb] =
                __builtin_amdgcn_mfma_f32_16x16x32_f16(f.w[gw * TN + t], f.x[rb * PLANES + p], acc[gw][t][rb], 0, 0, 0);
  };
  // One slot.  With the fragments read a step ahead: the slot's own were read in the step before, by every wavefront once
  // the barrier is passed, so it is free for the request ST slots ahead, and the barrier also says that every wavefront's
  // loads of the next slot have landed.  (The scheduling fences keep the products in front of the next step's wait.)
  auto step_ahead = [&](uint4* slot, const uint4* next, const Frags& now, Frags& then, bool live) {
    wait_loads<IN_FLIGHT>();
    barrier_only();
    request(slot);
    read(next, then);
    __builtin_amdgcn_sched_barrier(0);
    if (live) compute(now);
    __builtin_amdgcn_sched_barrier(0);
  };
  // Otherwise (large wavefront tiles): read and multiplied in the same step; the slot of the step before is free.  The
  // activations stay in registers, the weights pass through two, one fragment ahead of its products.  (The fences hold the
  // compiler to that: with a slot's fragments all in registers it spilled the load addresses, and fetching those inside the
  // loop waited for every load in flight, two of three slots.)
  auto step_direct = [&](const uint4* slot, uint4* freed, bool live) {
    wait_loads<IN_FLIGHT>();
    barrier_only();
    request(freed);
    if (!live) return;
    const uint4* lw = slot + fg * (GPW * TN) * 64 + lane;
    const uint4* lx = slot + (WF + rg * (RBW * PLANES)) * 64 + lane;
    f16x8_t w[2], x[RBW * PLANES];
    w[0] = __builtin_bit_cast(f16x8_t, lw[0]);
#pragma unroll
    for (int i = 0; i < RBW * PLANES; ++i) x[i] = __builtin_bit_cast(f16x8_t, lx[i << 6]);
#pragma unroll
    for (int i = 0; i < GPW * TN; ++i) {
      if (i + 1 < GPW * TN) w[(i + 1) & 1] = __builtin_bit_cast(f16x8_t, lw[(i + 1) << 6]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < PLANES; ++p)
#pragma unroll
        for (int rb = 0; rb < RBW; ++rb)
          acc[i / TN][i % TN][rb] =
              __builtin_amdgcn_mfma_f32_16x16x32_f16(w[i & 1], x[rb * PLANES + p], acc[i / TN][i % TN][rb], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  open_segment();
  request_first();
  for (int par = 0;; par ^= 1) {
    const int cur_tile = tile, cur_part = part_id, n = kp_end - kp;
    const int tf = cur_tile / row_tiles, rb_tile = (cur_tile - tf * row_tiles) * RBT, rbw = rb_tile + rg * RBW;
    const bool any_rows = rbw < real_rb;  // (otherwise this wavefront has nothing to store)
    // (lane numbers of their own for what happens once per tile: the addresses derived from them would otherwise be
    // formed ahead of the loop over tiles and held, or spilled, across the products)
    int ltid = tid, llane = lane;
    asm volatile("" : "+v"(ltid), "+v"(llane));
    // 1 / rms of the tile's input rows, one thread per row, while the first slots are on their way
    if (epi.ssq_in && ltid < RBT * 16) {
      const int r = min(rb_tile * 16 + ltid, RB * 16 - 1);
      const float2* src = reinterpret_cast<const float2*>(epi.ssq_in + (int64_t)r * epi.ssq_groups);
      float s = 0.f;
      const int n2 = epi.ssq_groups >> 1, per = (n2 + ssq_waves - 1) / ssq_waves;
      for (int w = 0; w < ssq_waves; ++w) {
        float p = 0.f;
#pragma unroll 16
        for (int g = w * per; g < min(n2, (w + 1) * per); ++g) p += src[g].x + src[g].y;
        s += p;
      }
      s_scale[par][ltid] = 1.0f / sqrtf(s * epi.inv_k + epi.eps);
    }
#pragma unroll
    for (int gw = 0; gw < GPW; ++gw)
#pragma unroll
      for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int rb = 0; rb < RBW; ++rb) acc[gw][t][rb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // (one exit, after whole turns of the ring: an exit behind every step would give every step accumulators of its own)
    if constexpr (AHEAD) {
      wait_loads<(ST - 1) * (WJ + XJ)>();
      barrier_only();
      read(ring0, fa);
      if constexpr (ST == 3) {
        for (int c = 0; c < n; c += 6) {
          step_ahead(ring0, ring1, fa, fb, true);
          step_ahead(ring1, ring2, fb, fa, c + 1 < n);
          step_ahead(ring2, ring0, fa, fb, c + 2 < n);
          step_ahead(ring0, ring1, fb, fa, c + 3 < n);
          step_ahead(ring1, ring2, fa, fb, c + 4 < n);
          step_ahead(ring2, ring0, fb, fa, c + 5 < n);
        }
      } else {
        for (int c = 0; c < n; c += ST) {
          step_ahead(ring0, ring1, fa, fb, true);
          step_ahead(ring1, ring2, fb, fa, c + 1 < n);
          step_ahead(ring2, ring3, fa, fb, c + 2 < n);
          step_ahead(ring3, ST > 4 ? ring4 : ring0, fb, fa, c + 3 < n);
          if constexpr (ST > 4) {
            step_ahead(ring4, ring5, fa, fb, c + 4 < n);
            step_ahead(ring5, ring0, fb, fa, c + 5 < n);
          }
        }
      }
    } else {
      for (int c = 0; c < n; c += ST) {
        step_direct(ring0, ST == 3 ? ring2 : ST == 4 ? ring3 : ring5, any_rows);
        step_direct(ring1, ring0, any_rows && c + 1 < n);
        step_direct(ring2, ring1, any_rows && c + 2 < n);
        if constexpr (ST > 3) step_direct(ring3, ring2, any_rows && c + 3 < n);
        if constexpr (ST > 4) step_direct(ring4, ring3, any_rows && c + 4 < n);
        if constexpr (ST > 4) step_direct(ring5, ring4, any_rows && c + 5 < n);
      }
    }
    wait_loads<0>();
    barrier_only();  // every wavefront has read its last slot, nothing is in flight: the ring is free
    asm volatile("" : "+v"(llane));
    item += step;
    const bool more = item < end;
    if (more) {
      open_segment();
      request_first();
    }

    // finish the tile, or hand this workgroup's part of it over
    bool finish = any_rows;
    if (cur_part >= 0 && finish) {
      constexpr int WT_ELEMS = GPW * TN * RBW * 256;  // a wavefront tile, in accumulator order
      constexpr int NF = GPW * TN * RBW, CF = S::ACC_REGS > 64 ? 2 : 4;  // its fragments; fragments summed together
      const int wt = rg * FGS + fg, rel = cur_tile - n_whole;
      auto slice = [&](int pt) {
        return slice_ref(part + ((int64_t)pt * rest + rel) * S::TILE_ELEMS + (int64_t)wt * WT_ELEMS, WT_ELEMS * 4);
      };
      if (EPI == EPI_RESIDUAL && !counters) {  // gemm_sum_slices_kernel does the rest
        float* own = part + ((int64_t)cur_part * rest + rel) * S::TILE_ELEMS + (int64_t)wt * WT_ELEMS + llane * 4;
#pragma unroll
        for (int i = 0; i < NF; ++i) *reinterpret_cast<f32x4_t*>(own + i * 256) = acc[i / (TN * RBW)][i / RBW % TN][i % RBW];
        if (!more) break;
        continue;
      }
      {
        const SliceRef own = slice(cur_part);
#pragma unroll
        for (int i = 0; i < NF; ++i) slice_store16(own, (i << 10) + (llane << 4), acc[i / (TN * RBW)][i / RBW % TN][i % RBW]);
      }
#ifdef DED_SPLITK_FENCES
      __atomic_thread_fence(__ATOMIC_RELEASE);
#else
      wait_loads<0>();  // the slice has been stored
#endif
      int prev = 0;
      if (llane == 0) {
        int* ticket = counters + rel * TILE_WAVES + wt;
        prev = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == parts - 1) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      prev = __builtin_amdgcn_readfirstlane(prev);
      asm volatile("" ::: "memory");
      finish = prev == parts - 1;
#ifdef DED_SPLITK_FENCES
      if (finish) __atomic_thread_fence(__ATOMIC_ACQUIRE);
#endif
      if (finish) {
        if (parts == 2) {  // the other part is added to the own (the same sum either way round)
          const SliceRef other = slice(1 - cur_part);
#pragma unroll
          for (int i = 0; i < NF; ++i) {
            acc[i / (TN * RBW)][i / RBW % TN][i % RBW] += slice_load16(other, (i << 10) + (llane << 4));
            if (S::ACC_REGS > 64 && i % 8 == 7) __builtin_amdgcn_sched_barrier(0);  // (registers for eight in flight)
          }
        } else {  // all parts in k order, four at a time (beyond the last part the last one is read again and not added)
#pragma unroll
          for (int c = 0; c < NF; c += CF) {
            f32x4_t sum[CF];
#pragma unroll
            for (int i = 0; i < CF; ++i) sum[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            for (int pt = 0; pt < parts; pt += 4) {
              f32x4_t v[4][CF];
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const SliceRef sl = slice(min(pt + q, parts - 1));
#pragma unroll
                for (int i = 0; i < CF; ++i) v[q][i] = slice_load16(sl, ((c + i) << 10) + (llane << 4));
              }
#pragma unroll
              for (int q = 0; q < 4; ++q)
                if (pt + q < parts) {
#pragma unroll
                  for (int i = 0; i < CF; ++i) sum[i] += v[q][i];
                }
            }
#pragma unroll
            for (int i = 0; i < CF; ++i) acc[(c + i) / (TN * RBW)][(c + i) / RBW % TN][(c + i) % RBW] = sum[i];
            if (S::ACC_REGS > 64) __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
    if (finish) {
      const float row_scale = epi.ssq_in ? s_scale[par][rg * (RBW * 16) + min(llane, RBW * 16 - 1)] : 1.f;
#pragma unroll
      for (int gw = 0; gw < GPW; ++gw) {
        const int ng = (tf * FGS + fg) * GPW + gw;
        if (ng < NG) run_epilogue<EPI, RBW, TN, true>(epi, ng, N, rbw, rbw, row_scale, llane, acc[gw]);
      }
    }
    if (!more) break;
  }
}

// The sums and the epilogue of tiles (128 features x RBW * 64 rows) whose slices the tile kernel has only stored: a wavefront per
// 64 features and 16 rows, so that all CUs share what the last workgroup of a tile would do alone.  Bound by reading the slices
// from the last-level cache and by its start: 144 rows x 4096 features in 8 ranges, 19 MB, 7.7 us; 256 rows, 34 MB, 10.2 us.
template <int RBW>
__global__ __launch_bounds__(256) void gemm_sum_slices_kernel(const float* __restrict__ part, int N, int row_tiles, int tiles, int parts,
                                                              GemmEpilogue epi) {
  using S = TileShape<1, 1, RBW>;
  const int lane = threadIdx.x & 63, w = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int NG = N / (16 * TN), ng = w % NG, rb = w / NG;
  if (rb * 16 >= epi.rows) return;
  const int rt = rb / S::RBT, rg = rb % S::RBT / RBW, tile = ng / S::FG * row_tiles + rt;
  const float* src = part + (int64_t)tile * S::TILE_ELEMS + (rg * S::FGS + ng % S::FGS) * (TN * RBW * 256) + rb % RBW * 256 + lane * 4;
  f32x4_t v[SUM_PARTS][TN], sum[TN][1];
#pragma unroll
  for (int p = 0; p < SUM_PARTS; ++p)
    if (p < parts) {
#pragma unroll
      for (int t = 0; t < TN; ++t) v[p][t] = *reinterpret_cast<const f32x4_t*>(src + (int64_t)p * tiles * S::TILE_ELEMS + t * (RBW * 256));
    }
#pragma unroll
  for (int t = 0; t < TN; ++t) sum[t][0] = v[0][t];
#pragma unroll
  for (int p = 1; p < SUM_PARTS; ++p)
    if (p < parts) {
#pragma unroll
      for (int t = 0; t < TN; ++t) sum[t][0] += v[p][t];
    }
  run_epilogue<EPI_RESIDUAL, 1>(epi, ng, N, rb, rb, 1.f, lane, sum);
}

// Sweep knob, compiled in only with -DDED_GEMM_TUNE_ENV (never in the library build): the environment variable
// DED_GEMM_TUNE="nwn,splits" forces the kernel shape (nwn 0 = stream kernel).
struct Tune {
  int nwn = -1, splits = 0;
  Tune() {
#ifdef DED_GEMM_TUNE_ENV
    if (const char* e = getenv("DED_GEMM_TUNE")) {
      int a = -1, b = 0;
      if (sscanf(e, "%d,%d", &a, &b) == 2 && a >= 0 && b >= 1) {
        nwn = a;
        splits = b;
      }
    }
#endif
  }
};

constexpr int kCUs = 256;
constexpr int kTickets = 1 << 16;  // arrival tickets that a launch may use

// relative cost of a shape: weight stream slowed down by activation reloads and uneven CU filling,
// plus the split-K slices that are written and read back inside the kernel
double shape_cost(int64_t w_bytes, int64_t slice_bytes, int wgs, double x_per_w, int splits) {
  int rounds = (wgs + kCUs - 1) / kCUs;
  double eff = (double)wgs / (double)(rounds * kCUs);
  double stream = (double)w_bytes * (1.0 + 0.35 * x_per_w) / eff;
  return stream + 2.0 * (double)slice_bytes * (splits > 1 ? splits : 0);
}

struct TileDims {
  int groups, row_blocks;  // 64-feature groups and 16-row blocks of a workgroup tile
};
TileDims tile_dims(int tile) {
  const int rbt[3] = {16, 12, 8};
  return TileDims{tile < TILE_128x256 ? 4 : 2, rbt[(tile - TILE_256x256) % 3]};
}
int row_tile_count(int tile, int rows_pad) { return (rows_pad / 16 + tile_dims(tile).row_blocks - 1) / tile_dims(tile).row_blocks; }
int64_t tile_count(int tile, int rows_pad, int N) {
  const int NG = (N + 16 * TN - 1) / (16 * TN), groups = tile_dims(tile).groups;
  return (int64_t)((NG + groups - 1) / groups) * row_tile_count(tile, rows_pad);
}
// whether the slices of a tile plan fit `part_elems` and its k ranges are not empty
bool tile_plan_ok(const GemmPlan& p, int rows_pad, int N, int K, int64_t part_elems) {
  if (p.tile < TILE_256x256 || p.tile > TILE_128x128 || p.splits < 1) return false;
  const TileDims t = tile_dims(p.tile);
  const int64_t tiles = tile_count(p.tile, rows_pad, N), rest = tiles - p.whole;
  if (p.whole == SUMMED_APART)
    return p.tile >= TILE_128x256 && p.splits >= 2 && p.splits <= std::min(SUM_PARTS, K / (32 * PD)) && N % 64 == 0 &&
           tiles * p.splits * t.groups * 64 * t.row_blocks * 16 <= part_elems;
  if (tiles * p.splits > (1 << 20) || p.whole < 0 || rest < 0) return false;
  if (p.splits == 1) return rest == 0;
  return rest > 0 && p.splits <= K / (32 * PD) && rest * TILE_WAVES <= kTickets &&
         rest * p.splits * t.groups * 64 * t.row_blocks * 16 <= part_elems;
}

// Into how many k ranges a product of 256 and more rows is summed: the first x_main groups of 256 features in `main`, the
// others in `rem`.  The shape (and what the context has room for) decides it, not the workgroup tile, so that a result has
// the same bits whichever tile runs.  The ranges are counted so that 256 x 128 (from 512 rows on also 256 x 256) tiles fill the chip's last round of
// one workgroup per CU: as few as it takes, or whole rounds unsplit and only a mostly empty last one split.
struct KRanges {
  int x_main, main, rem;
};
KRanges k_ranges(int rows, int N, int K, int max_splits) {
  const int NG = (N + 16 * TN - 1) / (16 * TN), groups = K / (32 * PD), X = (NG + 3) / 4;
  KRanges best{X, 1, 1};
  double best_cost = 1e300;
  for (int wide = 0; wide <= (rows >= 512 ? 1 : 0); ++wide) {
    const int Z = (rows + (wide ? 255 : 127)) / (wide ? 256 : 128), tiles = X * Z;
    const double slow = wide ? 1.0 : 1.15;
    for (int s = 1; s <= 4 && s <= max_splits && s <= groups; ++s) {
      const int wgs = tiles * s, rounds = (wgs + kCUs - 1) / kCUs;
      const double c = (double)rounds * kCUs / wgs * (1.0 + 0.15 * (s - 1)) * slow;
      if (c < best_cost) {
        best_cost = c;
        best = KRanges{X, s, 1};
      }
    }
    const int full = tiles / kCUs;
    if (max_splits >= 2 && full >= 1 && (full * kCUs) % Z == 0 && full * kCUs < tiles) {
      const int rem = tiles - full * kCUs, rs = std::min(std::min(4, groups), kCUs / rem);
      if (rs >= 2) {
        const double c = (full + (1.0 + 0.15 * (rs - 1)) / rs + 0.05) * kCUs / tiles * slow;
        if (c < best_cost) {
          best_cost = c;
          best = KRanges{full * kCUs / Z, 1, rs};
        }
      }
    }
  }
  return best;
}

// Tile of a launch whose sums have k ranges `r`.  Every tile shape is weighed with the time of one ring slot on a full chip
// (measured, in us: 7B-, 8B- and 13B-width projections, 128 - 2048 rows, random operands).  With fewer workgroups a slot is
// faster where the chip's memory bounds it more than the CU; with two planes and 256 rows and more it is not, and a partly
// filled round takes as long as a full one (gate/up in a step, us, by tile 256 x 256 / x 192 / x 128, 128 x 256 / x 192 /
// x 128: 7B shape, 512 rows 193 / 284 / 207, 221 / 221 / 177; 13B, 512 rows 250 / 383 / 262, 272 / 303 / 286, 2048 rows
// 976 / 962 / 894, 926 / 1001 / 1009).  A hand-over costs about 3 us and 1.5 us per 64 KB slice beyond
// the first, and 25 us more with 128 accumulators per lane (the other part is fetched eight fragments at a time: QKV of a
// 7B shape, 2048 rows, a third of it split, 350 us with 256 x 256 tiles, 337 with 256 x 128).
GemmPlan plan_tiles(const KRanges& r, int rows_pad, int N, int K, int planes, int64_t part_elems, double* us = nullptr) {
  constexpr double slot_us[3][6] = {{0.97, 0.74, 0.52, 0.50, 0.40, 0.31},    // one plane
                                    {1.80, 1.25, 0.86, 0.94, 0.70, 0.51},    // two planes, fewer than 256 rows
                                    {1.50, 1.19, 0.79, 0.84, 0.63, 0.47}};   // two planes, 256 rows and more
  const int kind = planes == 1 ? 0 : rows_pad < 256 ? 1 : 2;
  const int parts = r.main > 1 ? r.main : r.rem;
  GemmPlan best{0, 1, 1, 0, 0};
  double best_cost = 1e300;
  for (int tile = TILE_256x256; tile <= TILE_128x128; ++tile) {
    const TileDims t = tile_dims(tile);
    const int64_t tiles = tile_count(tile, rows_pad, N);
    const int64_t whole = r.main > 1 ? 0 : std::min<int64_t>(tiles, (int64_t)r.x_main * (4 / t.groups) * row_tile_count(tile, rows_pad));
    const int slots = K / 32;
    const double slot = slot_us[kind][tile - TILE_256x256], slice_64k = t.groups * t.row_blocks / 16.0;
    const GemmPlan p{0, 1, parts, tile, (int)whole};
    if (!tile_plan_ok(p, rows_pad, N, K, part_elems)) continue;
    double cost = 0.0;
    auto rounds = [&](int64_t items, int len) {
      const double fill = (double)(items % kCUs) / kCUs;
      cost += len * slot * ((double)(items / kCUs) + (fill > 0 ? kind == 2 ? 1.0 : 0.4 + 0.6 * fill : 0.0));
    };
    rounds(whole, slots);
    rounds((tiles - whole) * parts, (slots + parts - 1) / parts);
    if (parts > 1) cost += 3.0 + 1.5 * (parts - 1) * slice_64k + (tile == TILE_256x256 ? 25.0 : 0.0);
    if (cost < best_cost) {
      best_cost = cost;
      best = p;
    }
  }
  if (us) *us = best_cost;
  return best;
}

// Time of an unsplit wide launch of `wgs` workgroups whose row groups all have four blocks, in us: 8 us around the loop, and a turn
// of it (64 of k) that is longer the more of the chip streams weights.  (Groups of three are faster; 80 and 144 rows are taken for
// 128 and 192 here.)
double wide_us(int nwn, int wgs, int K) {
  constexpr double turn_us[5] = {0.0, 0.0, 0.905, 1.04, 1.24};
  return (wgs + kCUs - 1) / kCUs * 8.0 + K / 64 * turn_us[nwn] * wgs / kCUs;
}

template <int PLANES, int EPI>
bool launch_shape(const GemmPlan& plan, dim3 grid_stream, dim3 grid_wide, float* part, int64_t part_stride,
                  const uint4* xp, const uint4* wp, int RB, int N, int KT, int* counters, const GemmEpilogue& epi,
                  int nw, hipStream_t s) {
  const int splits = plan.splits;
#define DED_ARGS part, part_stride, xp, wp, RB, larger, N, KT, splits, counters, epi
  if (plan.tile) {
    const TileDims t = tile_dims(plan.tile);
    const int row_tiles = (RB + t.row_blocks - 1) / t.row_blocks;
    const int tiles = ((N + 16 * TN - 1) / (16 * TN) + t.groups - 1) / t.groups * row_tiles;
    const bool apart = plan.whole == SUMMED_APART;
    const int whole = apart ? 0 : plan.whole, items = whole + (tiles - whole) * splits;
    int* const tickets = apart ? nullptr : counters;
#define DED_TILE(ID, GPW, RBW)                                                                                       \
  case ID:                                                                                                           \
    hipLaunchKernelGGL((gemm_tile_kernel<PLANES, EPI, GPW, RBW>), dim3(std::min(kCUs, items)), dim3(512), 0, s, part, xp, \
                       wp, RB, N, KT, tiles, row_tiles, whole, splits, plan.ssq_waves, tickets, epi);                        \
    break;
    switch (plan.tile) {
      DED_TILE(TILE_256x256, 2, 4)
      DED_TILE(TILE_256x192, 2, 3)
      DED_TILE(TILE_256x128, 2, 2)
      DED_TILE(TILE_128x256, 1, 4)
      DED_TILE(TILE_128x192, 1, 3)
      DED_TILE(TILE_128x128, 1, 2)
    }
#undef DED_TILE
    if constexpr (PLANES == 1 && EPI == EPI_RESIDUAL) {
      if (apart) {
        const dim3 grid((N / 64 * (epi.rows / 16) + 3) / 4);
#define DED_SUM(RBW) hipLaunchKernelGGL((gemm_sum_slices_kernel<RBW>), grid, dim3(256), 0, s, part, N, row_tiles, tiles, splits, epi)
        if (plan.tile == TILE_128x256) DED_SUM(4);
        else if (plan.tile == TILE_128x192) DED_SUM(3);
        else DED_SUM(2);
#undef DED_SUM
      }
    }
    return true;
  }
  // the logits epilogues read a single plane only where the projection is matrix-bound (the tile kernel above)
  if constexpr (PLANES == 1 && (EPI == EPI_LOGITS || EPI == EPI_TOP2)) {
    return false;
  } else {
  const int rbs = (epi.rows + 15) / 16, groups = RB / 4, most = rbs > 3 * groups ? 4 : 3;
  const bool once = groups == 1;  // every weight byte is read once
  const int larger = rbs - groups * (most - 1);
#define DED_STREAM(NW, READS)                                                                                                        \
  {                                                                                                                                  \
    if (most == 4) hipLaunchKernelGGL((gemm_stream_kernel<NW, PLANES, EPI, READS, 4>), grid_stream, dim3(NW * 64), 0, s, DED_ARGS);  \
    else hipLaunchKernelGGL((gemm_stream_kernel<NW, PLANES, EPI, READS, 3>), grid_stream, dim3(NW * 64), 0, s, DED_ARGS);            \
  }
#define DED_WIDE(NWN, ONCE)                                                                                                          \
  {                                                                                                                                  \
    if (most == 4) hipLaunchKernelGGL((gemm_wide_kernel<NWN, PLANES, EPI, ONCE, 4>), grid_wide, dim3(NWN * 128), 0, s, DED_ARGS);    \
    else hipLaunchKernelGGL((gemm_wide_kernel<NWN, PLANES, EPI, ONCE, 3>), grid_wide, dim3(NWN * 128), 0, s, DED_ARGS);              \
  }
  if (plan.nwn == 0) {
    // (one or two wavefronts: short k, refilled at once whatever the launch; O of d = 1024, 192 rows, us, together / at once 10.6 / 10.3)
    const bool rounds = (int64_t)grid_stream.x * grid_stream.y * grid_stream.z > kCUs;
    if (nw == 4) {
      if (once) DED_STREAM(4, READ_ONCE) else if (rounds) DED_STREAM(4, READ_ROUNDS) else DED_STREAM(4, READ_SHARED)
    } else if (nw == 2) {
      if (once) DED_STREAM(2, READ_ONCE) else DED_STREAM(2, READ_SHARED)
    } else {
      if (once) DED_STREAM(1, READ_ONCE) else DED_STREAM(1, READ_SHARED)
    }
    return true;
  }
  if (plan.nwn == 4) {
    if (once) DED_WIDE(4, true) else DED_WIDE(4, false)
  } else if (plan.nwn == 3) {
    if (once) DED_WIDE(3, true) else DED_WIDE(3, false)
  } else if (plan.nwn == 2) {
    if (once) DED_WIDE(2, true) else DED_WIDE(2, false)
  } else {
    return false;
  }
#undef DED_STREAM
#undef DED_WIDE
#undef DED_ARGS
  return true;
  }
}

}  // namespace

GemmPlan bf16_gemm_plan(int sum_rows, int rows_pad, int N, int K, int planes, int max_splits, int64_t part_elems) {
  static const Tune tune;
  const int NG = (N + 16 * TN - 1) / (16 * TN), groups = K / (32 * PD), rg = sum_rows / 64;
  const int64_t w_bytes = (int64_t)NG * 64 * K * 2, slice = (int64_t)sum_rows * N * 4;
  if (sum_rows >= 256) {
    // No room for the slices: unsplit.  Asked for sum_rows, so that a ragged batch is summed like a full one: a tile whose
    // slices fit sum_rows fits fewer rows as well.
    KRanges r = k_ranges(sum_rows, N, K, max_splits);
    if (!plan_tiles(r, sum_rows, N, K, planes, part_elems).tile) r = k_ranges(sum_rows, N, K, 1);
    return plan_tiles(r, rows_pad, N, K, planes, part_elems);
  }
  GemmPlan best{0, 1, 1};
  double best_cost = 1e300;
  for (int nwn = 0; nwn <= 4; ++nwn) {
    if (tune.nwn >= 0 && nwn != tune.nwn) continue;
    if (nwn == 1) continue;  // a 1-wide tile is the stream kernel
    for (int s = 1; s <= 8 && s <= groups && s <= max_splits; ++s) {
      if (tune.nwn >= 0 && max_splits > 1 && s != std::min(tune.splits, groups)) continue;
      GemmPlan p{nwn, 1, s};
      double x_per_w;
      int wgs;
      if (nwn == 0) {
        p.nw = 4;
        while (p.nw > 1 && s * p.nw > groups) p.nw /= 2;
        wgs = NG * s * rg;
        x_per_w = planes;  // every wavefront reloads its own activations: 64 rows per 64 features
      } else {
        if (groups / s < 2) continue;  // each half needs at least two chunks
        wgs = ((NG + nwn - 1) / nwn) * s * rg;
        x_per_w = (double)planes / nwn + 0.7;  // + barriers and LDS traffic of the wide kernel (calibrated)
      }
      double c = shape_cost(w_bytes, slice, wgs, x_per_w, s);
      if (c < best_cost) {
        best_cost = c;
        best = p;
      }
    }
  }
  // 65 - 255 rows, an unsplit wide kernel: the halves of its k range can run as the two ranges of the tile kernel, added in
  // the same order.  Worth it where the wide kernel reads the weights in several rounds, or k is long against the tile
  // kernel's start-up and hand-over (5 us and 4.5 us per 64 features of the tile beyond plan_tiles' estimate).  Both sides
  // measured in steps, wide / tile, us, 80 - 97 - 128 rows and 144 - 176 - 192; * what the rule takes:
  //   gate/up  7B   57* - 60* - 63* / 69 - 70 - 70                (144 rows and more: split, the rule does not apply)
  //            8B   68* - 72* - 75* / 78 - 79 - 79                109 - 118 - 117 / 95* - 97* - 99*
  //            13B  85 - 89 - 92 / 89* - 90* - 91*                137 - 142 - 144 / 112* - 116* - 118*
  //            d = 2048, F = 8192  25 - 26 - 27 / 31* - 31* - 31*
  //   QKV      7B                                                 51 - 52 - 55 / 54* - 54* - 55*
  //            13B  53 - 56 - 58 / 58* - 59* - 60*                63 - 64 - 68 / 70* - 70* - 70*
  //   LM head of 32000 tokens
  //     d = 2048    45* - 47* - 47* / 49 - 50 - 51                67 - 72 - 73 / 65* - 67* - 68*
  //     d = 4096    83 - 83 - 84 / 79* - 84* - 85*                123 - 129 - 130 / 106* - 107* - 110*
  //     d = 5120    96 - 99 - 100 / 102* - 100* - 100*            157 - 161 - 158 / 121* - 124* - 125*
  //   of 128256     380 - 385 - 389 / 284* - 288* - 292*          548 - 557 - 558 / 380* - 389* - 395*
  // The estimates know groups of four only, so the rule takes the tile kernel too early where groups have three (QKV of the 13B
  // shape, 80 and 144 rows 10 %) and at d = 2048.
  if (rows_pad > 64 && best.nwn && best.splits == 1 && groups % 2 == 0) {
    double tile_us;
    GemmPlan p = plan_tiles(KRanges{0, 2, 1}, rows_pad, N, K, planes, part_elems, &tile_us);
    const int wgs = (NG + best.nwn - 1) / best.nwn * (rows_pad / 64);
    p.ssq_waves = 2 * best.nwn;
    if (p.tile && tile_us + 5.0 + 4.5 * tile_dims(p.tile).groups < wide_us(best.nwn, wgs, K)) return p;
  }
  return best;
}

// A narrow projection (O, down) has few tiles, so k is cut into many ranges, and the workgroup that finishes a tile last reads all of
// its slices, up to 800 KB at the ~60 GB/s that a CU draws, while the others have left.  Where there are three ranges or more the
// slices are added by a launch of their own that all CUs share.  (Two ranges: 8B shape, 600 rows, down 102 -> 108 us, 1024 rows
// 129 -> 126; the existing hand-over stays.)  Below 256 rows the skinny kernels are the faster where the weights are few: O of the 7B
// shape, 80 / 144 / 192 rows, us, stream / tile and sums 18.1 / 20.5, 24.9 / 26.4, 27.6 / 26.7, down of d = 2048, F = 8192 19.1 / 22.7,
// 22.8 / 25.7, 26.0 / 27.1; hence 64 MB of weights.  us, before / now:
//   down  7B   80 - 128 - 192 rows  34.0 - 37.5 - 56.6 / 32.9 - 35.2 - 41.4   320 - 512  61 - 75 / 50 - 62
//         8B                        41.1 - 45.9 - 68.8 / 35.6 - 40.2 - 47.4              68 - 85 / 58 - 72
//         13B                       48.1 - 58.4 - 70.2 / 42.7 - 46.7 - 54.9              80 - 97 / 68 - 86
//   O     7B                                                                             40 - 46 / 32 - 39
//         13B                                                                            47 - 60 / 39 - 49
// 256 rows in full rounds of the existing ranges (N = 4096: 64 tiles in four) stay with them: down takes 46 us there and 42 apart, O
// 28 and 29, and twice the slice bytes cost a 32-layer step at the chip's power limit more than that (prompt chunk of 256 rows, 8600 /
// 8950).  Where the ranges do not fill the chip (13B: O 59 / 35, down 80 / 58) the sums go apart.
// (A small tree beside one of 33 - 48 nodes, 64 packed rows that are summed like 128: 13B, down 34.1 / 36.6; 7B 35.0 / 27.9.)
GemmPlan bf16_gemm_plan_residual(int sum_rows, int rows_pad, int N, int K, int max_splits, int64_t part_elems) {
  auto apart = [&](int rows, int parts) {
    constexpr double slot_us[3] = {0.50, 0.40, 0.31};  // see plan_tiles
    GemmPlan best{0, 1, 1, 0, 0};
    double cost = 1e300;
    for (int tile = TILE_128x256; tile <= TILE_128x128; ++tile) {
      const GemmPlan p{0, 1, parts, tile, SUMMED_APART};
      const double c = row_tile_count(tile, rows) * slot_us[tile - TILE_128x256];
      if (c < cost && tile_plan_ok(p, rows, N, K, part_elems)) cost = c, best = p;
    }
    return best;
  };
  bool worth = sum_rows >= 256 || (sum_rows > 64 && (int64_t)N * K * 2 >= (64 << 20));
  if (sum_rows == 256) {
    const GemmPlan p = bf16_gemm_plan(sum_rows, sum_rows, N, K, 1, max_splits, part_elems);
    const int64_t items = p.whole + (tile_count(p.tile ? p.tile : TILE_128x128, sum_rows, N) - p.whole) * p.splits;
    worth = items * 10 < (items + kCUs - 1) / kCUs * kCUs * 9;  // a round less than nine tenths full
  }
  if (worth) {
    const int tiles = (N / 64 + 1) / 2 * ((sum_rows + 255) / 256);
    const int parts = std::min({kCUs / tiles, SUM_PARTS, max_splits, K / 512});  // (16 ring slots each, at least)
    // (room asked for sum_rows too, so that a ragged batch is summed like a full one)
    if (parts >= 3 && apart(sum_rows, parts).tile) {
      const GemmPlan p = apart(rows_pad, parts);
      if (p.tile) return p;
    }
  }
  return bf16_gemm_plan(sum_rows, rows_pad, N, K, 1, max_splits, part_elems);
}

int bf16_gemm_tiles(int rows_pad, int N, const GemmPlan& plan) {
  const int NG = (N + 16 * TN - 1) / (16 * TN);
  const int gx = plan.nwn == 0 ? NG : (NG + plan.nwn - 1) / plan.nwn;
  return gx * (rows_pad / 64);
}

bool bf16_gemm(float* part, int64_t part_stride, int64_t part_elems, const bf16_t* x_packed, const bf16_t* w_packed, int rows_pad,
               int N, int K, int planes, const GemmPlan& plan, int* counters, const GemmEpilogue& epi,
               hipStream_t s) {
  if (rows_pad <= 0 || rows_pad % 64 || N % 16 || K % (32 * PD) || (planes != 1 && planes != 2)) return false;
  const int RB = rows_pad / 16, KT = K / 32, groups = KT / PD;
  const int NG = (N + 16 * TN - 1) / (16 * TN);
  const int splits = plan.splits;
  if (splits < 1 || !counters) return false;
  if (plan.tile) {
    if (!tile_plan_ok(plan, rows_pad, N, K, part_elems)) return false;
  } else {
    if (splits > groups) return false;
    if (plan.nwn != 0 && groups / splits < 2) return false;
    if (plan.nwn < 0 || plan.nwn > 4) return false;
    if (splits > 1 && (part_stride < (int64_t)rows_pad * NG * 16 * TN || splits * part_stride > part_elems)) return false;
  }
  if ((epi.kind == EPI_RESIDUAL || epi.kind == EPI_QKV || epi.kind == EPI_SILU) && N % 64) return false;
  int nw = plan.nw >= 4 ? 4 : plan.nw >= 2 ? 2 : 1;
  while (nw > 1 && splits * nw > groups) nw /= 2;  // every wavefront needs at least one k group
  const uint4* xp = reinterpret_cast<const uint4*>(x_packed);
  const uint4* wp = reinterpret_cast<const uint4*>(w_packed);
  dim3 gs(NG, splits, RB / 4), gw(plan.nwn ? (NG + plan.nwn - 1) / plan.nwn : 1, splits, RB / 4);
#define DED_GO(P, E) return launch_shape<P, E>(plan, gs, gw, part, part_stride, xp, wp, RB, N, KT, counters, epi, nw, s)
  switch (epi.kind) {
    case EPI_LOGITS:
      if (planes == 2) DED_GO(2, EPI_LOGITS);
      if (plan.tile) DED_GO(1, EPI_LOGITS);
      return false;
    case EPI_TOP2:
      if (planes == 2) DED_GO(2, EPI_TOP2);
      if (plan.tile) DED_GO(1, EPI_TOP2);
      return false;
    case EPI_QKV:
      if (planes == 2) DED_GO(2, EPI_QKV);
      return false;
    case EPI_SILU:
      if (planes == 2) DED_GO(2, EPI_SILU);
      return false;
    case EPI_RESIDUAL:
      if (planes == 1) DED_GO(1, EPI_RESIDUAL);
      return false;
  }
#undef DED_GO
  return false;
}

static SlimRanges slim_ranges(const GemmPlan& p, int K) {
  const int groups = K / (32 * PD);
  if (p.nwn) return SlimRanges{p.splits, 2, groups, 0, 1, 2 * p.nwn};
  int nw = p.nw >= 4 ? 4 : p.nw >= 2 ? 2 : 1;
  while (nw > 1 && p.splits * nw > groups) nw /= 2;
  return SlimRanges{p.splits, nw, K / 32 / RING, RING, 0, nw};
}
bool bf16_gemm_slim_ok(const GemmPlan& plan, int K, int planes) {
  const SlimRanges r = slim_ranges(plan, K);
  // (two planes: up to 16 ranges x 8 KiB and the sums of squares of 32 rows x K / 64 groups in the CU's LDS)
  return !plan.tile && r.splits * r.per <= 16 && K % (32 * PD) == 0 && (planes == 1 || K <= 12288);
}

bool bf16_gemm_slim(const bf16_t* x_packed, const bf16_t* w_packed, int rows, int rows_pad, int N, int K, int planes,
                    const GemmPlan& plan, const GemmEpilogue& epi, hipStream_t s) {
  if (rows < 16 || rows > BF16_SLIM_ROWS || rows % 16 || rows_pad != 64 || N % 16 || !bf16_gemm_slim_ok(plan, K, planes)) return false;
  if (epi.ssq_in && epi.ssq_groups != K / 64 && epi.ssq_groups != K / 4) return false;
  if ((epi.kind == EPI_RESIDUAL || epi.kind == EPI_QKV || epi.kind == EPI_SILU) && N % 64) return false;
  const uint4* xp = reinterpret_cast<const uint4*>(x_packed);
  const uint4* wp = reinterpret_cast<const uint4*>(w_packed);
  const int RB = rows_pad / 16, NG = (N + 16 * TN - 1) / (16 * TN), rbn = rows / 16;
  const SlimRanges rg = slim_ranges(plan, K);
  const int ranges = rg.splits * rg.per;
  const size_t ssq_bytes = epi.ssq_in ? (size_t)rows * (K / 64 + 1 + rg.ssq_waves) * 4 : 0;
#define DED_SLIM(R, T, P, E, NW)                                                                                       \
  {                                                                                                                    \
    hipLaunchKernelGGL((gemm_slim_kernel<T, R, P, E, NW>), dim3(NG * (TN / T)), dim3(ranges * 64),                       \
                       (size_t)ranges * R * T * 1024 + ssq_bytes, s, xp, wp, RB, N, K / 32, rg, epi);                  \
    return true;                                                                                                       \
  }
#define DED_SLIM_ROWS(T, P, E, NW) { if (rbn == 1) DED_SLIM(1, T, P, E, NW) else DED_SLIM(2, T, P, E, NW) }
  // Paired epilogues: whole groups halve the activations fetched per weight, half groups make twice the workgroups.
  // 7B widths, 16 / 32 rows: QKV (192 groups) 21.8 / 27.6 us with whole groups, 25.1 / 32.0 with halves; gate/up (344
  // groups, more than one workgroup per CU) 37.8 / 45.6 and 35.9 / 49.2.
  const bool whole = NG >= 160 && (rows > 16 || NG <= kCUs) && ranges <= 8;
  if (planes == 2 && epi.kind == EPI_QKV) {
    if (whole) DED_SLIM_ROWS(4, 2, EPI_QKV, 8)
    if (ranges <= 8) DED_SLIM_ROWS(2, 2, EPI_QKV, 8)
    DED_SLIM_ROWS(2, 2, EPI_QKV, 16)
  }
  if (planes == 2 && epi.kind == EPI_SILU) {
    if (whole) DED_SLIM_ROWS(4, 2, EPI_SILU, 8)
    if (ranges <= 8) DED_SLIM_ROWS(2, 2, EPI_SILU, 8)
    DED_SLIM_ROWS(2, 2, EPI_SILU, 16)
  }
  if (planes == 2 && epi.kind == EPI_LOGITS) {
    if (ranges <= 8) DED_SLIM_ROWS(4, 2, EPI_LOGITS, 8)
    DED_SLIM_ROWS(4, 2, EPI_LOGITS, 16)
  }
  if (planes == 2 && epi.kind == EPI_TOP2) {
    if (ranges <= 8) DED_SLIM_ROWS(4, 2, EPI_TOP2, 8)
    DED_SLIM_ROWS(4, 2, EPI_TOP2, 16)
  }
  if (planes == 1 && epi.kind == EPI_RESIDUAL) {
    if (ranges <= 8) DED_SLIM_ROWS(1, 1, EPI_RESIDUAL, 8)
    DED_SLIM_ROWS(1, 1, EPI_RESIDUAL, 16)
  }
#undef DED_SLIM_ROWS
#undef DED_SLIM
  return false;
}

}  // namespace ded
