// Kernels used by both storage types: per-node argmax (with the logits' export), sampler, approval walk.
#include "ded_kernels.h"
#include "step_ends.h"

namespace ded {

// ------------------------------------------------------------------------------------------
// Measurement aid: a plain streaming read of a device buffer: every wavefront walks a contiguous region of its own
// with 16-byte non-temporal loads, four in flight per lane (the access pattern of the weight-streaming GEMMs; the
// non-temporal hint is worth ~12 % on this chip: 6.8 against 6.0 TB/s).  Its rate is the ceiling that a weight- or
// cache-streaming kernel can be held against on the same chip in the same run.  The XOR of everything read goes
// to sink[0] so that the loads cannot be dropped.
typedef unsigned probe_u32x4_t __attribute__((ext_vector_type(4)));
__device__ inline uint4 probe_load(const uint4* q) {
  const probe_u32x4_t r = __builtin_nontemporal_load(reinterpret_cast<const probe_u32x4_t*>(q));
  return make_uint4(r.x, r.y, r.z, r.w);
}
__global__ __launch_bounds__(256) void stream_read_kernel(const uint4* __restrict__ src, int64_t n_u4,
                                                          uint32_t* __restrict__ sink) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), n_waves = (int64_t)gridDim.x * 4;
  const int64_t per = n_u4 / n_waves / 256 * 256;  // 16-byte units per wavefront, whole turns of 4 x 64 only
  uint4 a = make_uint4(0, 0, 0, 0);
  const uint4* q = src + wave * per + lane;
  for (int64_t i = 0; i < per; i += 256) {
    const uint4 v0 = probe_load(q + i), v1 = probe_load(q + i + 64), v2 = probe_load(q + i + 128), v3 = probe_load(q + i + 192);
    a.x ^= v0.x ^ v1.x ^ v2.x ^ v3.x;
    a.y ^= v0.y ^ v1.y ^ v2.y ^ v3.y;
    a.z ^= v0.z ^ v1.z ^ v2.z ^ v3.z;
    a.w ^= v0.w ^ v1.w ^ v2.w ^ v3.w;
  }
  for (int64_t i = n_waves * per + wave * 64 + lane; i < n_u4; i += n_waves * 64) {  // what the regions leave over
    const uint4 v = src[i];
    a.x ^= v.x;
    a.y ^= v.y;
    a.z ^= v.z;
    a.w ^= v.w;
  }
  uint32_t x = a.x ^ a.y ^ a.z ^ a.w;
  for (int off = 32; off >= 1; off >>= 1) x ^= __shfl_xor(x, off);
  if (lane == 0 && x == 0x9e3779b9u) sink[0] = x;  // practically never true: the store is the data dependence
}

void launch_stream_read(const void* src, size_t bytes, uint32_t* sink, hipStream_t s) {
  const int64_t n = (int64_t)(bytes / 16);
  if (n <= 0) return;
  hipLaunchKernelGGL(stream_read_kernel, dim3(1024), dim3(256), 0, s, reinterpret_cast<const uint4*>(src), n, sink);
}

// ------------------------------------------------------------------------------------------
// Argmax with top-2 margin.  One workgroup per row; candidates are merged with a fixed rule
// (larger value wins, equal values -> lower index), so the result does not depend on the
// reduction order.
// ------------------------------------------------------------------------------------------
struct Top2 {
  float v1;
  int i1;
  float v2;
};

__device__ inline void top2_push(Top2& t, float v, int i) {
  if (v > t.v1 || (v == t.v1 && i < t.i1)) {
    t.v2 = t.v1;
    t.v1 = v;
    t.i1 = i;
  } else if (v > t.v2) {
    t.v2 = v;
  }
}

__device__ inline void top2_merge(Top2& a, const Top2& b) {
  if (b.v1 > a.v1 || (b.v1 == a.v1 && b.i1 < a.i1)) {
    a.v2 = fmaxf(a.v1, b.v2);
    a.v1 = b.v1;
    a.i1 = b.i1;
  } else {
    a.v2 = fmaxf(a.v2, b.v1);
  }
}

// NaN and +-inf: a row that holds one has no meaningful argmax; it is reported through the row's flag
__device__ inline int nonfinite(float v) { return !(fabsf(v) <= 3.402823466e38f); }

// combine the 256 threads' candidates of one row and write the row's verdict
__device__ inline void top2_block_finish(Top2 t, int bad, int32_t* amax, float* margin, int32_t* flag) {
  for (int off = 32; off >= 1; off >>= 1) {
    Top2 o;
    o.v1 = __shfl_xor(t.v1, off);
    o.i1 = __shfl_xor(t.i1, off);
    o.v2 = __shfl_xor(t.v2, off);
    top2_merge(t, o);
    bad |= __shfl_xor(bad, off);
  }
  __shared__ Top2 sh[4];
  __shared__ int sh_bad[4];
  int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sh[wave] = t;
    sh_bad[wave] = bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    Top2 r = sh[0];
    for (int w = 1; w < 4; ++w) top2_merge(r, sh[w]);
    amax[blockIdx.x] = r.i1;
    margin[blockIdx.x] = r.v1 - r.v2;
    flag[blockIdx.x] = sh_bad[0] | sh_bad[1] | sh_bad[2] | sh_bad[3];
  }
}

typedef float caller_f32x4_t __attribute__((ext_vector_type(4), aligned(4)));  // the caller's array: aligned to its elements only

// (the row goes to the caller from the same registers: as a launch of its own the copy read it once more)
__global__ __launch_bounds__(256) void argmax_kernel(const float* __restrict__ logits, int V, int32_t* __restrict__ amax,
                                                     float* __restrict__ margin, int32_t* __restrict__ flag,
                                                     float* __restrict__ export_to, int max_nodes,
                                                     const int32_t* __restrict__ seq_n, const int32_t* __restrict__ row0,
                                                     const int32_t* __restrict__ blk_seq) {
  const int r = blockIdx.x;
  const float* row = logits + (int64_t)r * V;
  float* out = nullptr;
  if (export_to) {
    const int b = blk_seq[r >> 4], node = r - row0[b];
    if (node < seq_n[b]) out = export_to + ((int64_t)b * max_nodes + node) * V;
  }
  Top2 t = {-INFINITY, 0x7fffffff, -INFINITY};
  int bad = 0;
  int nv4 = ((reinterpret_cast<uintptr_t>(row) & 15) == 0) ? (V / 4) : 0;
  const float4* row4 = reinterpret_cast<const float4*>(row);
  for (int i = threadIdx.x; i < nv4; i += 256) {
    float4 v = row4[i];
    if (out) *reinterpret_cast<caller_f32x4_t*>(out + 4 * i) = caller_f32x4_t{v.x, v.y, v.z, v.w};
    bad |= nonfinite(v.x) | nonfinite(v.y) | nonfinite(v.z) | nonfinite(v.w);
    top2_push(t, v.x, 4 * i);
    top2_push(t, v.y, 4 * i + 1);
    top2_push(t, v.z, 4 * i + 2);
    top2_push(t, v.w, 4 * i + 3);
  }
  for (int i = nv4 * 4 + threadIdx.x; i < V; i += 256) {
    const float v = row[i];
    if (out) out[i] = v;
    bad |= nonfinite(v);
    top2_push(t, v, i);
  }
  top2_block_finish(t, bad, amax, margin, flag);
}

void launch_argmax(const float* logits, const StepMeta& m, int V, int32_t* amax, float* margin, int32_t* flag, float* export_to,
                   int max_nodes, hipStream_t s) {
  if (m.rows <= 0) return;
  hipLaunchKernelGGL(argmax_kernel, dim3(m.rows), dim3(256), 0, s, logits, V, amax, margin, flag, export_to, max_nodes,
                     m.seq_n, m.row0, m.blk_seq);
}

// The same verdict from per-(row, 64-feature group) candidates that the LM-head GEMM's epilogue left instead of
// logits: part[r][g] = (top-1 value, its id, top-2 value, non-finite flag) as four 32-bit words.  The merge rule
// does not depend on the order, so the result equals argmax_kernel's on the materialised row bit for bit.
__global__ __launch_bounds__(256) void top2_reduce_kernel(const uint4* __restrict__ part, int groups,
                                                          int32_t* __restrict__ amax, float* __restrict__ margin,
                                                          int32_t* __restrict__ flag) {
  const uint4* row = part + (int64_t)blockIdx.x * groups;
  Top2 t = {-INFINITY, 0x7fffffff, -INFINITY};
  int bad = 0;
  for (int g = threadIdx.x; g < groups; g += 256) {
    const uint4 p = row[g];
    Top2 o = {__uint_as_float(p.x), (int)p.y, __uint_as_float(p.z)};
    top2_merge(t, o);
    bad |= (int)p.w;
  }
  top2_block_finish(t, bad, amax, margin, flag);
}

void launch_top2_reduce(const void* part, int groups, int rows, int32_t* amax, float* margin, int32_t* flag,
                        hipStream_t s) {
  if (rows <= 0) return;
  hipLaunchKernelGGL(top2_reduce_kernel, dim3(rows), dim3(256), 0, s, reinterpret_cast<const uint4*>(part), groups,
                     amax, margin, flag);
}

// ------------------------------------------------------------------------------------------
// Temperature / top-p sampling of the model's token at every node (stochastic approval, Sec. 2.4: a token
// is sampled from the model's distribution and compared with the draft; Sec. 4.4 varies temperature and
// top-p).  One workgroup per real row.  p_i = softmax(logits / T); the nucleus is the smallest set of most
// probable tokens reaching top_p, ties with its last member included; the token is the inverse CDF of the
// caller's uniform number over the nucleus in token-id order.
//
// Weights w_i = exp((l_i - max) / T) lie in [0, 1], so their bit patterns order like their values, and the nucleus is
// {bits(w) >= t*} with t* the largest threshold under which the set still reaches top_p.  t* is found digit by digit
// (11 + 10 + 10 bits): a histogram of WEIGHT per digit value, a suffix sum over its bins, and on into the bin where the
// sum crosses top_p.  Weights are added as 64-bit fixed point (units of 2^-40): integer sums do not depend on the order
// of their terms, so the histogram can be built with LDS atomics and is still reproducible, and a sum over the
// vocabulary is off by less than V 2^-40 (128256 tokens: 6e-8 against 64 bits, 1.5e-6 for sums in fp32).  A weight below
// 2^-40 of the largest counts as zero (beside such a total fp32 loses it below 2^-24).  Only the first digit looks at every
// token's weight; the later passes compare the logit with the bin's range first.
// Bound by reading the row (from L2 / last-level cache) five times and by the exponentials of the first histogram.
// Measured, 144 rows x 128256 tokens: 93 us; a bisection over global memory (34 passes), which served vocabularies beyond
// what LDS can hold before, took 1.2 ms for these rows.
constexpr int SAMPLE_THREADS = 1024, SAMPLE_WAVES = SAMPLE_THREADS / 64;
constexpr int SAMPLE_BINS = 1024;   // bits(w) <= bits(1.0f) = 0x3f800000: the first digit is at most 0x3f8
constexpr int SAMPLE_COPIES = 8;    // of the first histogram: neighbouring lanes often hit the same bin
constexpr int SAMPLE_SUBS = SAMPLE_THREADS / SAMPLE_WAVES;  // sub-blocks per wavefront in the inverse CDF

__device__ inline unsigned long long weight_fixed(float w) {  // w * 2^40, w in [0, 1]
  const float a = w * 256.0f;
  const unsigned hi = (unsigned)a;
  const unsigned lo = (unsigned)((a - (float)hi) * 4294967296.0f);  // the difference is exact and below 1
  return ((unsigned long long)hi << 32) + lo;
}
__device__ inline unsigned long long wave_sum_u64(unsigned long long v) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
__device__ inline unsigned long long wave_inclusive_u64(unsigned long long v) {
  const int lane = threadIdx.x & 63;
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned long long o = __shfl_up(v, off);
    if (lane >= off) v += o;
  }
  return v;
}
// sums of v over the threads before this one, and over all of them (sh: SAMPLE_WAVES entries; starts with a barrier)
__device__ inline unsigned long long block_exclusive_u64(unsigned long long v, unsigned long long* sh,
                                                         unsigned long long& total) {
  const unsigned long long inc = wave_inclusive_u64(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 63) sh[threadIdx.x >> 6] = inc;
  __syncthreads();
  unsigned long long before = 0, all = 0;
  for (int w = 0; w < SAMPLE_WAVES; ++w) {
    if (w < (int)(threadIdx.x >> 6)) before += sh[w];
    all += sh[w];
  }
  total = all;
  return before + inc - v;
}

__global__ __launch_bounds__(SAMPLE_THREADS) void sample_top_p_kernel(
    const float* __restrict__ logits, int64_t row_stride, int V, float inv_temp, float top_p,
    const float* __restrict__ uniform, const int32_t* __restrict__ seq_n, const int32_t* __restrict__ row0,
    const int32_t* __restrict__ blk_seq, const int32_t* __restrict__ flag, int32_t* __restrict__ token_out,
    int32_t* __restrict__ flag_out) {
  __shared__ unsigned long long hist[SAMPLE_COPIES * SAMPLE_BINS];
  __shared__ unsigned long long sh[SAMPLE_WAVES];
  __shared__ float sh_f[SAMPLE_WAVES];
  __shared__ int sh_bin, sh_sub;
  __shared__ unsigned long long sh_u64;
  const int r = blockIdx.x, seq = blk_seq[r >> 4];
  if (r - row0[seq] >= seq_n[seq]) return;  // padding row
  const float* row = logits + (int64_t)r * row_stride;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) flag_out[r] = flag[r];
  const float u = uniform[r];  // (host memory: requested here, needed at the end)
  const bool vec = (reinterpret_cast<uintptr_t>(row) & 15) == 0;
  auto load4 = [&](int i, float (&l)[4]) {  // past the end: no weight
    if (vec && i + 3 < V) {
      const float4 v = *reinterpret_cast<const float4*>(row + i);
      l[0] = v.x, l[1] = v.y, l[2] = v.z, l[3] = v.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) l[j] = i + j < V ? row[i + j] : -INFINITY;
    }
  };
  float m = -INFINITY;
#pragma unroll 4
  for (int i = tid * 4; i < V; i += SAMPLE_THREADS * 4) {
    float l[4];
    load4(i, l);
    m = fmaxf(m, fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3])));
  }
  for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  for (int i = tid; i < SAMPLE_COPIES * SAMPLE_BINS; i += SAMPLE_THREADS) hist[i] = 0;
  if (tid == 0) sh_bin = 0, sh_sub = 0, sh_u64 = 0;
  if (lane == 0) sh_f[wave] = m;
  __syncthreads();
  for (int w = 0; w < SAMPLE_WAVES; ++w) m = fmaxf(m, sh_f[w]);
  auto weight = [&](float l) {  // in [0, 1] whatever the row holds (a row with a NaN or an infinity is reported, not used)
    const float w = __expf((l - m) * inv_temp);
    return w >= 0.f ? fminf(w, 1.0f) : 0.f;
  };
  // logit below which the weight is certainly under `w` (the margin covers the rounding of exp and log)
  auto logit_floor = [&](float w) { return w > 0.f ? m + (__logf(w) - 1e-3f) / inv_temp - 1e-5f * fabsf(m) : -INFINITY; };

#pragma unroll 4
  for (int i = tid * 4; i < V; i += SAMPLE_THREADS * 4) {
    float l[4];
    load4(i, l);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float w = weight(l[j]);
      const unsigned long long q = weight_fixed(w);
      if (q) atomicAdd(&hist[(lane & (SAMPLE_COPIES - 1)) * SAMPLE_BINS + (__float_as_uint(w) >> 20)], q);
    }
  }
  __syncthreads();
  unsigned long long own = 0;
#pragma unroll
  for (int c = 0; c < SAMPLE_COPIES; ++c) own += hist[c * SAMPLE_BINS + tid];
  // Thread t stands for bin t of the digit.  The crossing bin is the highest one whose suffix sum (plus the weight above
  // the digit's range) reaches `need`: the one with  suffix >= need  and  suffix without it < need.
  unsigned long long Z = 0, above = 0, need = 0;
  auto crossing = [&](unsigned long long in_bin, bool first) {
    unsigned long long total;
    const unsigned long long before = block_exclusive_u64(in_bin, sh, total);
    if (first) {
      Z = total;
      need = (unsigned long long)ceil((double)top_p * (double)Z);
      need = need > Z ? Z : need < 1 ? 1 : need;
    }
    const unsigned long long beyond = above + (total - before - in_bin), with = beyond + in_bin;
    if (with >= need && beyond < need) {
      sh_bin = tid;
      sh_u64 = beyond;
    }
    __syncthreads();
    above = sh_u64;
    return (uint32_t)sh_bin;
  };
  uint32_t lo = crossing(own, true);  // digits found so far
  for (int shift = 10; shift >= 0; shift -= 10) {
    hist[tid] = 0;
    const float l_min = logit_floor(__uint_as_float(lo << (shift + 10)));
    __syncthreads();
    for (int i = tid * 4; i < V; i += SAMPLE_THREADS * 4) {
      float l[4];
      load4(i, l);
      if (fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3])) >= l_min) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float w = weight(l[j]);
          const uint32_t bits = __float_as_uint(w);
          if (bits >> (shift + 10) == lo) atomicAdd(&hist[(bits >> shift) & 1023u], weight_fixed(w));
        }
      }
    }
    __syncthreads();
    lo = (lo << 10) | crossing(hist[tid], false);
  }
  // Inverse CDF over the nucleus {bits(w) >= lo} in id order.  The ids are cut into 1024 sub-blocks of whole 256-id
  // groups, dealt to the wavefronts in turn; their sums locate the target's sub-block, which one wavefront walks.
  const float l_min = logit_floor(__uint_as_float(lo));
  auto nucleus_mass = [&](const float (&l)[4], unsigned long long (&q)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = 0;
    if (fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3])) >= l_min) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float w = weight(l[j]);
        if (__float_as_uint(w) >= lo) q[j] = weight_fixed(w);
      }
    }
  };
  const int groups = (V + 255) / 256, per_sub = (groups + SAMPLE_WAVES * SAMPLE_SUBS - 1) / (SAMPLE_WAVES * SAMPLE_SUBS);
  __syncthreads();
  for (int s = 0; s < SAMPLE_SUBS; ++s) {
    unsigned long long sum = 0;
    const int sub = s * SAMPLE_WAVES + wave, g0 = sub * per_sub;
    for (int gi = g0; gi < min(g0 + per_sub, groups); ++gi) {
      float l[4];
      unsigned long long q[4];
      load4(gi * 256 + lane * 4, l);
      nucleus_mass(l, q);
      sum += q[0] + q[1] + q[2] + q[3];
    }
    if (g0 < groups) sum = wave_sum_u64(sum);
    if (lane == 0) hist[sub] = sum;
  }
  __syncthreads();
  unsigned long long total;
  const unsigned long long mine = hist[tid], before = block_exclusive_u64(mine, sh, total);
  unsigned long long target = (unsigned long long)((double)u * (double)total);
  target = target < total ? target : total - 1;
  if (before <= target && target < before + mine) {
    sh_sub = tid;
    sh_u64 = before;
  }
  __syncthreads();
  if (wave != sh_sub % SAMPLE_WAVES) return;
  unsigned long long run = sh_u64;
  const int g0 = sh_sub * per_sub;
  for (int gi = g0; gi < min(g0 + per_sub, groups); ++gi) {
    float l[4];
    unsigned long long q[4];
    load4(gi * 256 + lane * 4, l);
    nucleus_mass(l, q);
    const unsigned long long sum = q[0] + q[1] + q[2] + q[3], inc = run + wave_inclusive_u64(sum);
    unsigned long long at = inc - sum;
    if (at <= target && target < inc) {  // exactly one lane of one group
      int pick = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (at <= target && target < at + q[j]) pick = j;
        at += q[j];
      }
      token_out[r] = gi * 256 + lane * 4 + pick;
    }
    run = __shfl(inc, 63);
  }
}

void launch_sample_top_p(const float* logits, int64_t row_stride, const StepMeta& m, int V, float temperature,
                         float top_p, const float* uniform, const int32_t* flag, int32_t* token_out, int32_t* flag_out,
                         hipStream_t s) {
  if (m.rows <= 0) return;
  hipLaunchKernelGGL(sample_top_p_kernel, dim3(m.rows), dim3(SAMPLE_THREADS), 0, s, logits, row_stride, V,
                     1.0f / temperature, top_p, uniform, m.seq_n, m.row0, m.blk_seq, flag, token_out, flag_out);
}

// ------------------------------------------------------------------------------------------
// One workgroup per sequence.
__global__ __launch_bounds__(256) void accept_walk_kernel(ApprovalWalk w) {
  __shared__ WalkShared sh;
  const int len = approval_walk(w, blockIdx.x, sh);
  report_walk(w, blockIdx.x, sh, len);
}
void launch_accept_walk(const ApprovalWalk& w, hipStream_t s) {
  hipLaunchKernelGGL(accept_walk_kernel, dim3(w.batch), dim3(256), 0, s, w);
}

}  // namespace ded
