// fp32 storage path: plain row-major buffers, cache [B][Hkv][cap][hd].  Contractions run on the fp32 matrix
// instructions (v_mfma_f32_16x16x4_f32: fp32 operands and accumulators, nothing is rounded to a shorter type); every
// reduction has a fixed order.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "ded_kernels.h"
#include "step_ends.h"

namespace ded {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float cache_v4f __attribute__((ext_vector_type(4), aligned(4)));  // the caller's cache: aligned to its elements only

__device__ inline float wave_sum(float v) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
__device__ inline float wave_max(float v) {
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

// block-wide reductions for 256 threads; `sh` needs 4 floats
__device__ inline float block_sum_256(float v, float* sh) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}
__device__ inline float block_max_256(float v, float* sh) {
  v = wave_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

// ------------------------------------------------------------------------------------------
// Operands of the projections lie in memory as the matrix instructions read them ("packed"): a matrix of R rows (features of
// a weight, tree rows of an activation) and K columns is cut into tiles of 16 rows x 16 k, 1 KiB each, the tiles of 16 rows
// one after the other along k.  Inside a tile lane = (k / 4 % 4) * 16 + row % 16 holds four consecutive k, so one load
// instruction of a wavefront fetches a whole tile from 1 KiB of contiguous memory, and a result tile of the 16x16x4
// instruction (lane = (feature / 4 % 4) * 16 + row) is stored as the next projection's input without a shuffle.  Row-major
// operands cost 16 rows x 64 bytes per load instruction, all 16 on the same memory channel where the row stride is a
// power of two.  K and the features are padded with zeros to whole tiles.
__host__ __device__ inline int tiles16(int n) { return (n + 15) / 16; }
__device__ inline int64_t packed_unit(int r, int k, int kt) {  // in units of four floats; kt = tiles16(K)
  return ((int64_t)(r >> 4) * kt + (k >> 4)) * 64 + ((k >> 2) & 3) * 16 + (r & 15);
}

// dst = packed W[n][k] * gain[k] (gain null: 1).  The RMSNorm gain of a projection's input multiplies here, once, instead of
// every input element in every workgroup: one fp32 rounding per product either way.
__global__ __launch_bounds__(256) void f32_pack_weight_kernel(float4* __restrict__ dst, const float* __restrict__ src,
                                                              const float* __restrict__ gain, int N, int K, int kt) {
  const int lane = threadIdx.x & 63, k = ((blockIdx.x * 4 + (threadIdx.x >> 6)) * 4 + (lane >> 4)) * 4;
  const int n = blockIdx.y * 16 + (lane & 15);
  if (k >= kt * 16) return;
  float v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = n < N && k + i < K ? src[(int64_t)n * K + k + i] : 0.f;
    if (gain && k + i < K) v[i] *= gain[k + i];
  }
  dst[((int64_t)blockIdx.y * kt + (k >> 4)) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
}
void f32_pack_weight(float* dst, const float* src, const float* gain, int N, int K, hipStream_t s) {
  const int kt = tiles16(K), nt = tiles16(N);
  for (int n0 = 0; n0 < nt; n0 += 32768) {  // (grid limit of the second dimension)
    const int n = std::min(nt - n0, 32768);
    hipLaunchKernelGGL(f32_pack_weight_kernel, dim3((kt + 3) / 4, n), dim3(256), 0, s,
                       reinterpret_cast<float4*>(dst) + (int64_t)n0 * kt * 64, src + (int64_t)n0 * 16 * K, gain, N - n0 * 16, K, kt);
  }
}

// ------------------------------------------------------------------------------------------
// x (packed) = emb[token]; a wavefront takes one tile of 16 rows x 16 dims.  The workgroups behind those of the embedding do
// the step's front work.
__global__ __launch_bounds__(256) void f32_embed_kernel(float4* __restrict__ x, const float* __restrict__ emb, StepFront f, int d,
                                                        int kt, int groups) {
  const int lane = threadIdx.x & 63, rb = blockIdx.x / groups;
  if (rb * 16 >= f.rows) {
    step_front(f, blockIdx.x - f.rows / 16 * groups);
    return;
  }
  const int c = (blockIdx.x - rb * groups) * 4 + (threadIdx.x >> 6), k = c * 16 + (lane >> 4) * 4;
  if (c >= kt) return;
  const float* src = emb + (int64_t)f.token[rb * 16 + (lane & 15)] * d + k;
  float v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = k + i < d ? src[i] : 0.f;
  x[((int64_t)rb * kt + c) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
}
void f32_embed(float* x, const float* emb, const StepFront& f, int d, hipStream_t s) {
  const int groups = (tiles16(d) + 3) / 4;
  hipLaunchKernelGGL(f32_embed_kernel, dim3(f.rows / 16 * groups + step_front_blocks(f)), dim3(256), 0, s,
                     reinterpret_cast<float4*>(x), emb, f, d, tiles16(d), groups);
}

// ------------------------------------------------------------------------------------------
// Projections with fused neighbours:  Y[r][n] = sum_k X[r][k] W[n][k], X optionally RMS-normalised on the way in, Y
// going into what the decoder does with it (F32_* in ded_kernels.h).  X and W are packed (above).
//
// A workgroup owns FT x RT tiles of 16 features x 16 rows; its 8 wavefronts take the k tiles in turn and meet in LDS.
// Operands go straight from memory to registers, D k tiles ahead; component j of a lane's 16 bytes is the operand of the
// j-th matrix instruction (both operands permute k alike).  Splitting k over the wavefronts is what fills the chip at the
// sizes of this path (a d = 256 model has 16 feature tiles per projection) and keeps the chain of dependent loads short.
// RMSNorm is applied as (W * gain) . x * (1 / rms): the wavefronts form sum(x^2) from the operands they load anyway.
// Bound by the fp32 matrix instructions (64 flop per cycle and SIMD) and, the smaller the tile the more, by the operands into
// each CU: 2 KiB per 32 cycles of matrix work with 1 x 1 tiles, 6 KiB per 256 with 4 x 2.  160 rows, K = 1024, us with
// row-major operands and the gain multiplied into every input / now: gate/up of N = 5632 37.6 / 17.2 (matrix instructions
// alone: 11.7), QKV of N = 3072 22.2 / 9.8, LM head of N = 8192 45.4 / 24.  Deeper rings are slower: 448 rows, gate/up,
// 4 x 2 tiles, 2 / 3 / 4 k tiles ahead: 42.5 / 44.9 / 98 (spilled); 2 x 2, 3 / 4 / 6: 45.4 / 50.7 / 54.6.
template <int FT, int RT, int D, int EPI>
__global__ __launch_bounds__(512, 4) void f32_mfma_gemm_kernel(F32Gemm g) {
  constexpr int NW = 8;
  constexpr bool NORM = EPI != F32_RESIDUAL, PAIRED = EPI == F32_SILU || EPI == F32_QKV;
  constexpr int UF = PAIRED ? FT / 2 : FT;  // a unit = a feature tile, or a pair of partner tiles (t, t + UF)
  static_assert(!PAIRED || FT % 2 == 0, "partner tiles come in pairs");
  static_assert(UF * RT <= NW, "one wavefront finishes one unit of one row block");
  __shared__ float4 red[NW][FT * RT][64];
  __shared__ float s_ss[NORM ? NW : 1][RT][16];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // (scalar: addresses are a scalar base and the lane)
  const unsigned lane = threadIdx.x & 63, m16 = lane & 15, quad = lane >> 4;
  const int nrb = g.rows / 16, kt = tiles16(g.K), half = g.hd / 2;
  // Workgroups go to the 8 XCDs in turn: every XCD gets a contiguous share of the feature units, the row groups of a unit
  // next to each other, so that a unit's weights come into one L2 only.
  const int n_rg = (nrb + RT - 1) / RT, xcd = blockIdx.x & 7, share = gridDim.x >> 3, rest = gridDim.x & 7;
  const int lin = xcd * share + min(xcd, rest) + (blockIdx.x >> 3);
  const int u0 = lin / n_rg * UF, rb0 = (lin - lin / n_rg * n_rg) * RT;
  const int n_units = EPI == F32_SILU ? tiles16(g.N / 2) : EPI == F32_QKV ? g.N / 32 : tiles16(g.N);
  // the feature tile of unit u (PAIRED: of its first partner) and its partner's
  auto tile_of = [&](int u, int second) {
    if (EPI == F32_SILU) return second * n_units + u;
    if (EPI == F32_QKV) {
      const int per = half / 16, hs = u / per;
      return hs * 2 * per + (u - hs * per) + second * per;
    }
    return u;
  };
  const char *wp[FT], *xp[RT];
#pragma unroll
  for (int t = 0; t < FT; ++t)
    wp[t] = reinterpret_cast<const char*>(g.W) + (int64_t)tile_of(min(u0 + t % UF, n_units - 1), t / UF) * kt * 1024;
#pragma unroll
  for (int t = 0; t < RT; ++t) xp[t] = reinterpret_cast<const char*>(g.X) + (int64_t)min(rb0 + t, nrb - 1) * kt * 1024;
  // what this wavefront finishes after the reduction
  const int fu = wave % UF, rt = wave / UF, u = u0 + fu, rb = rb0 + rt, r = rb * 16 + m16;
  const bool finishes = wave < UF * RT && u < n_units && rb < nrb;
  // (the residual's old values are requested first: they have arrived by then)
  const int64_t at = ((int64_t)rb * tiles16(g.N) + u) * 64 + lane;
  v4f old = v4f{0.f, 0.f, 0.f, 0.f};
  if (EPI == F32_RESIDUAL && finishes) old = reinterpret_cast<const v4f*>(g.Y)[at];
  v4f acc[FT][RT];
  float ss[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    ss[i] = 0.f;
#pragma unroll
    for (int t = 0; t < FT; ++t) acc[t][i] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  struct Chunk {
    v4f w[FT], x[RT];
  };
  auto load = [&](Chunk& q, int c) {
    const uint32_t off = (uint32_t)c * 1024 + lane * 16;
#pragma unroll
    for (int t = 0; t < FT; ++t) q.w[t] = *reinterpret_cast<const v4f*>(wp[t] + off);
#pragma unroll
    for (int t = 0; t < RT; ++t) q.x[t] = *reinterpret_cast<const v4f*>(xp[t] + off);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto compute = [&](const Chunk& q) {
    if (NORM) {
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        const v4f x = q.x[i];
        ss[i] += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int t = 0; t < FT; ++t)
#pragma unroll
        for (int j = 0; j < RT; ++j)
          acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(q.w[t][i], q.x[j][i], acc[t][j], 0, 0, 0);
  };
  // k tiles wave, wave + 8, ...: D in flight; the last turns load only what there is
  if (wave < kt) {
    const int n = (kt - wave + NW - 1) / NW;
    Chunk st[D];
#pragma unroll
    for (int i = 0; i < D; ++i) load(st[i], wave + min(i, n - 1) * NW);
    int c = 0;
    for (; c + 2 * D <= n; c += D) {
#pragma unroll
      for (int i = 0; i < D; ++i) {
        compute(st[i]);
        load(st[i], wave + (c + D + i) * NW);
      }
    }
#pragma unroll
    for (int i = 0; i < D; ++i)
      if (c + i < n) {
        compute(st[i]);
        if (c + D + i < n) load(st[i], wave + (c + D + i) * NW);
      }
#pragma unroll
    for (int i = 0; i < D; ++i)
      if (c + D + i < n) compute(st[i]);
  }
  // the wavefronts' k shares meet in LDS, added in wavefront order
#pragma unroll
  for (int t = 0; t < FT; ++t)
#pragma unroll
    for (int j = 0; j < RT; ++j) red[wave][t * RT + j][lane] = make_float4(acc[t][j][0], acc[t][j][1], acc[t][j][2], acc[t][j][3]);
  if (NORM) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      float v = ss[i];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (quad == 0) s_ss[wave][i][m16] = v;
    }
  }
  __syncthreads();
  if (!finishes) return;
  float scale = 1.f;
  if (NORM) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) v += s_ss[w][rt][m16];
    scale = 1.0f / sqrtf(v / (float)g.K + g.eps);
  }
  v4f y[PAIRED ? 2 : 1];
#pragma unroll
  for (int t = 0; t < (PAIRED ? 2 : 1); ++t) {
    v4f v = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float4 q = red[w][(t * UF + fu) * RT + rt][lane];
      v += v4f{q.x, q.y, q.z, q.w};
    }
    y[t] = NORM ? v * scale : v;
  }
  if (EPI == F32_RESIDUAL) {  // packed, like the old values
    reinterpret_cast<v4f*>(g.Y)[at] = y[0] + old;
  } else if (EPI == F32_STORE) {  // row-major
    const int n = u * 16 + quad * 4;
    float* dst = g.Y + (int64_t)r * g.N + n;
    if ((g.N & 3) == 0) {
      if (n < g.N) *reinterpret_cast<v4f*>(dst) = y[0];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (n + i < g.N) dst[i] = y[0][i];
    }
  } else if (EPI == F32_SILU) {  // packed: the down projection's input (features past F come out as 0)
    v4f h;
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = y[0][i] / (1.0f + expf(-y[0][i])) * y[PAIRED][i];
    reinterpret_cast<v4f*>(g.Y)[((int64_t)rb * n_units + u) * 64 + lane] = h;
  } else {  // F32_QKV: rotate queries and keys, queries stay in the row, keys and values go to cache slot P + node
    const int per = half / 16, hs = u / per, d0 = (u - hs * per) * 16 + quad * 4;
    const int b = g.m.blk_seq[rb], node = r - g.m.row0[b];
    const bool real = node < g.m.seq_n[b];
    v4f lo = y[0], hi = y[PAIRED];
    if (hs < g.H + g.Hkv) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 cs = g.tab[(int64_t)r * half + d0 + i];
        lo[i] = y[0][i] * cs.x - y[PAIRED][i] * cs.y;
        hi[i] = y[PAIRED][i] * cs.x + y[0][i] * cs.y;
      }
    }
    float* dst = nullptr;
    if (hs < g.H) {
      dst = g.Y + (int64_t)r * g.N + (int64_t)hs * g.hd;
    } else if (real) {
      const int kvh = hs < g.H + g.Hkv ? hs - g.H : hs - g.H - g.Hkv;
      dst = (hs < g.H + g.Hkv ? g.kc : g.vc) + (((int64_t)b * g.Hkv + kvh) * g.cap + g.m.seq_p[b] + node) * g.hd;
    }
    if (dst) {
      *reinterpret_cast<cache_v4f*>(dst + d0) = lo;
      *reinterpret_cast<cache_v4f*>(dst + d0 + half) = hi;
    }
  }
}

// Tiles per workgroup: the shape whose busiest CU is done first.  A workgroup takes `us` microseconds per 1024 of K of its CU
// (fitted to 16 - 448 rows, N = 256 - 16000, K = 256 - 3200; most launches within 10 %).  160 rows, us with 1 x 1 / 2 x 1 /
// 2 x 2 / 4 x 2 tiles: gate/up (N = 5632, K = 1024) - / 18.0 / 19.0 / 17.2, O (1024, 1024) 4.6 / 4.8 / 4.8 / 8.0, down
// (1024, 2816) 12.6 / 12.7 / 10.9 / 20, LM head (8192, 1024) 31 / 27.7 / 23.9 / 26.5; 448 rows, LM head 79 / 68.7 / 63.4 / 60.
void f32_gemm(const F32Gemm& g, hipStream_t s) {
  if (g.rows <= 0) return;
  const int nrb = g.rows / 16;
  const bool paired = g.kind == F32_SILU || g.kind == F32_QKV;
  const int units = g.kind == F32_SILU ? tiles16(g.N / 2) : g.kind == F32_QKV ? g.N / 32 : tiles16(g.N);
  auto groups = [&](int ft, int rt) {  // workgroups of ft x rt tiles
    const int uf = paired ? ft / 2 : ft;
    return (units + uf - 1) / uf * ((nrb + rt - 1) / rt);
  };
  static const struct {
    int ft, rt;
    double us;
  } shapes[] = {{1, 1, 1.55}, {2, 1, 2.45}, {2, 2, 4.45}, {4, 2, 8.3}};
  int FT = 2, RT = 1;
  double best = 1e300;
  for (const auto& sh : shapes) {
    if (paired && sh.ft == 1) continue;
    const double cost = sh.us * ((groups(sh.ft, sh.rt) + 255) / 256);
    if (cost < best) best = cost, FT = sh.ft, RT = sh.rt;
  }
#define DED_F32_GO(FT, RT, D, EPI) \
  hipLaunchKernelGGL((f32_mfma_gemm_kernel<FT, RT, D, EPI>), dim3(groups(FT, RT)), dim3(512), 0, s, g)
#define DED_F32_PAIRED(EPI)                    \
  if (FT == 4) DED_F32_GO(4, 2, 2, EPI);       \
  else if (RT == 2) DED_F32_GO(2, 2, 3, EPI);  \
  else DED_F32_GO(2, 1, 4, EPI)
#define DED_F32_PLAIN(EPI)                     \
  if (FT == 1) DED_F32_GO(1, 1, 4, EPI);       \
  else DED_F32_PAIRED(EPI)
  switch (g.kind) {
    case F32_STORE: DED_F32_PLAIN(F32_STORE); break;
    case F32_RESIDUAL: DED_F32_PLAIN(F32_RESIDUAL); break;
    case F32_SILU: DED_F32_PAIRED(F32_SILU); break;
    case F32_QKV: DED_F32_PAIRED(F32_QKV); break;
  }
#undef DED_F32_GO
#undef DED_F32_PAIRED
#undef DED_F32_PLAIN
}

// ------------------------------------------------------------------------------------------
// Rotate q (in place) and k, append k/v of real nodes to cache slot P + node (head dims below 32, whose rotary pairs do
// not fill two 16-feature tiles of the fused projection).
__global__ void f32_rope_kv_kernel(float* __restrict__ qkv, float* __restrict__ kc, float* __restrict__ vc,
                                   const float2* __restrict__ tab, const int32_t* __restrict__ seq_p,
                                   const int32_t* __restrict__ seq_n, const int32_t* __restrict__ row0,
                                   const int32_t* __restrict__ blk_seq, int H, int Hkv, int hd, int cap) {
  int r = blockIdx.x, hs = blockIdx.y;
  int b = blk_seq[r >> 4], node = r - row0[b];
  int half = hd / 2;
  int width = (H + 2 * Hkv) * hd;
  float* v = qkv + (int64_t)r * width + (int64_t)hs * hd;
  bool real = node < seq_n[b];
  int64_t slot = (int64_t)seq_p[b] + node;
  if (hs < H + Hkv) {
    float* dst = nullptr;
    if (hs >= H && real) dst = kc + (((int64_t)b * Hkv + (hs - H)) * cap + slot) * hd;
    for (int i = threadIdx.x; i < half; i += blockDim.x) {
      float2 cs = tab[(int64_t)r * half + i];
      float a = v[i], c = v[i + half];
      float ra = a * cs.x - c * cs.y;
      float rc = c * cs.x + a * cs.y;
      if (hs < H) {
        v[i] = ra;
        v[i + half] = rc;
      } else if (dst) {
        dst[i] = ra;
        dst[i + half] = rc;
      }
    }
  } else if (real) {
    float* dst = vc + (((int64_t)b * Hkv + (hs - H - Hkv)) * cap + slot) * hd;
    for (int i = threadIdx.x; i < hd; i += blockDim.x) dst[i] = v[i];
  }
}
void f32_rope_kv(float* qkv, float* kc, float* vc, const float2* tab, const StepMeta& m,
                 const ModelDims& md, hipStream_t s) {
  hipLaunchKernelGGL(f32_rope_kv_kernel, dim3(m.rows, md.H + 2 * md.Hkv), dim3(64), 0, s, qkv, kc, vc, tab,
                     m.seq_p, m.seq_n, m.row0, m.blk_seq, md.H, md.Hkv, md.hd, md.cap);
}

// ------------------------------------------------------------------------------------------
// Tree-masked attention for head dims below 16 (too short for a matrix instruction's tile), one workgroup per (row,
// query head).  Keys are taken in chunks of 1024:
// scores -> running max -> probabilities -> value accumulation (thread = (dim, key-part)).
// Needs hd <= 256 and 256 % hd == 0.
#define F32_ATT_CHUNK 1024
__global__ __launch_bounds__(256) void f32_tree_attention_kernel(
    float* __restrict__ o, const float* __restrict__ qkv, int q_stride, const float* __restrict__ kc,
    const float* __restrict__ vc, const uint64_t* __restrict__ mask, const int32_t* __restrict__ seq_p,
    const int32_t* __restrict__ seq_n, const int32_t* __restrict__ row0, const int32_t* __restrict__ blk_seq, int H,
    int Hkv, int hd, int cap) {
  __shared__ float sq[256];
  __shared__ float sp[F32_ATT_CHUNK];
  __shared__ float sred[4];
  __shared__ float sacc[256];
  int r = blockIdx.x, h = blockIdx.y;
  int b = blk_seq[r >> 4], node = r - row0[b];
  auto put = [&](int i, float v) {  // packed, the O projection's input
    const int k = h * hd + i;
    o[packed_unit(r, k, tiles16(H * hd)) * 4 + (k & 3)] = v;
  };
  int nb = seq_n[b];
  if (node >= nb) {
    for (int i = threadIdx.x; i < hd; i += 256) put(i, 0.f);
    return;
  }
  int P = seq_p[b];
  int T = P + nb;
  int g = (h * Hkv) / H;
  const float* K = kc + ((int64_t)b * Hkv + g) * cap * hd;
  const float* V = vc + ((int64_t)b * Hkv + g) * cap * hd;
  const uint64_t* mrow = mask + (int64_t)r * 4;
  for (int i = threadIdx.x; i < hd; i += 256) sq[i] = qkv[(int64_t)r * q_stride + (int64_t)h * hd + i];
  __syncthreads();
  float scale = 1.0f / sqrtf((float)hd);
  int parts = 256 / hd;
  int dim = threadIdx.x % hd, part = threadIdx.x / hd;
  float m_run = -INFINITY, l_run = 0.f, acc = 0.f;
  for (int c0 = 0; c0 < T; c0 += F32_ATT_CHUNK) {
    int cn = min(F32_ATT_CHUNK, T - c0);
    float lmax = -INFINITY;
    for (int j = threadIdx.x; j < cn; j += 256) {
      int key = c0 + j;
      bool vis = key < P;
      if (!vis) {
        int t = key - P;
        vis = (mrow[t >> 6] >> (t & 63)) & 1ull;
      }
      float sc = -INFINITY;
      if (vis) {
        const float* kr = K + (int64_t)key * hd;
        float d = 0.f;
        for (int i = 0; i < hd; ++i) d += sq[i] * kr[i];
        sc = d * scale;
      }
      sp[j] = sc;
      lmax = fmaxf(lmax, sc);
    }
    float cmax = block_max_256(lmax, sred);
    float m_new = fmaxf(m_run, cmax);
    float alpha = (m_run == -INFINITY) ? 0.f : expf(m_run - m_new);
    float lsum = 0.f;
    if (m_new != -INFINITY) {
      for (int j = threadIdx.x; j < cn; j += 256) {
        float sc = sp[j];
        float p = (sc == -INFINITY) ? 0.f : expf(sc - m_new);
        sp[j] = p;
        lsum += p;
      }
    } else {
      for (int j = threadIdx.x; j < cn; j += 256) sp[j] = 0.f;
    }
    float csum = block_sum_256(lsum, sred);  // also orders the sp[] writes before the reads below
    l_run = l_run * alpha + csum;
    acc *= alpha;
    for (int j = part; j < cn; j += parts) acc += sp[j] * V[(int64_t)(c0 + j) * hd + dim];
    m_run = m_new;
    __syncthreads();
  }
  sacc[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x < hd) {
    float t = 0.f;
    for (int p = 0; p < parts; ++p) t += sacc[p * hd + threadIdx.x];
    put(threadIdx.x, t / l_run);
  }
}
// Partial results of the kernel below travel between workgroups of one launch, which may sit on different XCDs: device-scope
// relaxed accesses that go through to the point of coherence, stores waited for before the ticket is taken, loads behind the
// ticket's return value (-DDED_SPLITK_FENCES: fences instead, as for the 16-bit path's split sums).
__device__ inline void part_store(float* p, float a, float b) {
  const unsigned long long v = (unsigned long long)__float_as_uint(b) << 32 | __float_as_uint(a);
#ifdef DED_SPLITK_FENCES
  *reinterpret_cast<unsigned long long*>(p) = v;
#else
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#endif
}
__device__ inline float2 part_load(const float* p) {
#ifdef DED_SPLITK_FENCES
  const unsigned long long v = *reinterpret_cast<const unsigned long long*>(p);
#else
  const unsigned long long v = __hip_atomic_load(reinterpret_cast<unsigned long long*>(const_cast<float*>(p)), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
#endif
  return make_float2(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
}
// whether this workgroup is the last of `splits` whose partial results lie in memory
__device__ inline bool last_of(int splits, int* ticket, int* s_flag) {
#ifdef DED_SPLITK_FENCES
  __atomic_thread_fence(__ATOMIC_RELEASE);
#else
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
  __syncthreads();
  if (threadIdx.x == 0) {
    const int prev = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (prev == splits - 1) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_flag = prev == splits - 1;
  }
  __syncthreads();
#ifdef DED_SPLITK_FENCES
  if (*s_flag) __atomic_thread_fence(__ATOMIC_ACQUIRE);
#endif
  return *s_flag != 0;
}
// Matrix-core form for head dims of 16 and more.  One workgroup per (16-row block, query head); its NW wavefronts take
// 16-key blocks in turn, each with an online soft-max of its own, and merge through LDS at the end.  S^T = K . Q^T leaves
// the scores of four consecutive keys (4 quad + i) of one row in a lane, which is the operand layout of the second
// product O^T = V^T . P^T when its i-th instruction takes keys 4 quad + i: no cross-lane traffic but the row maximum.
// The kernel above walks one row per workgroup, every lane along a key of its own (64 separate rows per load), and
// fetches K and V once per row; this one fetches them once per 16 rows.
// A workgroup takes one of up to F32_ATTN_SPLITS ranges of about 128 keys, one 16-key block per wavefront; the last one to finish
// adds the ranges in their order.  Bound by latencies (6 us from start to end for a single range of 24 keys: operands 2.8,
// products and soft-max 2.4, meeting of the wavefronts and hand-over) and, where a CU runs several ranges after one another, by
// the fp32 matrix instructions (2048 cycles per block for a head dim of 128).  Hence the list of items in place of a grid with
// empty workgroups, which the dispatcher spread so unevenly that some CUs ran two, and registers for two workgroups per CU:
// the values are requested behind the keys' products, the queries stay in LDS.
// us, per layer, 8 heads x 128, four trees of 160 rows: on prefixes of 512, 131, 300 and 17 keys unsplit 21, so 13.3 (12.4 with one
// workgroup per CU), on four prefixes of 512 keys 21 and 18.3 (21).
// A lane's feature m of value tiles 4 c .. 4 c + 3 stands for dims 64 c + 4 m .. + 3, so that it loads 16 bytes of a value row (one
// float per load instruction otherwise, 32 for a head dim of 128).
template <int HD>
__global__ __launch_bounds__(HD == 256 ? 256 : 512, HD == 256 ? 1 : 4) void f32_mfma_attention_kernel(
    float* __restrict__ o, const float* __restrict__ qkv, int q_stride, const float* __restrict__ kc,
    const float* __restrict__ vc, const uint64_t* __restrict__ mask, const int32_t* __restrict__ seq_p,
    const int32_t* __restrict__ seq_n, const int32_t* __restrict__ blk_seq, const int32_t* __restrict__ items, int H, int Hkv,
    int cap, int most,
    float* part_o, float* part_ml, int* tickets) {
  constexpr int NW = HD == 256 ? 4 : 8, DT = HD / 16, VEC = DT < 4 ? DT : 4;
  typedef float vec __attribute__((ext_vector_type(VEC), aligned(4)));
  __shared__ float4 s_o[NW][DT][64];
  __shared__ float2 s_ml[NW][16];
  __shared__ float4 s_q[DT][64];
  __shared__ int s_last;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m16 = lane & 15, quad = lane >> 4;
  const int h = blockIdx.x, item = items[blockIdx.y], rb = item / F32_ATTN_SPLITS, range = item % F32_ATTN_SPLITS;
  const int r = rb * 16 + m16, b = blk_seq[rb];
  const int P = seq_p[b], T = P + seq_n[b], kvh = h / (H / Hkv);
  const int splits = f32_attention_splits(T, most), blocks = (T + 15) / 16;
  const int k_begin = range * blocks / splits * 16, k_end = (range + 1) * blocks / splits * 16;
  const float* K = kc + ((int64_t)b * Hkv + kvh) * cap * HD;
  const float* V = vc + ((int64_t)b * Hkv + kvh) * cap * HD;
  const float* q = qkv + (int64_t)r * q_stride + (int64_t)h * HD;
  const uint64_t* mrow = mask + (int64_t)r * 4;
  const uint64_t w0 = mrow[0], w1 = mrow[1], w2 = mrow[2], w3 = mrow[3];
  const float scale = 1.0f / sqrtf((float)HD);
  // Whether a key counts is decided by the mask alone, never by its score's value: every finite score takes part, and a
  // NaN one has to reach the output (the maximum passes over it, its exponential does not).
  float m_run = -INFINITY, l_run = 0.f;  // l_run: this lane's keys only
  auto exponent_from = [](float v, float m) {
#pragma clang fp contract(off)  // (a product fused into the difference would leave the maximum's own rounding error there)
    return v - (m == -INFINITY ? 0.f : m);
  };
  v4f acc[DT];
#pragma unroll
  for (int c = 0; c < DT; ++c) acc[c] = v4f{0.f, 0.f, 0.f, 0.f};
  v4f kf[DT];
  auto load_keys = [&](int k0) {
    const float* kr = K + (int64_t)min(k0 + m16, T - 1) * HD + quad * 4;
#pragma unroll
    for (int c = 0; c < DT; ++c) kf[c] = *reinterpret_cast<const cache_v4f*>(kr + c * 16);
  };
  load_keys(k_begin + wave * 16);
  // the queries, the same for all wavefronts, stay in LDS: held by each they left registers for one workgroup per CU
  for (int c = wave; c < DT; c += NW) s_q[c][lane] = *reinterpret_cast<const float4*>(q + c * 16 + quad * 4);
  __syncthreads();
  for (int k0 = k_begin + wave * 16; k0 < k_end; k0 += NW * 16) {
    v4f sa = v4f{0.f, 0.f, 0.f, 0.f}, sb = sa;
#pragma unroll
    for (int c = 0; c < DT; ++c) {
      const float4 qc = s_q[c][lane];
      sa = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][0], qc.x, sa, 0, 0, 0);
      sb = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][1], qc.y, sb, 0, 0, 0);
      sa = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][2], qc.z, sa, 0, 0, 0);
      sb = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][3], qc.w, sb, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    float vf[4][DT];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float* vr = V + (int64_t)min(k0 + quad * 4 + j, T - 1) * HD + m16 * VEC;
#pragma unroll
      for (int c = 0; c < DT; c += VEC) {
        const vec v = *reinterpret_cast<const vec*>(vr + c * 16);
#pragma unroll
        for (int e = 0; e < VEC; ++e) vf[j][c + e] = v[e];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    float p[4], mx = -INFINITY;
    bool vis[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int key = k0 + quad * 4 + i, t = key - P;
      const uint64_t word = t < 64 ? w0 : t < 128 ? w1 : t < 192 ? w2 : w3;
      vis[i] = key < P || (key < T && ((word >> (t & 63)) & 1ull));
      p[i] = (sa[i] + sb[i]) * scale;
      mx = vis[i] ? fmaxf(mx, p[i]) : mx;
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx), alpha = expf(exponent_from(m_run, m_new));
    m_run = m_new;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = vis[i] ? expf(exponent_from(p[i], m_new)) : 0.f;
      sum += p[i];
    }
    l_run = l_run * alpha + sum;
#pragma unroll
    for (int c = 0; c < DT; ++c) {
      acc[c] *= alpha;
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[j][c], p[j], acc[c], 0, 0, 0);
    }
    load_keys(k0 + NW * 16);  // (past the end the last key again)
  }
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  if (quad == 0) s_ml[wave][m16] = make_float2(m_run, l_run);
#pragma unroll
  for (int c = 0; c < DT; ++c) s_o[wave][c][lane] = make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
  __syncthreads();
  float M = -INFINITY, L = 0.f, f[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, s_ml[w][m16].x);
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float2 ml = s_ml[w][m16];
    f[w] = expf(exponent_from(ml.x, M));
    L += ml.y * f[w];
  }
  float inv = 1.0f / L;
  const int64_t group = (int64_t)rb * H + h, part = group * most + range;
  for (int c = wave; c < DT; c += NW) {
    v4f v = v4f{0.f, 0.f, 0.f, 0.f};
    // dims c * 16 + quad * 4 + i, from where the wavefronts left them
#pragma unroll
    for (int w = 0; w < NW; ++w) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int dim = c * 16 + quad * 4 + i, m = dim % (16 * VEC) / VEC, t = dim / (16 * VEC) * VEC + dim % VEC;
        v[i] += reinterpret_cast<const float*>(&s_o[w][t][m / 4 * 16 + m16])[m % 4] * f[w];
      }
    }
    float4* out = reinterpret_cast<float4*>(o) + ((int64_t)rb * (H * DT) + h * DT + c) * 64 + lane;  // packed, the O projection's input
    if (splits == 1) {
      *out = make_float4(v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv);
    } else {
      float* p = part_o + ((part * DT + c) * 64 + lane) * 4;
      part_store(p, v[0], v[1]);
      part_store(p + 2, v[2], v[3]);
    }
  }
  if (splits == 1) return;
  if (wave == 0 && quad == 0) part_store(part_ml + (part * 16 + m16) * 2, M, L);
  if (!last_of(splits, tickets + group, &s_last)) return;
  float g[F32_ATTN_SPLITS];
  M = -INFINITY, L = 0.f;
  float2 ml[F32_ATTN_SPLITS];
#pragma unroll
  for (int z = 0; z < F32_ATTN_SPLITS; ++z)  // (past the last range it is read again, with no weight)
    ml[z] = part_load(part_ml + ((group * most + min(z, splits - 1)) * 16 + m16) * 2);
#pragma unroll
  for (int z = 0; z < F32_ATTN_SPLITS; ++z) M = fmaxf(M, ml[z].x);
#pragma unroll
  for (int z = 0; z < F32_ATTN_SPLITS; ++z) {
    g[z] = expf(exponent_from(ml[z].x, M));
    if (z < splits) L += ml[z].y * g[z];
  }
  inv = 1.0f / L;
  for (int c = wave; c < DT; c += NW) {
    float2 lo[F32_ATTN_SPLITS], hi[F32_ATTN_SPLITS];
#pragma unroll
    for (int z = 0; z < F32_ATTN_SPLITS; ++z) {
      const float* p = part_o + (((group * most + min(z, splits - 1)) * DT + c) * 64 + lane) * 4;
      lo[z] = part_load(p), hi[z] = part_load(p + 2);
    }
    v4f v = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int z = 0; z < F32_ATTN_SPLITS; ++z)
      if (z < splits) v += v4f{lo[z].x, lo[z].y, hi[z].x, hi[z].y} * g[z];
    reinterpret_cast<float4*>(o)[((int64_t)rb * (H * DT) + h * DT + c) * 64 + lane] =
        make_float4(v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv);
  }
}

void f32_tree_attention(float* o, const float* qkv, int q_stride, const float* kc, const float* vc,
                        const StepMeta& m, const ModelDims& md, int n_items, int most, float* part_o, float* part_ml, int* tickets,
                        hipStream_t s) {
#define DED_F32_ATTN(HD)                                                                                          \
  hipLaunchKernelGGL((f32_mfma_attention_kernel<HD>), dim3(md.H, n_items), dim3(HD == 256 ? 256 : 512), 0, s, o, \
                     qkv, q_stride, kc, vc, m.mask, m.seq_p, m.seq_n, m.blk_seq, m.attn_items, md.H, md.Hkv, md.cap, most, part_o, part_ml, \
                     tickets)
  switch (md.hd) {
    case 16: DED_F32_ATTN(16); return;
    case 32: DED_F32_ATTN(32); return;
    case 64: DED_F32_ATTN(64); return;
    case 128: DED_F32_ATTN(128); return;
    case 256: DED_F32_ATTN(256); return;
  }
#undef DED_F32_ATTN
  hipLaunchKernelGGL(f32_tree_attention_kernel, dim3(m.rows, md.H), dim3(256), 0, s, o, qkv, q_stride, kc, vc,
                     m.mask, m.seq_p, m.seq_n, m.row0, m.blk_seq, md.H, md.Hkv, md.hd, md.cap);
}

// ------------------------------------------------------------------------------------------
// Compaction: slot P + path[j] -> slot P + j for j = 0..len-1.  path is increasing with path[j] >= j,
// so each thread walks j upwards and only ever overwrites slots it has already consumed.  Every workgroup does the approval walk
// of its sequence itself; the first of the sequence reports it.
__global__ __launch_bounds__(256) void f32_kv_compact_kernel(float* const* __restrict__ kc, float* const* __restrict__ vc,
                                                             ApprovalWalk w, const int32_t* __restrict__ seq_p, int Hkv,
                                                             int hd, int cap) {
  __shared__ WalkShared sh;
  int layer = blockIdx.x, bh = blockIdx.y;
  int b = bh / Hkv;
  int P = seq_p[b];
  const int len = approval_walk(w, b, sh);
  if (layer == 0 && bh == b * Hkv) report_walk(w, b, sh, len);
  const int32_t* pth = sh.path;
  float* K = kc[layer] + (int64_t)bh * cap * hd;
  float* V = vc[layer] + (int64_t)bh * cap * hd;
  for (int i = threadIdx.x; i < hd; i += blockDim.x) {
    for (int j = 0; j < len; ++j) {
      int src = pth[j];
      if (src != j) {
        K[(int64_t)(P + j) * hd + i] = K[(int64_t)(P + src) * hd + i];
        V[(int64_t)(P + j) * hd + i] = V[(int64_t)(P + src) * hd + i];
      }
    }
  }
}
void f32_kv_compact(float* const* kc, float* const* vc, const ApprovalWalk& w, const StepMeta& m, const ModelDims& md, hipStream_t s) {
  hipLaunchKernelGGL(f32_kv_compact_kernel, dim3(md.n_layers, m.batch * md.Hkv), dim3(256), 0, s, kc, vc, w, m.seq_p, md.Hkv,
                     md.hd, md.cap);
}

// ------------------------------------------------------------------------------------------
__global__ void f32_kv_copy_kernel(float* __restrict__ cache, float* __restrict__ plain, int to_cache,
                                   int seq, int first, int n, int Hkv, int hd, int cap) {
  int j = blockIdx.x, g = blockIdx.y;
  float* c = cache + (((int64_t)seq * Hkv + g) * cap + first + j) * hd;
  float* p = plain + ((int64_t)g * n + j) * hd;
  for (int i = threadIdx.x; i < hd; i += blockDim.x) {
    if (to_cache) c[i] = p[i];
    else p[i] = c[i];
  }
}
void f32_kv_copy(float* cache, float* plain, bool to_cache, int seq, int first, int n,
                 const ModelDims& md, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(f32_kv_copy_kernel, dim3(n, md.Hkv), dim3(64), 0, s, cache, plain, to_cache ? 1 : 0, seq,
                     first, n, md.Hkv, md.hd, md.cap);
}

// zero the slots [first, first + n) of one sequence (keys and values)
__global__ void f32_kv_clear_kernel(float* __restrict__ kc, float* __restrict__ vc, int seq, int first, int Hkv,
                                    int hd, int cap) {
  int j = blockIdx.x, g = blockIdx.y;
  int64_t at = (((int64_t)seq * Hkv + g) * cap + first + j) * hd;
  for (int i = threadIdx.x; i < hd; i += blockDim.x) {
    kc[at + i] = 0.f;
    vc[at + i] = 0.f;
  }
}
void f32_kv_clear(float* kc, float* vc, int seq, int first, int n, const ModelDims& md, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(f32_kv_clear_kernel, dim3(n, md.Hkv), dim3(64), 0, s, kc, vc, seq, first, md.Hkv, md.hd, md.cap);
}

// k_tree / v_tree: [B][Hkv][max_nodes][hd] -> cache slot P + node
__global__ void f32_scatter_tree_kv_kernel(float* __restrict__ kc, float* __restrict__ vc,
                                           const float* __restrict__ kt, const float* __restrict__ vt,
                                           const int32_t* __restrict__ seq_p, const int32_t* __restrict__ seq_n,
                                           int Hkv, int hd, int cap, int max_nodes) {
  int node = blockIdx.x, bh = blockIdx.y;
  int b = bh / Hkv;
  if (node >= seq_n[b]) return;
  int64_t src = ((int64_t)bh * max_nodes + node) * hd;
  int64_t dst = ((int64_t)bh * cap + seq_p[b] + node) * hd;
  for (int i = threadIdx.x; i < hd; i += blockDim.x) {
    kc[dst + i] = kt[src + i];
    vc[dst + i] = vt[src + i];
  }
}
void f32_scatter_tree_kv(float* kc, float* vc, const float* k_tree, const float* v_tree,
                         const StepMeta& m, const ModelDims& md, int max_nodes, hipStream_t s) {
  hipLaunchKernelGGL(f32_scatter_tree_kv_kernel, dim3(max_nodes, m.batch * md.Hkv), dim3(64), 0, s, kc, vc,
                     k_tree, v_tree, m.seq_p, m.seq_n, md.Hkv, md.hd, md.cap, max_nodes);
}

// rows of real nodes from the caller's [B][max_nodes][width] to the padded [R][width] queries, and of the packed attention
// output to the caller
__global__ void f32_gather_rows_kernel(float* __restrict__ dst, const float* __restrict__ src,
                                       const int32_t* __restrict__ seq_n, const int32_t* __restrict__ row0,
                                       const int32_t* __restrict__ blk_seq, int max_nodes, int width, int to_padded) {
  int r = blockIdx.x;
  int b = blk_seq[r >> 4], node = r - row0[b];
  bool real = node < seq_n[b];
  int64_t pad = (int64_t)r * width, ext = ((int64_t)b * max_nodes + node) * width;
  for (int i = threadIdx.x; i < width; i += blockDim.x) {
    if (to_padded) dst[pad + i] = real ? src[ext + i] : 0.f;
    else if (real) dst[ext + i] = src[packed_unit(r, i, tiles16(width)) * 4 + (i & 3)];
  }
}
void f32_gather_rows(float* dst, const float* src, const StepMeta& m, int max_nodes, int width,
                     bool to_padded, hipStream_t s) {
  hipLaunchKernelGGL(f32_gather_rows_kernel, dim3(m.rows), dim3(256), 0, s, dst, src, m.seq_n, m.row0,
                     m.blk_seq, max_nodes, width, to_padded ? 1 : 0);
}

}  // namespace ded
