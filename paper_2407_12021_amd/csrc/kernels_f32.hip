// fp32 storage path: plain row-major buffers, cache [B][Hkv][cap][hd].  Contractions run on the fp32 matrix
// instructions (v_mfma_f32_16x16x4_f32: fp32 operands and accumulators, nothing is rounded to a shorter type); every
// reduction has a fixed order.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "ded_kernels.h"

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
__global__ void f32_embed_kernel(float* __restrict__ x, const float* __restrict__ emb,
                                 const int32_t* __restrict__ token, int d) {
  int r = blockIdx.x;
  const float* src = emb + (int64_t)token[r] * d;
  for (int i = threadIdx.x; i < d; i += blockDim.x) x[(int64_t)r * d + i] = src[i];
}
void f32_embed(float* x, const float* emb, const StepMeta& m, int d, hipStream_t s) {
  hipLaunchKernelGGL(f32_embed_kernel, dim3(m.rows), dim3(256), 0, s, x, emb, m.token, d);
}

// ------------------------------------------------------------------------------------------
// Projections with fused neighbours:  Y[r][n] = sum_k X[r][k] W[n][k], X optionally RMS-normalised on the way in, Y
// going into what the decoder does with it (F32_* in ded_kernels.h).
//
// A workgroup owns FT x RT tiles of 16 features x 16 rows; its 8 wavefronts split k in chunks of 32, taken in turn, and
// meet in LDS.  Operands go straight from memory to registers: a lane fetches 16 bytes of its feature (row), so four
// lanes cover 64 contiguous bytes of it, and component j of those registers is the operand of the j-th matrix
// instruction (both operands permute k alike).  Splitting k over the wavefronts is what fills the chip at the sizes of
// this path (a d = 256 model has 16 feature tiles per projection) and keeps the chain of dependent loads short.
// RMSNorm is applied as (x * gain) . W * (1 / rms): the wavefronts form sum(x^2) from the operands they load anyway.
// Bound by latency and L2 reads at these sizes, not by the matrix instructions.  Measured at 160 rows, gate/up of
// N = 5632, K = 1024: 34.5 us (about 480 us for one wavefront per feature walking the rows by vector arithmetic).
template <int FT, int RT, int EPI, bool VEC>
__global__ __launch_bounds__(512) void f32_mfma_gemm_kernel(F32Gemm g) {
  constexpr int NW = 8;
  constexpr bool NORM = EPI != F32_RESIDUAL;
  __shared__ float4 red[NW][FT * RT][64];
  __shared__ float s_ss[NORM ? NW : 1][RT][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m16 = lane & 15, quad = lane >> 4;
  const int bx = blockIdx.x, rb0 = blockIdx.y * RT, nrb = g.rows / 16, K = g.K;
  const int half = g.hd / 2;
  int n0[FT], n_end[FT];  // first feature of each tile and the end of its matrix part
#pragma unroll
  for (int t = 0; t < FT; ++t) {
    if (EPI == F32_SILU) {
      n0[t] = t * (g.N / 2) + bx * 16;
      n_end[t] = (t + 1) * (g.N / 2);
    } else if (EPI == F32_QKV) {
      const int per = half / 16, hs = bx / per, p = bx - hs * per;
      n0[t] = hs * g.hd + p * 16 + t * half;
      n_end[t] = g.N;
    } else {
      n0[t] = (bx * FT + t) * 16;
      n_end[t] = g.N;
    }
  }
  const float *wp[FT], *xp[RT];
#pragma unroll
  for (int t = 0; t < FT; ++t) wp[t] = g.W + (int64_t)min(n0[t] + m16, n_end[t] - 1) * K;
#pragma unroll
  for (int t = 0; t < RT; ++t) xp[t] = g.X + (int64_t)(min(rb0 + t, nrb - 1) * 16 + m16) * K;
  // four consecutive k of one row (VEC: K % 4 == 0, one 16-byte load); TAIL: zero past the row's end
  auto load4 = [&](const float* q, int k, auto tail) {
    constexpr bool TAIL = decltype(tail)::value;
    v4f v = v4f{0.f, 0.f, 0.f, 0.f};
    if constexpr (VEC) {
      if (!TAIL || k < K) v = *reinterpret_cast<const v4f*>(q + k);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (!TAIL || k + i < K) v[i] = q[k + i];
    }
    return v;
  };
  v4f acc[FT][RT];
  float ss[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    ss[r] = 0.f;
#pragma unroll
    for (int t = 0; t < FT; ++t) acc[t][r] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  struct Chunk {
    v4f w[FT][2], x[RT][2], gain[2];
  };
  auto load = [&](int c, auto tail) {
    Chunk q;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int k = c * 32 + j * 16 + quad * 4;
#pragma unroll
      for (int t = 0; t < FT; ++t) q.w[t][j] = load4(wp[t], k, tail);
#pragma unroll
      for (int t = 0; t < RT; ++t) q.x[t][j] = load4(xp[t], k, tail);
      if (NORM) q.gain[j] = load4(g.gain, k, tail);
    }
    return q;
  };
  auto compute = [&](Chunk& q) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (NORM) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          const v4f x = q.x[r][j];
          ss[r] += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
          q.x[r][j] = x * q.gain[j];
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < FT; ++t)
#pragma unroll
          for (int r = 0; r < RT; ++r)
            acc[t][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(q.w[t][j][i], q.x[r][j][i], acc[t][r], 0, 0, 0);
    }
  };
  // whole chunks: two in flight per wavefront (fetches past the share re-read its last chunk); what K leaves over goes
  // to the wavefront whose turn it would be
  const int n_full = K / 32, last = n_full - 1 - (n_full - 1 - wave) % NW;
  if (wave < n_full) {
    Chunk a = load(wave, std::false_type{});
    for (int c = wave;;) {
      Chunk b = load(min(c + NW, last), std::false_type{});
      compute(a);
      if ((c += NW) > last) break;
      a = load(min(c + NW, last), std::false_type{});
      compute(b);
      if ((c += NW) > last) break;
    }
  }
  if (K % 32 && wave == n_full % NW) {
    Chunk t = load(n_full, std::true_type{});
    compute(t);
  }
  // the wavefronts' k shares meet in LDS, added in wavefront order
#pragma unroll
  for (int t = 0; t < FT; ++t)
#pragma unroll
    for (int r = 0; r < RT; ++r) red[wave][t * RT + r][lane] = make_float4(acc[t][r][0], acc[t][r][1], acc[t][r][2], acc[t][r][3]);
  if (NORM) {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      float v = ss[r];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (quad == 0) s_ss[wave][r][m16] = v;
    }
  }
  __syncthreads();
  if (wave >= RT || rb0 + wave >= nrb) return;
  const int rt = wave, r = (rb0 + rt) * 16 + m16;
  float scale = 1.f;
  if (NORM) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) v += s_ss[w][rt][m16];
    scale = 1.0f / sqrtf(v / (float)K + g.eps);
  }
  float y[FT][4];
#pragma unroll
  for (int t = 0; t < FT; ++t) {
    v4f v = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float4 q = red[w][t * RT + rt][lane];
      v += v4f{q.x, q.y, q.z, q.w};
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) y[t][i] = NORM ? v[i] * scale : v[i];
  }
  // four consecutive outputs; 16-byte accesses where the row stride allows them
  auto put = [&](float* dst, const float (&v)[4], int n, int limit, bool aligned) {
    if (aligned && n + 3 < limit) {
      *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (n + i < limit) dst[i] = v[i];
    }
  };
  if (EPI == F32_STORE || EPI == F32_RESIDUAL) {
    const bool aligned = (g.N & 3) == 0;
#pragma unroll
    for (int t = 0; t < FT; ++t) {
      const int n = n0[t] + quad * 4;
      float* dst = g.Y + (int64_t)r * g.N + n;
      if (EPI == F32_RESIDUAL) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < g.N) y[t][i] += dst[i];
      }
      put(dst, y[t], n, g.N, aligned);
    }
  } else if (EPI == F32_SILU) {
    const int F = g.N / 2, f = bx * 16 + quad * 4;
    float h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = y[0][i] / (1.0f + expf(-y[0][i])) * y[FT - 1][i];
    put(g.Y + (int64_t)r * F + f, h, f, F, (F & 3) == 0);
  } else {  // F32_QKV: rotate queries and keys, queries stay in the row, keys and values go to cache slot P + node
    const int per = half / 16, hs = bx / per, d0 = (bx - hs * per) * 16 + quad * 4;
    const int b = g.m.blk_seq[r >> 4], node = r - g.m.row0[b];
    const bool real = node < g.m.seq_n[b];
    float lo[4], hi[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) lo[i] = y[0][i], hi[i] = y[FT - 1][i];
    if (hs < g.H + g.Hkv) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 cs = g.tab[(int64_t)r * half + d0 + i];
        lo[i] = y[0][i] * cs.x - y[FT - 1][i] * cs.y;
        hi[i] = y[FT - 1][i] * cs.x + y[0][i] * cs.y;
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
      *reinterpret_cast<cache_v4f*>(dst + d0) = cache_v4f{lo[0], lo[1], lo[2], lo[3]};
      *reinterpret_cast<cache_v4f*>(dst + d0 + half) = cache_v4f{hi[0], hi[1], hi[2], hi[3]};
    }
  }
}

// Tiles per workgroup by a cost fitted to a sweep (16 - 512 rows, the six shapes of the models above and the tiny one):
// a workgroup alone on its CU takes 3 us + K / 1024 * (1.1 us per operand tile it fetches + 0.85 us per tile product),
// and w workgroups per CU (counted in halves: the larger tiles run two at a time) take max(1, 0.95 w) times that.  160 rows: QKV (N = 3072, K = 1024) 34.6 us with 1 x 1 tiles,
// 18.7 with 2 x 2, 15.5 with 4 x 2; O (1024, 1024) 13.7 / 10.3 / 16.8; 512 rows, gate/up (5632, 1024): 88 us with 2 x 2,
// 74 with 2 x 4.  16 rows, d = 256: 3.7 us with 1 x 1, 5.1 with 2 x 2.
void f32_gemm(const F32Gemm& g, hipStream_t s) {
  if (g.rows <= 0) return;
  const int nrb = g.rows / 16;
  const bool vec = g.K % 4 == 0, paired = g.kind == F32_SILU || g.kind == F32_QKV;
  auto units = [&](int ft) {
    return g.kind == F32_SILU ? (g.N / 2 + 15) / 16 : g.kind == F32_QKV ? g.N / 32 : (g.N + 16 * ft - 1) / (16 * ft);
  };
  int FT = 2, RT = 2;
  if (vec) {
    static const int shapes[][2] = {{1, 1}, {2, 1}, {2, 2}, {2, 4}, {4, 2}};
    double best = 1e300;
    for (const auto& sh : shapes) {
      if (paired ? sh[0] != 2 : sh[0] == 2 && sh[1] == 1) continue;
      const double one = 3.0 + g.K / 1024.0 * (1.1 * (sh[0] + sh[1]) + 0.85 * sh[0] * sh[1]);
      const double per_cu = std::ceil(units(sh[0]) * ((nrb + sh[1] - 1) / sh[1]) / 128.0) / 2;
      const double cost = one * std::max(1.0, 0.95 * per_cu);
      if (cost < best) best = cost, FT = sh[0], RT = sh[1];
    }
  }
#define DED_F32_GO(FT, RT, EPI, VEC) \
  hipLaunchKernelGGL((f32_mfma_gemm_kernel<FT, RT, EPI, VEC>), dim3(units(FT), (nrb + RT - 1) / RT), dim3(512), 0, s, g)
#define DED_F32_PAIRED(EPI)                        \
  if (!vec) DED_F32_GO(2, 2, EPI, false);          \
  else if (RT == 1) DED_F32_GO(2, 1, EPI, true);   \
  else if (RT == 2) DED_F32_GO(2, 2, EPI, true);   \
  else DED_F32_GO(2, 4, EPI, true)
#define DED_F32_PLAIN(EPI)                         \
  if (!vec) DED_F32_GO(2, 2, EPI, false);          \
  else if (FT == 1) DED_F32_GO(1, 1, EPI, true);   \
  else if (FT == 4) DED_F32_GO(4, 2, EPI, true);   \
  else if (RT == 2) DED_F32_GO(2, 2, EPI, true);   \
  else DED_F32_GO(2, 4, EPI, true)
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
  float* out = o + ((int64_t)r * H + h) * hd;
  int nb = seq_n[b];
  if (node >= nb) {
    for (int i = threadIdx.x; i < hd; i += 256) out[i] = 0.f;
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
    out[threadIdx.x] = t / l_run;
  }
}
// Matrix-core form for head dims of 16 and more.  One workgroup per (16-row block, query head); its NW wavefronts take
// 16-key blocks in turn, each with an online soft-max of its own, and merge through LDS at the end.  S^T = K . Q^T leaves
// the scores of four consecutive keys (4 quad + i) of one row in a lane, which is the operand layout of the second
// product O^T = V^T . P^T when its i-th instruction takes keys 4 quad + i: no cross-lane traffic but the row maximum.
// The kernel above walks one row per workgroup, every lane along a key of its own (64 separate rows per load), and
// fetches K and V once per row; this one fetches them once per 16 rows.  Measured: four trees on prefixes of up to 512
// keys, 8 heads x 128, per layer 261 us before, 22 us now.
template <int HD>
__global__ __launch_bounds__(HD == 256 ? 256 : 512) void f32_mfma_attention_kernel(
    float* __restrict__ o, const float* __restrict__ qkv, int q_stride, const float* __restrict__ kc,
    const float* __restrict__ vc, const uint64_t* __restrict__ mask, const int32_t* __restrict__ seq_p,
    const int32_t* __restrict__ seq_n, const int32_t* __restrict__ row0, const int32_t* __restrict__ blk_seq, int H,
    int Hkv, int cap) {
  constexpr int NW = HD == 256 ? 4 : 8, DT = HD / 16;
  __shared__ float4 s_o[NW][DT][64];
  __shared__ float2 s_ml[NW][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m16 = lane & 15, quad = lane >> 4;
  const int h = blockIdx.y, r = blockIdx.x * 16 + m16, b = blk_seq[blockIdx.x];
  const int P = seq_p[b], T = P + seq_n[b], kvh = h / (H / Hkv);
  const float* K = kc + ((int64_t)b * Hkv + kvh) * cap * HD;
  const float* V = vc + ((int64_t)b * Hkv + kvh) * cap * HD;
  const float* q = qkv + (int64_t)r * q_stride + (int64_t)h * HD;
  v4f qf[DT];
#pragma unroll
  for (int c = 0; c < DT; ++c) qf[c] = *reinterpret_cast<const v4f*>(q + c * 16 + quad * 4);
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
  for (int k0 = wave * 16; k0 < T; k0 += NW * 16) {
    const float* kr = K + (int64_t)min(k0 + m16, T - 1) * HD + quad * 4;
    v4f kf[DT];
#pragma unroll
    for (int c = 0; c < DT; ++c) kf[c] = *reinterpret_cast<const cache_v4f*>(kr + c * 16);
    float vf[DT][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float* vr = V + (int64_t)min(k0 + quad * 4 + j, T - 1) * HD + m16;
#pragma unroll
      for (int c = 0; c < DT; ++c) vf[c][j] = vr[c * 16];
    }
    v4f sa = v4f{0.f, 0.f, 0.f, 0.f}, sb = sa;
#pragma unroll
    for (int c = 0; c < DT; ++c)
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        sa = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][j], qf[c][j], sa, 0, 0, 0);
        sb = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][j + 1], qf[c][j + 1], sb, 0, 0, 0);
      }
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
      for (int j = 0; j < 4; ++j) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][j], p[j], acc[c], 0, 0, 0);
    }
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
  const float inv = 1.0f / L;
  for (int c = wave; c < DT; c += NW) {
    v4f v = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float4 t = s_o[w][c][lane];
      v += v4f{t.x, t.y, t.z, t.w} * f[w];
    }
    *reinterpret_cast<float4*>(o + ((int64_t)r * H + h) * HD + c * 16 + quad * 4) =
        make_float4(v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv);
  }
}

void f32_tree_attention(float* o, const float* qkv, int q_stride, const float* kc, const float* vc,
                        const StepMeta& m, const ModelDims& md, hipStream_t s) {
#define DED_F32_ATTN(HD)                                                                                          \
  hipLaunchKernelGGL((f32_mfma_attention_kernel<HD>), dim3(m.rows / 16, md.H), dim3(HD == 256 ? 256 : 512), 0, s, o, \
                     qkv, q_stride, kc, vc, m.mask, m.seq_p, m.seq_n, m.row0, m.blk_seq, md.H, md.Hkv, md.cap)
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
// so each thread walks j upwards and only ever overwrites slots it has already consumed.
__global__ void f32_kv_compact_kernel(float* const* __restrict__ kc, float* const* __restrict__ vc,
                                      const int32_t* __restrict__ path, const int32_t* __restrict__ n_acc,
                                      const int32_t* __restrict__ seq_p, int Hkv, int hd, int cap, int stride) {
  int layer = blockIdx.x, bh = blockIdx.y;
  int b = bh / Hkv;
  int len = n_acc[b];
  int P = seq_p[b];
  const int32_t* pth = path + (int64_t)b * stride;
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
void f32_kv_compact(float* const* kc, float* const* vc, const int32_t* path, const int32_t* n_acc,
                    const StepMeta& m, const ModelDims& md, int stride, hipStream_t s) {
  hipLaunchKernelGGL(f32_kv_compact_kernel, dim3(md.n_layers, m.batch * md.Hkv), dim3(64), 0, s, kc, vc, path,
                     n_acc, m.seq_p, md.Hkv, md.hd, md.cap, stride);
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

// rows of real nodes between the caller's [B][max_nodes][width] and the padded [R][width] buffers
__global__ void f32_gather_rows_kernel(float* __restrict__ dst, const float* __restrict__ src,
                                       const int32_t* __restrict__ seq_n, const int32_t* __restrict__ row0,
                                       const int32_t* __restrict__ blk_seq, int max_nodes, int width, int to_padded) {
  int r = blockIdx.x;
  int b = blk_seq[r >> 4], node = r - row0[b];
  bool real = node < seq_n[b];
  int64_t pad = (int64_t)r * width, ext = ((int64_t)b * max_nodes + node) * width;
  for (int i = threadIdx.x; i < width; i += blockDim.x) {
    if (to_padded) dst[pad + i] = real ? src[ext + i] : 0.f;
    else if (real) dst[ext + i] = src[pad + i];
  }
}
void f32_gather_rows(float* dst, const float* src, const StepMeta& m, int max_nodes, int width,
                     bool to_padded, hipStream_t s) {
  hipLaunchKernelGGL(f32_gather_rows_kernel, dim3(m.rows), dim3(256), 0, s, dst, src, m.seq_n, m.row0,
                     m.blk_seq, max_nodes, width, to_padded ? 1 : 0);
}

}  // namespace ded
