// Internal launcher interface between the host scheduler (ded_api.hip) and the kernel files.
// Every launcher enqueues on the given stream and checks its shapes on the host first; the
// kernels themselves assume those shapes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ded {

// Device-resident description of the current step (one verification forward).
// The trees lie one after the other, each padded to whole blocks of 16 rows: row r = row0[b] + node, and every
// 16-row block belongs to one sequence.  (Padding all trees to the largest one instead made a ragged batch pay for
// rows nobody reads: 192 rows for trees of 37, 21 and 50 nodes where 144 do.)  n_step = the largest padded tree.
struct StepMeta {
  const int32_t* token;   // [R]   token id of the row (padding rows repeat the root token)
  const int32_t* parent;  // [R]   parent node index inside the sequence, -1 for root / padding
  const int32_t* depth;   // [R]
  const int32_t* pos;     // [R]   absolute position prefix_len + depth
  const uint64_t* mask;   // [R][4] ancestor-or-self bitmask over node indices (bit j = node j)
  const int32_t* seq_p;   // [B]   prefix_len per sequence
  const int32_t* seq_n;   // [B]   real tree rows per sequence
  const int32_t* row0;    // [B]   first row of the sequence (multiple of 16)
  const int32_t* blk_seq; // [rows / 16] sequence of each 16-row block
  const int32_t* attn_items;  // fp32 path: (16-row block, key range) pairs, block * F32_ATTN_SPLITS + range
  int32_t batch, n_step, rows;  // rows = sum of the padded tree sizes
};

struct ModelDims {
  int32_t n_layers, d, H, Hkv, hd, F, V, cap;
  float rope_base, eps;
};

// What the embedding kernels do beside the embedding (step_ends.h): the rotary table tab[r][i] = cos, sin of pos[r] *
// base^(-2i/hd), i < half = hd/2, and the copy of the step's description from pinned host memory to the device.  token and
// pos are read from the host's block, everything after from the device's.
struct StepFront {
  const uint4* meta_src;  // pinned host memory
  uint4* meta_dst;
  int units;  // 16 bytes each
  const int32_t *token, *pos;
  float2* tab;
  int rows, half;
  double neg2_over_hd_log2base;
};
// Approval walk (mode 0 greedy, mode 1 keep the whole chain), done by the kernels that compact the cache (step_ends.h).  The out_
// arrays are pinned host memory: out_n, out_flag [B], out_path, out_tok [B][stride].  If a real row of any sequence is
// flagged, every sequence gets out_n = 0, out_flag = 1.
struct ApprovalWalk {
  const int32_t *token, *parent, *seq_n, *row0, *amax, *row_flag;
  int batch, mode, stride;
  int32_t *out_n, *out_flag, *out_path, *out_tok;
};

// ---- shared (both dtypes) --------------------------------------------------------------
// Measurement aid: streams `bytes` (multiple of 16) of device memory through the CUs once.
void launch_stream_read(const void* src, size_t bytes, uint32_t* sink, hipStream_t s);
// Per-row argmax (lowest index on exact ties) and top-1 minus top-2 over V fp32 logits; flag[r] != 0 when the
// row holds a NaN or an infinity.  The rows of real nodes go to the caller's export_to [batch][max_nodes][V] too if it is not null.
void launch_argmax(const float* logits, const StepMeta& m, int V, int32_t* amax, float* margin, int32_t* flag, float* export_to,
                   int max_nodes, hipStream_t s);
// The same from the candidates the LM-head GEMM leaves with EPI_TOP2: part [rows][groups] x 16 bytes.
void launch_top2_reduce(const void* part, int groups, int rows, int32_t* amax, float* margin, int32_t* flag,
                        hipStream_t s);
// Temperature / top-p sample of every real row (inverse CDF of uniform[r] over the nucleus in id order) -> token_out[r].
// uniform and flag_out (the rows' flags once more) are pinned host memory.
void launch_sample_top_p(const float* logits, int64_t row_stride, const StepMeta& m, int V, float temperature,
                         float top_p, const float* uniform, const int32_t* flag, int32_t* token_out, int32_t* flag_out,
                         hipStream_t s);
// The walk alone, where there is nothing to compact.
void launch_accept_walk(const ApprovalWalk& w, hipStream_t s);

// ---- fp32 path (cache [B][Hkv][cap][hd], queries and logits row-major; weights and projection inputs "packed": tiles of
// 16 rows x 16 k, see kernels_f32.hip) ------------------------------------------------------
// floats of a packed matrix
inline int64_t f32_packed_floats(int64_t rows, int64_t k) { return (rows + 15) / 16 * ((k + 15) / 16) * 256; }
// dst = packed W[N][K] * gain[k] (gain null: 1)
void f32_pack_weight(float* dst, const float* src, const float* gain, int N, int K, hipStream_t s);
void f32_embed(float* x, const float* emb, const StepFront& f, int d, hipStream_t s);
// Y[r][n] = sum_k X[r][k] W[n][k] with a fused neighbour on either side.  All kinds but F32_RESIDUAL normalise their
// input rows, X[r] / sqrt(mean(x^2) + eps); the norm's gain is part of W.  X and W are packed.
enum {
  F32_STORE = 0,     // Y = result, row stride N
  F32_RESIDUAL = 1,  // Y += result, packed
  F32_SILU = 2,      // W = packed gate features, then packed up features, N / 2 each: Y = silu(gate) * up, packed
  F32_QKV = 3        // queries rotated into Y (row stride N), keys rotated / values into the cache; hd % 32 == 0
};
struct F32Gemm {
  int kind;
  float* Y;
  const float *X, *W;
  float eps;
  int rows, N, K;  // rows % 16 == 0
  // F32_QKV
  float *kc, *vc;
  const float2* tab;
  StepMeta m;
  int H, Hkv, hd, cap;
};
void f32_gemm(const F32Gemm& g, hipStream_t s);
void f32_rope_kv(float* qkv, float* kc, float* vc, const float2* tab, const StepMeta& m,
                 const ModelDims& md, hipStream_t s);
// Sequences of more than 256 keys are cut into up to `most` <= F32_ATTN_SPLITS key ranges (head dims of 16 and more); m.attn_items
// lists the n_items pairs of a 16-row block and one of its sequence's ranges.  part_o holds rows * H * most * hd floats,
// part_ml rows * H * most * 2, tickets rows / 16 * H zeroed ints (left zeroed); the first two are not used with most = 1.
// The sequence alone decides about its ranges (and the room the context has), not how full the chip is: a row's sums do not
// depend on its neighbours.  A range is one block of 16 keys per wavefront; two blocks in a row are faster than the hand-over
// (144 keys, 4 heads x 64: 7.0 us whole, 8.8 in two ranges; 560 keys, 8 heads x 128: 21 and 13.3 in five).
constexpr int F32_ATTN_SPLITS = 8;
__host__ __device__ inline int f32_attention_splits(int keys, int most) {
  const int s = keys > 256 ? (keys + 127) / 128 : 1;
  return s < most ? s : most;
}
void f32_tree_attention(float* o, const float* qkv, int q_stride, const float* kc, const float* vc,
                        const StepMeta& m, const ModelDims& md, int n_items, int most, float* part_o, float* part_ml, int* tickets,
                        hipStream_t s);
void f32_kv_compact(float* const* kc, float* const* vc, const ApprovalWalk& w, const StepMeta& m, const ModelDims& md, hipStream_t s);
// plain [Hkv][n][hd] <-> cache
void f32_kv_copy(float* cache, float* plain, bool to_cache, int seq, int first, int n,
                 const ModelDims& md, hipStream_t s);
void f32_kv_clear(float* kc, float* vc, int seq, int first, int n, const ModelDims& md, hipStream_t s);
void f32_scatter_tree_kv(float* kc, float* vc, const float* k_tree, const float* v_tree,
                         const StepMeta& m, const ModelDims& md, int max_nodes, hipStream_t s);
// q [B][max_nodes][H][hd] -> qkv-style rows [R][H*hd]; and the packed attention output -> [B][max_nodes][H][hd]
void f32_gather_rows(float* dst, const float* src, const StepMeta& m, int max_nodes, int width,
                     bool to_padded, hipStream_t s);

// ---- 16-bit path (bf16 weights in, f16 matrix-core operands; see bf16_layout.h) -----------------
// Operand-fragment layouts (units: 2-byte elements; a fragment = 64 lanes x 8 elements = 1 KiB):
//  PackW  W[N][K]   : frag (ng = n/64, kt = k/32, t = (n/16)%4) at (ng*(K/32)+kt)*4+t; lane = ((k%32)/8)*16 + n%16;
//                      elem k%8; N padded to a multiple of 64 with zero features
//  PackX  X[R][K]   : frag (kt, rb = r/16, plane hi/lo) at (kt*RB+rb)*2+plane; lane = ((k%32)/8)*16 + r%16; elem k%8
//  PackQ  per (b,kvh): frag (vrb, kk = hd/32, plane) at (vrb*4+kk)*2+plane, virtual row vr = g*(padded tree rows of b) + node
//  PackK  per (b,kvh): 32-key group kb; frag (kb, c, kk) at (kb*2+c)*4+kk; key%32 = q8*8 + c*4 + i
//                      -> lane = ((hdim%32)/8)*16 + q8*4 + i; elem hdim%8
//  PackVt per (b,kvh): frag (kb, hb = hdim/16) at kb*8+hb; lane = ((key%32)/8)*16 + hdim%16; elem key%8
typedef uint16_t bf16_t;

// How the features (rows) of a weight matrix are ordered inside PackW.  The paired orders put partner
// features into tiles t and t + 2 of one 64-feature group so that one wavefront holds both.
enum { PERM_NONE = 0, PERM_ROPE = 1 /* per head: dims i and i + 64 */, PERM_GATE_UP = 2 /* gate f and up f */ };
void bf16_pack_weight(bf16_t* dst, const bf16_t* src, int N, int K, int perm, hipStream_t s);
// x = emb[token]; y = (x * gain) as hi/lo f16 in PackX; ssq[r][g] = sum of x^2 over feature group g (64 wide)
void bf16_embed(float* x, bf16_t* y_packed, float* ssq, const bf16_t* emb, const float* gain, const StepFront& f,
                int rows_pad, int d, hipStream_t s);

// What a GEMM does with its result tile (fused epilogue).  RMSNorm is deferred: producers write
// x * gain and sum(x^2) per 64-feature group, consumers multiply their output rows by 1/rms.
enum { EPI_LOGITS = 0, EPI_QKV = 1, EPI_SILU = 2, EPI_RESIDUAL = 3, EPI_TOP2 = 4 };
struct GemmEpilogue {
  int kind;
  // row scale of the GEMM input (null: 1): scale[r] = rsqrt(sum_g ssq_in[r][g] * inv_k + eps)
  const float* ssq_in;
  int ssq_groups;
  float inv_k, eps;
  int rows;      // real rows (the rest up to rows_pad is padding)
  int rb_total;  // rows_pad / 16 of the PackX buffers
  // EPI_LOGITS: out[r][n] = scale * Y, and the rows of real nodes (seq_n, row0, blk_seq) in the caller's logits_out
  // [batch][max_nodes][N] too if it is not null; and what EPI_TOP2 leaves
  float* out;
  int64_t out_stride;
  float* logits_out;
  int max_nodes;
  // EPI_TOP2: instead of the logits, per (row, 64-feature group) the best value, its feature index, the second
  // best value and a non-finite flag: top2_part[r * top2_groups + group] (16 bytes each)
  void* top2_part;
  int top2_groups;
  // EPI_QKV: rotary embedding at the row's position, queries -> PackQ (hi/lo), keys / values -> cache
  bf16_t *q_packed, *k_cache, *v_cache;
  const float2* rope_tab;
  const int32_t *seq_p, *seq_n, *row0, *blk_seq;
  int n_step, H, Hkv, cap;
  // EPI_SILU: y_packed(hi) = silu(scale*gate) * (scale*up);  EPI_RESIDUAL: x += Y, y_packed = x*gain (hi/lo), ssq_out
  bf16_t* y_packed;
  float* x;
  const float* gain;
  float* ssq_out;
};

// Workgroup tiles of the tile kernel (features x rows).
enum {
  TILE_256x256 = 1, TILE_256x192, TILE_256x128, TILE_128x256, TILE_128x192, TILE_128x128
};
constexpr int SUMMED_APART = -1;
struct GemmPlan {
  int nwn;       // 0: stream kernel (one feature group per workgroup); 2..4: wide kernel, groups per workgroup
  int nw;        // stream kernel: wavefronts splitting the k range
  int splits;    // split-K slices
  int tile = 0;  // != 0: the tile kernel, with this workgroup tile
  int whole = 0; // tile kernel: that many tiles whole, the others with k split `splits` ways; SUMMED_APART: all split, the
                 // slices added by a launch of their own
  int ssq_waves = 1;  // tile kernel: shares in which a row's sums of squares are added
};
// sum_rows (a multiple of 64, >= rows_pad) decides into which k ranges the sums are split, rows_pad how they are run.
GemmPlan bf16_gemm_plan(int sum_rows, int rows_pad, int N, int K, int planes, int max_splits, int64_t part_elems);
// of a residual projection (one plane, EPI_RESIDUAL), whose sums may be added by a launch of their own
GemmPlan bf16_gemm_plan_residual(int sum_rows, int rows_pad, int N, int K, int max_splits, int64_t part_elems);
int bf16_gemm_tiles(int rows_pad, int N, const GemmPlan& plan);
// GEMM on the matrix cores with a fused epilogue (skinny and tile kernels).  planes = 2 uses X = hi + lo, planes = 1 only
// the hi plane.  rows_pad % 64 == 0, N % 16 == 0 (N % 64 for the paired epilogues), K % 128 == 0.  `part` (part_elems floats)
// takes the split sums: plan.splits slices of part_stride >= rows_pad * round_up(N, 64) floats, or the tile kernel's own
// slices; `counters` one zeroed int per output tile, eight per split tile of the tile kernel (left zeroed).  Returns false
// (nothing launched) on an unsupported shape.
bool bf16_gemm(float* part, int64_t part_stride, int64_t part_elems, const bf16_t* x_packed, const bf16_t* w_packed,
               int rows_pad, int N, int K, int planes, const GemmPlan& plan, int* counters, const GemmEpilogue& epi,
               hipStream_t s);
// Few rows (rows <= BF16_SLIM_ROWS, a multiple of 16): a workgroup takes the whole k range of few features; its wavefronts
// take the k ranges that `plan` (of 64 rows) gives the skinny kernels and their sums are added in the same order, so the
// result has the same bits.  EPI_RESIDUAL writes its sums of squares per 4 features here (epi.ssq_out[row][N / 4]), and
// epi.ssq_groups = d / 4 says that ssq_in holds those.  Returns false where the plan has more than 16 ranges.
constexpr int BF16_SLIM_ROWS = 32;
bool bf16_gemm_slim_ok(const GemmPlan& plan, int K, int planes);
bool bf16_gemm_slim(const bf16_t* x_packed, const bf16_t* w_packed, int rows, int rows_pad, int N, int K, int planes,
                    const GemmPlan& plan, const GemmEpilogue& epi, hipStream_t s);
// Tree-masked attention: split-KV partials (running max, sum, unnormalised output per key range), then - when
// there is more than one key range - the merge; the result is written as PackX(o), hi/lo, for the O projection.
// n_splits from bf16_attn_pick_splits.  part_o: [B][H][n_splits][n_step][hd] fp32, part_ml: [B][H][n_splits][n_step]
// float2 (max, sum).  q_planes: 2 = the queries are hi + lo pairs, 1 = their lo plane is known to be zero
// (queries given as bf16).  With q_plain / out_plain (q_planes = 1) the queries are read from, and the result written to,
// plain bf16 [batch][max_nodes][H][hd] arrays; q_packed and o_packed are then not touched.
int bf16_attn_pick_splits(const StepMeta& m, const ModelDims& md, int max_p, int64_t part_rows_cap);
// Query planes the model path hands to the attention: 2, except 1 (hi plane only) when 512 or more rows share each
// K / V byte (grouped query heads x tree rows per kv head): there the attention is bound by the matrix cores and the lo
// plane is a third of their work, while the keys are stored with the same 11-bit rounding anyway, so the score error
// grows by at most sqrt(2).
int bf16_attn_query_planes(const StepMeta& m, const ModelDims& md);
void bf16_tree_attention(bf16_t* o_packed, int rows_pad, const bf16_t* q_packed, const bf16_t* kc, const bf16_t* vc,
                         float* part_o, float2* part_ml, int n_splits, int q_planes, const StepMeta& m,
                         const ModelDims& md, hipStream_t s, const bf16_t* q_plain = nullptr,
                         bf16_t* out_plain = nullptr, int max_nodes = 0);
void bf16_kv_compact(bf16_t* const* kc, bf16_t* const* vc, const ApprovalWalk& w, const StepMeta& m, const ModelDims& md, hipStream_t s);
void bf16_kv_copy(bf16_t* kcache, bf16_t* vcache, bf16_t* k_plain, bf16_t* v_plain, bool to_cache,
                  int seq, int first, int n, const ModelDims& md, hipStream_t s);
void bf16_kv_clear(bf16_t* kcache, bf16_t* vcache, int seq, int first, int n, const ModelDims& md, hipStream_t s);
// m: the step's description in pinned host memory, `units` x 16 bytes of which go from meta_src to meta_dst beside the scatter;
// host_p, host_n: its prefix lengths and tree sizes for the host
void bf16_scatter_tree_kv(bf16_t* kc, bf16_t* vc, const bf16_t* k_tree, const bf16_t* v_tree, const StepMeta& m,
                          const void* meta_src, void* meta_dst, int units, const int32_t* host_p, const int32_t* host_n,
                          const ModelDims& md, int max_nodes, hipStream_t s);

}  // namespace ded
