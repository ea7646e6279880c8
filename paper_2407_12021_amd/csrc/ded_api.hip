// C ABI of the verification library: argument validation, workspace lay-out, and the fixed kernel
// sequence of one verification forward (Sec. 2.4) on the caller's stream.
#include "../../include/ded_verify.h"
#include "ded_kernels.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

using namespace ded;

namespace {

constexpr int kMaskWords = 4;   // ancestor bitmask words per row (max_nodes <= 256)
constexpr int kMaxNodes = 256;
constexpr int64_t kAttnPartRows = 1 << 17;  // split-KV partial rows the workspace reserves at least
constexpr int64_t kF32AttnPartFloats = 16 << 20;  // partial results of the fp32 attention: at most
constexpr size_t kMetaMirrorBytes = 1 << 20;  // of pinned slots for step descriptions (at least two slots, at most 16)
constexpr int kGemmCounters = 1 << 16;      // split-K arrival tickets (a GEMM with more output tiles runs unsplit)

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline int round_up(int v, int a) { return (v + a - 1) / a * a; }

enum KClass {
  KC_META = 0, KC_ROPE_TABLE, KC_EMBED, KC_GEMM_QKV, KC_QKV_EPILOGUE, KC_TREE_ATTN, KC_GEMM_O, KC_GEMM_GATE_UP,
  KC_GEMM_DOWN, KC_GEMM_LM_HEAD, KC_ARGMAX, KC_EXPORT, KC_WALK, KC_COMPACT, KC_LAYOUT, KC_SAMPLE, KC_TOP2_REDUCE, KC_COUNT
};
// (rope_table and export_logits count no launches: the embedding and the argmax do that work)
const char* const kClassNames[KC_COUNT] = {
    "meta_upload", "rope_table", "embed", "gemm_qkv", "qkv_rope_epilogue", "tree_attention", "gemm_o", "gemm_gate_up",
    "gemm_down", "gemm_lm_head", "argmax", "export_logits", "accept_walk", "kv_compact", "layout_convert", "sample_top_p",
    "top2_reduce"};

struct Carve {  // bump allocator over the workspace (base may be null when only sizing)
  char* base;
  size_t off = 0;
  explicit Carve(char* b) : base(b) {}
  template <typename T>
  T* take(size_t count) {
    off = align_up(off, 256);
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

}  // namespace

// Where the parts of a step's description sit inside the uploaded block, for `rows` tree rows of `batch` sequences.
struct MetaOffsets {
  size_t token = 0, parent = 0, depth = 0, pos = 0, mask = 0, p = 0, n = 0, row0 = 0, blk_seq = 0, attn_items = 0, bytes = 0;
  MetaOffsets() = default;
  MetaOffsets(int rows, int batch, bool f32) {
    auto take = [&](size_t count) {
      const size_t at = bytes;
      bytes = align_up(bytes + count, 64);
      return at;
    };
    token = take((size_t)rows * 4), parent = take((size_t)rows * 4), depth = take((size_t)rows * 4);
    pos = take((size_t)rows * 4), mask = take((size_t)rows * 8 * kMaskWords);
    p = take((size_t)batch * 4), n = take((size_t)batch * 4), row0 = take((size_t)batch * 4);
    blk_seq = take((size_t)rows / 16 * 4);
    if (f32) attn_items = take((size_t)rows / 16 * F32_ATTN_SPLITS * 4);
  }
};

// Scratch of ded_tree_attention_static: device memory that belongs to the library itself, for callers that
// cannot allocate and bring no workspace region of their own for it.  One copy per GPU, held until the
// process ends.  In host code the array's name is only a handle: its device address is resolved once per
// device (resolve_static_scratch) and that pointer is what kernels, copies and memsets receive.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static unsigned char* g_scratch_ptr[kMaxDevices] = {};
static std::mutex g_scratch_mutex;

// With `device` current: the address of this device's copy of `scratch` (null if the runtime refuses).
static unsigned char* resolve_static_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[device] = static_cast<unsigned char*>(p);
  }
  return g_scratch_ptr[device];
}

struct ded_ctx {
  ded_config cfg;
  ModelDims md;
  bool bf16 = false;
  hipStream_t stream = nullptr;
  int device = -1;                          // the device that was current at ded_verify_init
  unsigned char* static_scratch = nullptr;  // this device's copy of the library's own scratch array
  int max_n_pad = 0;    // max_nodes rounded up to 16
  int max_rows = 0;     // max_batch * max_n_pad
  int max_rows_pad = 0; // rounded up to 64

  // weights inside the workspace
  void* emb = nullptr;
  void* lm_head = nullptr;
  float* final_norm = nullptr;
  std::vector<void*> wqkv, wo, wgu, wdown;
  std::vector<float*> norm_attn, norm_ffn;
  // caches
  std::vector<void*> kc, vc;
  void** d_kc = nullptr;
  void** d_vc = nullptr;
  // activations
  float* x = nullptr;
  float* logits = nullptr;
  float2* rope_tab = nullptr;
  // fp32 path
  float *f_qkv = nullptr, *f_o = nullptr, *f_h = nullptr, *f_part_o = nullptr, *f_part_ml = nullptr;
  int* f_tickets = nullptr;
  int f_splits = 1;  // key ranges that f_part_o has room for
  int f_items = 0;   // of the pending step: workgroups per head of its attention
  // bf16 path
  bf16_t *y_p = nullptr, *o_p = nullptr, *h_p = nullptr, *q_p = nullptr;
  float* part = nullptr;
  int64_t part_elems = 0;
  float* ssq = nullptr;     // [rows_pad][d / 64] sum of squares of the residual stream per feature group
  int* counters = nullptr;  // split-K arrival tickets, one per output tile (kept at zero between launches)
  float* attn_part_o = nullptr;
  float2* attn_part_ml = nullptr;
  int64_t attn_part_rows = 0;
  void* top2_part = nullptr;  // [rows_pad][ceil(V / 64)] x 16 B: per-group candidates of the fused LM-head argmax
  // step meta (device + pinned host mirror, one contiguous block).  The mirror has several slots that calls take in turn, in
  // two halves: entering a half, a call waits for the calls that used it the last time round.
  char* d_meta = nullptr;
  char* h_meta = nullptr;  // the present slot
  size_t meta_bytes = 0;
  char *h_meta_slots = nullptr, *h_meta_slots_dev = nullptr;
  int meta_slots = 0, meta_slot = 0;
  char* h_meta_dev = nullptr;  // the present slot as kernels address it: the first kernel of a call reads it there
  hipEvent_t meta_ev[2] = {};  // what had been enqueued when the half was left
  bool meta_left[2] = {};
  MetaOffsets off;  // of the pending step: the block is packed to the step's own row count
  // results
  // (the three lie one after the other, packed to the step's rows: one copy brings them to the host)
  int32_t* d_amax = nullptr;
  float* d_margin = nullptr;
  int32_t* d_rowflag = nullptr;  // [rows] != 0: the row's logits hold a NaN or an infinity
  // pinned: amax | margin | row flags, or uniform numbers | row flags, or nacc | seqflag | path | acctok
  char *h_res = nullptr, *h_res_dev = nullptr;
  size_t res_bytes = 0;
  // state of the pending step
  bool pending = false;
  bool have_argmax = false;
  bool have_logits = false;    // the workspace holds the fp32 logits of the last step
  bool poisoned = false;       // the last step's tree slots may hold NaN / infinite K/V: cleared before they can be read
  bool sampling_seen = false;  // ded_sample has been used on this context: steps keep their logits from then on
  int batch = 0, n_step = 0, rows = 0;
  int max_p = 0;
  std::vector<int32_t> s_p, s_n, s_parent, s_row0;
  // profiling
  bool prof_on = false;
  std::vector<hipEvent_t> ev_pool;
  size_t ev_used = 0;
  struct Span { int cls; size_t e0, e1; };
  std::vector<Span> spans;
  double prof_ms[KC_COUNT] = {};
  int64_t prof_n[KC_COUNT] = {};

  StepMeta meta() const { return meta_at(d_meta); }
  // the step description inside a device copy of the meta block that starts at `base`
  StepMeta meta_at(const char* base) const {
    StepMeta m;
    m.token = reinterpret_cast<const int32_t*>(base + off.token);
    m.parent = reinterpret_cast<const int32_t*>(base + off.parent);
    m.depth = reinterpret_cast<const int32_t*>(base + off.depth);
    m.pos = reinterpret_cast<const int32_t*>(base + off.pos);
    m.mask = reinterpret_cast<const uint64_t*>(base + off.mask);
    m.seq_p = reinterpret_cast<const int32_t*>(base + off.p);
    m.seq_n = reinterpret_cast<const int32_t*>(base + off.n);
    m.row0 = reinterpret_cast<const int32_t*>(base + off.row0);
    m.blk_seq = reinterpret_cast<const int32_t*>(base + off.blk_seq);
    m.attn_items = reinterpret_cast<const int32_t*>(base + off.attn_items);
    m.batch = batch;
    m.n_step = n_step;
    m.rows = rows;
    return m;
  }
  size_t meta_units() const { return (off.bytes + 15) / 16; }  // (the blocks end on a multiple of 256 bytes)
  StepFront front() const {
    const StepMeta h = meta_at(h_meta_dev);
    StepFront f;
    f.meta_src = reinterpret_cast<const uint4*>(h_meta_dev);
    f.meta_dst = reinterpret_cast<uint4*>(d_meta);
    f.units = (int)meta_units();
    f.token = h.token, f.pos = h.pos;
    f.tab = rope_tab;
    f.rows = rows, f.half = md.hd / 2;
    f.neg2_over_hd_log2base = -2.0 / (double)md.hd * log2((double)md.rope_base);
    return f;
  }
};

namespace {

// ---------------------------------------------------------------------------------------------
bool config_ok(const ded_config* c) {
  if (!c) return false;
  if (c->n_layers < 0 || c->d_model <= 0 || c->n_heads <= 0 || c->n_kv_heads <= 0 || c->head_dim <= 0 ||
      c->vocab <= 0 || c->max_batch <= 0 || c->kv_capacity <= 0 || c->max_nodes <= 0)
    return false;
  if (c->n_layers > 0 && c->d_ffn <= 0) return false;
  if (c->n_heads % c->n_kv_heads) return false;
  if (c->max_nodes > kMaxNodes) return false;
  if (c->head_dim % 2) return false;
  if (!(c->rope_base > 0.f) || !(c->rms_eps >= 0.f)) return false;
  if ((int64_t)c->max_batch * round_up(c->max_nodes, 16) > (1 << 20)) return false;
  if (c->dtype == DED_F32) {
    if (c->head_dim > 256 || 256 % c->head_dim) return false;
    return true;
  }
  if (c->dtype == DED_BF16) {
    if (c->head_dim != 128) return false;
    if (c->d_model % 128 || c->vocab % 16 || c->kv_capacity % 64) return false;
    if (c->n_layers > 0 && c->d_ffn % 128) return false;
    return true;
  }
  return false;
}

struct Sizes {
  int max_n_pad, max_rows, max_rows_pad;
  size_t elem;  // bytes per stored element
};

Sizes sizes_of(const ded_config& c) {
  Sizes s;
  s.max_n_pad = round_up(c.max_nodes, 16);
  s.max_rows = c.max_batch * s.max_n_pad;
  s.max_rows_pad = round_up(s.max_rows, 64);
  s.elem = c.dtype == DED_BF16 ? 2 : 4;
  return s;
}

// Single description of the workspace; used for sizing (ctx == nullptr members untouched) and for init.
size_t carve_workspace(const ded_config& c, char* base, ded_ctx* ctx) {
  Sizes z = sizes_of(c);
  Carve w(base);
  const int64_t d = c.d_model, V = c.vocab, F = c.d_ffn;
  const int64_t qd = (int64_t)c.n_heads * c.head_dim, kvd = (int64_t)c.n_kv_heads * c.head_dim;
  const int64_t qkv_n = qd + 2 * kvd;
  const int L = c.n_layers;
  auto bytes = [&](int64_t n) { return (size_t)n * z.elem; };

  // matrices are re-laid-out: bf16 with the feature count padded to a multiple of 64, fp32 to whole tiles of 16 x 16
  auto wbytes = [&](int64_t n_out, int64_t k_in) {
    return c.dtype == DED_BF16 ? bytes((n_out + 63) / 64 * 64 * k_in) : (size_t)f32_packed_floats(n_out, k_in) * 4;
  };
  char* emb = w.take<char>(bytes(V * d));
  char* lm = w.take<char>(wbytes(V, d));
  float* fn = w.take<float>(d);
  if (ctx) {
    ctx->emb = emb;
    ctx->lm_head = lm;
    ctx->final_norm = fn;
    ctx->wqkv.assign(L, nullptr);
    ctx->wo.assign(L, nullptr);
    ctx->wgu.assign(L, nullptr);
    ctx->wdown.assign(L, nullptr);
    ctx->norm_attn.assign(L, nullptr);
    ctx->norm_ffn.assign(L, nullptr);
  }
  for (int l = 0; l < L; ++l) {
    char* a = w.take<char>(wbytes(qkv_n, d));
    char* b = w.take<char>(wbytes(d, qd));
    char* g = w.take<char>(c.dtype == DED_BF16 ? wbytes(2 * F, d) : 2 * wbytes(F, d));
    char* dn = w.take<char>(wbytes(d, F));
    float* na = w.take<float>(d);
    float* nf = w.take<float>(d);
    if (ctx) {
      ctx->wqkv[l] = a;
      ctx->wo[l] = b;
      ctx->wgu[l] = g;
      ctx->wdown[l] = dn;
      ctx->norm_attn[l] = na;
      ctx->norm_ffn[l] = nf;
    }
  }
  void** dkc = w.take<void*>(std::max(L, 1));
  void** dvc = w.take<void*>(std::max(L, 1));
  float* x = w.take<float>(c.dtype == DED_BF16 ? (int64_t)z.max_rows_pad * d : f32_packed_floats(z.max_rows_pad, d));
  float* logits = w.take<float>((int64_t)z.max_rows_pad * V);
  float2* tab = w.take<float2>((int64_t)z.max_rows * (c.head_dim / 2));
  if (ctx) {
    ctx->d_kc = dkc;
    ctx->d_vc = dvc;
    ctx->x = x;
    ctx->logits = logits;
    ctx->rope_tab = tab;
  }
  if (c.dtype == DED_F32) {
    float* qkv = w.take<float>((int64_t)z.max_rows_pad * qkv_n);
    float* o = w.take<float>(f32_packed_floats(z.max_rows_pad, qd));
    float* h = w.take<float>(f32_packed_floats(z.max_rows_pad, F));
    const int64_t range = (int64_t)z.max_rows * c.n_heads;  // (row, head) pairs of one key range
    const int splits = (int)std::max<int64_t>(1, std::min<int64_t>(F32_ATTN_SPLITS, kF32AttnPartFloats / (range * (c.head_dim + 2))));
    float* part_o = w.take<float>(splits > 1 ? range * splits * c.head_dim : 1);
    float* part_ml = w.take<float>(splits > 1 ? range * splits * 2 : 1);
    int* tickets = w.take<int>(range / 16);
    if (ctx) {
      ctx->f_qkv = qkv;
      ctx->f_o = o;
      ctx->f_h = h;
      ctx->f_part_o = part_o;
      ctx->f_part_ml = part_ml;
      ctx->f_tickets = tickets;
      ctx->f_splits = splits;
    }
  } else {
    // GEMM inputs and queries are kept as hi/lo pairs of f16: two planes each
    bf16_t* y = w.take<bf16_t>((int64_t)z.max_rows_pad * d * 2);
    bf16_t* o = w.take<bf16_t>((int64_t)z.max_rows_pad * qd * 2);
    bf16_t* h = w.take<bf16_t>((int64_t)z.max_rows_pad * std::max<int64_t>(F, 1) * 2);
    bf16_t* q = w.take<bf16_t>((int64_t)z.max_rows_pad * qd * 2);
    // split-K partials: at most 8 slices of 64 rows, or one slice of every row
    int64_t widest = std::max<int64_t>(std::max<int64_t>(qkv_n, 2 * F), std::max<int64_t>(d, round_up((int)V, 64)));
    int64_t part_elems = widest * std::max<int64_t>(8 * 64, z.max_rows_pad);
    float* part = w.take<float>(part_elems);
    float* ssq = w.take<float>((int64_t)z.max_rows_pad * (d / 64));
    int* counters = w.take<int>(kGemmCounters);
    int64_t arows = std::max<int64_t>(kAttnPartRows, (int64_t)z.max_rows * c.n_heads);
    float* apo = w.take<float>(arows * c.head_dim);
    float2* apm = w.take<float2>(arows);
    char* t2 = w.take<char>((size_t)z.max_rows_pad * ((V + 63) / 64) * 16);
    if (ctx) {
      ctx->top2_part = t2;
      ctx->y_p = y;
      ctx->o_p = o;
      ctx->h_p = h;
      ctx->q_p = q;
      ctx->part = part;
      ctx->part_elems = part_elems;
      ctx->ssq = ssq;
      ctx->counters = counters;
      ctx->attn_part_o = apo;
      ctx->attn_part_ml = apm;
      ctx->attn_part_rows = arows;
    }
  }
  // step meta block
  const size_t m = align_up(MetaOffsets(z.max_rows, c.max_batch, c.dtype == DED_F32).bytes, 256);
  char* dmeta = w.take<char>(m);
  int32_t* amax = w.take<int32_t>((int64_t)z.max_rows_pad * 3);  // and margins and flags, see ingest
  if (ctx) {
    ctx->d_meta = dmeta;
    ctx->meta_bytes = m;
    ctx->d_amax = amax;
  }
  return align_up(w.off, 256);
}

#define HIP_TRY(expr)                     \
  do {                                    \
    if ((expr) != hipSuccess) {           \
      (void)hipGetLastError();            \
      return DED_EHIP;                    \
    }                                     \
  } while (0)

// Profiling bracket around one launcher call.
struct ProfScope {
  ded_ctx* c;
  int cls;
  size_t e0 = 0;
  bool on;
  ProfScope(ded_ctx* ctx, int k) : c(ctx), cls(k), on(ctx->prof_on) {
    if (!on) return;
    e0 = next();
    (void)hipEventRecord(c->ev_pool[e0], c->stream);
  }
  ~ProfScope() {
    if (!on) return;
    size_t e1 = next();
    (void)hipEventRecord(c->ev_pool[e1], c->stream);
    c->spans.push_back({cls, e0, e1});
  }
  size_t next() {
    if (c->ev_used == c->ev_pool.size()) {
      hipEvent_t e;
      (void)hipEventCreate(&e);
      c->ev_pool.push_back(e);
    }
    return c->ev_used++;
  }
};

int prof_drain(ded_ctx* c) {
  if (c->spans.empty()) return DED_OK;
  HIP_TRY(hipStreamSynchronize(c->stream));
  for (auto& s : c->spans) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, c->ev_pool[s.e0], c->ev_pool[s.e1]) == hipSuccess) {
      c->prof_ms[s.cls] += ms;
      c->prof_n[s.cls] += 1;
    }
  }
  c->spans.clear();
  c->ev_used = 0;
  return DED_OK;
}

// ---------------------------------------------------------------------------------------------
// Host-side tree ingest: validation, depth, position, ancestor bitmask (mask[i] = mask[parent] | bit i).
int validate_step(const ded_config& cfg, int32_t batch, const int32_t* prefix_len, const int32_t* n_nodes,
                  const int32_t* parent, const int32_t* token, bool need_token) {
  if (batch < 1 || batch > cfg.max_batch) return DED_EINVAL;
  if (!prefix_len || !n_nodes || !parent || (need_token && !token)) return DED_EINVAL;
  for (int b = 0; b < batch; ++b) {
    int n = n_nodes[b], p = prefix_len[b];
    if (n < 1 || n > cfg.max_nodes || p < 0) return DED_EINVAL;
    if ((int64_t)p + n > cfg.kv_capacity) return DED_ECAP;
    const int32_t* par = parent + (int64_t)b * cfg.max_nodes;
    if (par[0] != -1) return DED_ETREE;
    for (int i = 1; i < n; ++i)
      if (par[i] < 0 || par[i] >= i) return DED_ETREE;
    if (need_token) {
      const int32_t* tok = token + (int64_t)b * cfg.max_nodes;
      for (int i = 0; i < n; ++i)
        if (tok[i] < 0 || tok[i] >= cfg.vocab) return DED_ETOKEN;
    }
  }
  return DED_OK;
}

// The description of a call, into the next slot of the pinned mirror.
int ingest(ded_ctx* c, int32_t batch, const int32_t* prefix_len, const int32_t* n_nodes, const int32_t* parent,
           const int32_t* token) {
  const ded_config& cfg = c->cfg;
  int nmax = 0, pmax = 0, rows = 0;
  c->s_row0.resize(batch);
  for (int b = 0; b < batch; ++b) {
    nmax = std::max(nmax, n_nodes[b]);
    pmax = std::max(pmax, prefix_len[b]);
    c->s_row0[b] = rows;
    rows += round_up(n_nodes[b], 16);
  }
  const int half = c->meta_slots / 2;
  c->meta_slot = (c->meta_slot + 1) % c->meta_slots;
  if (c->meta_slot % half == 0) {
    const int now = c->meta_slot / half, left = 1 - now;
    HIP_TRY(hipEventRecord(c->meta_ev[left], c->stream));
    c->meta_left[left] = true;
    if (c->meta_left[now]) HIP_TRY(hipEventSynchronize(c->meta_ev[now]));
  }
  c->h_meta = c->h_meta_slots + c->meta_slot * c->meta_bytes;
  c->h_meta_dev = c->h_meta_slots_dev + c->meta_slot * c->meta_bytes;
  c->batch = batch;
  c->n_step = round_up(nmax, 16);
  c->rows = rows;
  c->off = MetaOffsets(rows, batch, !c->bf16);
  c->d_margin = reinterpret_cast<float*>(c->d_amax + rows);
  c->d_rowflag = c->d_amax + 2 * (size_t)rows;
  c->max_p = pmax;
  c->s_p.assign(prefix_len, prefix_len + batch);
  c->s_n.assign(n_nodes, n_nodes + batch);
  c->s_parent.assign((size_t)batch * cfg.max_nodes, -1);
  int32_t* h_token = reinterpret_cast<int32_t*>(c->h_meta + c->off.token);
  int32_t* h_parent = reinterpret_cast<int32_t*>(c->h_meta + c->off.parent);
  int32_t* h_depth = reinterpret_cast<int32_t*>(c->h_meta + c->off.depth);
  int32_t* h_pos = reinterpret_cast<int32_t*>(c->h_meta + c->off.pos);
  uint64_t* h_mask = reinterpret_cast<uint64_t*>(c->h_meta + c->off.mask);
  int32_t* h_p = reinterpret_cast<int32_t*>(c->h_meta + c->off.p);
  int32_t* h_n = reinterpret_cast<int32_t*>(c->h_meta + c->off.n);
  int32_t* h_row0 = reinterpret_cast<int32_t*>(c->h_meta + c->off.row0);
  int32_t* h_blk = reinterpret_cast<int32_t*>(c->h_meta + c->off.blk_seq);
  int32_t* h_items = reinterpret_cast<int32_t*>(c->h_meta + c->off.attn_items);
  c->f_items = 0;
  for (int b = 0; b < batch; ++b) {
    const int32_t* par = parent + (int64_t)b * cfg.max_nodes;
    const int32_t* tok = token ? token + (int64_t)b * cfg.max_nodes : nullptr;
    const int n = n_nodes[b], P = prefix_len[b], row0 = c->s_row0[b], n_pad = round_up(n, 16);
    h_p[b] = P;
    h_n[b] = n;
    h_row0[b] = row0;
    for (int i = 0; i < n_pad; i += 16) h_blk[(row0 + i) / 16] = b;
    if (!c->bf16)
      for (int i = 0; i < n_pad; i += 16)
        for (int z = 0; z < f32_attention_splits(P + n, c->f_splits); ++z)
          h_items[c->f_items++] = (row0 + i) / 16 * F32_ATTN_SPLITS + z;
    for (int i = 0; i < n_pad; ++i) {
      const int r = row0 + i;
      uint64_t* mr = h_mask + (size_t)r * kMaskWords;
      if (i < n) {
        c->s_parent[(size_t)b * cfg.max_nodes + i] = par[i];
        h_parent[r] = par[i];
        h_token[r] = tok ? tok[i] : 0;
        if (i == 0) {
          h_depth[r] = 0;
          for (int w = 0; w < kMaskWords; ++w) mr[w] = 0;
        } else {
          const int pr = row0 + par[i];
          h_depth[r] = h_depth[pr] + 1;
          const uint64_t* mp = h_mask + (size_t)pr * kMaskWords;
          for (int w = 0; w < kMaskWords; ++w) mr[w] = mp[w];
        }
        mr[i >> 6] |= 1ull << (i & 63);
      } else {  // padding row: behaves like a copy of the root, never read back
        h_parent[r] = -1;
        h_token[r] = tok ? tok[0] : 0;
        h_depth[r] = 0;
        for (int w = 0; w < kMaskWords; ++w) mr[w] = 0;
        mr[0] = 1ull;
      }
      h_pos[r] = P + h_depth[r];
    }
  }
  return DED_OK;
}

inline int launch_status() { return hipGetLastError() == hipSuccess ? DED_OK : DED_EHIP; }

// ---------------------------------------------------------------------------------------------
void f32_attention(ded_ctx* c, const float* q, int q_stride, int layer, const StepMeta& m, hipStream_t s) {
  f32_tree_attention(c->f_o, q, q_stride, (const float*)c->kc[layer], (const float*)c->vc[layer], m, c->md, c->f_items, c->f_splits,
                     c->f_part_o, c->f_part_ml, c->f_tickets, s);
}

int forward_f32(ded_ctx* c) {
  const ModelDims& md = c->md;
  StepMeta m = c->meta();
  hipStream_t s = c->stream;
  const int d = md.d, qd = md.H * md.hd, kvd = md.Hkv * md.hd, qkv_n = qd + 2 * kvd, F = md.F;
  { ProfScope p(c, KC_EMBED); f32_embed(c->x, (const float*)c->emb, c->front(), d, s); }
  auto gemm = [&](int cls, int kind, float* y, const float* x, const void* w, int N, int K, int l) {
    F32Gemm g = {};
    g.kind = kind;
    g.Y = y, g.X = x, g.W = (const float*)w;
    g.eps = md.eps;
    g.rows = m.rows, g.N = N, g.K = K;
    if (kind == F32_QKV) {
      g.kc = (float*)c->kc[l], g.vc = (float*)c->vc[l], g.tab = c->rope_tab;
      g.m = m;
      g.H = md.H, g.Hkv = md.Hkv, g.cap = md.cap;
    }
    g.hd = md.hd;
    ProfScope p(c, cls);
    f32_gemm(g, s);
  };
  for (int l = 0; l < md.n_layers; ++l) {
    const bool fused = md.hd % 32 == 0;
    gemm(KC_GEMM_QKV, fused ? F32_QKV : F32_STORE, c->f_qkv, c->x, c->wqkv[l], qkv_n, d, l);
    if (!fused) { ProfScope p(c, KC_QKV_EPILOGUE); f32_rope_kv(c->f_qkv, (float*)c->kc[l], (float*)c->vc[l], c->rope_tab, m, md, s); }
    { ProfScope p(c, KC_TREE_ATTN); f32_attention(c, c->f_qkv, qkv_n, l, m, s); }
    gemm(KC_GEMM_O, F32_RESIDUAL, c->x, c->f_o, c->wo[l], d, qd, l);
    gemm(KC_GEMM_GATE_UP, F32_SILU, c->f_h, c->x, c->wgu[l], 2 * F, d, l);
    gemm(KC_GEMM_DOWN, F32_RESIDUAL, c->x, c->f_h, c->wdown[l], d, F, l);
  }
  gemm(KC_GEMM_LM_HEAD, F32_STORE, c->logits, c->x, c->lm_head, md.V, d, 0);
  return launch_status();
}

// After a step whose logits were not finite the K/V it appended (slots prefix_len .. prefix_len + n_nodes of every
// sequence, every layer) may be NaN or infinite.  Dead slots are still fetched by whole-tile loads (and multiplied
// by a zero weight), so they are zeroed before any later step can fetch them.
int clear_step_slots(ded_ctx* c) {
  for (int l = 0; l < c->md.n_layers; ++l)
    for (int b = 0; b < c->batch; ++b) {
      if (c->bf16) bf16_kv_clear((bf16_t*)c->kc[l], (bf16_t*)c->vc[l], b, c->s_p[b], c->s_n[b], c->md, c->stream);
      else f32_kv_clear((float*)c->kc[l], (float*)c->vc[l], b, c->s_p[b], c->s_n[b], c->md, c->stream);
    }
  c->poisoned = false;
  return launch_status();
}

// Rows that decide into which k ranges a step's projections are summed: those of its trees padded to the largest, so that
// the sums of a tree do not depend on how much its neighbours in the batch fall short of it.  (They do depend on the room
// that the context, sized by its max_batch and max_nodes, has for split sums.)
int sum_rows(const ded_ctx* c) { return round_up(c->batch * c->n_step, 64); }
GemmPlan plan_gemm(const ded_ctx* c, int rows_pad, int N, int K, int planes, bool residual = false) {
  const int rows = sum_rows(c);
  const int cap = (int)std::min<int64_t>(8, c->part_elems / ((int64_t)rows * round_up(N, 64)));
  GemmPlan plan = residual ? bf16_gemm_plan_residual(rows, rows_pad, N, K, std::max(cap, 1), c->part_elems)
                           : bf16_gemm_plan(rows, rows_pad, N, K, planes, std::max(cap, 1), c->part_elems);
  if (!plan.tile && bf16_gemm_tiles(rows, N, plan) > kGemmCounters) plan.splits = 1;
  return plan;
}
// Steps of few rows run the slim projections, all or none of them: their sums of squares come per 4 features and lie in
// the split-K buffer (at least 512 rows of d floats), which such a step has no other use for.
bool slim_step(const ded_ctx* c) {
  const ModelDims& md = c->md;
  if (c->rows > BF16_SLIM_ROWS) return false;
  const int qd = md.H * md.hd, qkv_n = qd + 2 * md.Hkv * md.hd;
  auto fits = [&](int N, int K, int planes) { return bf16_gemm_slim_ok(plan_gemm(c, 64, N, K, planes), K, planes); };
  auto fits_residual = [&](int N, int K) { return bf16_gemm_slim_ok(plan_gemm(c, 64, N, K, 1, true), K, 1); };
  return fits(md.V, md.d, 2) && (md.n_layers == 0 || (fits(qkv_n, md.d, 2) && fits_residual(md.d, qd) && fits(2 * md.F, md.d, 2) &&
                                                      fits_residual(md.d, md.F)));
}

// LM head of the 16-bit path on the final residual stream (c->y_p / c->ssq as the last layer left them): the per-group top-2
// candidates that the per-node argmax needs and, with want_logits, the fp32 logits, into the workspace and the rows of real nodes
// into the caller's logits_out too if it is not null (otherwise no logits reach memory).
bool lm_head_bf16(ded_ctx* c, bool want_logits, float* logits_out = nullptr) {
  const ModelDims& md = c->md;
  const int rows = c->rows, rows_pad = round_up(rows, 64), d = md.d;
  GemmEpilogue e = {};
  e.rows = rows;
  e.rb_total = rows_pad / 16;
  e.eps = md.eps;
  const bool slim = slim_step(c), fine = slim && md.n_layers > 0;  // without layers the embedding's sums are the last ones
  e.ssq_in = fine ? c->part : c->ssq;
  e.ssq_groups = fine ? d / 4 : d / 64;
  e.inv_k = 1.0f / (float)d;
  if (want_logits) {
    e.kind = EPI_LOGITS;
    e.out = c->logits;
    e.out_stride = md.V;
    e.logits_out = logits_out;
    e.max_nodes = c->cfg.max_nodes;
    const StepMeta m = c->meta();
    e.seq_n = m.seq_n;
    e.row0 = m.row0;
    e.blk_seq = m.blk_seq;
  } else {
    e.kind = EPI_TOP2;
  }
  e.top2_part = c->top2_part;
  e.top2_groups = (md.V + 63) / 64;
  // From 256 rows on the projection is bound by the matrix cores and reads the hi plane of its input alone: the lo
  // plane matters for what is carried through the layers, not here, where one rounding of the final normalised input
  // (2^-12 relative) moves a logit by ~2e-4.  Below, the weight stream bounds it and the lo product is free.
  const int planes = sum_rows(c) >= 256 ? 1 : 2;
  const GemmPlan plan = plan_gemm(c, rows_pad, md.V, d, planes);
  ProfScope p(c, KC_GEMM_LM_HEAD);
  if (slim) return bf16_gemm_slim(c->y_p, (const bf16_t*)c->lm_head, rows, rows_pad, md.V, d, planes, plan, e, c->stream);
  return bf16_gemm(c->part, (int64_t)rows_pad * round_up(md.V, 64), c->part_elems, c->y_p, (const bf16_t*)c->lm_head,
                   rows_pad, md.V, d, planes, plan, c->counters, e, c->stream);
}

int forward_bf16(ded_ctx* c, bool want_logits, float* logits_out) {
  const ModelDims& md = c->md;
  StepMeta m = c->meta();
  hipStream_t s = c->stream;
  const int d = md.d, qd = md.H * md.hd, kvd = md.Hkv * md.hd, qkv_n = qd + 2 * kvd, F = md.F, L = md.n_layers;
  const int rows_pad = round_up(m.rows, 64);
  bool ok = true;
  GemmEpilogue base = {};
  base.rows = m.rows;
  base.rb_total = rows_pad / 16;
  base.eps = md.eps;
  // planes: 2 = the input is consumed as hi + lo, 1 = hi only (enough for the O and down projections)
  const bool slim = slim_step(c);
  auto gemm = [&](int cls, const bf16_t* xp, const void* w, int N, int K, int planes, const GemmEpilogue& epi) {
    const GemmPlan plan = plan_gemm(c, rows_pad, N, K, planes, epi.kind == EPI_RESIDUAL);
    ProfScope p(c, cls);
    if (slim)
      ok = bf16_gemm_slim(xp, (const bf16_t*)w, m.rows, rows_pad, N, K, planes, plan, epi, s) && ok;
    else
      ok = bf16_gemm(c->part, (int64_t)rows_pad * round_up(N, 64), c->part_elems, xp, (const bf16_t*)w, rows_pad, N, K,
                     planes, plan, c->counters, epi, s) && ok;
  };
  // RMSNorm is deferred: whoever produces the residual stream also writes x * gain(next norm) as the next
  // GEMM input and sum(x^2) per 64 features; the consuming GEMM multiplies its output rows by 1/rms.
  auto normed_input = [&](GemmEpilogue& e, bool embedded = false) {
    const bool fine = slim && !embedded;
    e.ssq_in = fine ? c->part : c->ssq;
    e.ssq_groups = fine ? d / 4 : d / 64;
    e.inv_k = 1.0f / (float)d;
  };
  auto next_gain = [&](int l) { return l < L ? c->norm_attn[l] : c->final_norm; };
  { ProfScope p(c, KC_EMBED); bf16_embed(c->x, c->y_p, c->ssq, (const bf16_t*)c->emb, next_gain(0), c->front(), rows_pad, d, s); }
  for (int l = 0; l < L; ++l) {
    {
      GemmEpilogue e = base;
      e.kind = EPI_QKV;
      normed_input(e, l == 0);
      e.q_packed = c->q_p;
      e.k_cache = (bf16_t*)c->kc[l];
      e.v_cache = (bf16_t*)c->vc[l];
      e.rope_tab = c->rope_tab;
      e.seq_p = m.seq_p;
      e.seq_n = m.seq_n;
      e.row0 = m.row0;
      e.blk_seq = m.blk_seq;
      e.n_step = m.n_step;
      e.H = md.H;
      e.Hkv = md.Hkv;
      e.cap = md.cap;
      gemm(KC_GEMM_QKV, c->y_p, c->wqkv[l], qkv_n, d, 2, e);
    }
    int ns = bf16_attn_pick_splits(m, md, c->max_p, c->attn_part_rows);
    { ProfScope p(c, KC_TREE_ATTN);
      bf16_tree_attention(c->o_p, rows_pad, c->q_p, (const bf16_t*)c->kc[l], (const bf16_t*)c->vc[l], c->attn_part_o,
                          c->attn_part_ml, ns, bf16_attn_query_planes(m, md), m, md, s); }
    {
      GemmEpilogue e = base;
      e.kind = EPI_RESIDUAL;
      e.x = c->x;
      e.gain = c->norm_ffn[l];
      e.y_packed = c->y_p;
      e.ssq_out = slim ? c->part : c->ssq;
      gemm(KC_GEMM_O, c->o_p, c->wo[l], d, qd, 1, e);
    }
    {
      GemmEpilogue e = base;
      e.kind = EPI_SILU;
      normed_input(e);
      e.y_packed = c->h_p;
      gemm(KC_GEMM_GATE_UP, c->y_p, c->wgu[l], 2 * F, d, 2, e);
    }
    {
      GemmEpilogue e = base;
      e.kind = EPI_RESIDUAL;
      e.x = c->x;
      e.gain = next_gain(l + 1);
      e.y_packed = c->y_p;
      e.ssq_out = slim ? c->part : c->ssq;
      gemm(KC_GEMM_DOWN, c->h_p, c->wdown[l], d, F, 1, e);
    }
  }
  ok = lm_head_bf16(c, want_logits, logits_out) && ok;
  if (!ok) return DED_EINVAL;
  return launch_status();
}

}  // namespace

// =============================================================================================
extern "C" {

const char* ded_strerror(int code) {
  switch (code) {
    case DED_OK: return "ok";
    case DED_EINVAL: return "invalid argument or unsupported configuration";
    case DED_ETREE: return "malformed draft tree (parent[0] must be -1 and 0 <= parent[i] < i)";
    case DED_ETOKEN: return "token id outside the vocabulary";
    case DED_ECAP: return "prefix_len + n_nodes exceeds kv_capacity";
    case DED_ESTATE: return "call out of order";
    case DED_EHIP: return "HIP runtime failure";
    case DED_ENOMEM: return "workspace too small or host allocation failed";
    case DED_ENONFINITE: return "NaN or infinity in the logits of a tree node (weights or activations outside the half-precision operand range?)";
    default: return "unknown error";
  }
}

size_t ded_workspace_bytes(const ded_config* cfg) {
  if (!config_ok(cfg)) return 0;
  return carve_workspace(*cfg, nullptr, nullptr);
}

size_t ded_kv_layer_bytes(const ded_config* cfg) {
  if (!config_ok(cfg)) return 0;
  size_t elem = cfg->dtype == DED_BF16 ? 2 : 4;
  return (size_t)cfg->max_batch * cfg->n_kv_heads * cfg->kv_capacity * cfg->head_dim * elem;
}

int ded_validate_tree(const ded_config* cfg, int32_t batch, const int32_t* prefix_len, const int32_t* n_nodes,
                      const int32_t* parent, const int32_t* token) {
  if (!config_ok(cfg)) return DED_EINVAL;
  return validate_step(*cfg, batch, prefix_len, n_nodes, parent, token, true);
}

int ded_verify_init(const ded_config* cfg, const ded_weights* w, const ded_kv* kv, void* workspace,
                    size_t workspace_bytes, void* hip_stream, ded_ctx** out) {
  if (!out) return DED_EINVAL;
  *out = nullptr;
  if (!config_ok(cfg) || !w || !kv || !workspace) return DED_EINVAL;
  const int L = cfg->n_layers;
  if (!w->emb || !w->lm_head || !w->final_norm) return DED_EINVAL;
  if (L > 0 && (!w->wqkv || !w->wo || !w->wgate_up || !w->wdown || !w->norm_attn || !w->norm_ffn || !kv->k || !kv->v))
    return DED_EINVAL;
  for (int l = 0; l < L; ++l)
    if (!w->wqkv[l] || !w->wo[l] || !w->wgate_up[l] || !w->wdown[l] || !w->norm_attn[l] || !w->norm_ffn[l] ||
        !kv->k[l] || !kv->v[l])
      return DED_EINVAL;
  if (reinterpret_cast<uintptr_t>(workspace) % 256) return DED_EINVAL;
  size_t need = carve_workspace(*cfg, nullptr, nullptr);
  if (workspace_bytes < need) return DED_ENOMEM;

  ded_ctx* c = new (std::nothrow) ded_ctx();
  if (!c) return DED_ENOMEM;
  c->cfg = *cfg;
  c->bf16 = cfg->dtype == DED_BF16;
  c->stream = reinterpret_cast<hipStream_t>(hip_stream);
  // set-up of the library's own scratch array: resolved here, once per device, with the context's device current
  if (hipGetDevice(&c->device) != hipSuccess) {
    (void)hipGetLastError();
    delete c;
    return DED_EHIP;
  }
  c->static_scratch = resolve_static_scratch(c->device);
  if (!c->static_scratch) {
    delete c;
    return DED_EHIP;
  }
  c->md = ModelDims{cfg->n_layers, cfg->d_model, cfg->n_heads, cfg->n_kv_heads, cfg->head_dim,
                    cfg->d_ffn,    cfg->vocab,   cfg->kv_capacity, cfg->rope_base, cfg->rms_eps};
  Sizes z = sizes_of(*cfg);
  c->max_n_pad = z.max_n_pad;
  c->max_rows = z.max_rows;
  c->max_rows_pad = z.max_rows_pad;
  carve_workspace(*cfg, static_cast<char*>(workspace), c);
  c->kc.assign(kv->k, kv->k + L);
  c->vc.assign(kv->v, kv->v + L);

  auto fail = [&](int code) {
    ded_verify_free(c);
    return code;
  };
  int stride = cfg->max_nodes + 1;
  c->res_bytes = align_up((size_t)z.max_rows_pad * 12 + (size_t)cfg->max_batch * 4 * (2 + 2 * stride), 256);
  // (coherent: kernels read and write them while they run)
  const unsigned kind = hipHostMallocMapped | hipHostMallocCoherent;
  c->meta_slots = (int)std::max<size_t>(2, std::min<size_t>(16, kMetaMirrorBytes / c->meta_bytes) / 2 * 2);
  if (hipHostMalloc(reinterpret_cast<void**>(&c->h_meta_slots), c->meta_bytes * c->meta_slots, kind) != hipSuccess ||
      hipHostMalloc(reinterpret_cast<void**>(&c->h_res), c->res_bytes, kind) != hipSuccess ||
      hipHostGetDevicePointer(reinterpret_cast<void**>(&c->h_meta_slots_dev), c->h_meta_slots, 0) != hipSuccess ||
      hipHostGetDevicePointer(reinterpret_cast<void**>(&c->h_res_dev), c->h_res, 0) != hipSuccess) {
    (void)hipGetLastError();
    return fail(DED_EHIP);
  }
  memset(c->h_meta_slots, 0, c->meta_bytes * c->meta_slots);
  if (hipEventCreateWithFlags(&c->meta_ev[0], hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&c->meta_ev[1], hipEventDisableTiming) != hipSuccess) {
    (void)hipGetLastError();
    return fail(DED_EHIP);
  }
  hipStream_t s = c->stream;
  const int64_t d = cfg->d_model, V = cfg->vocab, F = cfg->d_ffn;
  const int64_t qd = (int64_t)cfg->n_heads * cfg->head_dim, kvd = (int64_t)cfg->n_kv_heads * cfg->head_dim;
  const int64_t qkv_n = qd + 2 * kvd;
#define INIT_TRY(expr)                  \
  do {                                  \
    if ((expr) != hipSuccess) {         \
      (void)hipGetLastError();          \
      return fail(DED_EHIP);            \
    }                                   \
  } while (0)
  // activations start from zero so that padding rows hold finite values
  {
    char* act0 = reinterpret_cast<char*>(c->d_kc);
    size_t act_bytes = need - (size_t)(act0 - static_cast<char*>(workspace));
    INIT_TRY(hipMemsetAsync(act0, 0, act_bytes, s));
  }
  // cache slots beyond the live range are read (and masked) by whole-tile loads: keep them finite
  for (int l = 0; l < L; ++l) {
    INIT_TRY(hipMemsetAsync(c->kc[l], 0, ded_kv_layer_bytes(cfg), s));
    INIT_TRY(hipMemsetAsync(c->vc[l], 0, ded_kv_layer_bytes(cfg), s));
  }
  if (L > 0) {
    INIT_TRY(hipMemcpyAsync(c->d_kc, c->kc.data(), sizeof(void*) * L, hipMemcpyHostToDevice, s));
    INIT_TRY(hipMemcpyAsync(c->d_vc, c->vc.data(), sizeof(void*) * L, hipMemcpyHostToDevice, s));
  }
  auto copy_gain = [&](float* dst, const float* src) {
    return hipMemcpyAsync(dst, src, sizeof(float) * d, hipMemcpyDeviceToDevice, s);
  };
  INIT_TRY(copy_gain(c->final_norm, w->final_norm));
  INIT_TRY(hipMemcpyAsync(c->emb, w->emb, (size_t)V * d * z.elem, hipMemcpyDeviceToDevice, s));
  if (!c->bf16) {
    // (packed with the gain of the norm before the projection)
    auto pack = [&](void* dst, const void* src, const float* gain, int64_t n, int64_t k) {
      f32_pack_weight((float*)dst, (const float*)src, gain, (int)n, (int)k, s);
    };
    pack(c->lm_head, w->lm_head, w->final_norm, V, d);
    for (int l = 0; l < L; ++l) {
      pack(c->wqkv[l], w->wqkv[l], w->norm_attn[l], qkv_n, d);
      pack(c->wo[l], w->wo[l], nullptr, d, qd);
      pack(c->wgu[l], w->wgate_up[l], w->norm_ffn[l], F, d);
      pack((float*)c->wgu[l] + f32_packed_floats(F, d), (const float*)w->wgate_up[l] + F * d, w->norm_ffn[l], F, d);
      pack(c->wdown[l], w->wdown[l], nullptr, d, F);
    }
    INIT_TRY(hipGetLastError());
  } else {
    bf16_pack_weight((bf16_t*)c->lm_head, (const bf16_t*)w->lm_head, (int)V, (int)d, PERM_NONE, s);
    for (int l = 0; l < L; ++l) {
      bf16_pack_weight((bf16_t*)c->wqkv[l], (const bf16_t*)w->wqkv[l], (int)qkv_n, (int)d, PERM_ROPE, s);
      bf16_pack_weight((bf16_t*)c->wo[l], (const bf16_t*)w->wo[l], (int)d, (int)qd, PERM_NONE, s);
      bf16_pack_weight((bf16_t*)c->wgu[l], (const bf16_t*)w->wgate_up[l], (int)(2 * F), (int)d, PERM_GATE_UP, s);
      bf16_pack_weight((bf16_t*)c->wdown[l], (const bf16_t*)w->wdown[l], (int)d, (int)F, PERM_NONE, s);
      INIT_TRY(copy_gain(c->norm_attn[l], w->norm_attn[l]));
      INIT_TRY(copy_gain(c->norm_ffn[l], w->norm_ffn[l]));
    }
    INIT_TRY(hipGetLastError());
  }
  INIT_TRY(hipStreamSynchronize(s));
#undef INIT_TRY
  *out = c;
  return DED_OK;
}

void ded_verify_free(ded_ctx* c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  for (hipEvent_t e : c->ev_pool) (void)hipEventDestroy(e);
  for (hipEvent_t e : c->meta_ev)
    if (e) (void)hipEventDestroy(e);
  if (c->h_meta_slots) (void)hipHostFree(c->h_meta_slots);
  if (c->h_res) (void)hipHostFree(c->h_res);
  delete c;
}

int ded_verify_step(ded_ctx* c, int32_t batch, const int32_t* prefix_len, const int32_t* n_nodes,
                    const int32_t* parent, const int32_t* token, float* logits_out) {
  if (!c) return DED_EINVAL;
  int rc = validate_step(c->cfg, batch, prefix_len, n_nodes, parent, token, true);
  if (rc != DED_OK) return rc;
  if (c->poisoned && (rc = clear_step_slots(c)) != DED_OK) return rc;
  rc = ingest(c, batch, prefix_len, n_nodes, parent, token);
  if (rc != DED_OK) return rc;
  c->pending = false;
  c->have_argmax = false;
  // the fp32 logits are materialised only for a caller that asks for them or samples from them
  const bool want_logits = !c->bf16 || logits_out != nullptr || c->sampling_seen;
  c->have_logits = false;
  rc = c->bf16 ? forward_bf16(c, want_logits, logits_out) : forward_f32(c);
  if (rc != DED_OK) return rc;
  StepMeta m = c->meta();
  if (c->bf16) {
    // the LM head has left every row's candidates, and the logits where they are wanted, the caller's rows among them
    ProfScope p(c, KC_TOP2_REDUCE);
    launch_top2_reduce(c->top2_part, (c->md.V + 63) / 64, m.rows, c->d_amax, c->d_margin, c->d_rowflag, c->stream);
  } else {
    ProfScope p(c, KC_ARGMAX);
    launch_argmax(c->logits, m, c->md.V, c->d_amax, c->d_margin, c->d_rowflag, logits_out, c->cfg.max_nodes, c->stream);
  }
  c->have_logits = want_logits;
  rc = launch_status();
  if (rc != DED_OK) return rc;
  c->pending = true;
  c->have_argmax = true;
  return DED_OK;
}

int ded_accept(ded_ctx* c, int32_t mode, int32_t* accepted_tokens, int32_t* n_accepted,
               int32_t* compaction_idx, int32_t* new_prefix_len) {
  if (!c || !accepted_tokens || !n_accepted || !compaction_idx || !new_prefix_len) return DED_EINVAL;
  if (mode != 0 && mode != 1) return DED_EINVAL;
  if (!c->pending) return DED_ESTATE;
  const int mn = c->cfg.max_nodes, stride = mn + 1, B = c->batch;
  if (mode == 1) {
    for (int b = 0; b < B; ++b)
      for (int i = 1; i < c->s_n[b]; ++i)
        if (c->s_parent[(size_t)b * mn + i] != i - 1) return DED_ETREE;
  }
  StepMeta m = c->meta();
  hipStream_t s = c->stream;
  // nacc | seqflag | path | acctok, written by the kernel and read below
  const int MB = c->cfg.max_batch;
  int32_t* h_n = reinterpret_cast<int32_t*>(c->h_res);
  int32_t *h_flag = h_n + MB, *h_path = h_flag + MB, *h_tok = h_path + (size_t)MB * stride;
  auto on_device = [&](int32_t* p) { return reinterpret_cast<int32_t*>(c->h_res_dev + (reinterpret_cast<char*>(p) - c->h_res)); };
  const ApprovalWalk w = {m.token, m.parent, m.seq_n, m.row0, c->d_amax, c->d_rowflag, B, mode, stride,
                          on_device(h_n), on_device(h_flag), on_device(h_path), on_device(h_tok)};
  if (c->md.n_layers > 0 && mode == 0) {
    ProfScope p(c, KC_COMPACT);
    if (c->bf16) bf16_kv_compact((bf16_t* const*)c->d_kc, (bf16_t* const*)c->d_vc, w, m, c->md, s);
    else f32_kv_compact((float* const*)c->d_kc, (float* const*)c->d_vc, w, m, c->md, s);
  } else {
    ProfScope p(c, KC_WALK);
    launch_accept_walk(w, s);
  }
  if (launch_status() != DED_OK) return DED_EHIP;
  HIP_TRY(hipStreamSynchronize(s));
  c->pending = false;
  for (int b = 0; b < B; ++b)
    if (h_flag[b]) {  // the walk kept nothing: every sequence's cache is as it was before the step
      int rc = clear_step_slots(c);
      return rc != DED_OK ? rc : DED_ENONFINITE;
    }
  for (int b = 0; b < B; ++b) {
    int len = h_n[b];
    if (len < 1 || len > c->s_n[b]) return DED_EHIP;
    n_accepted[b] = len;
    new_prefix_len[b] = c->s_p[b] + len;
    memcpy(accepted_tokens + (size_t)b * stride, h_tok + (size_t)b * stride, sizeof(int32_t) * len);
    memcpy(compaction_idx + (size_t)b * stride, h_path + (size_t)b * stride, sizeof(int32_t) * len);
  }
  return DED_OK;
}

int ded_sample(ded_ctx* c, float temperature, float top_p, const float* uniform) {
  if (!c || !uniform) return DED_EINVAL;
  if (!(temperature > 0.f) || !(top_p > 0.f) || !(top_p <= 1.f)) return DED_EINVAL;
  if (!c->pending || !c->have_argmax) return DED_ESTATE;
  const int mn = c->cfg.max_nodes, rows = c->rows;
  float* h_u = reinterpret_cast<float*>(c->h_res);  // nothing else is in flight on the pinned result block
  for (int b = 0; b < c->batch; ++b)
    for (int i = 0; i < round_up(c->s_n[b], 16); ++i) {
      float u = i < c->s_n[b] ? uniform[(size_t)b * mn + i] : 0.f;
      if (!(u >= 0.f) || !(u < 1.f)) return DED_EINVAL;
      h_u[c->s_row0[b] + i] = u;
    }
  // A step keeps its logits only if the caller asked for them or the context has sampled before; the first
  // sampled step of a context recomputes them from the final residual stream, which is still in place.
  c->sampling_seen = true;
  if (!c->have_logits) {
    if (!lm_head_bf16(c, true)) return DED_EINVAL;
    c->have_logits = true;
  }
  const int32_t* h_f = reinterpret_cast<int32_t*>(c->h_res) + rows;  // written by the kernel
  { ProfScope p(c, KC_SAMPLE);
    launch_sample_top_p(c->logits, c->md.V, c->meta(), c->md.V, temperature, top_p, reinterpret_cast<const float*>(c->h_res_dev),
                        c->d_rowflag, c->d_amax, reinterpret_cast<int32_t*>(c->h_res_dev) + rows, c->stream); }
  if (launch_status() != DED_OK) return DED_EHIP;
  HIP_TRY(hipStreamSynchronize(c->stream));  // h_res is free again
  for (int b = 0; b < c->batch; ++b)
    for (int i = 0; i < c->s_n[b]; ++i)
      if (h_f[c->s_row0[b] + i]) {
        c->poisoned = true;
        return DED_ENONFINITE;
      }
  return DED_OK;
}

int ded_get_argmax(ded_ctx* c, int32_t* argmax, float* margin) {
  if (!c || !argmax) return DED_EINVAL;
  if (!c->have_argmax) return DED_ESTATE;
  const int rows = c->rows, mn = c->cfg.max_nodes;
  const int32_t* h_a = reinterpret_cast<int32_t*>(c->h_res);
  const float* h_m = reinterpret_cast<float*>(c->h_res) + rows;
  const int32_t* h_f = h_a + 2 * (size_t)rows;
  HIP_TRY(hipMemcpyAsync(c->h_res, c->d_amax, sizeof(int32_t) * 3 * (size_t)rows, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  for (int b = 0; b < c->batch; ++b)
    for (int i = 0; i < c->s_n[b]; ++i)
      if (h_f[c->s_row0[b] + i]) {
        c->poisoned = true;
        return DED_ENONFINITE;
      }
  for (int b = 0; b < c->batch; ++b)
    for (int i = 0; i < c->s_n[b]; ++i) {
      argmax[(size_t)b * mn + i] = h_a[c->s_row0[b] + i];
      if (margin) margin[(size_t)b * mn + i] = h_m[c->s_row0[b] + i];
    }
  return DED_OK;
}

static int kv_copy_common(ded_ctx* c, int32_t layer, int32_t seq, int32_t first, int32_t n, void* kp, void* vp,
                          bool to_cache) {
  if (!c || layer < 0 || layer >= c->md.n_layers || seq < 0 || seq >= c->cfg.max_batch || first < 0 || n < 0)
    return DED_EINVAL;
  if ((int64_t)first + n > c->cfg.kv_capacity) return DED_ECAP;
  if (n == 0 || (!kp && !vp)) return DED_OK;
  ProfScope p(c, KC_LAYOUT);
  if (c->bf16) {
    bf16_kv_copy((bf16_t*)c->kc[layer], (bf16_t*)c->vc[layer], (bf16_t*)kp, (bf16_t*)vp, to_cache, seq, first, n,
                 c->md, c->stream);
  } else {
    if (kp) f32_kv_copy((float*)c->kc[layer], (float*)kp, to_cache, seq, first, n, c->md, c->stream);
    if (vp) f32_kv_copy((float*)c->vc[layer], (float*)vp, to_cache, seq, first, n, c->md, c->stream);
  }
  return launch_status();
}

int ded_kv_store(ded_ctx* c, int32_t layer, int32_t seq, int32_t first_slot, int32_t n, const void* k_plain,
                 const void* v_plain) {
  return kv_copy_common(c, layer, seq, first_slot, n, const_cast<void*>(k_plain), const_cast<void*>(v_plain), true);
}

int ded_kv_load(ded_ctx* c, int32_t layer, int32_t seq, int32_t first_slot, int32_t n, void* k_plain,
                void* v_plain) {
  return kv_copy_common(c, layer, seq, first_slot, n, k_plain, v_plain, false);
}

// Transient device buffers of one stand-alone attention call: the step description and the split-KV partials.
struct AttnScratch {
  char* d_meta;
  float* part_o;
  float2* part_ml;
  int64_t part_rows;
};

static int tree_attention_common(ded_ctx* c, int32_t layer, int32_t batch, const int32_t* prefix_len,
                                 const int32_t* n_nodes, const int32_t* parent, const void* q, const void* k_tree,
                                 const void* v_tree, void* out, bool st) {
  if (!c || !q || !k_tree || !v_tree || !out) return DED_EINVAL;
  if (layer < 0 || layer >= c->md.n_layers) return DED_EINVAL;
  int rc = validate_step(c->cfg, batch, prefix_len, n_nodes, parent, nullptr, false);
  if (rc != DED_OK) return rc;
  if (c->poisoned && (rc = clear_step_slots(c)) != DED_OK) return rc;
  const ModelDims& md = c->md;
  AttnScratch ws = {c->d_meta, c->attn_part_o, c->attn_part_ml, c->attn_part_rows};
  int ns = 1;
  if (c->bf16) {
    // the key-range count is the workspace path's in both variants, so both give the same bits
    int nmax = 0, pmax = 0, rows = 0;
    for (int b = 0; b < batch; ++b) {
      nmax = std::max(nmax, n_nodes[b]);
      pmax = std::max(pmax, prefix_len[b]);
      rows += round_up(n_nodes[b], 16);
    }
    StepMeta shape = {};
    shape.batch = batch;
    shape.n_step = round_up(nmax, 16);
    shape.rows = rows;
    ns = bf16_attn_pick_splits(shape, md, pmax, c->attn_part_rows);
    if (st) {  // carve the library's own array; a call that does not fit is refused before anything is enqueued
      const int64_t part_rows = (int64_t)batch * md.H * ns * shape.n_step;
      Carve w(reinterpret_cast<char*>(c->static_scratch));
      ws.d_meta = w.take<char>(c->meta_bytes);
      // counted with every call as documented, though the queries and the output are no longer re-laid-out: what is refused
      // does not change
      w.take<bf16_t>((int64_t)round_up(shape.rows, 64) * md.H * md.hd * 4);
      ws.part_o = w.take<float>(part_rows * md.hd);
      ws.part_ml = w.take<float2>(part_rows);
      ws.part_rows = part_rows;
      if (w.off > kStaticScratchBytes) return DED_ECAP;
    }
  } else if (st) {
    return DED_EINVAL;  // the fp32 path has no transient buffers of this kind
  }
  rc = ingest(c, batch, prefix_len, n_nodes, parent, nullptr);
  if (rc != DED_OK) return rc;
  c->pending = false;
  c->have_argmax = false;
  StepMeta m = c->meta_at(ws.d_meta);
  hipStream_t s = c->stream;
  const int mn = c->cfg.max_nodes, qd = md.H * md.hd;
  if (c->bf16) {
    const int rows_pad = round_up(m.rows, 64);
    { ProfScope p(c, KC_LAYOUT);
      bf16_scatter_tree_kv((bf16_t*)c->kc[layer], (bf16_t*)c->vc[layer], (const bf16_t*)k_tree, (const bf16_t*)v_tree,
                           c->meta_at(c->h_meta_dev), c->h_meta_dev, ws.d_meta, (int)c->meta_units(), c->s_p.data(), c->s_n.data(),
                           md, mn, s); }
    { ProfScope p(c, KC_TREE_ATTN);
      bf16_tree_attention(nullptr, rows_pad, nullptr, (const bf16_t*)c->kc[layer], (const bf16_t*)c->vc[layer], ws.part_o,
                          ws.part_ml, ns, 1, m, md, s, (const bf16_t*)q, (bf16_t*)out, mn); }
  } else {
    { ProfScope p(c, KC_META);
      HIP_TRY(hipMemcpyAsync(ws.d_meta, c->h_meta, c->off.bytes, hipMemcpyHostToDevice, s)); }
    { ProfScope p(c, KC_LAYOUT);
      f32_scatter_tree_kv((float*)c->kc[layer], (float*)c->vc[layer], (const float*)k_tree, (const float*)v_tree, m, md, mn, s);
      f32_gather_rows(c->f_qkv, (const float*)q, m, mn, qd, true, s); }
    { ProfScope p(c, KC_TREE_ATTN);
      f32_attention(c, c->f_qkv, qd, layer, m, s); }
    { ProfScope p(c, KC_LAYOUT); f32_gather_rows((float*)out, c->f_o, m, mn, qd, false, s); }
  }
  return launch_status();
}

int ded_tree_attention(ded_ctx* c, int32_t layer, int32_t batch, const int32_t* prefix_len,
                       const int32_t* n_nodes, const int32_t* parent, const void* q, const void* k_tree,
                       const void* v_tree, void* out) {
  return tree_attention_common(c, layer, batch, prefix_len, n_nodes, parent, q, k_tree, v_tree, out, false);
}

int ded_tree_attention_static(ded_ctx* c, int32_t layer, int32_t batch, const int32_t* prefix_len,
                              const int32_t* n_nodes, const int32_t* parent, const void* q, const void* k_tree,
                              const void* v_tree, void* out) {
  if (!c) return DED_EINVAL;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return DED_EHIP;
  }
  if (dev != c->device || !c->static_scratch) return DED_EINVAL;  // the array's address belongs to the context's device
  return tree_attention_common(c, layer, batch, prefix_len, n_nodes, parent, q, k_tree, v_tree, out, true);
}

size_t ded_static_scratch_bytes(void) { return kStaticScratchBytes; }

int ded_probe_stream_read(const void* device_buffer, size_t bytes, void* sink4, void* hip_stream) {
  if (!device_buffer || !sink4 || bytes < 16 || reinterpret_cast<uintptr_t>(device_buffer) % 16) return DED_EINVAL;
  launch_stream_read(device_buffer, bytes / 16 * 16, static_cast<uint32_t*>(sink4), reinterpret_cast<hipStream_t>(hip_stream));
  return launch_status();
}

int ded_profile_enable(ded_ctx* c, int32_t on) {
  if (!c) return DED_EINVAL;
  int rc = prof_drain(c);
  if (rc != DED_OK) return rc;
  if (on) {
    for (int i = 0; i < KC_COUNT; ++i) {
      c->prof_ms[i] = 0;
      c->prof_n[i] = 0;
    }
  }
  c->prof_on = on != 0;
  return DED_OK;
}

int ded_profile_read(ded_ctx* c, int32_t cap, const char** names, double* total_ms, int64_t* launches) {
  if (!c || cap < 0 || (cap > 0 && (!names || !total_ms || !launches))) return DED_EINVAL;
  int rc = prof_drain(c);
  if (rc != DED_OK) return rc;
  for (int i = 0; i < KC_COUNT && i < cap; ++i) {
    names[i] = kClassNames[i];
    total_ms[i] = c->prof_ms[i];
    launches[i] = c->prof_n[i];
  }
  return KC_COUNT;
}

}  // extern "C"
